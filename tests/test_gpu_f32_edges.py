"""The f32 FFN launch at the edges of its 32 x 32 work items, against the
oracle element by element: remainders on both sides of 32 and 64 rows, K
whose quarters are 16, 32 and 48 (short chunks only), 64 and 80 (a long chunk
and a remainder)."""

import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import F32_RTOL, assert_close, log, make_context, to_dev, to_host, upload_weights

pytestmark = pytest.mark.gpu

DEPTHS = [1, 31, 32, 33, 0, 63, 64, 65, 129]


@pytest.mark.parametrize("d,f", [(64, 128), (192, 64), (256, 320), (320, 192)])
def test_f32_edges_match_oracle(d, f):
    w = synth.Workload(f"f32_{d}_{f}", 116, d=d, f=f, E=len(DEPTHS), k=1, zipf_s=1.0, mode="rows",
                       depth_max=max(DEPTHS), act="f32", wdt="f32")
    g = np.random.default_rng(41)
    N = sum(DEPTHS)
    tok = g.permutation(N).astype(np.int32)
    gw = g.random(N, dtype=np.float32)
    x = g.standard_normal((N, d), dtype=np.float32)
    log(f"case f32 edges: depths {DEPTHS}, d={d} f={f}")
    ws = synth.all_expert_weights(w, 0, threads=4)
    ctx = make_context(w, max_tokens=N)
    dev_w = upload_weights(ctx, w, 0, ws)
    lq = oracle.LayerQueues(w.E, 1)
    keep, r0 = [], 0
    for e, n in enumerate(DEPTHS):
        if n:
            s = slice(r0, r0 + n)
            keep.append((to_dev(x[s], "f32"), to_dev(tok[s], "i32"), to_dev(gw[s], "f32")))
            ctx.enqueue_rows(0, e, *keep[-1], N)
            lq.enqueue_rows(e, x[s], tok[s], gw[s], N)
        r0 += n
    b = ctx.rebatch(0)
    y = to_host(ctx.expert_ffn(b))
    ctx.release(b)
    ctx.sync()
    st = assert_close(y, oracle.moe_layer(lq, ws, "f32", "f32")["y"], F32_RTOL, f"f32 d={d} f={f} y")
    log(f"case f32 edges d={d} f={f}: y {st}")
    del ctx, dev_w, keep

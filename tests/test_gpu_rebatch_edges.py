"""Re-batch at the edges of its paths: group counts on both sides of one wave
(64) and of the plan's workgroup (1024), empty experts first, last and in
runs, row lengths of less than, exactly and more than a pass of the gather.
Counts, offsets, row order and rows bit for bit; y (every tile's group)
against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import BF16_RTOL, assert_close, log, make_context, to_dev, to_host, upload_weights
from test_gpu_tile_families import _rows

pytestmark = pytest.mark.gpu

DEPTHS = [0, 0, 1, 64, 65, 0, 128, 129, 3, 256, 257, 17, 0, 2, 600, 40]


@pytest.mark.parametrize("E,d", [(1, 64), (2, 576), (16, 4096), (17, 4160), (63, 8256), (64, 512), (65, 576),
                                 (130, 4160), (1024, 64)])
def test_rebatch_edges(E, d):
    g = np.random.default_rng(70 + E)
    depths = [257] if E == 1 else [0, 300] if E == 2 else [DEPTHS[i % 16] for i in g.permutation(E)]
    if E >= 16:
        depths[0] = depths[-1] = 0
    w = synth.Workload(f"rebatch_{E}_{d}", 118, d=d, f=64, E=E, k=1, zipf_s=1.0, mode="rows", depth_max=max(depths))
    if E > 200:
        depths = [min(n, 130) for n in depths]
    N, per = _rows(w, depths, 72)
    log(f"case rebatch E={E} d={d}: {N} rows")
    ws = synth.all_expert_weights(w, 0, threads=8)
    ctx = make_context(w, max_tokens=N)
    dev_w = upload_weights(ctx, w, 0, ws)
    x = np.concatenate([p["x"] for p in per])
    tok = np.concatenate([p["token_ids"] for p in per])
    gw = np.concatenate([p["gate_w"] for p in per])
    lq = oracle.LayerQueues(E, 1)
    for e, p in enumerate(per):
        if depths[e]:
            lq.enqueue_rows(e, p["x"], p["token_ids"], p["gate_w"], N)
    t = (to_dev(x, "bf16"), to_dev(tok, "i32"), to_dev(gw, "f32"))
    off = np.concatenate([[0], np.cumsum(depths)]).astype(np.int32)
    for rep in range(2):
        ctx.enqueue_rows_grouped(0, depths, *t, N)
        b = ctx.rebatch(0)
        y = ctx.expert_ffn(b)
        assert np.array_equal(to_host(b.counts()), depths)
        assert np.array_equal(to_host(b.offsets()), off)
        assert np.array_equal(to_host(b.row_token())[:N], tok)
        assert np.array_equal(to_host(b.row_weight())[:N], gw)
        assert np.array_equal(to_host(b.x_perm())[:N], x)
        ctx.release(b)
    assert_close(oracle.bf16_to_f64(to_host(y)), oracle.moe_layer(lq, ws, "bf16", "bf16")["y"], BF16_RTOL, "y")
    ctx.sync()
    del ctx, dev_w

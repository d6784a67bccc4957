"""The FFN launch at the edges of its tiles, rounds and rings, against the
oracle element by element: remainders on both sides of 64, 128 and 256 rows,
column counts that end inside a 256-column tile, K of fewer, as many and more
steps than a ring has stages, launches of several rounds whose workgroups
chain tiles of one family and then change to the next, and tails whose tiles
are cut along K (reruns bit-identical)."""

import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import BF16_RTOL, assert_close, log, make_context, to_dev, to_host, upload_weights
from test_gpu_tile_families import _rows

pytestmark = pytest.mark.gpu

EDGES = [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 0, 320, 321, 384, 385]
CASES = {
    # K steps: gate/up 3, down 5; the last column tiles hold 64 of 128 / 192 of 256
    "narrow": (EDGES, 192, 320),
    # 2 and 1 steps
    "short": (EDGES, 128, 64),
    # 17 and 13 steps: chained tiles of an odd number of steps
    "odd": (EDGES, 1088, 832),
    # 9 rounds of gate/up tiles of all three families (f / 128 = 72 column
    # tiles), 24 and 144 steps in the two launches
    "rounds": ([1100, 700, 300, 200, 100, 90, 50, 20] * 2, 1536, 9216),
    # a tail of all three families over few CUs, up to 8 pieces
    "tail": ([300, 100, 30], 512, 4096),
}


@pytest.mark.parametrize("case,wdt", [(c, w) for c in sorted(CASES) for w in ("bf16", "fp8")])
def test_ffn_edges_match_oracle(case, wdt):
    depths, d, f = CASES[case]
    w = synth.Workload(f"edges_{case}_{wdt}", 115, d=d, f=f, E=len(depths), k=1, zipf_s=1.0, mode="rows",
                       depth_max=max(depths), wdt=wdt)
    N, per = _rows(w, depths, 31)
    log(f"case edges {case}/{wdt}: depths {depths}, d={d} f={f}")
    ws = synth.all_expert_weights(w, 0, threads=8)
    ctx = make_context(w, max_tokens=N)
    dev_w = upload_weights(ctx, w, 0, ws)
    lq = oracle.LayerQueues(w.E, 1)
    keep = []
    for e, ex in enumerate(per):
        if depths[e]:
            keep.append((e, (to_dev(ex["x"], "bf16"), to_dev(ex["token_ids"], "i32"), to_dev(ex["gate_w"], "f32"))))
            lq.enqueue_rows(e, ex["x"], ex["token_ids"], ex["gate_w"], N)
    ys = []
    for rep in range(2):
        for e, t in keep:
            ctx.enqueue_rows(0, e, *t, N)
        b = ctx.rebatch(0)
        ys.append(to_host(ctx.expert_ffn(b)))
        ctx.release(b)
    ctx.sync()
    st = assert_close(oracle.bf16_to_f64(ys[0]), oracle.moe_layer(lq, ws, "bf16", wdt)["y"], BF16_RTOL,
                      f"edges {case}/{wdt} y")
    assert np.array_equal(ys[0], ys[1]), "results differ between runs"
    log(f"case edges {case}/{wdt}: y {st}, bit-identical rerun")
    del ctx, dev_w, keep

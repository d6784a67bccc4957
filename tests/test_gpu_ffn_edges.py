"""The FFN launch at the edges of its tiles, rounds and rings, against the
oracle element by element: remainders on both sides of 64, 128 and 256 rows,
column counts that end inside a 256-column tile, K of fewer, as many and more
steps than a ring has stages, launches of several rounds whose workgroups
chain tiles of one family and then change to the next, and tails whose tiles
are cut into column halves and along K (reruns bit-identical).  How the tails
are cut is a choice of the cost model; test_ffn_cut_host.py holds CUTS to it on
256 CUs."""

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
    # a tail of all three families over few CUs: gate/up 8 steps, down 64
    "tail": ([300, 100, 30], 512, 4096),
    # column halves, last ones that hold 64 columns, and none: 4.5 tiles of 128
    # features, 2.25 of 256 columns
    "halves": ([60, 340], 576, 576),
    # halves in pieces, in the down and in the gate/up launch
    "halves_pieces_down": ([300, 128], 576, 4160),
    "halves_pieces_gate_up": ([300, 128], 4160, 576),
    # whole tiles in pieces: all families at once, and 128-row tiles alone
    "whole_pieces": (([200, 100, 40] * 11)[:32], 320, 5120),
    "whole_pieces_128": ([100] * 34, 320, 5120),
    # more pieces would need more than the partial sums' area
    "area": ([520] * 19, 64, 6144),
}
# per launch (gate/up, down): column halves or not, and the families whose
# tiles or halves are cut into pieces
CUTS = {
    "halves": ((2, ()), (2, ())),
    "halves_pieces_down": ((2, ()), (2, (0, 1, 2))),
    "halves_pieces_gate_up": ((2, (0, 1, 2)), (2, ())),
    "whole_pieces": (None, (1, (0, 1, 2))),
    "whole_pieces_128": (None, (1, (1,))),
    "tail": ((2, ()), (2, (0, 1, 2))),
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

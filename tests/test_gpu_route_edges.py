"""Routing and queue append at the edges of the one-launch path for small
fragments (32 and 128 tokens), with larger fragments before, between and
after them in the same queues: routing, counts, row order and positions equal
to the oracle's, on tie-heavy logits too."""

import numpy as np
import pytest

import synth
from gpu_helpers import check_routing_and_queues, log, make_context, oracle_routed_layer, run_routed_layer, upload_weights

pytestmark = pytest.mark.gpu

FRAGS = [1, 31, 32, 200, 33, 63, 64, 65, 127, 128, 129, 2, 2100, 8]


@pytest.mark.parametrize("E,k,renorm,ties", [(5, 1, True, False), (8, 2, True, False), (13, 4, False, False),
                                             (32, 8, True, True), (33, 3, False, True), (64, 6, True, False),
                                             (64, 8, False, True)])
def test_fragment_sizes_match_oracle(E, k, renorm, ties):
    T = sum(FRAGS)
    w = synth.Workload(f"route_{E}_{k}", 117, d=64, f=64, E=E, k=k, zipf_s=1.0, renorm=renorm, tokens=(T,))
    g = np.random.default_rng(51 + E)
    log(f"case route E={E} k={k} renorm={renorm} ties={ties}: fragments {FRAGS}")
    frags = []
    for n in FRAGS:
        lg = g.standard_normal((n, E), dtype=np.float32)
        if ties:
            lg = np.round(lg)
        frags.append({"x": synth.round_to_bf16_bits(g.standard_normal((n, w.d), dtype=np.float32)), "logits": lg})
    ws = synth.all_expert_weights(w, 0, threads=4)
    ctx = make_context(w, max_tokens=T)
    dev_w = upload_weights(ctx, w, 0, ws)
    for rep in range(2):
        got = run_routed_layer(ctx, w, 0, frags)
        check_routing_and_queues(w, got, oracle_routed_layer(w, frags, ws, full_ffn=False))
    del ctx, dev_w

"""Pool merge and release at row lengths around a workgroup's pass (8 elements
per thread, 256 threads, two groups in flight): with top-1 routing and
renormalised weights a token's pool row is its expert row, so the released
rows are the FFN's rows bit for bit, and the pool is clean for a second use
of the same ids."""

import pytest
import torch

from gpu_helpers import log
from paper_2505_08944_amd import Context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 2048, 2112, 4096, 4160, 8256])
def test_released_rows_are_the_expert_rows(d, act):
    T, E, f = 37, 3, 64
    log(f"case pool d={d} {act}")
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    dt = torch.bfloat16 if act == "bf16" else torch.float32
    ctx = Context(1, E, d, f, 1, act=act, wdt=act, max_tokens_per_layer=T + 3, token_pool=True)
    W = [[(torch.randn(s, generator=g, device="cuda") * 0.05).to(dt) for s in ((f, d), (f, d), (d, f))]
         for _ in range(E)]
    for e in range(E):
        ctx.set_expert_weights(0, e, *W[e])
    out = torch.full((T + 3, d), 7.0, device="cuda", dtype=dt)
    ready = torch.empty(T + 3, device="cuda", dtype=torch.int32)
    for rep in range(2):
        x = torch.randn((T, d), generator=g, device="cuda").to(dt)
        lg = torch.randn((T, E), generator=g, device="cuda")
        ids = torch.randperm(T + 3, generator=g, device="cuda")[:T].to(torch.int32)
        ctx.route_enqueue_ids(0, x, lg, ids)
        want = out.clone()
        for e in range(E):
            b = ctx.rebatch_expert(0, e)
            y = ctx.expert_ffn(b)
            n = int(b.counts()[e])
            want[b.row_token()[:n].long()] = y[:n]
            ctx.pool_accumulate(b, y)
            ctx.release(b)
        ctx.pool_release(0, out, ready)
        assert torch.equal(out, want), f"rep {rep}"
        claimed = torch.zeros(T + 3, dtype=torch.int32, device="cuda")
        claimed[ids.long()] = 1
        assert torch.equal(ready, claimed)
        ctx.sync()
    del ctx, W

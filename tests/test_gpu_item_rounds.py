"""Prefill calls whose work items outnumber the compute units: every item is taken, by whichever workgroup's turn it is.  A sequence's items are
the same whether it is alone or in a batch, so a batch must give the bits of its sequences one by one (those stay within one round)."""
import math

import pytest
import torch

from paper_2604_12452_amd import lca

pytestmark = pytest.mark.gpu


def _batch(mode, B, L, H, S, g, w, dtype, up=False):
    gen = torch.Generator(device="cuda").manual_seed(100 * L + H)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(dtype)
    mla = mode == lca.MODE_MLA
    d_pool, d_sel = (512, 64) if mla else (128, 128)
    d_qk = d_pool + d_sel if mla else d_sel
    desc = lambda n: lca.Desc(B=n, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, mode=mode, dtype=lca.BF16 if dtype == torch.bfloat16 else lca.F16)
    Q = rnd(B, L, H, d_qk) / math.sqrt(d_qk)
    pool, sel = (rnd(B, L, d_pool), rnd(B, L, d_sel)) if mla else (rnd(B, L, S, d_pool), rnd(B, L, S, d_sel))
    W = rnd(H, 128, d_pool) / math.sqrt(d_pool) if up else None
    pool_rep, sel_rep, anchor, _ = lca.alloc_condensed(desc(B))
    ws = lca.alloc_workspace(desc(B))
    lca.condense(desc(B), Q, pool, sel, pool_rep, sel_rep, anchor, None, ws)

    def run(lo, n):
        O = torch.full((n, L, H, 128 if up else d_pool), math.nan, dtype=dtype, device="cuda")
        lse = torch.full((n, L, H), math.nan, device="cuda")
        a = [x[lo:lo + n].contiguous() for x in (Q, pool, sel, pool_rep, sel_rep)]
        if up:
            lca.prefill_attn_up(desc(n), *a, W, O, lse, ws)
        else:
            lca.prefill_attn(desc(n), *a, O, lse, ws)
        return O, lse

    O, lse = run(0, B)
    assert bool(O.isfinite().all()) and bool(lse.isfinite().all())
    return run, O, lse


@pytest.mark.parametrize("B,L,H,S,g,w,dtype", [
    (2, 1025, 32, 8, 16, 256, torch.bfloat16),      # 272 items: one more round for 16 workgroups
    (3, 1000, 28, 4, 32, 512, torch.float16),       # 336, four (sequence, KV head) pairs per sequence
    (9, 500, 32, 8, 8, 100, torch.bfloat16),        # 576: two rounds and a quarter
    (5, 600, 12, 4, 16, 64, torch.float16),         # 160: every workgroup one item or none
    (8, 2000, 16, 4, 16, 128, torch.bfloat16),      # 1024: four full rounds
    (11, 310, 5, 1, 16, 64, torch.bfloat16),        # 77
    (131, 130, 8, 2, 16, 64, torch.float16),        # 786, an odd number of pairs per round
])
def test_gqa_batches_of_many_items(B, L, H, S, g, w, dtype):
    run, O, lse = _batch(lca.MODE_GQA, B, L, H, S, g, w, dtype)
    for b in range(0, B, max(1, B // 12)):
        O1, lse1 = run(b, 1)
        assert torch.equal(O[b], O1[0]) and torch.equal(lse[b], lse1[0]), b

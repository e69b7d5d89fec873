"""Prefill calls whose work items outnumber the compute units: every item is taken, by whichever workgroup's turn it is.  A sequence's items are
the same whether it is alone or in a batch, so a batch must give the bits of its sequences one by one (those stay within one round)."""
import math

import pytest
import torch

from paper_2604_12452_amd import lca
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def _batch(mode, B, L, H, S, g, w, dtype, up=False, spike=False):
    gen = torch.Generator(device="cuda").manual_seed(100 * L + H)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(dtype)
    mla = mode == lca.MODE_MLA
    d_pool, d_sel = (512, 64) if mla else (128, 128)
    d_qk = d_pool + d_sel if mla else d_sel
    desc = lambda n: lca.Desc(B=n, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, mode=mode, dtype=lca.BF16 if dtype == torch.bfloat16 else lca.F16)
    Q = rnd(B, L, H, d_qk) / math.sqrt(d_qk)
    pool, sel = (rnd(B, L, d_pool), rnd(B, L, d_sel)) if mla else (rnd(B, L, S, d_pool), rnd(B, L, S, d_sel))
    if spike:                                       # one late key and one old one score 60 nats and more above the rest: the item is repeated from exact maxima
        Q[..., :d_pool] += 2.0 * (e := torch.nn.functional.normalize(rnd(d_pool).float(), dim=0)).to(dtype)
        pool[:, L // 10] = pool[:, L * 7 // 10] = (50.0 * e).to(dtype)
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


MANY = [      # (too many items for the form that halves them)
    (40, 100, 16, 1, 16, 48, torch.bfloat16, False), (9, 333, 16, 4, 8, 64, torch.float16, False), (60, 161, 6, 1, 4, 32, torch.bfloat16, False),
    (90, 129, 3, 1, 16, 16, torch.float16, False), (30, 200, 16, 16, 16, 64, torch.bfloat16, True), (33, 97, 16, 2, 3, 0, torch.float16, True),
    (70, 40, 20, 1, 4, 3, torch.bfloat16, False), (600, 5, 2, 1, 1, 2, torch.bfloat16, False), (130, 140, 2, 2, 16, 48, torch.float16, True),
]


@pytest.mark.parametrize("spike", [False, True])
@pytest.mark.parametrize("B,L,H,S,g,w,dtype,up", MANY)
def test_mla_batches_of_many_items(B, L, H, S, g, w, dtype, up, spike):
    """The kernel for many items against the one for few (which the oracle's tests cover at these sizes): both are held to the same tolerance against exact
    values, so they may differ by twice that."""
    run, O, lse = _batch(lca.MODE_MLA, B, L, H, S, g, w, dtype, up, spike)
    name = "bf16" if dtype == torch.bfloat16 else "f16"
    for b in range(0, B, max(1, B // 8)):
        O1, lse1 = run(b, 1)
        x, y = O[b].double(), O1[0].double()
        err = ((x - y).abs().amax(-1) / y.abs().amax(-1).clamp_min(1e-6)).amax().item()
        assert err <= 2 * hp.TOL[name], (b, err)
        assert (lse[b] - lse1[0]).abs().amax().item() <= 1e-3 * max(1.0, lse1.abs().amax().item()), b     # (fp32 sums of 16-bit products in two orders)

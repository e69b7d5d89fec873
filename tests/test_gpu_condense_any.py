"""The any-width condensation kernel (condense_any_kernel): rows held in registers and rows read again, one 16-byte piece per row
to more pieces than lanes, group sizes that are no power of two, every reduce strategy; and the summary query over more
(position, head) pairs than one round of loads and more pieces than one workgroup."""
import pytest

from paper_2604_12452_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,mode,d_pool,d_sel,g,H,S,n_q", [
    ("bf16", inputs.MODE_GQA, 64, 64, 16, 16, 4, 0),        # 8 pieces per row, held
    ("bf16", inputs.MODE_GQA, 64, 64, 8, 8, 4, 0),          # one load holds the group, and the last group size that it does
    ("f16", inputs.MODE_MLA, 64, 56, 9, 8, 2, 0),           # two loads
    ("bf16", inputs.MODE_GQA, 64, 64, 32, 8, 4, 0),         # four loads, and the last size
    ("f32", inputs.MODE_GQA, 32, 32, 33, 8, 4, 0),          # five
    ("bf16", inputs.MODE_MLA, 512, 64, 24, 16, 1, 0),       # 24 rows of 64 pieces: read again
    ("f16", inputs.MODE_MLA, 512, 64, 5, 4, 2, 3),
    ("f32", inputs.MODE_GQA, 520, 32, 16, 4, 2, 0),         # 130 pieces per row: more than lanes
    ("f32", inputs.MODE_MLA, 8, 4, 64, 6, 1, 50),           # one and two pieces per row, the largest group
    ("bf16", inputs.MODE_GQA, 8, 136, 1, 40, 2, 30),        # one-token groups; 600 pairs of 17 pieces in the summary query
    ("f16", inputs.MODE_MLA, 256, 32, 16, 40, 1, 40),       # 1600 pairs: four rounds of loads
])
def test_any_width_condensation(oracle, dtype, mode, d_pool, d_sel, g, H, S, n_q):
    wl = inputs.Workload("any", B=2, L=11 * g + 60, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=17, n_q=n_q, dtype=dtype, mode=mode, seed=800 + g + H)
    print(f"[case] {wl}", flush=True)
    Q, POOL, SEL = inputs.gen_all(wl)
    run = hp.GpuRun(wl, Q, POOL, SEL).condense(alpha=True)
    hp.check_condense(oracle, wl, run, inputs.to_f64(Q[:, wl.L - wl.nq:], wl.dtype), inputs.to_f64(POOL, wl.dtype), inputs.to_f64(SEL, wl.dtype))


@pytest.mark.parametrize("pool_reduce,sel_reduce", [(2, 1), (4, 4), (3, 2), (1, 4)])
@pytest.mark.parametrize("dtype,d_pool,d_sel,g", [("bf16", 512, 64, 16), ("f32", 520, 64, 24), ("f16", 64, 32, 3)])
@pytest.mark.parametrize("mode", [inputs.MODE_MLA, inputs.MODE_GQA])
def test_strategies_at_layer_widths(oracle, mode, dtype, d_pool, d_sel, g, pool_reduce, sel_reduce):
    from paper_2604_12452_amd import lca
    import torch
    wl = inputs.Workload("any_reduce", B=1, L=15 * g, H=4, S=1, d_pool=d_pool, d_sel=d_sel, g=g, w=30, dtype=dtype, mode=mode, seed=900 + g)
    Q, POOL, SEL = inputs.gen_all(wl)
    Qf, POOLf, SELf = (inputs.to_f64(x, dtype) for x in (Q, POOL, SEL))
    od = hp.oracle_desc(oracle, wl, pool_reduce=pool_reduce, sel_reduce=sel_reduce)
    ref = oracle.condense(od, oracle.summary_query(od, Qf[:, wl.L - wl.nq:]), POOLf, SELf)
    d = hp.lca_desc(wl, pool_reduce=pool_reduce, sel_reduce=sel_reduce)
    pool_rep, sel_rep, anchor, _ = lca.alloc_condensed(d)
    lca.condense(d, hp.to_dev(Q, dtype), hp.to_dev(POOL, dtype), hp.to_dev(SEL, dtype), pool_rep, sel_rep, anchor, None, lca.alloc_workspace(d))
    torch.cuda.synchronize()
    clear = ref["margin"] > hp.ANCHOR_MARGIN
    assert (anchor.cpu().numpy()[clear] == ref["anchor"][clear]).all()
    # (norms and scores of rows are far apart on these inputs wherever the margin is clear)
    assert hp.vec_rel_err(hp.from_dev(pool_rep, dtype)[clear], ref["pool_rep"][clear]) <= hp.TOL[dtype]
    assert hp.vec_rel_err(hp.from_dev(sel_rep, dtype)[clear], ref["sel_rep"][clear]) <= hp.TOL[dtype]

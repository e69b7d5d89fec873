"""The kernels for many work items and many groups against the oracle, at sizes where the rules send a call there: short prompts, which most tests are made of, have
forms of their own.  Scales, biases, ties, an empty window, every head layout."""
import math

import numpy as np
import pytest

from paper_2604_12452_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def _inputs(wl, ties):
    Q, POOL, SEL = inputs.gen_all(wl)
    if ties:                                       # the rows of a group alike, in pairs
        POOL[:, 1:wl.L // 2 * 2:2], SEL[:, 1:wl.L // 2 * 2:2] = POOL[:, 0:wl.L // 2 * 2:2], SEL[:, 0:wl.L // 2 * 2:2]
    return (Q, POOL, SEL), tuple(inputs.to_f64(x, wl.dtype) for x in (Q, POOL, SEL))


# B, L, H, S, g, w, dtype, scale, logit bias of the representatives, ties, up-projection
MLA = [
    (40, 100, 16, 1, 16, 48, "bf16", 1.0, 0.0, False, False), (40, 100, 16, 1, 16, 48, "f16", 0.3, 0.0, False, False),
    (9, 333, 16, 4, 8, 0, "f16", 1.0, 0.0, False, False), (60, 161, 6, 1, 4, 32, "bf16", 3.0, 0.0, False, False),
    (90, 129, 3, 1, 16, 16, "f16", 1.0 / math.sqrt(576.0), 0.0, False, False), (30, 200, 16, 16, 16, 64, "bf16", 1.0, math.log(16.0), False, False),
    (70, 40, 20, 1, 4, 3, "bf16", 1.0, 0.0, True, False), (300, 5, 4, 1, 1, 2, "bf16", 1.0, 0.0, False, False),
    (33, 97, 16, 2, 3, 0, "f16", 1.0, 0.0, False, True), (130, 140, 2, 2, 16, 48, "bf16", 1.0, math.log(16.0), False, True),
    (1, 60, 128, 2, 16, 16, "bf16", 1.0, 0.0, False, False), (1, 70, 64, 1, 16, 16, "f16", 1.0, 0.0, False, True),       # many heads: undivided whatever the length
]

# half items that some workgroups take two of (of one, two and four heads), and row blocks without a later half
HALVES = [
    (1, 1300, 16, 16, 32, 1200, "bf16", 1.0, math.log(32.0), False, False), (2, 640, 16, 16, 8, 500, "f16", 1.0, 0.1, False, True),
    (1, 560, 32, 16, 16, 400, "bf16", 3.0, 0.1, False, False), (1, 1250, 16, 1, 16, 512, "f16", 1.0, 0.0, False, False),
    (5, 60, 20, 20, 4, 16, "bf16", 1.0, 0.0, True, False), (3, 64, 19, 19, 16, 3, "f16", 0.3, 0.1, False, True),
]


@pytest.mark.parametrize("B,L,H,S,g,w,dtype,scale,bias,ties,up", MLA + HALVES)
def test_mla_prefill(oracle, B, L, H, S, g, w, dtype, scale, bias, ties, up):
    import torch
    from paper_2604_12452_amd import lca
    wl = inputs.Workload("many", B=B, L=L, H=H, S=S, d_pool=512, d_sel=64, g=g, w=w, dtype=dtype, scale=scale, seed=B + L)
    print(f"[case] {wl}", flush=True)
    arrays, (Qf, POOLf, SELf) = _inputs(wl, ties)
    run = hp.GpuRun(wl, *arrays, rep_logit_bias=bias).condense()
    ref, differ = hp.check_condense(oracle, wl, run, Qf[:, L - wl.nq:], POOLf, SELf)
    rows = np.unique(np.r_[0:L:7, L - 1, w:min(w + 2 * g, L):3]).astype(np.int32)
    if not up:
        run.prefill()
        hp.check_prefill(oracle, wl, run, rows, Qf[:, rows], POOLf, SELf, ref, differ, bias=bias)
        if bias == 0.0:
            run.dense()
            hp.check_dense(oracle, wl, run, rows, Qf[:, rows], POOLf, SELf)
        return
    W = inputs.to_storage(np.random.default_rng(L).standard_normal((H, 128, 512)) / np.sqrt(512.0), dtype)
    O = torch.full((B, L, H, 128), float("nan"), dtype=lca.torch_dtype(run.desc), device="cuda")
    lse = torch.full((B, L, H), float("nan"), dtype=torch.float32, device="cuda")
    lca.prefill_attn_up(run.desc, run.Q, run.POOL, run.SEL, run.pool_rep, run.sel_rep, hp.to_dev(W, dtype), O, lse, run.ws)
    got = hp.from_dev(O[:, rows.tolist()], dtype)
    od = hp.oracle_desc(oracle, wl, rep_logit_bias=bias)
    latent, lse_ref = oracle.lca_attn_rows(od, rows, Qf[:, rows], POOLf, SELf, hp.from_dev(run.pool_rep, dtype), hp.from_dev(run.sel_rep, dtype), want_lse=True)
    assert np.isfinite(got).all()
    assert hp.vec_rel_err(got, oracle.up_project(latent, inputs.to_f64(W, dtype))) <= hp.TOL[dtype]
    assert np.abs(lse[:, rows.tolist()].cpu().numpy() - lse_ref).max() <= hp.LSE_TOL[dtype]


# kernel, dtype, mode, d_pool, d_sel, H, S, g, w, L, B, n_q, scale, ties
GROUPS = [
    ("condense_mfma_kernel", "bf16", inputs.MODE_MLA, 512, 64, 16, 16, 16, 0, 770, 3, 0, 1.0, False), ("condense_mfma_kernel", "f16", inputs.MODE_MLA, 512, 64, 16, 8, 32, 40, 2000, 6, 3, 3.0, False),
    ("condense_mfma_kernel", "bf16", inputs.MODE_MLA, 512, 64, 32, 16, 16, 64, 900, 3, 0, 0.04, True),
    ("condense_any_kernel", "f16", inputs.MODE_GQA, 64, 64, 8, 4, 8, 5, 1620, 4, 0, 1.0, False), ("condense_any_kernel", "bf16", inputs.MODE_GQA, 128, 128, 8, 4, 5, 0, 1100, 4, 9, 3.0, False),
    ("condense_reg_kernel", "f32", inputs.MODE_MLA, 128, 32, 4, 1, 16, 128, 1024, 60, 0, 1.0, False), ("condense_any_kernel", "bf16", inputs.MODE_GQA, 96, 112, 6, 6, 24, 16, 1500, 6, 0, 1.0, True),
    ("condense_any_kernel", "f32", inputs.MODE_MLA, 8, 4, 6, 1, 64, 0, 200, 300, 50, 1.0, False), ("condense_any_kernel", "f16", inputs.MODE_GQA, 32, 64, 8, 8, 1, 3, 500, 1, 0, 0.04, False), ("condense_any_kernel", "bf16", inputs.MODE_MLA, 256, 32, 8, 2, 64, 7, 9000, 8, 0, 1.0, False),
    ("condense_reg_kernel", "bf16", inputs.MODE_GQA, 128, 128, 16, 8, 16, 0, 3300, 2, 0, 1.0, False), ("condense_reg_kernel", "f16", inputs.MODE_GQA, 128, 128, 14, 2, 32, 100, 9000, 4, 0, 3.0, True),
]


@pytest.mark.parametrize("kernel,dtype,mode,d_pool,d_sel,H,S,g,w,L,B,n_q,scale,ties", GROUPS)
def test_condensation(oracle, kernel, dtype, mode, d_pool, d_sel, H, S, g, w, L, B, n_q, scale, ties):
    wl = inputs.Workload("groups", B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, n_q=n_q, dtype=dtype, mode=mode, scale=scale, seed=L + g)
    print(f"[case] {wl}", flush=True)
    arrays, (Qf, POOLf, SELf) = _inputs(wl, ties)
    run = hp.GpuRun(wl, *arrays).condense(alpha=True)
    hp.check_condense(oracle, wl, run, Qf[:, L - wl.nq:], POOLf, SELf)

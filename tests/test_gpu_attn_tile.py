"""The tiled attention kernel (csrc/attn_tile.hip): every instantiation (element type, width class, one or two blocks of
query rows per wavefront) at ragged sizes on every row against the oracle, and entries a row does not see left out of it
even when they are not finite."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2604_12452_amd import inputs
from tests import helpers as hp
from tests.test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,mode,d_pool,d_sel,L,g,w,H,S,B", [
    # widths at the edges of the classes (64, 128, 256, 512 value columns; whole and partial fragment chunks)
    ("bf16", inputs.MODE_GQA, 64, 64, 131, 4, 10, 8, 2, 1),
    ("f16", inputs.MODE_GQA, 72, 64, 67, 16, 5, 3, 3, 2),        # just past a class in the pooled part, one head per set
    ("bf16", inputs.MODE_GQA, 128, 120, 90, 8, 20, 10, 2, 1),    # five heads per set: a block of 16 rows is not whole tokens
    ("f16", inputs.MODE_MLA, 96, 32, 75, 8, 0, 4, 1, 1),         # no window: rows whose last token closes a group see no raw token
    ("bf16", inputs.MODE_MLA, 256, 32, 150, 16, 33, 4, 1, 1),
    ("bf16", inputs.MODE_GQA, 384, 64, 70, 8, 9, 2, 1, 1),
    ("f32", inputs.MODE_GQA, 64, 64, 131, 4, 10, 6, 2, 2),
    ("f32", inputs.MODE_GQA, 100, 60, 67, 16, 5, 3, 3, 1),       # multiples of four, not of sixteen
    ("f32", inputs.MODE_MLA, 256, 32, 90, 8, 20, 4, 1, 1),
    ("f32", inputs.MODE_MLA, 512, 64, 70, 8, 9, 2, 1, 1),
    ("f32", inputs.MODE_MLA, 128, 32, 16, 4, 3, 4, 1, 1),        # fewer tiles than wavefronts
    ("f32", inputs.MODE_GQA, 416, 64, 70, 8, 9, 4, 2, 1),        # key and value rows apart: two wavefronts' areas take 141 KB ...
    ("f32", inputs.MODE_GQA, 512, 64, 130, 4, 60, 2, 1, 2),      # ... of LDS
    ("f16", inputs.MODE_MLA, 256, 32, 150, 16, 33, 4, 1, 1),
    ("f16", inputs.MODE_GQA, 384, 64, 70, 8, 9, 2, 1, 1),
    ("f16", inputs.MODE_GQA, 64, 64, 131, 4, 10, 8, 2, 1),
    # as many rows as two blocks per wavefront take, which only heads up to 64 wide have: with them ...
    ("bf16", inputs.MODE_GQA, 64, 64, 1030, 16, 40, 16, 4, 2),
    ("f16", inputs.MODE_GQA, 64, 64, 1030, 16, 40, 16, 4, 2),
    ("f32", inputs.MODE_GQA, 64, 32, 1025, 8, 17, 16, 4, 2),
    # ... and one block each all the same
    ("f16", inputs.MODE_GQA, 128, 96, 1037, 32, 21, 32, 8, 1),
    ("f32", inputs.MODE_MLA, 128, 32, 2053, 16, 50, 16, 1, 1),
    # no instantiation: the row-by-row kernel
    ("f32", inputs.MODE_GQA, 520, 32, 40, 4, 5, 2, 1, 1),
])
def test_every_instantiation_all_rows(oracle, dtype, mode, d_pool, d_sel, L, g, w, H, S, B):
    wl = inputs.Workload("tile", B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, dtype=dtype, mode=mode, seed=700 + L + d_pool)
    _full_parity(oracle, wl)


# mode, d_pool, d_sel, L, g, w, H, S, B, wavefronts
LATE_CASES = [
    (inputs.MODE_MLA, 256, 64, 19, 4, 64, 3, 1, 1, 2),         # two tiles
    (inputs.MODE_MLA, 256, 64, 31, 8, 13, 4, 1, 2, 2),
    (inputs.MODE_MLA, 192, 128, 301, 16, 40, 2, 2, 1, 4),      # halves of four, one of which sees nothing of the first rows
    (inputs.MODE_MLA, 264, 56, 301, 64, 130, 1, 1, 1, 4),      # a partial last column block
    (inputs.MODE_MLA, 256, 64, 1030, 16, 0, 16, 4, 1, 1),      # as many workgroups as one wavefront each
    (inputs.MODE_GQA, 512, 64, 100, 16, 8, 32, 32, 3, 1),      # wide rows, few tiles, more workgroups than CUs
]


@pytest.mark.parametrize("mode,d_pool,d_sel,L,g,w,H,S,B,waves", LATE_CASES)
def test_the_second_form_of_the_512_column_class(oracle, mode, d_pool, d_sel, L, g, w, H, S, B, waves):
    _full_parity(oracle, inputs.Workload("late", B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, dtype="f32", mode=mode, seed=800 + L + d_pool))


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("dtype,mode,d_pool,d_sel,H,S", [("f32", inputs.MODE_MLA, 128, 32, 4, 1), ("bf16", inputs.MODE_GQA, 64, 64, 4, 2),
                                                         ("f16", inputs.MODE_GQA, 64, 64, 4, 2)])
def test_entries_a_row_does_not_see_never_reach_it(bad, dtype, mode, d_pool, d_sel, H, S):
    """One value of the pooled component of token 37 is not finite (what sits behind a padded prompt, say): rows before it must
    come out as without it, rows from it on show it in that column (nothing is condensed here: w >= L)."""
    import torch
    wl = inputs.Workload("nonfinite", B=1, L=60, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=4, w=64, dtype=dtype, mode=mode, seed=9, n_q=1)
    Q, POOL, SEL = inputs.gen_all(wl)
    clean, run = (hp.GpuRun(wl, Q, POOL, SEL).condense() for _ in range(2))
    run.POOL.view(1, 60, -1, d_pool)[0, 37, :, 3] = bad
    clean.prefill()
    run.prefill()
    a, b = (hp.from_dev(r.O, dtype) for r in (clean, run))
    assert hp.vec_rel_err(b[:, :37], a[:, :37]) <= hp.TOL[dtype]
    assert torch.equal(run.lse[:, :37].isfinite(), torch.ones_like(run.lse[:, :37], dtype=torch.bool))
    assert not np.isfinite(b[0, 37:, :, 3]).any()


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_probabilities_enter_the_second_product_whole(dtype):
    """The 24 bits of a probability: 512 sets of one head, three tokens, two of which have logit 0 and values that cancel the leading
    22 bits of the third's contribution p = exp(x), so that the output is what is left of p.

    Bound on the error of p, relative to 1 (x in (-1/2, 0)): the factor log2(e) and its product with x round once each (2^-25 + 2^-25
    of at most 0.72, times ln 2 p: 2^-25), the exponential by at most one unit (2^-24), the three terms' sum by at most one unit of
    its largest value per addition (3 * 2^-24); together below 2^-21.6.  Largest seen: 2^-24.0 (fp16 in two parts: 2^-21.4)."""
    import torch
    from paper_2604_12452_amd import lca
    n, V = 512, 2.0 ** 14
    rng = np.random.default_rng(3)
    x = -rng.uniform(0.02, 0.5, n).astype(np.float32)
    x = inputs.to_f64(inputs.to_storage(x, dtype), dtype)                # the logit itself: one product of x and 1
    p = np.exp(x)
    parts = []
    for _ in range(2):                                                   # leading parts of p in the storage type
        parts.append(inputs.to_f64(inputs.to_storage((p - sum(parts)).astype(np.float32), dtype), dtype))
    Q, K, Vals = np.zeros((1, 3, n, 64)), np.zeros((1, 3, n, 64)), np.zeros((1, 3, n, 64))
    Q[..., 0] = 1.0
    K[0, 2, :, 0] = x
    Vals[0, 0], Vals[0, 1], Vals[0, 2] = -V * parts[0][:, None], -V * parts[1][:, None], V
    dev = [hp.to_dev(inputs.to_storage(a.astype(np.float32), dtype), dtype) for a in (Q, Vals, K)]
    d = lca.Desc(B=1, L=3, H=n, S=n, d_pool=64, d_sel=64, g=4, w=64, n_q=1, mode=lca.MODE_GQA,
                 dtype={"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}[dtype])
    O = torch.empty(1, 3, n, 64, dtype=lca.torch_dtype(d), device="cuda")
    lse = torch.empty(1, 3, n, dtype=torch.float32, device="cuda")
    lca.dense_attn(d, *dev, O, lse, lca.alloc_workspace(d))
    got = hp.from_dev(O, dtype)[0, 2] * (2.0 + p[:, None]) / V           # p - parts[0] - parts[1]
    err = np.abs(got - (p - parts[0] - parts[1])[:, None]).max()
    print(f"  largest error of p: 2^{np.log2(err):.2f}", flush=True)
    assert err <= 2.0 ** -21.6
    assert np.abs(lse[0, 2].cpu().numpy() - np.log(2.0 + p)).max() <= 4e-7


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("scale", [1.0, -1.0, 0.0])
@pytest.mark.parametrize("L,d_pool,B", [(15, 64, 1), (31, 64, 2), (60, 128, 1), (300, 128, 1), (300, 64, 1), (2100, 64, 40)])
@pytest.mark.parametrize("step", [0.16, 0.18, 1.0])
def test_rising_logits_over_one_to_eight_wavefronts(oracle, dtype, scale, L, d_pool, B, step):
    """Every entry's logit lies `step` above the one before: 7.4 binades per tile of 32 entries, which the reference of the exponentials does
    not follow, 8.3 and 46, which it does.  Up to 15 entries are one tile and wavefront, 300 split over eight in fp32, and 40 sequences of 2100
    take two.  Tolerance: the stated bar (the largest logit is 2100, whose last fp32 bit is 1.2e-4: rows from 1000 on are left to the test below)."""
    wl = inputs.Workload("rising", B=B, L=L, H=1, S=1, d_pool=d_pool, d_sel=64, g=4, w=4096, dtype=dtype, mode=inputs.MODE_GQA, seed=5, n_q=1, scale=scale)
    print(f"[case] {wl} step {step}", flush=True)
    rng = np.random.default_rng(L)
    Qf, Kf = np.zeros((B, L, 1, 64)), np.zeros((B, L, 1, 64))
    Qf[..., 0] = 1.0
    Kf[..., 0] = (step * np.arange(L) * (-1.0 if scale < 0 else 1.0))[None, :, None]
    arrays = [inputs.to_storage(a.astype(np.float32), dtype) for a in (Qf, rng.standard_normal((B, L, 1, d_pool)), Kf)]
    run = hp.GpuRun(wl, *arrays)
    run.dense()
    rows = np.unique(np.concatenate([np.arange(0, min(L, 1000), max(1, L // 60)), [min(L, 1000) - 1]])).astype(np.int32)
    wide = [inputs.to_f64(a[:1], dtype) for a in arrays]
    ref, _ = oracle.dense_attn_rows(hp.oracle_desc(oracle, replace(wl, B=1)), rows, wide[0][:, rows], wide[1], wide[2], want_lse=True)
    got = hp.from_dev(run.O_dense, dtype)
    assert hp.vec_rel_err(got[:1, rows], ref) <= hp.TOL[dtype]
    assert np.isfinite(got).all()


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("scale", [1.0, -1.0])
@pytest.mark.parametrize("step", [0.16, 0.18, 1.0])
def test_rising_logits_in_long_rows_of_the_last_sequence(oracle, dtype, scale, step):
    """The same in the rows with the most tiles, first and last sequence, and their lse.  A logit of up to 2100 is good to 2^-13 (its fp32 product with the
    scale and log2 e), which is what a probability and lse lose besides the type's bar; at steps below one 16-bit storage rounds the keys
    themselves, the same for the oracle."""
    B, L = 40, 2100
    wl = inputs.Workload("rising", B=B, L=L, H=1, S=1, d_pool=64, d_sel=64, g=4, w=4096, dtype=dtype, mode=inputs.MODE_GQA, seed=5, n_q=1, scale=scale)
    print(f"[case] {wl} step {step}", flush=True)
    rng = np.random.default_rng(L)
    Qf, Kf = np.zeros((B, L, 1, 64)), np.zeros((B, L, 1, 64))
    Qf[..., 0] = 1.0
    Kf[..., 0] = (step * np.arange(L) * (-1.0 if scale < 0 else 1.0))[None, :, None]
    arrays = [inputs.to_storage(a.astype(np.float32), dtype) for a in (Qf, rng.standard_normal((B, L, 1, 64)), Kf)]
    run = hp.GpuRun(wl, *arrays)
    run.dense()
    rows = np.unique(np.concatenate([np.arange(7, L, 97), np.arange(L - 3, L)])).astype(np.int32)
    got, lse = hp.from_dev(run.O_dense, dtype), run.lse_dense.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all() and np.isfinite(lse).all()
    for b in (0, B - 1):
        wide = [inputs.to_f64(a[b:b + 1], dtype) for a in arrays]
        ref, ref_lse = oracle.dense_attn_rows(hp.oracle_desc(oracle, replace(wl, B=1)), rows, wide[0][:, rows], wide[1], wide[2], want_lse=True)
        assert hp.vec_rel_err(got[b:b + 1, rows], ref) <= hp.TOL[dtype] + 2.0 ** -12
        assert np.abs(lse[b:b + 1, rows] - ref_lse).max() <= 2.0 ** -12


def _peaked(dtype, a, scale, L=60, at=(20, 45), seed=4):
    """(run, values, lse) of plain attention where every query is `a` in all 64 columns and so are the keys of the tokens `at`, with the scale's sign;
    the other keys are zero."""
    from paper_2604_12452_amd import lca
    import torch
    rng = np.random.default_rng(seed)
    Q, K = np.full((1, L, 2, 64), a), np.zeros((1, L, 1, 64))
    K[0, list(at)] = -a if scale < 0 else a
    V = inputs.to_f64(inputs.to_storage(rng.standard_normal((1, L, 1, 64)).astype(np.float32), dtype), dtype)
    d = lca.Desc(B=1, L=L, H=2, S=1, d_pool=64, d_sel=64, g=4, w=2 * L, n_q=1, mode=lca.MODE_GQA, scale=scale,
                 dtype={"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}[dtype])
    dev = [hp.to_dev(inputs.to_storage(x.astype(np.float32), dtype), dtype) for x in (Q, V, K)]
    O = torch.empty(1, L, 2, 64, dtype=lca.torch_dtype(d), device="cuda")
    lse = torch.empty(1, L, 2, dtype=torch.float32, device="cuda")
    lca.dense_attn(d, *dev, O, lse, lca.alloc_workspace(d))
    return hp.from_dev(O, dtype)[0], V[0, :, 0], lse[0].cpu().numpy().astype(np.float64)


def _check_peaked(dtype, logit, got, V, lse, at, lse_tol):
    """Rows against the weighted mean of the values they see: exp(logit) for the tokens `at`, one for the others."""
    for t in range(len(V)):
        z = np.array([logit if i in at else 0.0 for i in range(t + 1)])
        p = np.exp(z - z.max())
        ref = (p / p.sum()) @ V[:t + 1]
        assert hp.vec_rel_err(got[t], np.broadcast_to(ref, got[t].shape)) <= hp.TOL[dtype], t
        want = z.max() + np.log(p.sum())
        assert np.abs(lse[t] - want).max() <= lse_tol * max(1.0, abs(want)), (t, lse[t], want)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("scale", [1.0, -0.25])
@pytest.mark.parametrize("logit", [2.0e3, 4.0e6, 4.67e7, 1.5e9, 6.0e10])
def test_two_keys_with_very_large_logits(dtype, scale, logit):
    """Where a unit in the last place of a logit is several binades of its exponential: from 2^26 in base 2 on, the fp16 parts of a probability that is
    not taken from the logit as it was rounded hold less than its whole (4.67e7 is 2^26 log 2; at 6e10 the unit is 2^13).  The two keys' logits
    are equal, so the rows are means of values.
    lse: 64 additions of products, the factor and its product round once each, 66 times 2^-24."""
    a = inputs.to_f64(inputs.to_storage(np.array([np.sqrt(logit / (64 * abs(scale)))], dtype=np.float32), dtype), dtype)[0]
    print(f"[case] {dtype} scale {scale} logit {logit}", flush=True)
    got, V, lse = _peaked(dtype, a, scale)
    _check_peaked(dtype, 64 * a * a * abs(scale), got, V, lse, (20, 45), 66 * 2.0 ** -24)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("scale,a", [(0.0, 1.0e18), (-0.0, 1.0e18), (0.0, 1.0), (2.0e-39, 1.0e18), (-2.0e-39, 1.0e18), (3.0e-38, 2.0e17), (1.0e-37, 1.5e18)])
def test_products_up_to_the_largest_number_and_a_scale_of_nothing(dtype, scale, a):
    """A scale of zero makes every entry count alike whatever the products are (64 a a = 6.4e37), and one below the least normal number is used as it is."""
    a = inputs.to_f64(inputs.to_storage(np.array([a], dtype=np.float32), dtype), dtype)[0]
    print(f"[case] {dtype} scale {scale} a {a}", flush=True)
    got, V, lse = _peaked(dtype, a, scale)
    _check_peaked(dtype, 64 * a * a * abs(float(np.float32(scale))), got, V, lse, (20, 45), 1e-5)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_scale_zero_leaves_what_is_no_number(sign):
    """A scale of zero times an infinity is no number: rows whose query, or one of whose keys, is not finite are none."""
    import torch
    from paper_2604_12452_amd import lca
    d = lca.Desc(B=1, L=40, H=2, S=1, d_pool=64, d_sel=64, g=4, w=64, n_q=1, mode=lca.MODE_GQA, scale=0.0, dtype=lca.F32)
    Q, K, V = torch.ones(1, 40, 2, 64, device="cuda"), torch.ones(1, 40, 1, 64, device="cuda"), torch.randn(1, 40, 1, 64, device="cuda")
    Q[0, 5, 0, 3], Q[0, 6, 1, 9], K[0, 20, 0, 7] = float("inf"), -float("inf"), sign * float("inf")
    O = torch.empty(1, 40, 2, 64, device="cuda")
    lca.dense_attn(d, Q, V, K, O, None, lca.alloc_workspace(d))
    bad = ~O.isfinite().all(-1)[0]
    want = torch.zeros(40, 2, dtype=torch.bool, device="cuda")
    want[5, 0] = want[6, 1] = True
    want[20:] = True
    assert torch.equal(bad, want)
    mean = V[0, :, 0].cumsum(0) / torch.arange(1, 41, device="cuda")[:, None]
    assert (O[0, 7:20] - mean[7:20, None]).abs().max() <= 1e-5

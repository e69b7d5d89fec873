"""The online cache update by group size and row width: one row to eight rows per wavefront, groups that the wavefronts do not divide,
rows that take one, two or more 16-byte pieces per lane, with the summary query computed inside the kernel and before it."""
import numpy as np
import pytest

from paper_2604_12452_amd import inputs
from tests import helpers as hp
from tests.test_gpu_cache_update import Cache, _storage, _update_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,d_pool,d_sel,H,S,dtype", [
    (inputs.MODE_GQA, 128, 128, 14, 2, "f16"),       # one piece per lane, summary inside
    (inputs.MODE_GQA, 520, 64, 6, 3, "bf16"),        # 73 pieces: two per lane
    (inputs.MODE_MLA, 512, 64, 5, 1, "bf16"),        # summary in a kernel of its own
    (inputs.MODE_MLA, 128, 32, 4, 2, "f32"),
    (inputs.MODE_GQA, 256, 256, 4, 2, "f32"),        # 128 pieces, the most two per lane hold
    (inputs.MODE_GQA, 1024, 8, 4, 2, "bf16"),        # 129 pieces: one wavefront, rows read again
])
@pytest.mark.parametrize("g", [1, 7, 16, 17, 64])
def test_cache_update_rows(oracle, mode, d_pool, d_sel, H, S, dtype, g):
    B, w, m_before = 2, 9, 3
    k_cap = w + g + 2
    k_start = (k_cap - g // 2) % k_cap                         # the ring wraps inside the group
    wl = inputs.Workload("update_rows", B=B, L=w + (m_before + 1) * g, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, dtype=dtype, mode=mode,
                         seed=0, scale=1.0 / np.sqrt(d_pool + d_sel if mode == inputs.MODE_MLA else d_sel))
    print(f"[case] {wl}", flush=True)
    rng = np.random.default_rng(77 + g)
    cache = Cache(wl, m_cap=m_before + 2, k_cap=k_cap, k_start=k_start, rng=rng)
    cache.push(w + g)
    q_recent = _storage(rng, (B, g, H, wl.d_qk), dtype, sigma=2.0)
    _update_and_check(oracle, cache, wl.L, q_recent, m_before)


@pytest.mark.parametrize("mode,d_pool,d_sel,H,S,dtype", [
    (inputs.MODE_GQA, 128, 128, 14, 2, "f16"), (inputs.MODE_MLA, 512, 64, 5, 1, "bf16"), (inputs.MODE_GQA, 1024, 8, 4, 2, "bf16"),
])
@pytest.mark.parametrize("g,bad", [(7, [0]), (16, [1, 3]), (33, [32]), (16, list(range(16)))])
def test_rows_whose_score_is_not_a_number_are_no_anchor(mode, d_pool, d_sel, H, S, dtype, g, bad):
    """The anchor is the best of the rows whose score is a number (the first row if none is); the pooled row is not a number then."""
    import torch
    from paper_2604_12452_amd import lca
    wl = inputs.Workload("nan", B=2, L=5 + g, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=5, dtype=dtype, mode=mode, seed=0)
    rng = np.random.default_rng(5 + g)
    cache = Cache(wl, m_cap=1, k_cap=g + 6, k_start=4, rng=rng)
    cache.push(5 + g)
    for i in bad:
        cache.sel_tail[:, :, (4 + i) % cache.k_cap, 1] = float("nan")
    q = _storage(rng, (2, g, H, wl.d_qk), dtype)
    d = hp.lca_desc(wl)
    lca.cache_update(d, cache.layout(), hp.to_dev(q, dtype), cache.pool_tail, cache.sel_tail, cache.pool_rep, cache.sel_rep, cache.anchor,
                     lca.alloc_workspace(d))
    torch.cuda.synchronize()
    pool, sel = cache.tail_rows(0, g)
    qbar = inputs.to_f64(q, dtype).reshape(2, g, S, H // S, -1).mean((1, 3))
    for b in range(2):
        for s in range(S):
            p = s if mode == inputs.MODE_GQA else 0
            key = sel[b, p] if mode == inputs.MODE_GQA else np.concatenate([pool[b, p], sel[b, p]], -1)
            score = key @ qbar[b, s]
            want = int(np.nanargmax(score)) if len(bad) < g else 0
            assert int(cache.anchor[b, s, 0]) == want
            np.testing.assert_array_equal(hp.from_dev(cache.sel_rep, dtype)[b, s, 0], sel[b, p, want])
            assert np.isnan(hp.from_dev(cache.pool_rep, dtype)[b, s, 0]).all()

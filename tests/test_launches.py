"""Which kernel a call takes, at the sizes where a rule changes its mind (seen on the CPU, launches.py)."""
import pytest

from paper_2604_12452_amd import lca
from tests import launches as t


def _mla(**kw):
    return lca.Desc(**{**dict(B=1, L=8192, H=16, S=1, d_pool=512, d_sel=64, g=16, w=1024), **kw})


def _gqa(**kw):
    return lca.Desc(**{**dict(B=1, L=8192, H=32, S=8, d_pool=128, d_sel=128, g=16, w=1024, mode=lca.MODE_GQA), **kw})


@pytest.mark.parametrize("desc,wide", [
    (_mla(), True), (_gqa(), True), (_gqa(d_pool=512, d_sel=512), True), (_gqa(d_pool=256, d_sel=256, dtype=lca.F32), True),
    (_gqa(d_pool=1024, d_sel=8), False), (_mla(dtype=lca.F32), False), (_gqa(d_pool=260, d_sel=256, dtype=lca.F32), False),
    (_gqa(d_pool=1024, d_sel=1024, dtype=lca.F32, g=64, L=1024 + 64), False),
])
def test_cache_update_by_row_width(desc, wide):
    """Rows of up to 128 16-byte pieces: eight wavefronts per group; wider ones: four that split rows and columns."""
    last = t.cache_update(desc)[-1]
    assert (last.kernel.split("<")[0], last.block) == (("cache_update_wide_kernel", 512) if wide else ("cache_update_rows_kernel", 256))
    assert last.grid == desc.B * desc.S


@pytest.mark.parametrize("desc,tiles,wgs", [
    (_mla(L=1), 1, 1), (_mla(L=256), 16, 1), (_mla(L=257), 17, 5), (_mla(L=70, B=81), 5, 1), (_mla(L=237, w=128, B=63), 10, 1), (_mla(L=1024), 64, 16),
    (_gqa(L=512), 16, 1), (_gqa(L=513), 17, 5), (_gqa(L=155, w=128, B=4, H=8), 6, 1), (_gqa(L=300, B=40), 10, 1), (_gqa(L=1600, w=2000, B=40), 50, 1),
])
@pytest.mark.parametrize("q8", [False, True])
def test_decode_step_by_cache_length(desc, tiles, wgs, q8):
    """Up to 16 tiles (16 entries each at 512 + 64, 32 at 128 / 128) one workgroup per (sequence, set) takes them all and there is nothing to
    merge; so it is where the pairs alone fill the chip."""
    bn = 16 if desc.mode == lca.MODE_MLA else 32
    assert -(-desc.m // bn) + -(-desc.k // bn) == tiles
    run = t.decode(desc, q8)
    assert run[0].grid == desc.B * desc.S * wgs
    assert len(run) == (1 if wgs == 1 else 2)


def _odd(**kw):
    return lca.Desc(**{**dict(B=1, L=500, H=8, S=1, d_pool=256, d_sel=32, g=16, w=128), **kw})


@pytest.mark.parametrize("desc,waves", [
    (_odd(), 4), (_odd(L=1500), 2), (_odd(d_pool=64, L=20), 1), (_odd(d_pool=64, L=40), 2), (_odd(d_pool=128, d_sel=64, L=90), 4),
    (_odd(d_pool=512, d_sel=64, H=2, dtype=lca.F32), 4), (_odd(d_pool=512, d_sel=64, H=16, dtype=lca.F32), 2),
    (_odd(d_pool=512, d_sel=64, H=32, L=4000, dtype=lca.F32), 1), (_odd(dtype=lca.F32, H=4, L=100), 4), (_odd(dtype=lca.F32, H=16), 2),
    (_odd(d_pool=416, d_sel=64, S=2, L=90, mode=lca.MODE_GQA, dtype=lca.F32), 2), (_odd(d_pool=512, d_sel=64, S=8, L=900, mode=lca.MODE_GQA, dtype=lca.F32), 1),
])
def test_tiled_attention_wavefronts(desc, waves):
    """As many as LDS and the registers leave room for at this grid, no more than there are tiles; never more LDS than a CU has."""
    (run,) = t.prefill(desc)
    assert run.kernel.startswith("attn_tile_kernel")
    assert run.block == 64 * waves and run.lds <= 160 * 1024


@pytest.mark.parametrize("kw,most", [
    (dict(d_pool=512, d_sel=64, dtype=lca.F32), 18), (dict(d_pool=512, d_sel=64, dtype=lca.F32, mode=lca.MODE_GQA), 40),
    (dict(d_pool=256, d_sel=32, dtype=lca.F32), 8), (dict(d_pool=128, d_sel=32, dtype=lca.F32), 4), (dict(d_pool=64, d_sel=64, dtype=lca.F32, mode=lca.MODE_GQA), 3),
    (dict(d_pool=512, d_sel=64, mode=lca.MODE_GQA), 7), (dict(d_pool=128, d_sel=64, mode=lca.MODE_GQA, dtype=lca.F16), 2),
])
def test_rows_that_see_few_entries_are_taken_one_by_one(kw, most):
    for L, w, g in ((most, 100, 4), (10 * most, most - 2, 64), (most + 4, most - 2, 2)):         # the longest row sees `most` entries, or more
        run = t.prefill(_odd(H=1, L=L, w=w, g=g, **kw))
        seen = max((max(0, i + 1 - w) // g) + i + 1 - max(0, i + 1 - w) // g * g for i in range(L))
        assert (run[0].kernel.split("<")[0] == "attn_simple_kernel") == (min(L, max(0, L - w) // g + w + g - 1) <= most), (L, w, g, seen)
        assert seen <= most or run[0].kernel.startswith("attn_tile_kernel")
    assert t.prefill(_odd(H=1, L=most + 1, w=100, **kw))[0].kernel.startswith("attn_tile_kernel")
    assert t.prefill(_odd(L=most + 1, **kw), dense=True)[0].kernel.startswith("attn_tile_kernel")
    many = 8192 // most + 1
    assert t.prefill(_odd(H=many, L=most, w=100, **kw))[0].kernel.startswith("attn_tile_kernel")      # more rows than wavefronts on the chip


@pytest.mark.parametrize("kw,held", [
    (dict(d_pool=64, d_sel=64, g=8, mode=lca.MODE_GQA), "1, 1"), (dict(d_pool=64, d_sel=56, g=9), "4, 4"), (dict(d_pool=64, d_sel=64, g=32, mode=lca.MODE_GQA), "4, 4"),
    (dict(d_pool=32, d_sel=32, g=33, dtype=lca.F32), "16, 4"), (dict(d_pool=512, d_sel=64, g=1, pool_reduce=lca.REDUCE_MEAN), "1, 1"),
    (dict(d_pool=512, d_sel=64, g=24), "16, 4"), (dict(d_pool=8, d_sel=8, g=64), "1, 1"),
    (dict(d_pool=1024, d_sel=1024, g=1, mode=lca.MODE_GQA, dtype=lca.F32), "1, 1"),      # (more pieces than lanes: nothing is held)
])
def test_any_width_condensation_by_rows_held(kw, held):
    """The form of the any-width kernel whose registers hold the group's rows, and no more (of a batch with too many groups for one launch)."""
    run = t.condense(_odd(L=1000, B=400, **kw))
    assert run[1].kernel.startswith("condense_any_kernel") and run[1].kernel.endswith(held + ">")


@pytest.mark.parametrize("desc,waves", [
    (_mla(), 16), (_mla(n_q=1), 4), (_mla(n_q=2, H=17), 16), (_mla(H=1), 4), (_mla(B=102), 16), (_mla(B=103), 4), (_gqa(B=33, H=64, n_q=3), 16),
    (_gqa(n_q=4), 4), (_gqa(n_q=5), 16),
])
def test_summary_query_wavefronts(desc, waves):
    """Four wavefronts where there are at most 16 rows (queries x heads of a set) or 512 workgroups, else sixteen."""
    assert t.condense(desc)[0].block == 64 * waves


@pytest.mark.parametrize("desc,heads", [
    (_mla(H=128, L=143, B=4), 1), (_mla(H=128, L=511, B=4, w=512), 1), (_mla(H=128, L=944, B=2, w=128, g=8), 1), (_mla(H=128, L=512), 4),
    (_mla(H=128, L=513), 4), (_mla(H=128, L=581, w=128), 1), (_mla(H=128, L=60000), 4), (_mla(H=64, L=206, B=4), 4), (_mla(H=32, L=100), 4),
    (_mla(H=132, S=2, L=300, B=3), 1), (_mla(H=132, S=2, L=300), 2),
])
def test_up_projection_items(desc, heads):
    """Heads of a work item, which has 128 / heads rows: one where the matrices of more than 64 heads weigh more than the few tiles of many
    items."""
    for run, h in ((t.mla_items(desc, up=True), heads), (t.mla_items(desc), 4 if desc.H // desc.S % 4 == 0 else 2 if desc.H // desc.S % 2 == 0 else 1)):
        assert (run[0], 1 << run[2]) == (-(-desc.L * h // 128), h)


@pytest.mark.parametrize("desc,run", [
    (_mla(L=281), 0), (_mla(L=2048), 0), (_mla(L=2049), 3), (_mla(L=300, H=128), 0), (_mla(L=640, H=64), 1), (_mla(L=1100, H=64), 2), (_mla(L=2100, H=64), 3),
    (_mla(L=8192), 3), (_mla(L=131072), 3), (_mla(L=2048, S=16), 0), (_mla(L=2049, S=16), 1), (_mla(L=800, H=12, S=2, B=3), 0), (_mla(L=1000, H=12, S=2, B=3), 2),
])
def test_mla_query_blocks_of_an_xcd(desc, run):
    """256 rows at a time, fewer while that leaves an XCD without work, one block while there is a CU for every item."""
    assert t.mla_items(desc)[1] == run


def test_decode_split_cases_are_where_they_claim_to_be():
    from tests.test_gpu_decode_splits import CASES
    for dtype, mode, B, L, H, S, g, w, wgs in CASES:
        d_pool, d_sel = (512, 64) if mode == lca.MODE_MLA else (128, 128)
        run = t.decode(lca.Desc(B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, mode=mode, dtype={"bf16": lca.BF16, "f16": lca.F16}[dtype]))
        assert run[0].grid == B * S * wgs, (dtype, mode, B, L, wgs, run)
        merge = "" if wgs == 1 else "decode_merge_kernel" if wgs > 64 else "decode_merge_few_kernel"
        assert [k.kernel.split("<")[0] for k in run[1:]] == ([merge] if merge else [])


@pytest.mark.parametrize("H,S", [(1, 1), (7, 1), (8, 1), (16, 1), (14, 2), (32, 4)])
@pytest.mark.parametrize("B", [1, 2, 4, 11, 60])
def test_decode_results_fit_in_the_workspace(H, S, B):
    """One partial result per workgroup, for any length: around every change of the number of workgroups."""
    for L in [*range(16, 5000, 61), 3072, 3073, 4096, 20000, 131072]:
        d = _mla(B=B, L=L, H=H, S=S, w=1 << 20)
        run = t.decode(d)
        if len(run) > 1:
            assert run[0].grid * (H // S) * (512 + 2) * 4 <= lca.workspace_size(d), (L, run)


def test_tiled_attention_cases_cover_every_instantiation():
    from tests import test_gpu_attn_tile as cases
    (mark,) = [m for m in cases.test_every_instantiation_all_rows.pytestmark if m.name == "parametrize"]
    seen = set()
    for dtype, mode, d_pool, d_sel, L, g, w, H, S, B in mark.args[1]:
        d = lca.Desc(B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, mode=mode, dtype={"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}[dtype])
        seen |= {t.prefill(d)[0].kernel, t.prefill(d, dense=True)[0].kernel}
    built = {"unsigned short": 5, "f16_t": 5, "float": 5}
    for T, n in built.items():
        assert len([k for k in seen if k.startswith(f"attn_tile_kernel<{T},")]) == n, (T, sorted(seen))


@pytest.mark.parametrize("B,L,H,S,g,w,dtype,waves", [
    (2, 1086, 16, 1, 1, 512, lca.F32, 4), (1, 2230, 16, 1, 1, 256, lca.F32, 4), (1, 2500, 16, 1, 1, 256, lca.F32, 4), (1, 2600, 16, 1, 1, 256, lca.F32, 2),
    (2, 1086, 16, 1, 16, 512, lca.F32, 2), (1, 2500, 16, 4, 16, 512, lca.BF16, 2),
])
def test_wavefronts_of_two_row_blocks(B, L, H, S, g, w, dtype, waves):
    """Half of them from four workgroups per CU on, from five where a workgroup has more than 64 tiles."""
    (run,) = t.prefill(lca.Desc(B=B, L=L, H=H, S=S, d_pool=64, d_sel=64, g=g, w=w, mode=lca.MODE_GQA, dtype=dtype))
    assert "4, 2, 2, 2, 1" in run.kernel or "4, 4, 2, 1, 2" in run.kernel, run
    assert run.block == 64 * waves, run


def test_second_form_cases_are_where_they_claim_to_be():
    from tests import test_gpu_attn_tile as cases
    for mode, d_pool, d_sel, L, g, w, H, S, B, waves in cases.LATE_CASES:
        (run,) = t.prefill(lca.Desc(B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, mode=mode, dtype=lca.F32))
        assert run.kernel.startswith("attn_tile_kernel<float, 32, 36, 1, 1, 9, true>") and run.block == 64 * waves, (run, L, waves)
    for d in (lca.Desc(B=1, L=70, H=2, S=1, d_pool=512, d_sel=64, g=8, w=9, dtype=lca.F32), lca.Desc(B=1, L=600, H=32, S=32, d_pool=512, d_sel=64, g=8, w=9, mode=lca.MODE_GQA, dtype=lca.F32)):
        assert t.prefill(d)[0].kernel.startswith("attn_tile_kernel<float, 32, 36, 1, 1, 9, false>")


@pytest.mark.parametrize("desc,shared", [
    (_mla(L=256), True), (_mla(L=1024), True), (_mla(L=4001), True), (_mla(L=131072), True), (_mla(L=1500, B=20), False), (_mla(L=131072, B=32), False),
    (_mla(L=150, B=60), True), (_mla(L=1500, B=300), False),
])
@pytest.mark.parametrize("q8", [False, True])
def test_mla_decode_step_tiles_shared_by_the_wavefronts(desc, shared, q8):
    """Up to two tiles per wavefront, four in a workgroup with a sequence of its own: fewer pass the barriers than the merge costs."""
    run = t.decode(desc, q8)
    name = run[0].kernel                                       # (the last template argument; the demangler gives up on some of these names)
    assert (name.endswith(", true>") or "Lb1EEEv" in name, name.endswith(", false>") or "Lb0EEEv" in name) == (shared, not shared), name


def test_q8_steps_are_where_they_claim_to_be():
    from tests.test_gpu_decode_splits import Q8_STEPS
    for B, L, H, g, w, steps in Q8_STEPS:
        d = _mla(B=B, L=L, H=H, g=g, w=w)
        run = t.decode(d, True)
        tiles = -(-d.m // 16) + -(-d.k // 16)
        assert -(-tiles // (4 * run[0].grid // B)) == steps, (L, tiles, run)


@pytest.mark.parametrize("desc,halves", [
    (_mla(L=1), True), (_mla(L=1024), True), (_mla(L=1025), True), (_mla(L=1600), True), (_mla(L=1900), False), (_mla(L=2048), False), (_mla(L=3000), False),
    (_mla(L=8192), False), (_mla(H=8, L=2048), True), (_mla(H=8, L=3000), False), (_mla(H=1, L=16384), True), (_mla(H=1, L=32768), True), (_mla(H=2, L=12000), False),
    (_mla(B=2, L=1000), True), (_mla(B=3, L=1000), False), (_mla(B=16, L=64), True), (_mla(B=17, L=64), False), (_mla(B=3, L=400), True), (_mla(B=64, L=64), False),
    (_mla(S=16, L=1024), True), (_mla(S=16, L=4096), False), (_mla(H=3, L=5000), True),
])
@pytest.mark.parametrize("up", [False, True])
def test_mla_items_halved_while_they_are_few(desc, halves, up):
    """Two workgroups' worth of every item while each finds a CU of its own, or a second round that is short."""
    run = t.prefill(desc, up=up)[-1]
    assert run.kernel.startswith("attn_mla_kernel_halves" if halves else "attn_mla_kernel<"), run
    n_qb, run_log2, hw = t.mla_items(desc, up=up)
    deal = 8 << run_log2                             # (the query blocks are dealt out to the XCDs in whole rounds)
    items = -(-n_qb * desc.B // deal) * deal * (desc.H >> hw) * (2 if halves else 1)
    assert run.grid == min(256, items) and run.block == 256


@pytest.mark.parametrize("desc,halves", [
    (_mla(H=64, L=1), True), (_mla(H=64, L=256), True), (_mla(H=64, L=257), False), (_mla(H=64, B=8, L=32), True), (_mla(H=64, B=9, L=32), False), (_mla(H=128, L=1), False),
    (_mla(H=32, L=512), True), (_mla(H=32, L=900), True), (_mla(H=32, L=900, w=64), False), (_mla(H=6, S=2, B=2, L=1024), True), (_mla(H=6, S=2, B=2, L=1188, w=64, g=32), False), (_mla(H=66, L=50), False),
    (_mla(S=16, L=1877, w=2048), True), (_mla(S=16, L=1700), False), (_mla(H=32, S=16, L=1024), True), (_mla(H=32, S=16, L=1024, w=64), False), (_mla(H=40, L=378), False), (_mla(H=40, B=3, L=75), False),
    (_mla(H=20, S=20, L=64), True), (_mla(H=20, S=20, L=65), False), (_mla(H=33, S=33, L=64), False), (_mla(H=12, S=12, B=2, L=1003, w=4096), True),
])
@pytest.mark.parametrize("up", [False, True])
def test_mla_items_halved_while_an_xcd_has_cus_for_them(desc, halves, up):
    """The heads of a row block are one XCD's, which has 32 CUs for them, or whose second round is short; with the up-projection no more than 63 heads."""
    run = t.prefill(desc, up=up)[-1]
    assert run.kernel.startswith("attn_mla_kernel_halves" if halves and not (up and desc.H >= 64) else "attn_mla_kernel<"), run


def test_mla_batches_are_where_they_claim_to_be():
    from tests.test_gpu_item_rounds import MANY
    for B, L, H, S, g, w, _, up in MANY:
        for n, name in ((B, "attn_mla_kernel<"), (1, "attn_mla_kernel_halves")):
            assert t.prefill(_mla(B=n, L=L, H=H, S=S, g=g, w=w), up=up)[-1].kernel.startswith(name), (B, L, n)


@pytest.mark.parametrize("desc,one", [
    (_gqa(L=1040), True), (_gqa(L=7168), True), (_gqa(L=7200), False), (_gqa(L=8192, H=28, S=4), True), (_gqa(H=28, S=4, g=32, L=17000), True),
    (_gqa(H=28, S=4, g=32, L=18000), False), (_gqa(B=3, L=2000, H=16, S=4), True), (_gqa(L=2000, H=128, S=4), False), (_mla(L=1500), False), (_mla(L=1500, H=2), False),
    (_mla(L=3000, S=16), True), (_mla(L=3100, S=16), False), (_mla(L=2000, H=4, S=4, g=32), True), (_odd(), True), (_odd(g=32), False), (_odd(dtype=lca.F32, d_pool=128, H=8), True),
    (_odd(dtype=lca.F32, d_pool=128, H=9), False), (_odd(d_pool=64, d_sel=64, H=16, S=4, mode=lca.MODE_GQA), True), (_odd(d_pool=64, d_sel=64, S=2, mode=lca.MODE_GQA), True),
    (_odd(d_pool=64, d_sel=64, S=2, g=8, mode=lca.MODE_GQA), True), (_odd(d_pool=64, d_sel=64, S=2, g=7, mode=lca.MODE_GQA), False), (_odd(d_pool=64, d_sel=64, S=4, g=7, mode=lca.MODE_GQA), True),
    (_gqa(H=8, S=1, g=4, w=0, L=8192), True), (_gqa(H=8, S=1, g=4, w=0, L=8196), False), (_gqa(H=8, S=1, g=5, w=0, L=10240), True),
    (_gqa(H=5, S=1, g=4, w=0, L=800), False), (_gqa(H=6, S=1, g=4, w=0, L=800), True), (_gqa(H=6, S=2, g=4, w=0, L=800, n_q=8), True), (_gqa(H=5, S=1, g=4, w=0, L=800, sel_reduce=1), True),
    (_gqa(H=4, S=1, g=5, w=0, L=800), True), (_odd(d_pool=128, H=5, g=4, dtype=lca.F32), False), (_odd(d_pool=128, H=6, g=4, dtype=lca.F32), True), (_gqa(H=1, S=1, w=0, L=800), True), (_gqa(H=1, S=1, g=8, w=0, L=800), True),
    (_odd(d_pool=128, H=4, S=2, g=4, dtype=lca.F32), True), (_odd(H=2, g=4), True), (_odd(d_pool=128, H=16, S=8, g=1, L=390, dtype=lca.F32), True),
    (_odd(d_pool=128, H=16, S=8, g=1, L=513, dtype=lca.F32), False), (_odd(d_pool=128, H=4, S=2, g=1, L=1178, dtype=lca.F32), False),
    (_odd(d_pool=64, d_sel=64, S=2, B=2, mode=lca.MODE_GQA), True), (_odd(L=8192, g=64, d_pool=512, d_sel=64, S=4), False), (_odd(d_pool=1024, d_sel=8, S=8, mode=lca.MODE_GQA), False),
])
def test_condensation_in_one_launch(desc, one):
    """Few groups whose queries every workgroup can read for itself."""
    run = t.condense(desc)
    assert [k.kernel.split("<")[0] for k in run][:1] == (["condense_one_kernel"] if one else ["summary_query_kernel"]) and len(run) == (1 if one else 2), run
    if one:
        assert run[0].grid == -(-desc.m // 8) * desc.S * desc.B and run[0].block == 512


def test_one_launch_condensations_are_where_they_claim_to_be():
    from tests.test_gpu_condense_one import CASES
    for dtype, mode, d_pool, d_sel, H, S, g, w, L, n_q, pr, sr, B in CASES:
        for n, first in ((1, "condense_one_kernel"), (B, "summary_query_kernel")):
            d = lca.Desc(B=n, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, n_q=n_q, mode=mode, dtype={"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}[dtype],
                         pool_reduce=pr, sel_reduce=sr)
            assert t.condense(d)[0].kernel.startswith(first), (mode, d_pool, d_sel, H, S, g, L, n)


def test_cases_without_a_number_are_where_they_claim_to_be():
    from tests.test_gpu_condense_one import NAN_CASES
    names = []
    for dtype, mode, d_pool, d_sel, H, S, n_q, sr, B in NAN_CASES:
        d = lca.Desc(B=B, L=64, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=16, w=0, n_q=n_q, mode=mode, sel_reduce=sr, dtype={"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}[dtype])
        names.append(t.condense(d)[-1].kernel.split("<")[0])
    assert names == ["condense_one_kernel"] * 3 + ["condense_any_kernel"] * 3 + ["condense_reg_kernel"]


def test_cases_of_many_items_are_where_they_claim_to_be():
    from tests.test_gpu_many_items import GROUPS, HALVES, MLA
    for B, L, H, S, g, w, dtype, scale, bias, ties, up in HALVES:
        run = t.prefill(_mla(B=B, L=L, H=H, S=S, g=g, w=w, dtype={"bf16": lca.BF16, "f16": lca.F16}[dtype]), up=up)[-1]
        assert run.kernel.startswith("attn_mla_kernel_halves") and run.grid == 256, (B, L, H, run)
    for B, L, H, S, g, w, dtype, scale, bias, ties, up in MLA:
        d = _mla(B=B, L=L, H=H, S=S, g=g, w=w, dtype={"bf16": lca.BF16, "f16": lca.F16}[dtype])
        for kw in (dict(up=True),) if up else (dict(), dict(dense=True)):
            assert t.prefill(d, **kw)[-1].kernel.startswith("attn_mla_kernel<"), (B, L, H)
    for kernel, dtype, mode, d_pool, d_sel, H, S, g, w, L, B, n_q, scale, ties in GROUPS:
        d = lca.Desc(B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, n_q=n_q, mode=mode, dtype={"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}[dtype])
        assert kernel in t.condense(d)[-1].kernel, (L, g, t.condense(d))

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

"""The binding's native marshalling (binding/bind.cpp): it takes calls with plain tensors, leaves everything else to lca.py, and the two ways
call the library alike."""
import numpy as np
import pytest

from paper_2604_12452_amd import inputs, lca
from tests import helpers as hp

pytestmark = pytest.mark.gpu


class _Counted:
    """The native module with the statuses its functions returned."""
    def __init__(self, bind):
        self.bind, self.seen = bind, []

    def __getattr__(self, name):
        def call(*args):
            self.seen.append((name, getattr(self.bind, name)(*args)))
            return self.seen[-1][1]
        return call


def _step(desc, layout, t):
    """Update, quantisation and both decode steps, prefill and dense: every call the native marshalling knows but the up-projection."""
    import torch
    dt = lca.torch_dtype(desc)
    pr, sr, an, al = lca.alloc_condensed(desc, alpha=True)
    O = torch.empty(desc.B, desc.L, desc.H, desc.d_pool, dtype=dt, device="cuda")
    lse = torch.empty(desc.B, desc.L, desc.H, device="cuda")
    Od = torch.empty_like(O)
    lca.condense(desc, t["Q"], t["POOL"], t["SEL"], pr, sr, an, al, t["ws"])
    lca.prefill_attn(desc, t["Q"], t["POOL"], t["SEL"], pr, sr, O, lse, t["ws"])
    lca.dense_attn(desc, t["Q"], t["POOL"], t["SEL"], Od, None, t["ws"])
    cap_p, cap_s = (torch.zeros(desc.B, desc.S, layout.m_cap, n, dtype=dt, device="cuda") for n in (desc.d_pool, desc.d_sel))
    an2 = torch.zeros(desc.B, desc.S, layout.m_cap, dtype=torch.int32, device="cuda")
    cap_p[:, :, :desc.m], cap_s[:, :, :desc.m] = pr, sr
    lca.cache_update(desc, layout, t["recent"], t["pt"], t["st"], cap_p, cap_s, an2, t["ws"])
    o = [torch.empty(desc.B, desc.H, desc.d_pool, dtype=dt, device="cuda") for _ in range(3)]
    lca.decode_attn_cached(desc, layout, t["q"], cap_p, cap_s, t["pt"], t["st"], o[0], t["ws"])
    lca.decode_attn(desc, t["q"], pr, sr, t["pt"][:, :, :desc.k].contiguous(), t["st"][:, :, :desc.k].contiguous(), o[1], t["ws"])
    p8, s8 = (torch.zeros(x.shape, dtype=torch.uint8, device="cuda") for x in (cap_p, cap_s))
    sc = torch.ones(desc.B, desc.S, layout.m_cap, 2, device="cuda")
    lca.quantize_cache(desc, layout, cap_p, cap_s, p8, s8, sc)
    lca.decode_attn_q8(desc, layout, t["q"], p8, s8, sc, t["pt"], t["st"], o[2], t["ws"])
    return [pr, sr, an, al, O, lse, Od, cap_p, cap_s, an2, *o, p8, s8, sc]


@pytest.mark.parametrize("dtype", [lca.BF16, lca.F16])
@pytest.mark.parametrize("mode,d_pool,d_sel,S", [(lca.MODE_MLA, 512, 64, 1), (lca.MODE_GQA, 128, 128, 2)])
def test_both_ways_call_the_library_alike(monkeypatch, dtype, mode, d_pool, d_sel, S):
    import torch
    lca.load()
    assert lca._bind is not None, "the native marshalling was not built"
    d = lca.Desc(B=2, L=96, H=4, S=S, d_pool=d_pool, d_sel=d_sel, g=8, w=32, mode=mode, dtype=dtype)
    lay = lca.CacheLayout(m_cap=d.m + 2, k_cap=d.w + 2 * d.g, k_start=5)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    rn = lambda *s: (0.3 * torch.randn(*s, generator=gen, device="cuda")).to(lca.torch_dtype(d))
    P, dq = d.kv_heads, d.d_qk
    kv = lambda n: (2, 96, n) if mode == lca.MODE_MLA else (2, 96, P, n)
    t = dict(Q=rn(2, 96, 4, dq), POOL=rn(*kv(d_pool)), SEL=rn(*kv(d_sel)), recent=rn(2, 8, 4, dq), q=rn(2, 4, dq), pt=rn(2, P, lay.k_cap, d_pool),
             st=rn(2, P, lay.k_cap, d_sel), ws=lca.alloc_workspace(d))
    counted = _Counted(lca._bind)
    monkeypatch.setattr(lca, "_bind", counted)
    native = _step(d, lay, t)
    assert [s for _, s in counted.seen] == [0] * 8 and len({n for n, _ in counted.seen}) == 8, counted.seen
    monkeypatch.setattr(lca, "_bind", None)
    plain = _step(d, lay, t)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    monkeypatch.setattr(lca, "_bind", counted)
    with torch.cuda.stream(side):
        current = _step(d, lay, t)                   # the current stream is asked for on every call
    torch.cuda.synchronize()
    for stream in (side, side.cuda_stream):
        out = torch.empty_like(native[6])
        torch.cuda.synchronize()
        lca.dense_attn(d, t["Q"], t["POOL"], t["SEL"], out, None, t["ws"], stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(out, native[6])
    for a, *others in zip(native, plain, current):
        for b in others:
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_what_it_leaves_to_python():
    """Raw addresses, tensor subclasses, views that are not contiguous, sizes past any integer and descriptors of another class."""
    import torch
    lca.load()
    d = lca.Desc(B=1, L=64, H=2, S=1, d_pool=64, d_sel=64, g=4, w=8, mode=lca.MODE_GQA)
    t = dict(Q=torch.zeros(1, 64, 2, 64, dtype=torch.bfloat16, device="cuda"), K=torch.zeros(1, 64, 1, 64, dtype=torch.bfloat16, device="cuda"),
             O=torch.zeros(1, 64, 2, 64, dtype=torch.bfloat16, device="cuda"), ws=lca.alloc_workspace(d))
    call = lambda desc=d, Q=t["Q"], K=t["K"], O=t["O"], ws=t["ws"], stream=None: lca._bind.dense_attn(desc, Q, K, K, O, None, ws, stream)
    assert call() == 0

    class Sub(torch.Tensor):
        pass

    class Other(lca.Desc):
        pass

    wide = torch.zeros(1, 64, 2, 128, dtype=torch.bfloat16, device="cuda")[..., ::2]
    for kw in (dict(Q=t["Q"].data_ptr()), dict(Q=t["Q"].as_subclass(Sub)), dict(Q=wide), dict(Q=t["Q"].float()), dict(O=t["O"][:, :63]), dict(O=None), dict(ws=None),
               dict(Q=t["Q"].cpu()), dict(desc=Other(**d.__dict__)), dict(desc=lca.Desc(**{**d.__dict__, "scale": np.float32(1)})),
               dict(desc=lca.Desc(**{**d.__dict__, "L": 1 << 40})), dict(desc=lca.Desc(**{**d.__dict__, "B": 2 ** 31 - 1, "L": 2 ** 31 - 1, "H": 2 ** 30})),
               dict(desc=None), dict(stream="none")):
        assert call(**kw) == -1, kw
    torch.cuda.synchronize()

"""How a decode step is split over workgroups: one, two and four tiles per wavefront, caches whose pairs (sequence, set) fill the chip
alone, more partial results than the merge's one-group form takes, and fewer tiles than wavefronts."""
import numpy as np
import pytest

from paper_2604_12452_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu


# ..., workgroups per (sequence, set); tests/test_launches.py checks these on the CPU, so that a changed rule cannot move the cases
CASES = [
    ("bf16", inputs.MODE_MLA, 1, 37, 16, 1, 4, 20, 1),              # fewer tiles than wavefronts of one workgroup
    ("bf16", inputs.MODE_MLA, 1, 1024, 16, 1, 16, 1024, 16),        # one tile per wavefront, the merge's one-group form at its limit
    ("f16", inputs.MODE_MLA, 2, 3100, 16, 1, 1, 100, 25),           # two tiles per wavefront, the last one ragged
    ("f16", inputs.MODE_MLA, 2, 2200, 16, 1, 1, 100, 35),           # one, the last workgroup with tiles for three of its wavefronts
    ("bf16", inputs.MODE_MLA, 1, 16400, 16, 1, 2, 16, 65),          # one more than a wavefront has lanes: the merge for any number
    ("bf16", inputs.MODE_MLA, 20, 1500, 4, 1, 1, 30, 6),            # four tiles per wavefront
    ("bf16", inputs.MODE_MLA, 130, 300, 2, 1, 2, 30, 1),            # more than half as many sequences as CUs: one workgroup each
    ("bf16", inputs.MODE_MLA, 1, 512, 16, 1, 16, 512, 8),           # 8 and 9 partial results: on both sides of eight rows per thread
    ("f16", inputs.MODE_MLA, 1, 520, 7, 1, 16, 1024, 9),
    ("bf16", inputs.MODE_MLA, 1, 2100, 16, 1, 16, 4096, 33),        # one more than 32
    ("bf16", inputs.MODE_MLA, 3, 2060, 16, 1, 16, 4096, 17),        # the first with four groups, of two tiles per wavefront
    ("bf16", inputs.MODE_MLA, 1, 8300, 16, 1, 16, 9000, 65),
    ("bf16", inputs.MODE_GQA, 1, 6100, 28, 4, 1, 40, 48),
    ("f16", inputs.MODE_GQA, 3, 2900, 14, 2, 2, 33, 12),
    ("bf16", inputs.MODE_GQA, 33, 400, 8, 4, 2, 64, 1),             # 132 pairs
    ("bf16", inputs.MODE_MLA, 1, 256, 16, 1, 16, 300, 1),           # 16 and 17 tiles: the longest cache of one workgroup, the shortest of several
    ("f16", inputs.MODE_MLA, 1, 257, 16, 1, 16, 300, 5),
    ("bf16", inputs.MODE_GQA, 2, 512, 8, 2, 16, 600, 1),
    ("f16", inputs.MODE_GQA, 2, 513, 8, 2, 16, 600, 5),
    ("bf16", inputs.MODE_MLA, 1, 7000, 16, 1, 16, 9000, 55),        # the merge's fourth group has work, and all of it
    ("f16", inputs.MODE_MLA, 1, 8192, 16, 1, 16, 9000, 64),
    ("bf16", inputs.MODE_MLA, 1, 1030, 16, 1, 16, 9000, 17),        # one tile per wavefront and more results than 16: the first, the last, and one workgroup too many
    ("f16", inputs.MODE_MLA, 2, 2048, 16, 1, 16, 9000, 32),
    ("bf16", inputs.MODE_MLA, 4, 1460, 8, 1, 16, 9000, 23),
    ("bf16", inputs.MODE_MLA, 4, 1480, 16, 1, 16, 9000, 12),
    ("f16", inputs.MODE_MLA, 1, 3072, 16, 1, 16, 9000, 48),         # the most results, of few workgroups and of few heads; one more workgroup, or one more head, than that
    ("bf16", inputs.MODE_MLA, 1, 3073, 16, 1, 16, 9000, 25),
    ("bf16", inputs.MODE_MLA, 4, 3072, 7, 1, 16, 9000, 48),
    ("f16", inputs.MODE_MLA, 4, 1480, 7, 1, 16, 9000, 24),
    ("bf16", inputs.MODE_MLA, 2, 2200, 14, 2, 16, 9000, 35),
    ("f16", inputs.MODE_MLA, 4, 1480, 8, 1, 16, 9000, 12),
]


@pytest.mark.parametrize("dtype,mode,B,L,H,S,g,w", [c[:-1] for c in CASES])
def test_decode_step_splits(oracle, dtype, mode, B, L, H, S, g, w):
    import torch
    from paper_2604_12452_amd import lca
    d_pool, d_sel = (512, 64) if mode == inputs.MODE_MLA else (128, 128)
    wl = inputs.Workload("splits", B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, dtype=dtype, mode=mode)
    print(f"[case] {wl}", flush=True)
    desc = hp.lca_desc(wl)
    rng = np.random.default_rng(31 + L)
    P, dq = desc.kv_heads, desc.d_qk
    def draw(*shape, std=1.0):
        return inputs.to_storage(rng.standard_normal(shape, dtype=np.float32) * np.float32(std), dtype)
    host = dict(q=draw(B, H, dq, std=dq ** -0.5), pool_rep=draw(B, S, desc.m, d_pool), sel_rep=draw(B, S, desc.m, d_sel),
                pool_tail=draw(B, P, desc.k, d_pool), sel_tail=draw(B, P, desc.k, d_sel))
    dev = {n: hp.to_dev(x, dtype) for n, x in host.items()}
    O = torch.full((B, H, d_pool), float("nan"), dtype=lca.torch_dtype(desc), device="cuda")
    ws = torch.full((lca.workspace_size(desc),), 0xFF, dtype=torch.uint8, device="cuda")      # NaN patterns: nothing may be read before it is written
    lca.decode_attn(desc, dev["q"], dev["pool_rep"], dev["sel_rep"], dev["pool_tail"], dev["sel_tail"], O, ws)
    torch.cuda.synchronize()
    ref = oracle.decode_attn(hp.oracle_desc(oracle, wl), *(inputs.to_f64(host[n], dtype) for n in ("q", "pool_rep", "sel_rep", "pool_tail", "sel_tail")))
    err = hp.vec_rel_err(hp.from_dev(O, dtype), ref)
    print(f"  decode err {err:.2e}", flush=True)
    assert err <= hp.TOL[dtype]


@pytest.mark.parametrize("dtype,ulp", [("bf16", 2.0 ** -7), ("f16", 2.0 ** -10)])
@pytest.mark.parametrize("k", [30, 60])
def test_gqa_output_is_the_sum_divided_once(dtype, ulp, k):
    """One workgroup, equal logits (a zero query): the output is the mean of the k value rows.  Half of them are a number of the
    16-bit type and half the next one, so the mean lies exactly between the two and rounds to the even one; a product with a rounded
    1 / k lands beside the tie and misses it in four columns of ten."""
    import torch
    from paper_2604_12452_amd import lca
    d = lca.Desc(B=1, L=k, H=4, S=2, d_pool=128, d_sel=128, g=16, w=64, mode=lca.MODE_GQA, dtype={"bf16": lca.BF16, "f16": lca.F16}[dtype])
    j = np.arange(128) * (1 if dtype == "bf16" else 8) + np.arange(128) % 2
    low = 1.0 + ulp * j
    v = np.tile(low, (1, 2, k, 1))
    v[:, :, k // 2:] += ulp
    dev = [hp.to_dev(inputs.to_storage(a.astype(np.float32), dtype), dtype) for a in (np.zeros((1, 4, 128)), v, np.ones((1, 2, k, 128)))]
    O = torch.empty(1, 4, 128, dtype=lca.torch_dtype(d), device="cuda")
    lca.decode_attn(d, dev[0], None, None, dev[1], dev[2], O, lca.alloc_workspace(d))
    np.testing.assert_array_equal(hp.from_dev(O, dtype)[0], np.tile(np.where(j % 2 == 0, low, low + ulp), (4, 1)))


# ..., tiles per wavefront: one and two (shared by the wavefronts of a workgroup), three and four in a workgroup that has the sequence to itself, four otherwise
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,L,H,g,w,steps", [(1, 30, 16, 4, 64, 1), (2, 150, 7, 4, 200, 3), (1, 250, 16, 4, 300, 4), (1, 600, 16, 4, 700, 1), (1, 2205, 5, 2, 90, 1), (1, 6300, 5, 2, 90, 2), (20, 1500, 4, 1, 30, 4)])
@pytest.mark.parametrize("late", [0.0, 100.0])
def test_mla_step_over_shared_tiles(oracle, dtype, B, L, H, g, w, steps, late):
    """Partial last tiles and steps, and (late) logits that rise past any fixed reference in the last third of the raw tail, so that a workgroup of two steps
    or more that has them in a later one runs its tiles again from exact maxima (in one step the reference is the exact maximum); with sequences whose
    caches end in a tile of one entry."""
    import torch
    from paper_2604_12452_amd import lca
    wl = inputs.Workload("shared", B=B, L=L, H=H, S=1, d_pool=512, d_sel=64, g=g, w=w, dtype=dtype, mode=inputs.MODE_MLA)
    print(f"[case] {wl} late {late}", flush=True)
    desc = hp.lca_desc(wl)
    rng = np.random.default_rng(7 + L)
    def draw(*shape, std=1.0):
        x = rng.standard_normal(shape, dtype=np.float32) * np.float32(std)
        return x
    host = dict(q=draw(B, H, 576, std=576 ** -0.5), pool_rep=draw(B, 1, desc.m, 512), sel_rep=draw(B, 1, desc.m, 64),
                pool_tail=draw(B, 1, desc.k, 512), sel_tail=draw(B, 1, desc.k, 64))
    if late:
        host["sel_tail"][:, :, desc.k - max(1, desc.k // 3):] *= late
    host = {n: inputs.to_storage(x, dtype) for n, x in host.items()}
    dev = {n: hp.to_dev(x, dtype) for n, x in host.items()}
    O = torch.full((B, H, 512), float("nan"), dtype=lca.torch_dtype(desc), device="cuda")
    ws = torch.full((lca.workspace_size(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    lca.decode_attn(desc, dev["q"], dev["pool_rep"], dev["sel_rep"], dev["pool_tail"], dev["sel_tail"], O, ws)
    torch.cuda.synchronize()
    ref = oracle.decode_attn(hp.oracle_desc(oracle, wl), *(inputs.to_f64(host[n], dtype) for n in ("q", "pool_rep", "sel_rep", "pool_tail", "sel_tail")))
    assert hp.vec_rel_err(hp.from_dev(O, dtype), ref) <= hp.TOL[dtype]


# B, L, H, g, w, steps of a workgroup: codes and tail in one workgroup, codes alone and then both in several, one step each (twice), four unshared
Q8_STEPS = [(1, 250, 16, 4, 100, 3), (2, 280, 7, 4, 230, 4), (1, 6300, 5, 2, 90, 2), (1, 600, 16, 2, 200, 1), (1, 2205, 5, 2, 90, 1), (20, 1500, 4, 1, 30, 4)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,L,H,g,w,steps", Q8_STEPS)
@pytest.mark.parametrize("late", [None, "tail", "codes"])
def test_mla_q8_step_over_shared_tiles(oracle, dtype, B, L, H, g, w, steps, late):
    """The same over 8-bit representatives, whose tiles are converted in place one step behind their request: logits that rise past the first step's maximum
    in the raw tail, or among the representatives."""
    import torch
    from oracle import q8
    from paper_2604_12452_amd import lca
    wl = inputs.Workload("shared_q8", B=B, L=L, H=H, S=1, d_pool=512, d_sel=64, g=g, w=w, dtype=dtype, mode=inputs.MODE_MLA)
    print(f"[case] {wl} late {late}", flush=True)
    desc = hp.lca_desc(wl)
    m, k = desc.m, desc.k
    rng = np.random.default_rng(11 + L)
    draw = lambda *shape, std=1.0: rng.standard_normal(shape, dtype=np.float32) * np.float32(std)
    host = dict(q=draw(B, H, 576, std=576 ** -0.5), pool_rep=draw(B, 1, m, 512), sel_rep=draw(B, 1, m, 64), pool_tail=draw(B, 1, k, 512), sel_tail=draw(B, 1, k, 64))
    if late == "tail":
        host["sel_tail"][:, :, k - max(1, k // 3):] *= 400.0
    if late == "codes":
        host["sel_rep"][:, :, 80:96] *= 400.0                # the sixth tile
    dev = {n: hp.to_dev(inputs.to_storage(x, dtype), dtype) for n, x in host.items()}
    codes = [torch.zeros(dev[n].shape, dtype=torch.uint8, device="cuda") for n in ("pool_rep", "sel_rep")]
    scales = torch.ones(B, 1, m, 2, device="cuda")
    lca.quantize_cache(desc, None, dev["pool_rep"], dev["sel_rep"], *codes, scales)
    O = torch.full((B, H, 512), float("nan"), dtype=lca.torch_dtype(desc), device="cuda")
    ws = torch.full((lca.workspace_size(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    lca.decode_attn_q8(desc, None, dev["q"], *codes, scales, dev["pool_tail"], dev["sel_tail"], O, ws)
    again = torch.full_like(O, float("nan"))
    lca.decode_attn_q8(desc, None, dev["q"], *codes, scales, dev["pool_tail"], dev["sel_tail"], again, ws)
    torch.cuda.synchronize()
    assert torch.equal(O.view(torch.int16), again.view(torch.int16))
    sc = scales.cpu().numpy().astype(np.float64)
    reps = [q8.dequantize_rows(c.cpu().numpy(), sc[..., i]) for i, c in enumerate(codes)]
    q, pt, st = (hp.from_dev(dev[n], dtype) for n in ("q", "pool_tail", "sel_tail"))
    assert hp.vec_rel_err(hp.from_dev(O, dtype), oracle.decode_attn(hp.oracle_desc(oracle, wl), q, *reps, pt, st)) <= hp.TOL[dtype]
    if (late == "tail" and steps > 1 and B < 20) or (late == "codes" and steps == 2):
        # some workgroup's later step holds a logit out of reach of the maximum of its first four tiles (bf16: 2^100, fp16: 65504)
        z = np.einsum("bhd,bed->bhe", q, np.concatenate([np.concatenate([reps[0], reps[1]], -1), np.concatenate([pt, st], -1)], 2)[:, 0]) * wl.scale * 1.4426950408889634
        tiles = [z[..., i:min(i + 16, m)] for i in range(0, m, 16)] + [z[..., i:i + 16] for i in range(m, m + k, 16)]
        wg = [tiles[i:i + 4 * steps] for i in range(0, len(tiles), 4 * steps)]
        top = lambda ts: np.concatenate(ts, -1).max(-1)
        assert max((top(ts[4:]) - top(ts[:4])).max() for ts in wg if len(ts) > 4) > (100 if dtype == "bf16" else 16)

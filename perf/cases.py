"""The workloads whose speed this repository watches: what a serving or evaluation program calls liblca for.

A case is one layer's call (or the few calls of one step) through ``paper_2604_12452_amd.lca``, over the shapes of the
repository's benchmark configurations and the sizes around them: short and long prompts, one sequence and batches, ragged
lengths, both 16-bit types and fp32, the MLA and the GQA widths and narrower heads, prefill, decode and the online cache
update, the 16-bit and the 8-bit cache.

  what = "prefill"  lca.condense + lca.prefill_attn (or, with up, lca.prefill_attn_up) on B prompts of L tokens
  what = "decode"   lca.decode_attn_cached (q8: lca.decode_attn_q8) for the L-th token of B sequences, tail in a ring
  what = "update"   the decode step on which a group is due: lca.cache_update, with q8 lca.quantize_cache of the new row,
                    then the decode step
"""
import math

import torch

from paper_2604_12452_amd import lca

_MODE = {"mla": lca.MODE_MLA, "gqa": lca.MODE_GQA}
_DTYPE = {"bf16": lca.BF16, "f16": lca.F16, "f32": lca.F32}
_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_ROOM = 3                    # spare groups in a growing cache (m_cap = m + _ROOM, k_cap = w + (1 + _ROOM) g)


def _case(name, what, mode, dtype, B, L, H, S, d_pool, d_sel, g=16, w=1024, up=False, q8=False, lse=False):
    return dict(name=name, what=what, mode=mode, dtype=dtype, B=B, L=L, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=g, w=w, up=up, q8=q8, lse=lse)


def listed():
    return [
        # One user, a conversation of a few thousand tokens: the latency of a single decode step.
        _case("decode_mla_one", "decode", "mla", "bf16", 1, 4001, 16, 1, 512, 64),
        # A full serving batch of long contexts (configuration 4's layer): bound by reading the caches.
        _case("decode_mla_batch", "decode", "mla", "bf16", 32, 131072, 16, 1, 512, 64),
        # The same for the GQA layer (configuration 5's), from the 8-bit copy of its representatives.
        _case("decode_gqa_q8", "decode", "gqa", "bf16", 32, 65536, 32, 8, 128, 128, q8=True),
        # Every g-th step of a small GQA batch: the online update, then the step (L - w divisible by g).
        _case("update_gqa", "update", "gqa", "f16", 5, 1024 + 16 * 937, 28, 4, 128, 128),
        # The fp32 configuration: the whole path in single precision at its small shape.
        _case("prefill_f32", "prefill", "mla", "f32", 1, 1024, 4, 1, 128, 32, w=128, lse=True),
        # A layer with narrow heads (64 / 64), which no width-specific kernel is built for.
        _case("prefill_narrow", "prefill", "gqa", "bf16", 1, 2500, 16, 4, 64, 64, w=512),
        # A chat prompt, mostly inside the local window: little work, the first-token latency of short requests.
        _case("prefill_mla_chat", "prefill", "mla", "bf16", 1, 1500, 16, 1, 512, 64),
        # Configuration 2: one 8K prompt.
        _case("prefill_mla_8k", "prefill", "mla", "bf16", 1, 8192, 16, 1, 512, 64),
        # Two ragged documents in fp16, one condensed set per head, value up-projection fused.
        _case("prefill_mla_up", "prefill", "mla", "f16", 2, 20011, 16, 16, 512, 64, up=True),
        # The headline: one 128K prompt through the MLA layer (configuration 4).
        _case("prefill_mla_128k", "prefill", "mla", "bf16", 1, 131072, 16, 1, 512, 64),
        # A batch of ragged prompts through a GQA layer with 7 heads per KV head, coarser groups, fp16.
        _case("prefill_gqa_ragged", "prefill", "gqa", "f16", 3, 5003, 28, 4, 128, 128, g=32, lse=True),
        # Configuration 5: one 64K prompt through the GQA layer.
        _case("prefill_gqa_64k", "prefill", "gqa", "bf16", 1, 65536, 32, 8, 128, 128),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    while True:
        what = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "update"])
        c = _case("", what, rng.choice(["mla", "gqa"]), rng.choice(["bf16", "bf16", "f16"]), 1, 0, 0, 1, 0, 0, g=rng.choice([8, 16, 16, 32]),
                  w=rng.choice([512, 1024, 1024, 2048]))
        del c["name"]
        if c["mode"] == "mla":
            c["H"], c["S"], c["d_pool"], c["d_sel"] = rng.choice([8, 16, 16]), 1, 512, 64
        else:
            (c["H"], c["S"]), c["d_pool"], c["d_sel"] = rng.choice([(32, 8), (28, 4), (16, 4)]), 128, 128
        if what == "prefill":
            c["lse"] = rng.random() < 0.3
            if rng.random() < 0.3:            # fp32, or widths without a kernel of their own
                c["dtype"], c["mode"], c["H"], c["S"], c["d_pool"], c["d_sel"] = rng.choice([
                    ("f32", "mla", 4, 1, 128, 32), ("f32", "mla", 8, 1, 128, 32), ("bf16", "gqa", 16, 4, 64, 64), ("f16", "gqa", 8, 8, 64, 64),
                    ("bf16", "mla", 8, 1, 256, 32)])
                c["w"] = rng.choice([128, 256, 512])
                c["L"] = _log_int(rng, 100, 4096)
            elif c["mode"] == "mla":
                c["L"] = _log_int(rng, 100, 131072)
                c["S"] = rng.choice([1, 1, 1, c["H"]])
                c["up"] = rng.random() < 0.3
            else:
                c["L"] = _log_int(rng, 100, 65536)
            c["B"] = rng.choice([1, 1, 2, 3]) if c["L"] <= 20000 else 1
        else:
            c["B"], c["L"] = _log_int(rng, 1, 32), _log_int(rng, 600, 131072)
            c["q8"] = rng.random() < 0.35
            if what == "update":
                c["L"] = c["w"] + c["g"] * max(1, (c["L"] - c["w"]) // c["g"])
        wk = work(c)
        # never dearer than the largest listed case of its kind (paths without a matrix-core kernel count for more)
        rate = 200.0 if c["what"] == "prefill" and _is_general(c) else 1.0
        if wk["flops"] * rate <= 24e12 and wk["bytes"] <= 5e9:
            return c


def _is_general(case):
    return case["dtype"] == "f32" or (case["d_pool"], case["d_sel"]) not in ((512, 64), (128, 128))


# ---------------------------------------------------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------------------------------------------------
def _rows(case):
    m = max(0, (case["L"] - case["w"]) // case["g"])
    return m, case["L"] - m * case["g"]


def _d_qk(case):
    return case["d_pool"] + case["d_sel"] if case["mode"] == "mla" else case["d_sel"]


def _desc(case):
    return lca.Desc(B=case["B"], L=case["L"], H=case["H"], S=case["S"], d_pool=case["d_pool"], d_sel=case["d_sel"], g=case["g"], w=case["w"],
                    mode=_MODE[case["mode"]], dtype=_DTYPE[case["dtype"]])


def _visible(t, g, w):
    """Representatives that query position t sees."""
    return max(0, (t + 1 - w) // g)


def work(case):
    B, L, H, S, g, w = (case[k] for k in ("B", "L", "H", "S", "g", "w"))
    m, k = _rows(case)
    elt = 4 if case["dtype"] == "f32" else 2
    P = 1 if case["mode"] == "mla" else S
    row, dq, dv = case["d_pool"] + case["d_sel"], _d_qk(case), case["d_pool"]
    if case["what"] == "prefill":
        pairs = 0
        for u in range(0, L - w + 1, g) if L > w else ():      # positions t = w - 1 + u see u / g representatives, g positions alike
            n = min(g, L - (w - 1 + u))
            j, t0 = u // g, w - 1 + u
            pairs += n * j + n * (t0 + 1 - j * g) + n * (n - 1) // 2
        first = min(L, max(w - 1, 0))
        pairs += first * (first + 1) // 2
        flops = 2.0 * (dq + dv) * pairs * B * H + 2.0 * (dq + dv) * B * S * m * g
        d_out = 128 if case["up"] else dv
        if case["up"]:
            flops += 2.0 * B * L * H * dv * d_out
        nbytes = B * L * (P * row + H * (dq + d_out)) * elt + B * S * m * (row * elt + 4) + (H * d_out * dv * elt if case["up"] else 0)
        nbytes += B * L * H * 4 if case["lse"] else 0
        return {"bytes": nbytes, "flops": flops}
    rep = row + 8 if case["q8"] else row * elt
    nbytes = B * (S * m * rep + P * k * row * elt + H * (dq + dv) * elt)
    flops = 2.0 * (dq + dv) * B * H * (m + k)
    if case["what"] == "update":
        nbytes += B * g * (P * row + H * dq) * elt + B * S * (row * elt + 4)
        flops += 2.0 * (dq + dv) * B * S * g
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Largest differences seen between two summation orders or softmax references of the same kernels, four times over.
    # A representative's anchor may differ only at near-ties of two scores.
    return {"f32": {"rel": 1e-5, "max": 4e-4, "differ": 1e-3}, "f16": {"rel": 2e-3, "max": 0.1, "differ": 1e-3},
            "bf16": {"rel": 1e-2, "max": 0.4, "differ": 1e-3}}[case["dtype"]]


# ---------------------------------------------------------------------------------------------------------------------
# inputs: locally redundant sequences (AR(1) along the tokens), unit-variance position keys, rotated GQA keys
# ---------------------------------------------------------------------------------------------------------------------
def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _ar1(gen, n, lead, width, rho=0.9):
    """[*lead, n, *width], x_t = rho x_{t-1} + N(0, 1) (to 256 taps)."""
    x = _randn(gen, *lead, n, *width)
    axis, k = len(lead), 1
    while k < min(n, 256):
        y = x.clone()
        y.narrow(axis, k, n - k).add_(x.narrow(axis, 0, n - k), alpha=rho ** k)
        x, k = y, 2 * k
    return x


def _rope(x, pos, theta=500000.0):
    """Rotary embedding of the last axis at positions pos (one per index of axis 1)."""
    d = x.shape[-1]
    inv = theta ** (-torch.arange(0, d, 2, device="cuda", dtype=torch.float32) / d)
    ang = (pos.to(torch.float32)[:, None] * inv).reshape(1, len(pos), *([1] * (x.dim() - 3)), d // 2)
    z = torch.view_as_complex(x.reshape(*x.shape[:-1], d // 2, 2).contiguous()) * torch.polar(torch.ones_like(ang), ang)
    return torch.view_as_real(z).reshape(x.shape)


def _sequence(gen, case, n, pos):
    """(pooled, selected) components of n cached tokens: [B, n, (S,) d]."""
    if case["mode"] == "mla":
        return _ar1(gen, n, (case["B"],), (case["d_pool"],)), _randn(gen, case["B"], n, case["d_sel"])
    return (_ar1(gen, n, (case["B"],), (case["S"], case["d_pool"])),
            _rope(_ar1(gen, n, (case["B"],), (case["S"], case["d_sel"])), pos))


def _queries(gen, case, *lead):
    d = _d_qk(case)
    return (_randn(gen, *lead, case["H"], d) / math.sqrt(d)).to(_TORCH[case["dtype"]])


def _quantise(x):
    """E4M3 codes and one power-of-two scale per row (largest magnitude of the row in (224, 448])."""
    big = x.float().abs().amax(-1)
    scale = torch.exp2(torch.ceil(torch.log2(big / 448.0)))
    scale = torch.where(big > 0, scale, torch.ones_like(scale))
    return (x.float() / scale[..., None]).to(torch.float8_e4m3fn).view(torch.uint8), scale


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) + 1)
    dt = _TORCH[case["dtype"]]
    B, L, H, S, g, w = (case[k] for k in ("B", "L", "H", "S", "g", "w"))
    d = _desc(case)
    m, k = _rows(case)
    st = {"case": case, "desc": d, "ws": lca.alloc_workspace(d)}
    if case["what"] == "prefill":
        pool, sel = _sequence(gen, case, L, torch.arange(L, device="cuda"))
        st["pool"], st["sel"] = pool.to(dt), sel.to(dt)
        st["Q"] = torch.cat([_queries(gen, case, 1, L) for _ in range(B)])
        st["pool_rep"], st["sel_rep"], st["anchor"], _ = lca.alloc_condensed(d)
        if case["up"]:
            st["W"] = (_randn(gen, H, 128, case["d_pool"]) / math.sqrt(case["d_pool"])).to(dt)
        st["O"] = torch.empty(B, L, H, 128 if case["up"] else case["d_pool"], dtype=dt, device="cuda")
        st["lse"] = torch.empty(B, L, H, device="cuda") if case["lse"] else None
        return st
    # a cache that has been growing: room for a few more groups, the raw tail somewhere in its ring
    lay = lca.CacheLayout(m_cap=m + _ROOM, k_cap=w + (1 + _ROOM) * g, k_start=0)
    lay.k_start = (5 * g) % lay.k_cap if m else 0
    due = case["what"] == "update"
    n_tail = w + g if due else k              # the ring holds the group about to be condensed as well
    P = 1 if case["mode"] == "mla" else S
    rep, srep = [], []
    for s in range(S):                        # one set at a time: representatives are sequences like the tokens'
        one = dict(case, S=1)
        p, q = _sequence(gen, one, lay.m_cap, torch.arange(lay.m_cap, device="cuda") * g)
        rep.append(p.reshape(B, lay.m_cap, -1).to(dt))
        srep.append(q.reshape(B, lay.m_cap, -1).to(dt))
    st["pool_rep"], st["sel_rep"] = torch.stack(rep, 1), torch.stack(srep, 1)
    tp, ts = _sequence(gen, case, n_tail, torch.arange(L - n_tail, L, device="cuda"))
    ring = (lay.k_start + torch.arange(n_tail, device="cuda")) % lay.k_cap
    for key, t in (("pool_tail", tp), ("sel_tail", ts)):
        t = t.reshape(B, n_tail, P, -1).transpose(1, 2).to(dt)
        st[key] = torch.zeros(B, P, lay.k_cap, t.shape[-1], dtype=dt, device="cuda")
        st[key][:, :, ring] = t
    st["after"] = lca.CacheLayout(lay.m_cap, lay.k_cap, (lay.k_start + g) % lay.k_cap) if due else lay
    st["layout"], st["anchor"] = lay, torch.zeros(B, S, lay.m_cap, dtype=torch.int32, device="cuda")
    st["recent"] = _queries(gen, case, B, g) if due else None
    st["q"] = st["recent"][:, -1].contiguous() if due else _queries(gen, case, B)
    st["O"] = torch.empty(B, H, case["d_pool"], dtype=dt, device="cuda")
    if case["q8"]:
        st["pool_q8"], a = _quantise(st["pool_rep"])
        st["sel_q8"], b = _quantise(st["sel_rep"])
        st["scales"] = torch.stack([a, b], -1).contiguous()
    st["m"] = m
    return st


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(st):
    c, d, ws = st["case"], st["desc"], st["ws"]
    if c["what"] == "prefill":
        lca.condense(d, st["Q"], st["pool"], st["sel"], st["pool_rep"], st["sel_rep"], st["anchor"], None, ws)
        if c["up"]:
            lca.prefill_attn_up(d, st["Q"], st["pool"], st["sel"], st["pool_rep"], st["sel_rep"], st["W"], st["O"], st["lse"], ws)
        else:
            lca.prefill_attn(d, st["Q"], st["pool"], st["sel"], st["pool_rep"], st["sel_rep"], st["O"], st["lse"], ws)
        return {"O": st["O"], "lse": st["lse"], "pool_rep": st["pool_rep"], "sel_rep": st["sel_rep"], "anchor": st["anchor"]}
    out = {"O": st["O"]}
    if c["what"] == "update":
        lca.cache_update(d, st["layout"], st["recent"], st["pool_tail"], st["sel_tail"], st["pool_rep"], st["sel_rep"], st["anchor"], ws)
        if c["q8"]:
            lca.quantize_cache(d, st["after"], st["pool_rep"], st["sel_rep"], st["pool_q8"], st["sel_q8"], st["scales"], st["m"] - 1)
            out.update(pool_q8=st["pool_q8"], sel_q8=st["sel_q8"], scales=st["scales"])
        out.update(pool_rep=st["pool_rep"], sel_rep=st["sel_rep"], anchor=st["anchor"])
    if c["q8"]:
        lca.decode_attn_q8(d, st["after"], st["q"], st["pool_q8"], st["sel_q8"], st["scales"], st["pool_tail"], st["sel_tail"], st["O"], ws)
    else:
        lca.decode_attn_cached(d, st["after"], st["q"], st["pool_rep"], st["sel_rep"], st["pool_tail"], st["sel_tail"], st["O"], ws)
    return out


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------------
def _condense64(qbar, pool, sel, g, mla, dt):
    """One set's groups: qbar [d_qk]; pool, sel [m g, d] in float64 -> pooled [m, d], stored form of it, selected, anchor."""
    m = pool.shape[0] // g
    key = torch.cat([pool, sel], -1) if mla else sel
    score = (key @ qbar).reshape(m, g)
    alpha = torch.softmax(score, -1)
    pooled = torch.einsum("jr,jrd->jd", alpha, pool.reshape(m, g, -1))
    pick = score.argmax(-1)
    anchor = torch.arange(m, device="cuda") * g + pick
    return pooled, pooled.to(dt).double(), sel[anchor], anchor.to(torch.int32)


def _attend64(q, key, val, seen):
    """q [n, d], key / val [e, d] in float64, seen [n, e] or None -> (output [n, d_v], lse [n])."""
    z = q @ key.T
    if seen is not None:
        z.masked_fill_(~seen, -math.inf)
    top = z.amax(-1, keepdim=True)
    z.sub_(top).exp_()
    s = z.sum(-1, keepdim=True)
    return (z @ val) / s, (top + s.log())[:, 0]


def exact(case, seed):
    st = prepare(case, seed)
    B, L, H, S, g, w = (case[k] for k in ("B", "L", "H", "S", "g", "w"))
    mla, dt, hs = case["mode"] == "mla", _TORCH[case["dtype"]], H // S
    m, k = _rows(case)

    def keys(pool, sel):
        return torch.cat([pool, sel], -1) if mla else sel

    if case["what"] == "prefill":
        O = torch.empty(st["O"].shape, dtype=torch.float64, device="cuda")
        lse = torch.empty(B, L, H, dtype=torch.float64, device="cuda")
        pool_rep = torch.empty(B, S, m, case["d_pool"], dtype=torch.float64, device="cuda")
        sel_rep = torch.empty(B, S, m, case["d_sel"], dtype=torch.float64, device="cuda")
        anchor = torch.empty(B, S, m, dtype=torch.int32, device="cuda")
        for b in range(B):
            for s in range(S):
                pool = (st["pool"][b] if mla else st["pool"][b, :, s]).double()
                sel = (st["sel"][b] if mla else st["sel"][b, :, s]).double()
                heads = slice(s * hs, (s + 1) * hs)
                stored = torch.empty(0, case["d_pool"], dtype=torch.float64, device="cuda")
                if m:
                    qbar = st["Q"][b, L - g:, heads].double().mean((0, 1))
                    pool_rep[b, s], stored, sel_rep[b, s], anchor[b, s] = _condense64(qbar, pool[:m * g], sel[:m * g], g, mla, dt)
                rep_key, raw_key = keys(stored, sel_rep[b, s]), keys(pool, sel)
                step = max(64, min(L, (1 << 26) // (hs * (m + w + 64 * g))))
                for t0 in range(0, L, step):
                    t1 = min(L, t0 + step)
                    n_rep, raw0 = _visible(t1 - 1, g, w), _visible(t0, g, w) * g
                    t = torch.arange(t0, t1, device="cuda")[:, None]
                    mt = torch.clamp((t + 1 - w) // g, min=0)
                    j, i = torch.arange(n_rep, device="cuda"), torch.arange(raw0, t1, device="cuda")
                    seen = torch.cat([j < mt, (i >= mt * g) & (i <= t)], -1)
                    q = st["Q"][b, t0:t1, heads].double().reshape((t1 - t0) * hs, -1)
                    o, l = _attend64(q, torch.cat([rep_key[:n_rep], raw_key[raw0:t1]]), torch.cat([stored[:n_rep], pool[raw0:t1]]),
                                     seen.repeat_interleave(hs, 0))
                    o = o.reshape(t1 - t0, hs, -1)
                    if case["up"]:
                        o = torch.stack([o[:, h] @ st["W"][s * hs + h].double().T for h in range(hs)], 1)
                    O[b, t0:t1, heads], lse[b, t0:t1, heads] = o, l.reshape(t1 - t0, hs)
        return {"O": O, "lse": lse if case["lse"] else None, "pool_rep": pool_rep, "sel_rep": sel_rep, "anchor": anchor}

    lay = st["layout"]
    pool_rep, sel_rep = st["pool_rep"].double(), st["sel_rep"].double()
    read_p, read_s, anchor = pool_rep.clone(), sel_rep.clone(), st["anchor"].clone()
    n_tail = st["case"]["w"] + g if case["what"] == "update" else k
    ring = (lay.k_start + torch.arange(n_tail, device="cuda")) % lay.k_cap
    tail_p, tail_s = st["pool_tail"][:, :, ring].double(), st["sel_tail"][:, :, ring].double()
    out = {}
    if case["what"] == "update":
        for b in range(B):
            for s in range(S):
                p = 0 if mla else s
                qbar = st["recent"][b, :, s * hs:(s + 1) * hs].double().mean((0, 1))
                one, stored, selected, a = _condense64(qbar, tail_p[b, p, :g], tail_s[b, p, :g], g, mla, dt)
                pool_rep[b, s, m - 1], read_p[b, s, m - 1], anchor[b, s, m - 1] = one[0], stored[0], a[0] + (m - 1) * g
                sel_rep[b, s, m - 1] = read_s[b, s, m - 1] = selected[0]
        tail_p, tail_s = tail_p[:, :, g:], tail_s[:, :, g:]
        out.update(pool_rep=pool_rep, sel_rep=sel_rep, anchor=anchor)
    if case["q8"]:
        both = []
        for x in (read_p, read_s):
            code, scale = _quantise(x.to(dt))
            both.append((code, scale, code.view(torch.float8_e4m3fn).double() * scale.double()[..., None]))
        read_p, read_s = both[0][2], both[1][2]
        if case["what"] == "update":
            out.update(pool_q8=both[0][0], sel_q8=both[1][0], scales=torch.stack([both[0][1], both[1][1]], -1).double())
    O = torch.empty(B, H, case["d_pool"], dtype=torch.float64, device="cuda")
    for b in range(B):
        for s in range(S):
            p = 0 if mla else s
            pool, sel = torch.cat([read_p[b, s, :m], tail_p[b, p]]), torch.cat([read_s[b, s, :m], tail_s[b, p]])
            O[b, s * hs:(s + 1) * hs] = _attend64(st["q"][b, s * hs:(s + 1) * hs].double(), keys(pool, sel), pool, None)[0]
    out["O"] = O
    return out

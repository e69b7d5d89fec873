#!/usr/bin/env python3
"""Benchmark of the LCA prefill hot path on one MI355X.

One "step" = one pass of the whole hot path over one batch of synthetic input that is already
resident in HBM: lca_condense (summary query + group condensation) followed by lca_prefill_attn.
Workload = the 128K configuration (batch 1, 16 heads, d_c = 512, d_R = 64, bf16, g = 16, w = 1024,
one condensed set shared by the heads — the setting whose cache sizes match the paper's).
Prints ONE JSON line: prefill tokens/s, the roofline of the dominant kernel (attention, bf16 MFMA),
and the CPU oracle timed on a bounded sample of the same workload.  The dense MLA baseline, the
condensation kernel's HBM rate, KV-cache bytes and the g = 32 / per-head-set variants go in "extra".
"""
from __future__ import annotations

import argparse
import math
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0


def pair_count(L: int, w: int, g: int, rows=None) -> int:
    """Visible (query, key) pairs per head: sum over rows t of m_t + (t + 1 - m_t g)."""
    t = np.arange(L, dtype=np.int64) if rows is None else np.asarray(rows, dtype=np.int64)
    mt = np.maximum(0, (t + 1 - w) // g)
    return int((mt + t + 1 - mt * g).sum())


def condense_bytes(wl, m: int) -> int:
    """Algorithmic HBM bytes of one condensation over m groups: groups read once, representatives + anchors written."""
    row = (wl.d_pool + wl.d_sel) * 2
    return wl.B * wl.kv_heads * m * wl.g * row + wl.B * wl.S * m * (row + 4) + wl.nq * wl.H * wl.d_qk * 2


def time_kernel(fn, iters: int, warmup: int, behind=None):
    """Average duration (ms) of fn's GPU work, HIP events on the current stream.  `behind`: a long-running launch
    enqueued in front of the first event, so that the host has queued every timed call before the GPU reaches the
    first one -- for calls so short (a few microseconds) that the host would otherwise submit them more slowly than
    the GPU runs them, and the events would time the host."""
    import torch
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    if behind is not None:
        behind()
    a.record()
    for _ in range(iters):
        fn()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) / iters


N_ROT = 3   # copies an HBM-bound kernel's inputs rotate through when it is timed back to back, so that no call finds its
            # input in the 256 MB memory-side cache left there by the call before


def rotating(make_call, n=N_ROT):
    """make_call(i) -> a zero-argument callable over copy i of the inputs; returns a callable that cycles through them."""
    calls = [make_call(i) for i in range(n)]
    state = {"i": 0}

    def fn():
        calls[state["i"] % n]()
        state["i"] += 1
    return fn


def measured_ceilings(torch, lca, behind):
    """What this chip sustains at the two operations the roofline fractions are read against, from the library's two
    probes: one pass over 151 MB (the bytes one 128K condensation reads) out of HBM, inputs rotated so that no call
    finds them in the memory-side cache, and back-to-back bf16 matrix-core products on every SIMD (the clock the chip
    settles at under that load is part of the figure).  The published peaks stay the denominators of `roofline`."""
    n_words = 151 * (1 << 20) // 4
    bufs = [torch.randint(-2 ** 31, 2 ** 31 - 1, (n_words,), dtype=torch.int32, device="cuda") for _ in range(N_ROT + 1)]
    sums = torch.empty(lca.PROBE_WORDS, dtype=torch.int32, device="cuda")
    ms_read = time_kernel(rotating(lambda i: (lambda: lca.probe_hbm_read(bufs[i], sums)), n=N_ROT + 1), 24, 4, behind=behind)
    del bufs
    out = torch.empty(lca.PROBE_MFMA_FLOATS, dtype=torch.float32, device="cuda")
    iters = 50000
    waves = lca.probe_mfma_bf16(iters, out)
    # pattern 1: operands with every mantissa bit in use, as a kernel's real data (the clock under load depends on it); pattern 0:
    # small integers (the probe's checkable form), which toggle few bits and run faster
    ms_mfma = time_kernel(lambda: lca.probe_mfma_bf16(iters, out, pattern=1), 5, 1)
    ms_mfma_int = time_kernel(lambda: lca.probe_mfma_bf16(iters, out, pattern=0), 5, 1)
    fl = waves * iters * 4 * 32768.0
    return {"hbm_read_TBps": n_words * 4 / (ms_read * 1e-3) / 1e12, "hbm_read_bytes": n_words * 4, "ms_hbm_read": ms_read,
            "mfma_bf16_TFLOPs": fl / (ms_mfma * 1e-3) / 1e12, "ms_mfma": ms_mfma,
            "mfma_bf16_small_integer_operands_TFLOPs": fl / (ms_mfma_int * 1e-3) / 1e12, "mfma_wavefronts": waves}


def cpu_baseline(wl, Q, POOL, SEL, n_rows: int, gpu_anchor=None, gpu_sel_rep=None):
    """The fp64 oracle as it stands, timed on the host cores, on a bounded sample of the workload:
    the full condensation plus n_rows evenly spaced query rows (all heads); extrapolated to a full
    prefill by the sampled rows' share of the visible (query, key) pairs.  Between the two timed calls
    the oracle's cache is brought to what the parity bar compares against (as the GPU tests do): the
    representatives rounded once to the 16-bit storage type, and a group whose top two scores lie
    within the anchor margin takes the GPU's choice."""
    import oracle
    from paper_2604_12452_amd import inputs
    oracle.build()
    d = oracle.Desc(B=wl.B, L=wl.L, H=wl.H, S=wl.S, d_pool=wl.d_pool, d_sel=wl.d_sel, g=wl.g, w=wl.w, n_q=wl.n_q,
                    mode=wl.mode, scale=wl.scale)
    POOLf, SELf = inputs.to_f64(POOL, wl.dtype), inputs.to_f64(SEL, wl.dtype)
    rows = (np.arange(n_rows) * wl.L // n_rows + wl.L // (2 * n_rows)).astype(np.int32)
    Qr = inputs.to_f64(Q[:, rows], wl.dtype)
    Qt = inputs.to_f64(Q[:, wl.L - wl.nq:], wl.dtype)
    t0 = time.perf_counter()
    c = oracle.condense(d, oracle.summary_query(d, Qt), POOLf, SELf)
    t1 = time.perf_counter()
    pool_rep = inputs.to_f64(inputs.to_storage(c["pool_rep"], wl.dtype), wl.dtype)
    sel_rep = c["sel_rep"].copy()
    near_ties = 0
    if gpu_anchor is not None and c["anchor"].size:
        differ = gpu_anchor != c["anchor"]
        if (differ & (c["margin"] > 1e-3)).any():
            raise RuntimeError("GPU anchors differ from the oracle's above the score margin")
        near_ties = int(differ.sum())
        sel_rep[differ] = gpu_sel_rep[differ]
    t1b = time.perf_counter()
    O = oracle.lca_attn_rows(d, rows, Qr, POOLf, SELf, pool_rep, sel_rep)
    t2 = time.perf_counter()
    t_cond, t_attn = t1 - t0, t2 - t1b
    share = pair_count(wl.L, wl.w, wl.g, rows) / pair_count(wl.L, wl.w, wl.g)
    full_s = t_cond + t_attn / share
    return {
        "value": wl.B * wl.L / full_s, "unit": "tokens/s", "cores": oracle.num_threads(), "kind": "oracle",
        "sample": f"full condensation ({t_cond:.2f} s) + {n_rows} evenly spaced query rows x {wl.H} heads "
                  f"({t_attn:.2f} s, {share:.3e} of all visible pairs), extrapolated to the whole prefill",
    }, rows, O, near_ties


PROFILES = {"cfg4": "lca_prefill_cfg4_128k.md", "cfg5": "lca_prefill_cfg5_gqa_64k.md", "cfg3": "lca_prefill_cfg3_32k.md",
            "cfg2": "lca_prefill_cfg2_8k.md", "cfg4+S=16": "lca_prefill_cfg4_128k_per_head_sets.md", "cfg4+g=32": "lca_prefill_cfg4_128k_g32.md",
            "cfg4/decode": "lca_decode_cfg4_mla_128k.md", "cfg5/decode": "lca_decode_cfg5_gqa_64k.md"}


def kernel_sources_sha256() -> str:
    """Hash of the HIP sources the library is built from (file names and contents, sorted): the stamp a profile
    summary carries, so that a summary made from other kernels than the tree's is recognised."""
    import hashlib
    csrc = os.path.join(os.path.dirname(os.path.abspath(__file__)), "paper_2604_12452_amd", "csrc")
    h = hashlib.sha256()
    for name in sorted(os.listdir(csrc)):
        if name.endswith((".hip", ".h")):
            h.update(name.encode() + b"\0" + open(os.path.join(csrc, name), "rb").read() + b"\0")
    return h.hexdigest()[:16]


def profiled_traffic(config, kernel):
    """HBM bytes per launch of `kernel` (fetched + written, counters scaled by the copy-kernel calibration) as
    recorded in the committed rocprofv3 summary of this configuration (its line `traffic_bytes <kernel> <bytes>`).
    None when there is no summary, or when the summary's `sources_sha256` stamp is not the hash of the kernel sources
    in this tree (the kernels changed after it was made).  The counters need the profiler, so they cannot be read
    inside this run."""
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "profiles", PROFILES.get(config, ""))
    traffic, stamp = None, None
    try:
        for line in open(path):
            f = line.split()
            if len(f) == 3 and f[0] == "traffic_bytes" and f[1] == kernel:
                traffic = float(f[2])
            if len(f) == 2 and f[0] == "sources_sha256":
                stamp = f[1]
    except (OSError, ValueError):
        return None
    return traffic if stamp == kernel_sources_sha256() else None


def deviation_report(run, d, wl, torch, lca):
    """lca_deviation_stats on the cache the run holds (Theorem 1's delta_k, delta_v, measured as in the appendix on
    empirical per-token deviations), and the theorem's right-hand side V (exp(2 Q delta_k scale) - 1) + delta_v with
    Q, V the largest query and value norms of the inputs and delta_k, delta_v the largest deviations (norms in the space
    attention works in: absorbed keys [c; k^R], latent values).  The norms are plain reductions over the inputs."""
    stats = torch.zeros((d.B, d.S, 6), dtype=torch.float32, device="cuda")
    ms_dev = time_kernel(lambda: lca.deviation_stats(d, run.POOL, run.SEL, run.pool_rep, run.sel_rep, stats, run.ws), 5, 1)
    st = stats.cpu().numpy().astype(np.float64)
    mean = st.mean(axis=(0, 1))
    dk, dv = float(st[..., 2].max()), float(st[..., 5].max())
    q_norm = float(torch.linalg.vector_norm(run.Q, dim=-1, dtype=torch.float32).max())
    v_norm = float(torch.linalg.vector_norm(run.POOL, dim=-1, dtype=torch.float32).max())
    expo = 2.0 * q_norm * dk * wl.scale
    return {"mean_dk": float(mean[0]), "mean_dk_rel": float(mean[1]), "max_dk": dk, "mean_dv": float(mean[3]),
            "mean_dv_rel": float(mean[4]), "max_dv": dv, "ms": ms_dev,
            "theorem1": {"Q": q_norm, "V": v_norm, "delta_k": dk, "delta_v": dv, "scale": wl.scale, "exponent_2_Q_dk_scale": expo,
                         "rhs": (v_norm * math.expm1(expo) + dv) if expo < 700 else float("inf"),
                         "note": "hard bound for the variant that counts a representative g times (rep_logit_bias = ln g); "
                                 "Algorithm 1 counts it once"}}


def error_vs_dense(O_lca, O_dense, rows, torch):
    """|| O_dense - O_LCA ||_2 per (sequence, sampled row, head): largest, mean, and mean relative to || O_dense ||_2."""
    idx = torch.as_tensor(np.asarray(rows, dtype=np.int64), device=O_lca.device)
    a, b = O_lca[:, idx].float(), O_dense[:, idx].float()
    err, ref = (a - b).norm(dim=-1), b.norm(dim=-1)
    return {"rows": int(idx.numel()), "max": float(err.max()), "mean": float(err.mean()),
            "mean_rel": float((err / ref.clamp_min(1e-20)).mean()), "max_rel": float((err / ref.clamp_min(1e-20)).max())}


def decode_bench(wl, lca, hp, torch, tdt):
    """One decode step of 32 sequences over their condensed caches (HBM-bound). Cache contents are random
    (torch.randn on the device): only the time matters here, parity is covered by the GPU tests."""
    B = 32
    wd = wl.with_(B=B, L=wl.L + 1)
    desc = hp.lca_desc(wd)
    m, k = desc.m, desc.k
    mk = lambda *shape: torch.randn(shape, dtype=tdt, device="cuda")
    caches = [(mk(B, wd.S, m, wd.d_pool), mk(B, wd.S, m, wd.d_sel), mk(B, wd.kv_heads, k, wd.d_pool), mk(B, wd.kv_heads, k, wd.d_sel))
              for _ in range(N_ROT)]
    pool_rep, sel_rep, pool_tail, sel_tail = caches[0]
    q = mk(B, wd.H, wd.d_qk) * 0.1
    O = torch.empty((B, wd.H, wd.d_pool), dtype=tdt, device="cuda")
    wu = wl.with_(B=B, L=wd.w + (m + 1) * wd.g)                     # the next length at which an update is due
    du = hp.lca_desc(wu)
    ws = torch.empty(max(lca.workspace_size(desc), lca.workspace_size(du), 256), dtype=torch.uint8, device="cuda")
    ms = time_kernel(rotating(lambda i: (lambda: lca.decode_attn(desc, q, *caches[i], O, ws))), 21, 3)
    nbytes = B * (wd.S * m + wd.kv_heads * k) * (wd.d_pool + wd.d_sel) * 2
    out = {"B": B, "L": wd.L, "m": m, "k": k, "ms_decode_step": ms, "algorithmic_bytes": nbytes,
           "GBps": nbytes / (ms * 1e-3) / 1e9, "frac_of_hbm_peak": nbytes / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS}
    if (wd.mode == 0 and wd.d_pool == 512 and wd.d_sel == 64) or (wd.mode == 1 and wd.d_pool == 128 and wd.d_sel == 128):
        # the same step over 8-bit representatives (E4M3 codes + row scales; the tail stays 16-bit)
        q8c = [(torch.empty_like(c[0], dtype=torch.uint8), torch.empty_like(c[1], dtype=torch.uint8),
                torch.empty((B, wd.S, m, 2), dtype=torch.float32, device="cuda")) for c in caches]
        out["ms_quantize_cache"] = time_kernel(
            rotating(lambda i: (lambda: lca.quantize_cache(desc, None, caches[i][0], caches[i][1], *q8c[i]))), 9, 3)
        ms8 = time_kernel(rotating(lambda i: (lambda: lca.decode_attn_q8(desc, None, q, *q8c[i], caches[i][2], caches[i][3], O, ws))), 21, 3)
        nb8 = B * (wd.S * m * (wd.d_pool + wd.d_sel + 8) + wd.kv_heads * k * (wd.d_pool + wd.d_sel) * 2)
        out["q8"] = {"ms_decode_step": ms8, "algorithmic_bytes": nb8, "GBps": nb8 / (ms8 * 1e-3) / 1e9,
                     "frac_of_hbm_peak": nb8 / (ms8 * 1e-3) / 1e9 / PEAK_HBM_GBS, "speedup_vs_16bit_cache": ms / ms8,
                     "cache_bytes_per_sequence": wd.S * m * (wd.d_pool + wd.d_sel + 8) + wd.kv_heads * k * (wd.d_pool + wd.d_sel) * 2}
        del q8c
    del caches
    # the same step over a growing cache (spare rows, ring tail that wraps), and the online update that runs every g-th step
    m_cap, k_cap = m + 64, wd.w + wd.g
    lay = lca.CacheLayout(m_cap=m_cap, k_cap=k_cap, k_start=k_cap - 100)
    pool_rep2, sel_rep2 = mk(B, wd.S, m_cap, wd.d_pool), mk(B, wd.S, m_cap, wd.d_sel)
    pool_ring, sel_ring = mk(B, wd.kv_heads, k_cap, wd.d_pool), mk(B, wd.kv_heads, k_cap, wd.d_sel)
    out["ms_decode_step_cached"] = time_kernel(
        lambda: lca.decode_attn_cached(desc, lay, q, pool_rep2, sel_rep2, pool_ring, sel_ring, O, ws), 20, 3)
    q_recent = mk(B, wd.g, wd.H, wd.d_qk) * 0.1
    anchor = torch.zeros((B, wd.S, m_cap), dtype=torch.int32, device="cuda")
    # (two short kernels per call: timed behind a millisecond of fills, or the events would time the host's submissions)
    blocker = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    out["ms_cache_update"] = time_kernel(
        lambda: lca.cache_update(du, lay, q_recent, pool_ring, sel_ring, pool_rep2, sel_rep2, anchor, ws), 20, 3,
        behind=lambda: [blocker.fill_(i) for i in range(4)])
    del blocker
    out["ms_decode_step_amortised"] = out["ms_decode_step_cached"] + out["ms_cache_update"] / wd.g
    return out


def sweep_bench(wl, args, lca, hp, torch, inputs, tdt):
    """Speed and cache size over the method's knobs at the workload's shapes (the paper's ablations of the
    pooling strategy, Table 5; of the group size, the window and the number of summary queries, Table 8 and
    the sensitivity figures): one line per setting with condensation and attention time, tokens/s, the
    attention kernel's rate and the bytes of the emitted cache."""
    Q, POOL, SEL = inputs.gen_all(wl)
    run = hp.GpuRun(wl, Q, POOL, SEL)
    O = torch.empty((wl.B, wl.L, wl.H, wl.d_v), dtype=tdt, device="cuda")
    names = {lca.REDUCE_WEIGHTED: "weighted", lca.REDUCE_MEAN: "mean", lca.REDUCE_MAXSEL: "maxsel", lca.REDUCE_MAXPOOL: "maxpool"}
    settings = [dict(g=g) for g in (4, 8, 16, 32)] + [dict(w=w) for w in (512, 2048, 4096)] + [dict(n_q=n) for n in (8, 32)]
    settings += [dict(pool_reduce=pr, sel_reduce=sr) for pr, sr in ((lca.REDUCE_MEAN, lca.REDUCE_MEAN), (lca.REDUCE_MAXPOOL, lca.REDUCE_MAXPOOL),
                                                                    (lca.REDUCE_MAXSEL, lca.REDUCE_MAXSEL), (lca.REDUCE_WEIGHTED, lca.REDUCE_WEIGHTED))]
    rows = []
    for kw in settings:
        w2 = wl.with_(**{k: v for k, v in kw.items() if k in ("g", "w", "n_q")})
        d2 = hp.lca_desc(w2, **{k: v for k, v in kw.items() if k.endswith("_reduce")})
        pr, sr, an, _ = lca.alloc_condensed(d2)
        ws2 = lca.alloc_workspace(d2)
        mc = time_kernel(lambda: lca.condense(d2, run.Q, run.POOL, run.SEL, pr, sr, an, None, ws2), 10, 2)
        ma = time_kernel(lambda: lca.prefill_attn(d2, run.Q, run.POOL, run.SEL, pr, sr, O, None, ws2), args.steps, 1)
        db, cb = lca.cache_bytes(d2)
        fl = 2.0 * (w2.d_qk + w2.d_v) * w2.B * w2.H * pair_count(w2.L, w2.w, w2.g)
        label = dict(g=w2.g, w=w2.w, n_q=w2.nq, pool=names.get(d2.pool_reduce, "weighted"), sel=names.get(d2.sel_reduce, "maxsel"))
        rows.append({**label, "ms_condense": mc, "ms_attn": ma, "tokens_per_s": w2.B * w2.L / ((mc + ma) * 1e-3),
                     "attn_TFLOPs": fl / (ma * 1e-3) / 1e12, "condense_GBps": condense_bytes(w2, d2.m) / (mc * 1e-3) / 1e9,
                     "kv_cache_bytes_lca": cb, "kv_cache_saved_frac": 1.0 - cb / db})
        del pr, sr, an, ws2
    return rows


def length_bench(wl0, lengths, args, lca, hp, torch, inputs, tdt):
    """The hot path over the sequence length at the workload's other shapes -- the paper's efficiency analysis (section 5.3: the
    kernel's latency against the dense baseline as the context grows, up to a million tokens).  Per length: fresh seeded inputs of
    the same recipe, condensation and attention timed, the dense baseline timed where a launch stays under a second (L <= 128K;
    beyond that the ratio of visible pairs, which is what the speed-up tends to at equal efficiency), the emitted cache's bytes,
    and 32 evenly spaced rows x all heads compared with the oracle."""
    out = []
    for L in lengths:
        wl = wl0.with_(L=L, name=f"{wl0.name.split('+')[0]}+L={L}")
        Q, POOL, SEL = inputs.gen_all(wl)
        run = hp.GpuRun(wl, Q, POOL, SEL)
        d = run.desc
        run.pool_rep, run.sel_rep, run.anchor, _ = lca.alloc_condensed(d)
        O = torch.empty((d.B, d.L, d.H, d.d_pool), dtype=tdt, device="cuda")

        def f_cond():
            lca.condense(d, run.Q, run.POOL, run.SEL, run.pool_rep, run.sel_rep, run.anchor, None, run.ws)

        def f_attn():
            lca.prefill_attn(d, run.Q, run.POOL, run.SEL, run.pool_rep, run.sel_rep, O, None, run.ws)

        f_cond()
        pairs, pairs_dense = pair_count(wl.L, wl.w, wl.g), wl.L * (wl.L + 1) // 2
        flops = 2.0 * (wl.d_qk + wl.d_v) * wl.B * wl.H * pairs
        n_attn = max(2, min(args.steps, int(400e-3 / (flops / 1.2e15))))          # about 0.4 s of attention per length
        ma = time_kernel(f_attn, n_attn, 1)
        mc = time_kernel(f_cond, 10, 2, behind=f_attn)
        row = {"L": L, "m": d.m, "ms_condense": mc, "ms_attn": ma, "tokens_per_s": wl.B * wl.L / ((mc + ma) * 1e-3),
               "attn_TFLOPs": flops / (ma * 1e-3) / 1e12, "attn_frac_of_mfma_peak": flops / (ma * 1e-3) / 1e12 / PEAK_BF16_TFLOPS,
               "dense_over_lca_visible_pairs": pairs_dense / pairs}
        db, cb = lca.cache_bytes(d)
        row["kv_cache_bytes_dense"], row["kv_cache_bytes_lca"], row["kv_cache_saved_frac"] = db, cb, 1.0 - cb / db
        _, rows, O_ref, near_ties = cpu_baseline(wl, Q, POOL, SEL, 32, run.anchor.cpu().numpy(), hp.from_dev(run.sel_rep, wl.dtype))
        O_gpu = hp.from_dev(O[:, rows.tolist()], wl.dtype)
        num = np.abs(O_gpu - O_ref).max(axis=-1)
        row["parity_max_rel_err_sampled_rows"] = float((num / np.maximum(np.abs(O_ref).max(axis=-1), 1e-6)).max())
        row["parity_anchor_near_ties"] = near_ties
        if L <= 131072:
            md = time_kernel(lambda: lca.dense_attn(d, run.Q, run.POOL, run.SEL, O, None, run.ws), 2 if L > 32768 else 5, 1)
            row["ms_dense_mla_attn"], row["speedup_vs_dense_mla"] = md, md / (mc + ma)
        else:
            row["ms_dense_mla_attn"], row["speedup_vs_dense_mla"] = None, None
        print(f"[lengths] L={L}: attention {ma:.3f} ms, condensation {mc * 1e3:.1f} us, parity {row['parity_max_rel_err_sampled_rows']:.2e}",
              file=sys.stderr, flush=True)
        out.append(row)
        del run, O, Q, POOL, SEL, O_gpu, O_ref
        torch.cuda.empty_cache()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", default="cfg4", help="cfg2 | cfg3 | cfg4 (default, the metric's workload) | cfg5 (GQA + decode step)")
    ap.add_argument("--oracle-rows", type=int, default=4096)
    ap.add_argument("--no-extra", action="store_true", help="skip dense baseline and variants (profiling runs)")
    ap.add_argument("--decode-only", action="store_true", help="time only the decode step of 32 sequences over their condensed caches")
    ap.add_argument("--dtype", default="bf16", choices=["bf16", "f16"],
                    help="16-bit element type of the inputs, the cache and the output (the metric is quoted on bf16)")
    ap.add_argument("--set", action="append", default=[], metavar="FIELD=INT",
                    help="override an integer field of the configuration's workload (B, L, H, S, g, w, n_q), e.g. --config cfg5 "
                         "--set H=28 --set S=4 --set L=131072 for the head layout of the GQA model the paper reports on")
    ap.add_argument("--sweep", action="store_true",
                    help="time the prefill over group sizes, windows, numbers of summary queries and pooling strategies instead")
    ap.add_argument("--lengths", default=None, metavar="L1,L2,...",
                    help="time the hot path at these sequence lengths (the workload's other shapes kept) instead of the default run")
    ap.add_argument("--pmc-calib", action="store_true",
                    help="also run one 1 GiB device-to-device copy, the known-size kernel the HBM counters are scaled by")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on ONE GPU; --gpus above 1 is not supported (no collectives in this path)")

    import torch
    from paper_2604_12452_amd import device as hp
    from paper_2604_12452_amd import inputs, lca

    if not torch.cuda.is_available():
        sys.exit("bench.py: no GPU visible")
    lca.load()   # fails loudly when liblca.so is missing
    wl = inputs.configs()[args.config].with_(dtype=args.dtype)
    if args.set:
        over = {k: int(v) for k, v in (kv.split("=") for kv in args.set)}
        assert set(over) <= {"B", "L", "H", "S", "g", "w", "n_q"}, over
        wl = wl.with_(name=wl.name + "+" + ",".join(args.set), **over)
    tdt = torch.bfloat16 if args.dtype == "bf16" else torch.float16
    prof_key = args.config + ("+" + ",".join(sorted(args.set)) if args.set else "")       # a summary exists for few of the overrides
    if args.pmc_calib:
        src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        dst.copy_(src)            # reads 1 GiB, writes 1 GiB
        torch.cuda.synchronize()
        del src, dst
    if args.decode_only:
        dec = decode_bench(wl, lca, hp, torch, tdt)
        dec_kernel = "decode_mla_kernel" if wl.mode == inputs.MODE_MLA else "decode_gqa_mfma_kernel"
        print(json.dumps({"metric": f"LCA decode step over the condensed cache ({wl.name})", "value": dec["ms_decode_step"], "unit": "ms",
                          "n_gpus": 1, "higher_is_better": False, "dtype": args.dtype, "data": "synthetic",
                          "roofline": {"bound": "hbm", "kernel": dec_kernel + " (lca_decode_attn)", "achieved": dec["GBps"], "peak": PEAK_HBM_GBS,
                                       "unit": "GB/s", "frac": dec["frac_of_hbm_peak"],
                                       "traffic": profiled_traffic(prof_key + "/decode", dec_kernel) if args.dtype == "bf16" else None}, "extra": dec}))
        return
    if args.sweep:
        print(json.dumps({"metric": f"LCA prefill over the method's settings ({wl.name} shapes)", "unit": "tokens/s", "n_gpus": 1,
                          "steps": args.steps, "dtype": args.dtype, "data": "synthetic", "sweep": sweep_bench(wl, args, lca, hp, torch, inputs, tdt)}))
        return
    if args.lengths:
        res = length_bench(wl, [int(x) for x in args.lengths.split(",")], args, lca, hp, torch, inputs, tdt)
        tol = 1e-2 if args.dtype == "bf16" else 2e-3
        print(json.dumps({"metric": f"LCA prefill over the sequence length ({wl.name} shapes)", "unit": "tokens/s", "n_gpus": 1, "steps": args.steps,
                          "dtype": args.dtype, "data": "synthetic", "lengths": res}))
        if not all(r["parity_max_rel_err_sampled_rows"] <= tol for r in res):
            sys.exit("bench.py: sampled rows differ from the oracle by more than the tolerance")
        return
    t_gen = time.perf_counter()
    Q, POOL, SEL = inputs.gen_all(wl)
    t_gen = time.perf_counter() - t_gen

    run = hp.GpuRun(wl, Q, POOL, SEL)
    d = run.desc
    mla = wl.mode == inputs.MODE_MLA
    run.pool_rep, run.sel_rep, run.anchor, _ = lca.alloc_condensed(d)
    O = torch.empty((d.B, d.L, d.H, d.d_pool), dtype=tdt, device="cuda")

    def f_cond():
        lca.condense(d, run.Q, run.POOL, run.SEL, run.pool_rep, run.sel_rep, run.anchor, None, run.ws)

    def f_attn():
        lca.prefill_attn(d, run.Q, run.POOL, run.SEL, run.pool_rep, run.sel_rep, O, None, run.ws)

    def step():
        f_cond()
        f_attn()

    # ---- the timed region: W warm-up steps, then exactly K steps between synchronisations ----
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps
    tokens_per_s = wl.B * wl.L / (ms_per_step * 1e-3)

    # ---- per-kernel durations (HIP events on the launch stream) ----
    ms_attn = time_kernel(f_attn, args.steps, 1)
    # (condensation alone, back to back, on rotating copies of its 170 MB of input: in the step above the attention
    # kernel's gigabytes flush the memory-side cache between two condensations anyway)
    rot = [(run.POOL, run.SEL)] + [(run.POOL.clone(), run.SEL.clone()) for _ in range(N_ROT - 1)]
    ms_cond = time_kernel(rotating(lambda i: (lambda: lca.condense(d, run.Q, rot[i][0], rot[i][1], run.pool_rep, run.sel_rep, run.anchor,
                                                                    None, run.ws))), 21, 3, behind=f_attn)
    del rot
    # the same call over a single group (without any group nothing is launched).  At 512 + 64 with one or two sets that is the fixed part of the call above: the same
    # two launches.  With more sets and in the GQA configuration a call of few groups is one launch of another kernel, and the figure is that kernel's
    d_one = hp.lca_desc(wl.with_(w=wl.L - wl.g))
    ws_one, (rep_one, srep_one, anchor_one, _) = lca.alloc_workspace(d_one), lca.alloc_condensed(d_one)
    ms_one = time_kernel(lambda: lca.condense(d_one, run.Q, run.POOL, run.SEL, rep_one, srep_one, anchor_one, None, ws_one), 21, 3, behind=f_attn)
    del ws_one
    pairs = pair_count(wl.L, wl.w, wl.g)
    flops = 2.0 * (wl.d_qk + wl.d_v) * wl.B * wl.H * pairs
    tflops = flops / (ms_attn * 1e-3) / 1e12
    cbytes = condense_bytes(wl, d.m)

    extra = {
        "ms_condense": ms_cond, "ms_attn": ms_attn,
        "condense_algorithmic_bytes": cbytes, "condense_GBps": cbytes / (ms_cond * 1e-3) / 1e9,
        "condense_frac_of_hbm_peak": cbytes / (ms_cond * 1e-3) / 1e9 / PEAK_HBM_GBS,
        "ms_condense_one_group": ms_one,
        "attn_algorithmic_flops": flops, "input_generation_s": t_gen,
    }
    dense_b, cond_b = lca.cache_bytes(d)
    extra["kv_cache_bytes_dense"], extra["kv_cache_bytes_lca"] = dense_b, cond_b
    extra["kv_cache_saved_frac"] = 1.0 - cond_b / dense_b

    # ---- per-token deviations of the emitted cache (Theorem 1's delta_k, delta_v; the statistic of the paper's Tables 9-10) ----
    extra["deviation"] = deviation_report(run, d, wl, torch, lca)
    extra["deviation"]["note"] = f"synthetic AR(1) rho={wl.rho} inputs, not model activations"

    # ---- parity spot-check + CPU baseline on a bounded sample ----
    base, rows, O_ref, near_ties = cpu_baseline(wl, Q, POOL, SEL, args.oracle_rows, run.anchor.cpu().numpy(),
                                                hp.from_dev(run.sel_rep, wl.dtype))
    O_gpu = hp.from_dev(O[:, rows.tolist()], wl.dtype)
    num = np.abs(O_gpu - O_ref).max(axis=-1)
    extra["parity_max_rel_err_sampled_rows"] = float((num / np.maximum(np.abs(O_ref).max(axis=-1), 1e-6)).max())
    extra["parity_anchor_near_ties"] = near_ties    # groups where the GPU took the other of two scores within 1e-3

    if not args.no_extra:
        # context for the MFMA roofline fraction: what the vendor library's plain bf16 GEMM reaches on this chip right now
        # (the chip clocks down under matrix-core load; no part of the product path)
        ga = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
        gb = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
        ms_gemm = time_kernel(lambda: torch.matmul(ga, gb), 10, 2)
        extra["context_library_gemm_bf16_8192_TFLOPs"] = 2.0 * 8192 ** 3 / (ms_gemm * 1e-3) / 1e12
        del ga, gb
        extra["measured_ceilings"] = measured_ceilings(torch, lca, f_attn)
        extra["measured_ceilings"]["attn_frac_of_measured_mfma"] = flops / (ms_attn * 1e-3) / 1e12 / extra["measured_ceilings"]["mfma_bf16_TFLOPs"]
        extra["measured_ceilings"]["condense_call_frac_of_measured_read"] = (
            cbytes / (ms_cond * 1e-3) / 1e12 / extra["measured_ceilings"]["hbm_read_TBps"])
        # in-run dense MLA baseline (same kernel engine, plain causal mask)
        O2 = torch.empty_like(O)
        n_dense = 2 if wl.L > 65536 else 5
        ms_dense = time_kernel(lambda: lca.dense_attn(d, run.Q, run.POOL, run.SEL, O2, None, run.ws), n_dense, 1)
        dflops = 2.0 * (wl.d_qk + wl.d_v) * wl.B * wl.H * (wl.L * (wl.L + 1) // 2)
        extra.update({"ms_dense_mla_attn": ms_dense, "dense_TFLOPs": dflops / (ms_dense * 1e-3) / 1e12,
                      "speedup_vs_dense_mla": ms_dense / ms_per_step, "dense_tokens_per_s": wl.B * wl.L / (ms_dense * 1e-3)})
        # what the condensation costs in accuracy on these inputs: || O_dense - O_LCA ||_2 per (row, head) on the sampled rows,
        # beside the right-hand side of Theorem 1 computed from the deviations measured above
        extra["deviation"]["attention_error_vs_dense"] = error_vs_dense(O, O2, rows, torch)
        if mla:
            # the same report on latents as redundant as the method assumes (section 4.1; the paper measures 2-5 % relative
            # deviations on model activations, appendix Tables 9-10): AR(1) with rho = 0.9999, everything else unchanged
            wr = wl.with_(rho=0.9999)
            kv = inputs.gen_kv_all(wr)
            keep = (run.POOL, run.SEL)
            run.POOL, run.SEL = hp.to_dev(np.stack([p for p, _ in kv]), wl.dtype), hp.to_dev(np.stack([s for _, s in kv]), wl.dtype)
            f_cond()
            f_attn()
            rep = deviation_report(run, d, wr, torch, lca)
            lca.dense_attn(d, run.Q, run.POOL, run.SEL, O2, None, run.ws)
            rep["attention_error_vs_dense"] = error_vs_dense(O, O2, rows, torch)
            rep["note"] = "synthetic AR(1) rho=0.9999 latents (strongly redundant neighbours), same queries and RoPE keys"
            extra["deviation_redundant_latents"] = rep
            run.POOL, run.SEL = keep
            f_cond()
            f_attn()              # O and the cache are the workload's own again
        del O2
        if mla:
            # the value up-projection fused into the attention kernel's epilogue (Eq. 5's W^UV), next to the separate pass it saves:
            # the library's batched GEMM over the stored latent output
            W_up = (torch.randn((wl.H, 128, wl.d_pool), dtype=torch.float32, device="cuda") / wl.d_pool ** 0.5).to(tdt)
            O_up = torch.empty((d.B, d.L, d.H, 128), dtype=tdt, device="cuda")
            ms_up = time_kernel(lambda: lca.prefill_attn_up(d, run.Q, run.POOL, run.SEL, run.pool_rep, run.sel_rep, W_up, O_up, None, run.ws),
                                max(3, args.steps // 2), 1)
            Wt = W_up.transpose(1, 2).contiguous()                                     # [H, d_pool, 128]
            Oh = O.view(d.B * d.L, d.H, wl.d_pool).transpose(0, 1)                     # [H, B L, d_pool], strided view
            ms_proj = time_kernel(lambda: torch.bmm(Oh, Wt), 5, 2)
            extra["fused_up_projection"] = {"ms_attn_up": ms_up, "ms_attn": ms_attn, "ms_separate_projection_library_gemm": ms_proj,
                                            "output_bytes": d.B * d.L * d.H * 128 * 2, "latent_output_bytes": d.B * d.L * d.H * wl.d_pool * 2}
            del W_up, O_up, Wt, Oh
        # variants: g = 32, and one condensed set per head (S = H)
        for tag, kw in ((("g32", dict(g=32)), ("per_head_sets", dict(S=wl.H))) if mla else ()):
            w2 = wl.with_(**kw)
            d2 = hp.lca_desc(w2)
            pr, sr, an, _ = lca.alloc_condensed(d2)
            ws2 = lca.alloc_workspace(d2)
            fc = lambda: lca.condense(d2, run.Q, run.POOL, run.SEL, pr, sr, an, None, ws2)
            fa = lambda: lca.prefill_attn(d2, run.Q, run.POOL, run.SEL, pr, sr, O, None, ws2)
            mc, ma = time_kernel(fc, 10, 2), time_kernel(fa, max(3, args.steps // 2), 1)
            db, cb = lca.cache_bytes(d2)
            fl = 2.0 * (w2.d_qk + w2.d_v) * w2.B * w2.H * pair_count(w2.L, w2.w, w2.g)
            extra[tag] = {"ms_condense": mc, "ms_attn": ma, "tokens_per_s": w2.B * w2.L / ((mc + ma) * 1e-3),
                          "attn_TFLOPs": fl / (ma * 1e-3) / 1e12, "condense_GBps": condense_bytes(w2, d2.m) / (mc * 1e-3) / 1e9,
                          "kv_cache_bytes_lca": cb, "kv_cache_saved_frac": 1.0 - cb / db}
            del pr, sr, an

    if not mla and not args.no_extra:
        extra["decode"] = decode_bench(wl, lca, hp, torch, tdt)

    out = {
        "metric": "LCA prefill tokens/s at 128K (MLA, 16 heads) + speedup vs dense MLA" if args.config == "cfg4"
        else f"LCA prefill tokens/s ({wl.name})",
        "value": tokens_per_s, "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": args.dtype, "data": "synthetic",
        "config": {"workload": (f"{wl.name}: B={wl.B} L={wl.L} H={wl.H} d_c={wl.d_pool} d_R={wl.d_sel} g={wl.g} w={wl.w} "
                                f"S={wl.S} {args.dtype}, AR(1) rho=0.9 latents, RoPE keys, Gaussian queries; one attention layer") if mla else
                               (f"{wl.name}: GQA B={wl.B} L={wl.L} H={wl.H} KV heads={wl.S} d={wl.d_sel} g={wl.g} w={wl.w} {args.dtype}, "
                                f"AR(1) keys/values, RoPE theta {wl.theta:g}; one attention layer"),
                   "step": "lca_condense + lca_prefill_attn"},
        "roofline": {"bound": "mfma", "kernel": ("attn_mla_kernel" if mla else "attn_gqa64_kernel") + " (lca_prefill_attn)", "achieved": tflops,
                     "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s", "frac": tflops / PEAK_BF16_TFLOPS,
                     "traffic": profiled_traffic(prof_key, "attn_mla_kernel" if mla else "attn_gqa64_kernel") if args.dtype == "bf16" else None},
        "cpu_baseline": base,
        "extra": extra,
    }
    print(json.dumps(out))
    tol = {"bf16": 1e-2, "f16": 2e-3}[args.dtype]
    if not extra["parity_max_rel_err_sampled_rows"] <= tol:
        sys.exit(f"bench.py: the sampled rows differ from the oracle by {extra['parity_max_rel_err_sampled_rows']:.3e} "
                 f"(allowed {tol:g}): the numbers above are not valid")


if __name__ == "__main__":
    main()

// One query row of the attention by one wavefront, entry by entry, in fp32: any widths, any scale, and no arithmetic on an
// entry the row does not see.  The kernel of attn_simple.hip is this and nothing else; the tiled kernel of attn_tile.hip
// comes back to it for rows whose result is not finite.
//
// Row t attends representatives j < m_t and raw tokens m_t*g <= i <= t (section 4.3, Eq. 10 with the
// per-query partition of appendix A.2), or every token i <= t in dense mode (section 3, Eq. 5).
#pragma once
#include "lca_internal.h"

namespace lca {
namespace attn_row {

constexpr int WAVE = 64;
constexpr int MAXD = 1024;   // largest d_qk / d_v handled (validated by the API)

template <typename T> __device__ __forceinline__ float ldf(const T *p);
template <> __device__ __forceinline__ float ldf<uint16_t>(const uint16_t *p) { return __uint_as_float(((uint32_t)*p) << 16); }
template <> __device__ __forceinline__ float ldf<f16_t>(const f16_t *p) { return f16_bits_to_float(p->bits); }
template <> __device__ __forceinline__ float ldf<float>(const float *p) { return *p; }

template <typename T> __device__ __forceinline__ void stf(T *p, float v);
template <> __device__ __forceinline__ void stf<uint16_t>(uint16_t *p, float v)
{
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    *p = (uint16_t)(u >> 16);
}
template <> __device__ __forceinline__ void stf<f16_t>(f16_t *p, float v) { p->bits = float_to_f16_bits(v); }
template <> __device__ __forceinline__ void stf<float>(float *p, float v) { *p = v; }

template <typename T> struct RowParams {
    const T *Q, *POOL, *SEL, *pool_rep, *sel_rep;
    T *O;
    float *lse;
    int L, H, S, P, d_pool, d_sel, mla, g, w, m, dense;
    float scale, rep_bias;
};

template <typename T> RowParams<T> row_params(const AttnArgs &a)
{
    const Dims &d = a.d;
    return RowParams<T>{(const T *)a.Q, (const T *)a.POOL, (const T *)a.SEL, (const T *)a.pool_rep, (const T *)a.sel_rep, (T *)a.O, a.lse,
                        d.L, d.H, d.S, d.P, d.d_pool, d.d_sel, d.mode == LCA_MODE_MLA, d.g, d.w, d.m, a.dense, d.scale, d.rep_logit_bias};
}

// LDS of the calling wavefront: q_s[d_qk] and p_s[64].  row = ((b * L) + t) * H + h.  NCOL: output columns a lane holds, >= d_pool / 64.
template <typename T, int NCOL>
__device__ __forceinline__ void attend_row(const RowParams<T> &k, long row, float *q_s, float *p_s, int lane)
{
    const int h = (int)(row % k.H), t = (int)((row / k.H) % k.L), b = (int)(row / ((long)k.H * k.L));
    const int s = h / (k.H / k.S), p = k.mla ? 0 : s;
    const int d_pool = k.d_pool, d_sel = k.d_sel, d_qk = k.mla ? d_pool + d_sel : d_sel;
    const int NV = (d_pool + WAVE - 1) / WAVE;   // output columns per lane (<= NCOL)

    __builtin_amdgcn_wave_barrier();
    for (int x = lane; x < d_qk; x += WAVE) q_s[x] = ldf(k.Q + (size_t)row * d_qk + x);
    __builtin_amdgcn_wave_barrier();

    const int mt = (k.dense || t + 1 <= k.w) ? 0 : (t + 1 - k.w) / k.g;     // visible representatives
    const int n_raw = t + 1 - mt * k.g;
    const int n = mt + n_raw;

    float acc[NCOL];
#pragma unroll
    for (int i = 0; i < NCOL; ++i) acc[i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    for (int e0 = 0; e0 < n; e0 += WAVE) {
        const int e = e0 + lane;
        float logit = -INFINITY;
        const T *vrow = nullptr;
        if (e < n) {
            const T *prow, *srow;
            float bias = 0.f;
            if (e < mt) {
                const size_t r = ((size_t)b * k.S + s) * k.m + e;
                prow = k.pool_rep + r * d_pool;
                srow = k.sel_rep + r * d_sel;
                bias = k.rep_bias;
            } else {
                const size_t i = (size_t)(mt * k.g + (e - mt));
                prow = k.POOL + (((size_t)b * k.L + i) * k.P + p) * d_pool;
                srow = k.SEL + (((size_t)b * k.L + i) * k.P + p) * d_sel;
            }
            float a = 0.f;
            if (k.mla)
                for (int x = 0; x < d_pool; ++x) a = fmaf(q_s[x], ldf(prow + x), a);
            const int qoff = k.mla ? d_pool : 0;
            for (int x = 0; x < d_sel; ++x) a = fmaf(q_s[qoff + x], ldf(srow + x), a);
            logit = k.scale * a + bias;
            vrow = prow;
        }
        float cmax = logit;
        for (int mask = 32; mask >= 1; mask >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, mask, WAVE));
        const float m_new = fmaxf(m_run, cmax);         // finite: every chunk holds at least one entry
        const float corr = __expf(m_run - m_new);
        const float pe = e < n ? __expf(logit - m_new) : 0.f;
        float psum = pe;
        for (int mask = 32; mask >= 1; mask >>= 1) psum += __shfl_xor(psum, mask, WAVE);
        l_run = l_run * corr + psum;
        m_run = m_new;
        __builtin_amdgcn_wave_barrier();
        p_s[lane] = pe;
        __builtin_amdgcn_wave_barrier();
        const int cnt = min(WAVE, n - e0);
#pragma unroll
        for (int i = 0; i < NCOL; ++i) acc[i] *= corr;
        for (int c = 0; c < cnt; ++c) {
            const unsigned long long vaddr = __shfl((unsigned long long)vrow, c, WAVE);
            const T *vr = reinterpret_cast<const T *>(vaddr);
            const float pc = p_s[c];
#pragma unroll
            for (int i = 0; i < NCOL; ++i) {
                const int x = i * WAVE + lane;
                if (i < NV && x < d_pool) acc[i] = fmaf(pc, ldf(vr + x), acc[i]);
            }
        }
    }
    const float inv = 1.f / l_run;
#pragma unroll
    for (int i = 0; i < NCOL; ++i) {
        const int x = i * WAVE + lane;
        if (i < NV && x < d_pool) stf(k.O + (size_t)row * d_pool + x, acc[i] * inv);
    }
    if (k.lse != nullptr && lane == 0) k.lse[row] = m_run + __logf(l_run);
}

}  // namespace attn_row
}  // namespace lca

// Online cache update during decoding (section 4.3 of the paper, "Decoding and Online Cache Update"): the g
// oldest raw tokens of the tail ring are condensed into one more representative — importance scores against
// the mean query of the last n_q tokens (Eq. 6), softmax-weighted pooling of the pooled component (Eq. 7),
// the selected component copied from the arg-max token (Eq. 8; lowest index on ties).
//
// g rows of at most 2 KB each: the step is bound by launch latency, one round trip to memory and the instructions of the
// wavefronts that work on the group (one wavefront alone issues for 8 us at 16 rows of 512 + 64), not by bandwidth, and runs
// once every g decode steps.  So a workgroup of eight wavefronts shares a group's rows (cache_update_wide_kernel), and
// where 16 chunks of 16 bytes hold a summary query the same launch computes it; wider ones (MLA: 295 KB of queries) keep the
// condensation's summary_query_kernel, whose workgroups share them.  The call, back to back in a graph, before (summary kernel,
// then one wavefront per group) / now: 28 heads over 4 KV heads 128 + 128, five sequences 8.8 / 6.0 us, g = 32 12.4 / 7.8 us;
// 16 heads, one set, 512 + 64 13.4 / 8.6 us at one sequence, 13.9 / 9.2 us at 32, g = 32 32.8 / 10.9 us.
// The summary query inside at 512 + 64 (five blocks of chunks one after another): 16.2 us with one wavefront per group.
// Rows of more than 128 pieces do not fit two pieces per lane: cache_update_rows_kernel.  (One wavefront per (sequence, set)
// that reads its rows again took longer: the call at fp32 512 + 64, one sequence, g = 4 / 16 / 64:
// 10.7 / 22.5 / 73.5 us so, 8.0 / 13.1 / 35.6 us by four.)
#include "group_rows.h"

namespace lca {
namespace {

using namespace group_rows;

struct UpdParams {
    const float *qbar;
    const void *pool_tail, *sel_tail;
    void *pool_rep, *sel_rep;
    int32_t *anchor;
    int S, d_pool, d_sel, g, m, mla, m_cap, k_cap, k_start;
    float scale;
};

// Four wavefronts per (sequence, set), any widths: the wavefronts split the g rows for the scores, the threads split the columns for the
// pooled row; every row is read again for it (from the caches), with as many loads in flight as there are rows.
// dynamic LDS: qbar[d_qk] then score[g]
constexpr int ROWS_THREADS = 256;
template <typename T>
__global__ __launch_bounds__(ROWS_THREADS) void cache_update_rows_kernel(const UpdParams kp)
{
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE, bs = blockIdx.x;
    const int d_pool = kp.d_pool, d_sel = kp.d_sel, mla = kp.mla, g = kp.g, d_qk = mla ? d_pool + d_sel : d_sel;
    float *const qbar = lds, *const score = lds + d_qk;
    for (int col = tid; col < d_qk; col += ROWS_THREADS) qbar[col] = kp.qbar[(size_t)bs * d_qk + col];
    __syncthreads();

    auto ring_row = [&](int i) { const int r = kp.k_start + i; return r >= kp.k_cap ? r - kp.k_cap : r; };
    const size_t src = mla ? bs / kp.S : bs;                 // (sequence, KV head) whose ring is read
    const T *const pool = (const T *)kp.pool_tail + src * kp.k_cap * d_pool, *const sel = (const T *)kp.sel_tail + src * kp.k_cap * d_sel;

    // scores of the g oldest tail tokens: key = [pooled ; selected] (MLA, absorbed form) or the selected component (GQA)
    for (int i = wave; i < g; i += ROWS_THREADS / WAVE) {
        const int r = ring_row(i);
        float a = 0.f;
        if (mla)
            for (int col = lane; col < d_pool; col += WAVE) a += qbar[col] * Elt<T>::ld(pool + (size_t)r * d_pool + col);
        for (int col = lane; col < d_sel; col += WAVE) a += qbar[(mla ? d_pool : 0) + col] * Elt<T>::ld(sel + (size_t)r * d_sel + col);
        a = lanes::over_group<WAVE>(a, lanes::Sum());
        if (lane == 0) score[i] = a * kp.scale;
    }
    __syncthreads();

    // group softmax and arg-max (every thread redundantly: g <= 64 values; a score that is not a number is never the largest)
    float mx = -INFINITY;
    int best = 0;
    for (int i = 0; i < g; ++i)
        if (score[i] > mx) { mx = score[i]; best = i; }
    float z = 0.f;
    for (int i = 0; i < g; ++i) z += __expf(score[i] - mx);
    const float inv_z = 1.f / z;

    // pooled component: softmax-weighted sum; selected component: the arg-max token's, copied
    const size_t unit = (size_t)bs * kp.m_cap + (kp.m - 1);
    for (int col = tid; col < d_pool; col += ROWS_THREADS) {
        float a = 0.f;
        for (int i = 0; i < g; ++i) a += __expf(score[i] - mx) * inv_z * Elt<T>::ld(pool + (size_t)ring_row(i) * d_pool + col);
        Elt<T>::st((T *)kp.pool_rep + unit * d_pool + col, a);
    }
    const T *const from = sel + (size_t)ring_row(best) * d_sel;
    for (int col = tid; col < d_sel; col += ROWS_THREADS) ((T *)kp.sel_rep)[unit * d_sel + col] = from[col];
    if (kp.anchor != nullptr && tid == 0) kp.anchor[unit] = (kp.m - 1) * g + best;
}

// Eight wavefronts, for rows of up to 128 16-byte pieces (both components): wavefront w holds rows w, w + 8, .. of
// the group whole, piece l and l + 64 in lane l, all requested at once; it scores its rows, every wavefront then evaluates the
// softmax, and the weighted rows are added up over the wavefronts in LDS.  SUMMARY: the summary query is computed here too, by
// the whole workgroup, while the rows are on their way.  UPD_ROWS: rows of a wavefront, g / 8 rounded up to 2 or 8.
constexpr int UPD_WAVES = 8, UPD_PIECES = 2 * WAVE;
struct WideParams {
    UpdParams u;
    const void *q_recent;
    int H, n_q;
};
template <typename T, bool SUMMARY, int UPD_ROWS>
__global__ __launch_bounds__(UPD_WAVES *WAVE) void cache_update_wide_kernel(const WideParams wp)
{
    constexpr int EPC = Elt<T>::EPC;
    const UpdParams &kp = wp.u;
    __shared__ SummaryPart<T, UPD_WAVES> part;
    __shared__ float summary[SUMMARY ? SQ_CHUNKS * EPC : 1];
    __shared__ float score[WAVE];
    __shared__ __attribute__((aligned(16))) float sums[UPD_WAVES][UPD_PIECES * EPC];
    const int lane = threadIdx.x & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), bs = blockIdx.x;
    const int d_pool = kp.d_pool, d_sel = kp.d_sel, mla = kp.mla, g = kp.g, d_qk = mla ? d_pool + d_sel : d_sel;
    const int n_pool = d_pool / EPC, n_all = n_pool + d_sel / EPC;
    const size_t src = mla ? bs / kp.S : bs;                 // (sequence, KV head) whose ring is read
    const T *const pool = (const T *)kp.pool_tail + src * kp.k_cap * d_pool, *const sel = (const T *)kp.sel_tail + src * kp.k_cap * d_sel;

    uintx4 held[UPD_ROWS][2];
#pragma unroll
    for (int i = 0; i < UPD_ROWS; ++i) {
        const int row = wave + i * UPD_WAVES;
        int r = kp.k_start + row;
        r = r >= kp.k_cap ? r - kp.k_cap : r;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = lane + j * WAVE;
            held[i][j] = uintx4{0, 0, 0, 0};
            if (row < g && c < n_all) {
                const T *p = c < n_pool ? pool + (size_t)r * d_pool + c * EPC : sel + (size_t)r * d_sel + (c - n_pool) * EPC;
                held[i][j] = *reinterpret_cast<const uintx4 *>(p);
            }
        }
    }

    const float *qb = kp.qbar + (size_t)bs * d_qk;
    if constexpr (SUMMARY) {
        const int hps = wp.H / kp.S;
        const T *const rows = (const T *)wp.q_recent + ((size_t)(bs / kp.S) * wp.n_q * wp.H + (size_t)(bs % kp.S) * hps) * d_qk;
        summary_columns<UPD_WAVES>(rows, wp.H, hps, d_qk, wp.n_q, 0, part, summary);
        __syncthreads();
        qb = summary;
    }
    // scores (Eq. 6): the pieces that are keys, against theirs of the summary query
    float a[UPD_ROWS];
#pragma unroll
    for (int i = 0; i < UPD_ROWS; ++i) a[i] = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = lane + j * WAVE, col = mla ? c * EPC : (c - n_pool) * EPC;
        if (c < n_all && col >= 0) {
            float q[EPC], f[EPC];
#pragma unroll
            for (int e = 0; e < EPC; ++e) q[e] = qb[col + e];
#pragma unroll
            for (int i = 0; i < UPD_ROWS; ++i) {
                unpack4<T>(held[i][j], f);
#pragma unroll
                for (int e = 0; e < EPC; ++e) a[i] = fmaf(f[e], q[e], a[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < UPD_ROWS; ++i)
        if (i * UPD_WAVES < g) a[i] = lanes::over_group<WAVE>(a[i], lanes::Sum());
#pragma unroll
    for (int i = 0; i < UPD_ROWS; ++i)
        if (lane == 0) score[wave + i * UPD_WAVES] = a[i];
    __syncthreads();
    const float mine = lane < g ? kp.scale * score[lane] : -INFINITY;       // lane r: the score of row r
    float bmax;
    // (a score that is not a number anchors nothing; it does reach the weights, and through them the whole pooled row)
    const int best = wave_argmax(mine == mine ? mine : -INFINITY, g, &bmax);
    const float p = lane < g ? __expf(mine - bmax) : 0.f;
    const float alpha = p / lanes::over_group<WAVE>(p, lanes::Sum());

    // pooled component: the weighted rows (Eq. 7), this wavefront's first, then over the wavefronts
    const size_t unit = (size_t)bs * kp.m_cap + (kp.m - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = lane + j * WAVE;
        float acc[EPC], f[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
#pragma unroll
        for (int i = 0; i < UPD_ROWS; ++i) {
            const int row = wave + i * UPD_WAVES;
            if (row < g) {
                const float w = readlane_f(alpha, row);
                unpack4<T>(held[i][j], f);
#pragma unroll
                for (int e = 0; e < EPC; ++e) acc[e] = fmaf(w, f[e], acc[e]);
            }
        }
        if (c < n_pool) {
#pragma unroll
            for (int e = 0; e < EPC; e += 4) *reinterpret_cast<float4 *>(&sums[wave][c * EPC + e]) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
        }
    }
    // selected component: the anchor's row (Eq. 8), from the wavefront that holds it
    if (wave == best % UPD_WAVES) {
#pragma unroll
        for (int i = 0; i < UPD_ROWS; ++i)
            if (i == best / UPD_WAVES) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int c = lane + j * WAVE - n_pool;
                    if (c >= 0 && c < n_all - n_pool) *reinterpret_cast<uintx4 *>((T *)kp.sel_rep + unit * d_sel + c * EPC) = held[i][j];
                }
            }
        if (kp.anchor != nullptr && lane == 0) kp.anchor[unit] = (kp.m - 1) * g + best;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < n_pool; c += UPD_WAVES * WAVE) {
        float acc[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = sums[0][c * EPC + e];
#pragma unroll
        for (int w = 1; w < UPD_WAVES; ++w)
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] += sums[w][c * EPC + e];
        *reinterpret_cast<uintx4 *>((T *)kp.pool_rep + unit * d_pool + c * EPC) = pack4<T>(acc);
    }
}

template <typename T>
hipError_t run(const UpdateArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    const UpdParams kp{a.qbar, a.pool_tail, a.sel_tail, a.pool_rep, a.sel_rep, a.anchor, d.S, d.d_pool, d.d_sel, d.g, d.m,
                       d.mode == LCA_MODE_MLA ? 1 : 0, a.m_cap, a.k_cap, a.k_start, d.scale};
    const bool wide = (d.d_pool + d.d_sel) / Elt<T>::EPC <= UPD_PIECES, summary = wide && d.d_qk <= SQ_CHUNKS * Elt<T>::EPC;
    const WideParams wp{kp, a.q_recent, d.H, d.n_q};
    const unsigned grid = d.B * d.S;
    if (!summary) {
        // the n_q recent queries are, to the summary-query kernel, a sequence of n_q tokens of which it averages the last n_q
        const hipError_t e = launch_summary_query(d, a.q_recent, d.n_q, a.qbar, st);
        if (e != hipSuccess) return e;
    }
    if (wide) {
        const bool few = d.g <= 2 * UPD_WAVES;
        if (summary && few) cache_update_wide_kernel<T, true, 2><<<grid, UPD_WAVES * WAVE, 0, st>>>(wp);
        else if (summary) cache_update_wide_kernel<T, true, 8><<<grid, UPD_WAVES * WAVE, 0, st>>>(wp);
        else if (few) cache_update_wide_kernel<T, false, 2><<<grid, UPD_WAVES * WAVE, 0, st>>>(wp);
        else cache_update_wide_kernel<T, false, 8><<<grid, UPD_WAVES * WAVE, 0, st>>>(wp);
        return hipGetLastError();
    }
    cache_update_rows_kernel<T><<<grid, ROWS_THREADS, (size_t)(d.d_qk + d.g) * sizeof(float), st>>>(kp);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_cache_update(const UpdateArgs &a, hipStream_t st)
{
    return a.d.dtype == LCA_BF16 ? run<uint16_t>(a, st) : a.d.dtype == LCA_F16 ? run<f16_t>(a, st) : run<float>(a, st);
}

}  // namespace lca

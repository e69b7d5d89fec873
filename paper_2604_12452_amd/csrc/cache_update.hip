// Online cache update during decoding (section 4.3 of the paper, "Decoding and Online Cache Update"): the g
// oldest raw tokens of the tail ring are condensed into one more representative — importance scores against
// the mean query of the last n_q tokens (Eq. 6), softmax-weighted pooling of the pooled component (Eq. 7),
// the selected component copied from the arg-max token (Eq. 8; lowest index on ties).
//
// The summary query comes from the condensation's own summary_query_kernel (the g recent queries are a
// sequence of length n_q to it).  Then one wavefront per (sequence, set) does what the any-width condensation does with a
// group (group_rows.h), its rows being rows of the ring.  g rows of at most 2 KB each — the step is bound by launch latency and
// one round trip to memory, not by bandwidth, and runs once every g decode steps; one wavefront per workgroup, so that
// the few there are sit on CUs of their own.  The call: 16.5 -> 13.6 us at
// one sequence and 22.2 -> 14.8 us at 32 (512 + 64, 16 heads), 11.1 -> 9.0 us at five (28 heads over 4 KV heads), scalar loads before.
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

template <typename T>
__global__ __launch_bounds__(WAVE) void cache_update_kernel(const UpdParams kp)
{
    constexpr int EPC = Elt<T>::EPC;
    __shared__ float per_row[2][WAVE];
    const int lane = threadIdx.x, bs = blockIdx.x, d_pool = kp.d_pool, d_sel = kp.d_sel, mla = kp.mla;
    const size_t src = mla ? bs / kp.S : bs;                 // (sequence, KV head) whose ring is read
    Rows<T, 16> pool;
    Rows<T, 4> sel;
    pool.init((const T *)kp.pool_tail + src * kp.k_cap * d_pool, d_pool, d_pool / EPC, kp.g, lane, kp.k_start, kp.k_cap);
    sel.init((const T *)kp.sel_tail + src * kp.k_cap * d_sel, d_sel, d_sel / EPC, kp.g, lane, kp.k_start, kp.k_cap);
    pool.request();
    sel.request();
    const size_t unit = (size_t)bs * kp.m_cap + (kp.m - 1);
    condense_group<T>(pool, sel, kp.qbar + (size_t)bs * (mla ? d_pool + d_sel : d_sel), mla, d_pool, kp.g, kp.scale, LCA_REDUCE_WEIGHTED,
                      LCA_REDUCE_MAXSEL, (T *)kp.pool_rep + unit * d_pool, (T *)kp.sel_rep + unit * d_sel,
                      kp.anchor != nullptr ? kp.anchor + unit : nullptr, (kp.m - 1) * kp.g, nullptr, per_row[0], per_row[1], lane);
}

template <typename T>
hipError_t run(const UpdateArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    const UpdParams kp{a.qbar, a.pool_tail, a.sel_tail, a.pool_rep, a.sel_rep, a.anchor, d.S, d.d_pool, d.d_sel, d.g, d.m,
                       d.mode == LCA_MODE_MLA ? 1 : 0, a.m_cap, a.k_cap, a.k_start, d.scale};
    cache_update_kernel<T><<<d.B * d.S, WAVE, 0, st>>>(kp);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_cache_update(const UpdateArgs &a, hipStream_t st)
{
    // the n_q recent queries are, to the summary-query kernel, a sequence of n_q tokens of which it averages the last n_q
    const hipError_t e = launch_summary_query(a.d, a.q_recent, a.d.n_q, a.qbar, st);
    if (e != hipSuccess) return e;
    return a.d.dtype == LCA_BF16 ? run<uint16_t>(a, st) : a.d.dtype == LCA_F16 ? run<f16_t>(a, st) : run<float>(a, st);
}

}  // namespace lca

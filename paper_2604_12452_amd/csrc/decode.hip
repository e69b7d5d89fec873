// Decode step over a condensed cache (section 4.3, decoding paragraph): one new query per sequence
// and head attends the m representatives and the k raw tail rows.  HBM-bound: every cache byte is
// read once with 16-byte coalesced loads; the query heads of a set share the rows they read.
//
//   decode_split_kernel   one workgroup per (sequence, set, split of the entries): LPR lanes per row,
//                         64/LPR rows per wavefront step, online softmax per lane group, then one
//                         merge per workgroup; writes (max, sum, unnormalised output) partials.
//   decode_merge_kernel   merges the splits and writes O.
// The MLA and GQA layer widths have matrix-core kernels of their own (decode_mla.hip, decode_gqa_mfma.hip), which
// share the merge kernel; decode_split_kernel serves the other instantiated shapes.
#include "lanes.h"
#include "lca_internal.h"

namespace lca {
namespace {

constexpr int WAVE = 64;
constexpr int NWAVE = 4;
constexpr int TARGET_BLOCKS = 2048;   // ~8 workgroups per CU

template <typename T> struct DElt;
template <> struct DElt<uint16_t> {
    static constexpr int EPC = 8;
    __device__ static float ld(const uint16_t *p) { return __uint_as_float(((uint32_t)*p) << 16); }
    __device__ static void unpack(const uint4 &c, float *f)
    {
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    __device__ static void st(uint16_t *p, float v)
    {
        uint32_t u = __float_as_uint(v);
        u += 0x7FFFu + ((u >> 16) & 1u);
        *p = (uint16_t)(u >> 16);
    }
};
template <> struct DElt<f16_t> {
    static constexpr int EPC = 8;
    __device__ static float ld(const f16_t *p) { return f16_bits_to_float(p->bits); }
    __device__ static void unpack(const uint4 &c, float *f)
    {
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = f16_bits_to_float((uint16_t)w[i]);
            f[2 * i + 1] = f16_bits_to_float((uint16_t)(w[i] >> 16));
        }
    }
    __device__ static void st(f16_t *p, float v) { p->bits = float_to_f16_bits(v); }
};
template <> struct DElt<float> {
    static constexpr int EPC = 4;
    __device__ static float ld(const float *p) { return *p; }
    __device__ static void unpack(const uint4 &c, float *f)
    {
        f[0] = __uint_as_float(c.x); f[1] = __uint_as_float(c.y); f[2] = __uint_as_float(c.z); f[3] = __uint_as_float(c.w);
    }
    __device__ static void st(float *p, float v) { *p = v; }
};

constexpr int pow2_at_least(int x) { int p = 1; while (p < x) p <<= 1; return p; }

// partial layout in the workspace: [B][S][splits][HPS][DP + 2] floats = (max, sum, acc[DP])
template <typename T, int DP, int DS, bool MLA, int HPS>
__global__ __launch_bounds__(WAVE *NWAVE) void decode_split_kernel(const T *__restrict__ q, const T *__restrict__ pool_rep,
                                                                   const T *__restrict__ sel_rep, const T *__restrict__ pool_tail,
                                                                   const T *__restrict__ sel_tail, float *__restrict__ part, int S, int P,
                                                                   int m, int k, int splits, float scale, float rep_bias, int m_cap,
                                                                   int k_cap, int k_start)
{
    constexpr int EPC = DElt<T>::EPC;
    constexpr int DQK = MLA ? DP + DS : DS;
    constexpr int NCP = DP / EPC, NCS = DS / EPC;
    constexpr int NROW = NCP + NCS;                       // chunks of a [pool | sel] row
    constexpr int LPR = pow2_at_least(NROW) > WAVE ? WAVE : pow2_at_least(NROW);   // lanes per row
    constexpr int RPW = WAVE / LPR;                       // rows per wavefront step
    constexpr int NSLOT = (NROW + LPR - 1) / LPR;
    constexpr int H = HPS;

    __shared__ __attribute__((aligned(16))) T q_s[H * DQK];
    __shared__ float comb[H * (DP + 2)];

    const int tid = threadIdx.x, wave = tid / WAVE, lane = tid % WAVE, sub = lane % LPR, grp = lane / LPR;
    const int split = blockIdx.x % splits, s = (blockIdx.x / splits) % S, b = blockIdx.x / (splits * S);
    const int p = MLA ? 0 : s;
    const int n = m + k;
    const int per = (n + splits - 1) / splits;
    const int e_lo = split * per, e_hi = min(n, e_lo + per);

    for (int x = tid; x < H * DQK; x += WAVE * NWAVE) q_s[x] = q[((size_t)b * S + s) * H * DQK + x];   // heads of set s are contiguous
    __syncthreads();

    bool is_pool[NSLOT], is_sel[NSLOT];
    int col[NSLOT];
#pragma unroll
    for (int sl = 0; sl < NSLOT; ++sl) {
        const int c = sl * LPR + sub;
        is_pool[sl] = c < NCP;
        is_sel[sl] = c >= NCP && c < NROW;
        col[sl] = is_pool[sl] ? c * EPC : (c - NCP) * EPC;
    }

    float mr[H], lr[H], acc[H][NSLOT][EPC];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        mr[h] = -INFINITY;
        lr[h] = 0.f;
#pragma unroll
        for (int sl = 0; sl < NSLOT; ++sl)
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[h][sl][e] = 0.f;
    }

    for (int base = e_lo + wave * RPW; base < e_hi; base += NWAVE * RPW) {
        const int e = base + grp;
        const bool valid = e < e_hi;
        const int ec = valid ? e : e_hi - 1;
        const T *prow, *srow;
        if (ec < m) {
            prow = pool_rep + (((size_t)b * S + s) * m_cap + ec) * DP;
            srow = sel_rep + (((size_t)b * S + s) * m_cap + ec) * DS;
        } else {
            int r = k_start + (ec - m);                         // the tail is a ring of k_cap rows
            r = r >= k_cap ? r - k_cap : r;
            prow = pool_tail + (((size_t)b * P + p) * k_cap + r) * DP;
            srow = sel_tail + (((size_t)b * P + p) * k_cap + r) * DS;
        }
        uint4 data[NSLOT];
#pragma unroll
        for (int sl = 0; sl < NSLOT; ++sl) {
            data[sl] = make_uint4(0, 0, 0, 0);
            if (is_pool[sl]) data[sl] = *reinterpret_cast<const uint4 *>(prow + col[sl]);
            else if (is_sel[sl]) data[sl] = *reinterpret_cast<const uint4 *>(srow + col[sl]);
        }
        float f[NSLOT][EPC];
#pragma unroll
        for (int sl = 0; sl < NSLOT; ++sl) DElt<T>::unpack(data[sl], f[sl]);
        float dot[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            float a = 0.f;
#pragma unroll
            for (int sl = 0; sl < NSLOT; ++sl) {
                const bool used = MLA ? (is_pool[sl] || is_sel[sl]) : is_sel[sl];
                if (used) {
                    const int qoff = is_pool[sl] ? col[sl] : (MLA ? DP + col[sl] : col[sl]);
#pragma unroll
                    for (int x = 0; x < EPC; ++x) a = fmaf(f[sl][x], DElt<T>::ld(&q_s[h * DQK + qoff + x]), a);
                }
            }
#pragma unroll
            for (int mask = LPR / 2; mask >= 1; mask >>= 1) a += __shfl_xor(a, mask, WAVE);
            dot[h] = a;
        }
        const float bias = ec < m ? rep_bias : 0.f;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const float logit = valid ? fmaf(dot[h], scale, bias) : -INFINITY;
            const float m_new = fmaxf(mr[h], logit);
            const float m_eff = m_new == -INFINITY ? 0.f : m_new;
            const float corr = __expf(mr[h] - m_eff);
            const float pe = __expf(logit - m_eff);
            lr[h] = lr[h] * corr + pe;
            mr[h] = m_new;
#pragma unroll
            for (int sl = 0; sl < NSLOT; ++sl)
                if (sl * LPR < NCP) {
#pragma unroll
                    for (int x = 0; x < EPC; ++x) acc[h][sl][x] = fmaf(pe, f[sl][x], acc[h][sl][x] * corr);
                }
        }
    }

    // merge the lane groups of this wavefront (they hold the same columns for different rows)
#pragma unroll
    for (int h = 0; h < H; ++h) {
#pragma unroll
        for (int mask = LPR; mask < WAVE; mask <<= 1) {
            const float om = __shfl_xor(mr[h], mask, WAVE), ol = __shfl_xor(lr[h], mask, WAVE);
            const float m_new = fmaxf(mr[h], om);
            const float m_eff = m_new == -INFINITY ? 0.f : m_new;
            const float ca = __expf(mr[h] - m_eff), cb = __expf(om - m_eff);
            lr[h] = lr[h] * ca + ol * cb;
#pragma unroll
            for (int sl = 0; sl < NSLOT; ++sl)
                if (sl * LPR < NCP) {
#pragma unroll
                    for (int x = 0; x < EPC; ++x) acc[h][sl][x] = acc[h][sl][x] * ca + __shfl_xor(acc[h][sl][x], mask, WAVE) * cb;
                }
            mr[h] = m_new;
        }
    }
    // merge the wavefronts one after another through LDS
    for (int wv = 0; wv < NWAVE; ++wv) {
        if (wave == wv && grp == 0) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                float *cm = comb + h * (DP + 2);
                float ca = 1.f, cb = 0.f, m_new = mr[h], l_new = lr[h];
                if (wv > 0) {
                    const float om = cm[0], ol = cm[1];
                    m_new = fmaxf(mr[h], om);
                    const float m_eff = m_new == -INFINITY ? 0.f : m_new;
                    ca = __expf(mr[h] - m_eff);
                    cb = __expf(om - m_eff);
                    l_new = lr[h] * ca + ol * cb;
                }
#pragma unroll
                for (int sl = 0; sl < NSLOT; ++sl)
                    if (sl * LPR < NCP && is_pool[sl]) {
#pragma unroll
                        for (int x = 0; x < EPC; ++x) {
                            float *dst = cm + 2 + col[sl] + x;
                            *dst = acc[h][sl][x] * ca + (wv > 0 ? *dst * cb : 0.f);
                        }
                    }
                // every lane of the group computed the same (m_new, l_new); write after all lanes have read cm[0..1]
                __builtin_amdgcn_wave_barrier();
                if (sub == 0) { cm[0] = m_new; cm[1] = l_new; }
            }
        }
        __syncthreads();
    }
    float *dst = part + ((((size_t)b * S + s) * splits + split) * H) * (DP + 2);
    for (int x = tid; x < H * (DP + 2); x += WAVE * NWAVE) dst[x] = comb[x];
}

// One workgroup per (b, set, head-in-set): blockIdx.x = (b*S + s)*HPS + h.  The weights of the splits,
// exp(max_sp - max) / sum, are computed once into LDS; then thread (group, column pair) sums every MERGE_GROUPS-th run of eight
// splits' rows with 8-byte loads, eight of them in flight, and the groups' sums are added in order through LDS.  DP is even;
// rows start 8 bytes into a (DP + 2)-float record, so 8 bytes is the alignment there is.  For more than 64 splits (one or two
// lonely caches, or decode_split_kernel's many); fewer go to decode_merge_few_kernel.
constexpr int MERGE_THREADS = 256, MERGE_GROUPS = 4;
template <typename T>
__global__ __launch_bounds__(MERGE_THREADS *MERGE_GROUPS) void decode_merge_kernel(const float *__restrict__ part, T *__restrict__ O, int HPS, int DP, int splits)
{
    extern __shared__ float wgt[];                        // [splits], then [MERGE_GROUPS - 1][DP] partial sums
    __shared__ float red[MERGE_THREADS * MERGE_GROUPS / WAVE];
    const size_t bs = blockIdx.x / HPS;
    const int h = blockIdx.x % HPS, tid = threadIdx.x, group = tid / MERGE_THREADS;
    const float *base = part + (bs * splits * HPS + h) * (size_t)(DP + 2);
    const size_t stride = (size_t)HPS * (DP + 2);
    auto block_reduce = [&](float v, bool is_max) {
        v = is_max ? lanes::over_group<WAVE>(v, lanes::Max()) : lanes::over_group<WAVE>(v, lanes::Sum());
        __syncthreads();                                  // red[] free again
        if ((tid & (WAVE - 1)) == 0) red[tid / WAVE] = v;
        __syncthreads();
        float r = red[0];
        for (int i = 1; i < MERGE_THREADS * MERGE_GROUPS / WAVE; ++i) r = is_max ? fmaxf(r, red[i]) : r + red[i];
        return r;
    };
    float mx = -INFINITY;
    for (int sp = tid; sp < splits; sp += MERGE_THREADS * MERGE_GROUPS) mx = fmaxf(mx, base[sp * stride]);
    mx = block_reduce(mx, true);
    float l = 0.f;
    for (int sp = tid; sp < splits; sp += MERGE_THREADS * MERGE_GROUPS) {
        const float e = __expf(base[sp * stride] - mx);
        wgt[sp] = e;
        l += base[sp * stride + 1] * e;
    }
    l = block_reduce(l, false);                           // (its barriers also publish wgt[])
    const float inv = 1.f / l;
    float *const psum = wgt + splits;
    for (int x0 = 0; x0 < DP; x0 += 2 * MERGE_THREADS) {
        const int x = x0 + 2 * (tid % MERGE_THREADS);
        float a0 = 0.f, a1 = 0.f;
        const float *col = base + 2 + x;
        if (x < DP) {
            int sp = 8 * group;
            for (; sp + 8 <= splits; sp += 8 * MERGE_GROUPS) {
                float2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float2 *>(col + (sp + u) * stride);
#pragma unroll
                for (int u = 0; u < 8; ++u) { a0 = fmaf(v[u].x, wgt[sp + u], a0); a1 = fmaf(v[u].y, wgt[sp + u], a1); }
            }
            for (int i = sp; i < splits && i < sp + 8; ++i) {        // (the last run, shorter than eight, is one group's)
                const float2 v = *reinterpret_cast<const float2 *>(col + i * stride);
                a0 = fmaf(v.x, wgt[i], a0);
                a1 = fmaf(v.y, wgt[i], a1);
            }
        }
        if (group > 0 && x < DP) { psum[(group - 1) * DP + x] = a0; psum[(group - 1) * DP + x + 1] = a1; }
        __syncthreads();
        if (group == 0 && x < DP)
            for (int i = 0; i < MERGE_GROUPS - 1; ++i) { a0 += psum[i * DP + x]; a1 += psum[i * DP + x + 1]; }
        if (group == 0 && x < DP) {
            DElt<T>::st(O + (size_t)blockIdx.x * DP + x, a0 * inv);
            DElt<T>::st(O + (size_t)blockIdx.x * DP + x + 1, a1 * inv);
        }
    }
}
// The same for up to 64 splits and 512 columns, in one round trip to memory: lane l of every wavefront reads the maximum and the sum
// of split l and finds the weights by itself, and the up to SPAN rows that a thread adds up are requested before that.
// GROUPS groups of wavefronts take SPAN splits each.  Bound by launch latency and that round trip: with the
// reductions over LDS barriers and the rows requested after them the kernel took 4.0 us of a step of 13.9 (one sequence, 512 + 64).
// Eight rows per thread where that is enough, so that short steps request no more than there is; four groups above sixteen
// splits.  Together with the merge inside the split kernels (all reads in flight, nothing rescaled before it is written), the
// step before / now, back to back in a graph: 512 + 64, 16 heads, B = 1, L = 700 13.2 / 11.2 us, 4001 13.9 / 12.1, 131072 16.3 / 15.6;
// B = 8, 4001 16.0 / 14.1; B = 32, 131072 66.4 / 65.1; 28 heads over 4 KV heads, B = 5, L = 16016 9.7 / 8.5; 32 over 8, B = 1,
// L = 65536 10.6 / 9.0.
template <typename T, int GROUPS, int SPAN>
__global__ __launch_bounds__(MERGE_THREADS *GROUPS) void decode_merge_few_kernel(const float *__restrict__ part, T *__restrict__ O, int HPS, int DP, int splits)
{
    __shared__ float2 psum[GROUPS > 1 ? GROUPS - 1 : 1][MERGE_THREADS];
    const size_t bs = blockIdx.x / HPS;
    const int h = blockIdx.x % HPS, lane = threadIdx.x & (WAVE - 1), per_group = blockDim.x / GROUPS;
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / per_group), x = 2 * (threadIdx.x % per_group);
    const float *base = part + (bs * splits * HPS + h) * (size_t)(DP + 2);
    const size_t stride = (size_t)HPS * (DP + 2);
    const float2 ml = lane < splits ? *reinterpret_cast<const float2 *>(base + lane * stride) : float2{-INFINITY, 0.f};
    const int sp0 = group * SPAN;
    float2 v[SPAN];
#pragma unroll
    for (int u = 0; u < SPAN; ++u)
        v[u] = sp0 + u < splits && x < DP ? *reinterpret_cast<const float2 *>(base + 2 + x + (sp0 + u) * stride) : float2{0.f, 0.f};
    const float mx = lanes::over_group<WAVE>(ml.x, lanes::Max());
    const float e = lane < splits ? __expf(ml.x - mx) : 0.f;
    const float l = lanes::over_group<WAVE>(lane < splits ? ml.y * e : 0.f, lanes::Sum());
    float2 sum = float2{0.f, 0.f};
#pragma unroll
    for (int u = 0; u < SPAN; ++u)
        if (sp0 + u < splits) {
            const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e), sp0 + u));
            sum.x = fmaf(v[u].x, w, sum.x);
            sum.y = fmaf(v[u].y, w, sum.y);
        }
    if constexpr (GROUPS > 1) {
        if (group > 0) psum[group - 1][x / 2] = sum;
        __syncthreads();
        if (group > 0) return;
#pragma unroll
        for (int i = 0; i < GROUPS - 1; ++i) { sum.x += psum[i][x / 2].x; sum.y += psum[i][x / 2].y; }
    }
    const float inv = 1.f / l;
    if (x < DP) {
        DElt<T>::st(O + (size_t)blockIdx.x * DP + x, sum.x * inv);
        DElt<T>::st(O + (size_t)blockIdx.x * DP + x + 1, sum.y * inv);
    }
}
template <typename T> void launch_merge(const DecodeArgs &a, int splits, hipStream_t st)
{
    const Dims &d = a.d;
    const unsigned grid = d.B * d.H;
    const int hps = d.H / d.S;
    if (splits <= WAVE && d.d_pool <= 2 * MERGE_THREADS) {
        const int threads = (d.d_pool / 2 + WAVE - 1) / WAVE * WAVE;       // two columns each
        if (splits <= 8) decode_merge_few_kernel<T, 1, 8><<<grid, threads, 0, st>>>(a.part, (T *)a.O, hps, d.d_pool, splits);
        else if (splits <= 16) decode_merge_few_kernel<T, 1, 16><<<grid, threads, 0, st>>>(a.part, (T *)a.O, hps, d.d_pool, splits);
        else decode_merge_few_kernel<T, 4, 16><<<grid, threads * 4, 0, st>>>(a.part, (T *)a.O, hps, d.d_pool, splits);
    } else {
        decode_merge_kernel<T><<<grid, MERGE_THREADS * MERGE_GROUPS, (splits + (MERGE_GROUPS - 1) * d.d_pool) * sizeof(float), st>>>(a.part, (T *)a.O, hps, d.d_pool, splits);
    }
}

template <typename T, int DP, int DS, bool MLA, int HPS>
hipError_t run(const DecodeArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    decode_split_kernel<T, DP, DS, MLA, HPS><<<d.B * d.S * a.splits, WAVE * NWAVE, 0, st>>>(
        (const T *)a.q, (const T *)a.pool_rep, (const T *)a.sel_rep, (const T *)a.pool_tail, (const T *)a.sel_tail, a.part, d.S, d.P, d.m,
        d.k, a.splits, d.scale, d.rep_logit_bias, a.m_cap, a.k_cap, a.k_start);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_merge<T>(a, a.splits, st);
    return hipGetLastError();
}

// 0 when no instantiation exists
int shape_id(const Dims &d)
{
    const int hps = d.H / d.S;
    const bool mla = d.mode == LCA_MODE_MLA;
    const bool b16 = d.dtype == LCA_BF16 || d.dtype == LCA_F16;    // the 16-bit types share the shapes; the launcher picks the type
    if (b16 && mla && d.d_pool == 512 && d.d_sel == 64 && (hps == 1 || hps == 16)) return 200 + hps;
    if (d.dtype == LCA_F32 && mla && d.d_pool == 128 && d.d_sel == 32 && (hps == 1 || hps == 4)) return 300 + hps;
    return 0;
}

}  // namespace

bool decode_supported(const Dims &d) { return decode_mla_supported(d) || decode_gqa_mfma_supported(d) || shape_id(d) != 0; }

int decode_splits(const Dims &d)
{
    if (decode_mla_supported(d)) return decode_mla_parts(d);
    if (decode_gqa_mfma_supported(d)) return decode_gqa_mfma_parts(d);
    const int n = d.m + d.k;
    int splits = (TARGET_BLOCKS + d.B * d.S - 1) / (d.B * d.S);
    const int max_splits = (n + 63) / 64;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    return splits;
}

size_t decode_workspace_bytes(const Dims &d)
{
    if (!decode_supported(d)) return 0;
    int records = decode_splits(d);
    if (decode_mla_supported(d) || decode_gqa_mfma_supported(d)) {
        // One result per workgroup of four wavefronts.  The size asked for is that of four results for every four wavefronts of four
        // tiles each, at most 4 * 256 in all (rounded up per pair): never less than the workgroups of the rule in use need.
        const int bn = decode_mla_supported(d) ? 16 : 32, tiles = (d.m + bn - 1) / bn + (d.k + bn - 1) / bn;
        const int target = (256 + d.B * d.S - 1) / (d.B * d.S), most = (tiles + 15) / 16;
        const int wgs = target < most ? target : most;
        records = 4 * (wgs < 1 ? 1 : wgs);
    }
    return (size_t)d.B * d.S * records * (d.H / d.S) * (d.d_pool + 2) * sizeof(float);
}

hipError_t launch_decode(const DecodeArgs &a, hipStream_t st)
{
    if (decode_mla_supported(a.d)) {     // matrix-core kernel at the MLA widths, then the common merge
        const hipError_t e = launch_decode_mla(a, st);
        if (e != hipSuccess) return e;
        const int wgs = a.splits / 4;    // one partial result per workgroup of four wavefronts
        if (wgs == 1) return hipSuccess; // ... unless a workgroup had a (sequence, set) to itself: then it wrote O
        if (a.d.dtype == LCA_F16)
            launch_merge<f16_t>(a, wgs, st);
        else
            launch_merge<uint16_t>(a, wgs, st);
        return hipGetLastError();
    }
    if (decode_gqa_mfma_supported(a.d)) {     // matrix-core kernel at the GQA widths, then the common merge
        const hipError_t e = launch_decode_gqa_mfma(a, st);
        if (e != hipSuccess) return e;
        const int wgs = a.splits / 4;
        if (wgs == 1) return hipSuccess; // a workgroup had a (sequence, KV head) to itself and wrote O
        if (a.d.dtype == LCA_F16)
            launch_merge<f16_t>(a, wgs, st);
        else
            launch_merge<uint16_t>(a, wgs, st);
        return hipGetLastError();
    }
    const bool f16 = a.d.dtype == LCA_F16;
    switch (shape_id(a.d)) {
    case 201: return f16 ? run<f16_t, 512, 64, true, 1>(a, st) : run<uint16_t, 512, 64, true, 1>(a, st);
    case 216: return f16 ? run<f16_t, 512, 64, true, 16>(a, st) : run<uint16_t, 512, 64, true, 16>(a, st);
    case 301: return run<float, 128, 32, true, 1>(a, st);
    case 304: return run<float, 128, 32, true, 4>(a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lca

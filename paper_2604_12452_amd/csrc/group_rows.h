// Pieces shared by the condensation kernels and the online cache update: element conversions, and the rows of one group
// spread over a wavefront.
#pragma once
#include "lanes.h"
#include "lca_internal.h"

namespace lca {
namespace group_rows {

constexpr int WAVE = 64;

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }   // round to nearest even

template <typename T> struct Elt;
template <> struct Elt<uint16_t> {      // bf16 bit patterns
    static constexpr int EPC = 8;        // elements per 16-byte chunk
    __device__ static float ld(const uint16_t *p) { return bf16_bits_to_float(*p); }
    __device__ static void st(uint16_t *p, float v) { *p = float_to_bf16_bits(v); }
    __device__ static void unpack(const uint4 &c, float *f)
    {
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    __device__ static uint4 pack(const float *f)
    {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = (uint32_t)float_to_bf16_bits(f[2 * i]) | ((uint32_t)float_to_bf16_bits(f[2 * i + 1]) << 16);
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
};
template <> struct Elt<f16_t> {         // fp16 bit patterns
    static constexpr int EPC = 8;
    __device__ static float ld(const f16_t *p) { return f16_bits_to_float(p->bits); }
    __device__ static void st(f16_t *p, float v) { p->bits = float_to_f16_bits(v); }
    __device__ static void unpack(const uint4 &c, float *f)
    {
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = f16_bits_to_float((uint16_t)w[i]);
            f[2 * i + 1] = f16_bits_to_float((uint16_t)(w[i] >> 16));
        }
    }
    __device__ static uint4 pack(const float *f)
    {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = (uint32_t)float_to_f16_bits(f[2 * i]) | ((uint32_t)float_to_f16_bits(f[2 * i + 1]) << 16);
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
};
template <> struct Elt<float> {
    static constexpr int EPC = 4;
    __device__ static float ld(const float *p) { return *p; }
    __device__ static void st(float *p, float v) { *p = v; }
    __device__ static void unpack(const uint4 &c, float *f)
    {
        f[0] = __uint_as_float(c.x); f[1] = __uint_as_float(c.y); f[2] = __uint_as_float(c.z); f[3] = __uint_as_float(c.w);
    }
    __device__ static uint4 pack(const float *f)
    {
        return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    }
};

__device__ __forceinline__ float readlane_f(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Lane r < rows holds v_r, the others -inf; returns the row with the largest v (lowest row on ties; numbers only, row 0 if there is none).
__device__ __forceinline__ int wave_argmax(float v, int rows, float *vmax_out)
{
    const float vmax = lanes::over_group<WAVE>(v, lanes::Max());
    if (vmax_out) *vmax_out = vmax;
    // (rows only: where no row is a number the maximum is the -inf of the lanes behind them)
    const unsigned long long at = __builtin_amdgcn_ballot_w64(v == vmax) & (~0ull >> (WAVE - rows));
    return at != 0 ? __builtin_ctzll(at) : 0;
}

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ void unpack4(const uintx4 &c, float *f) { Elt<T>::unpack(make_uint4(c[0], c[1], c[2], c[3]), f); }
template <typename T> __device__ __forceinline__ uintx4 pack4(const float *f)
{
    const uint4 u = Elt<T>::pack(f);
    return uintx4{u.x, u.y, u.z, u.w};
}

// The rows of one component of a group, spread over a wavefront.
template <typename T, int N> struct Rows {
    const T *base;
    size_t stride;           // elements between rows
    int chunks, g;           // 16-byte pieces per row, rows
    int shift;               // log2 of the lanes per row
    int row0, c0;            // this lane's first row and piece
    bool held_all;           // one piece per lane and row, all of them in `held` ...
    bool requested;          // ... once they have been asked for
    uintx4 held[N];

    // log2 of the lanes that a row of `ch` pieces takes; loads that g such rows take
    __host__ __device__ __forceinline__ static int row_shift(int ch) { return ch <= 1 ? 0 : ch > 32 ? 6 : 32 - __builtin_clz(ch - 1); }
    __host__ __device__ __forceinline__ static int loads(int ch, int gg) { return (gg + (WAVE >> row_shift(ch)) - 1) >> (6 - row_shift(ch)); }

    __device__ __forceinline__ void init(const T *b, size_t st, int ch, int gg, int lane)
    {
        base = b; stride = st; chunks = ch; g = gg;
        shift = row_shift(ch);
        row0 = lane >> shift; c0 = lane & ((1 << shift) - 1);
        held_all = ch <= WAVE && loads(ch, gg) <= N;
        requested = false;
    }
    __device__ __forceinline__ int rows_per_load() const { return WAVE >> shift; }
    __device__ __forceinline__ const uintx4 *at(int row, int c) const { return reinterpret_cast<const uintx4 *>(base + row * stride + c * Elt<T>::EPC); }
    __device__ __forceinline__ uintx4 fetch(int row, int c) const { return row < g && c < chunks ? *at(row, c) : uintx4{0, 0, 0, 0}; }
    __device__ __forceinline__ void request()
    {
        if (!held_all) return;
        requested = true;
#pragma unroll
        for (int i = 0; i < N; ++i) held[i] = i * rows_per_load() < g ? fetch(row0 + i * rows_per_load(), c0) : uintx4{0, 0, 0, 0};
    }
    // out[row] = per-row sums over the columns of term(element values, first column), plus `add`[row] if there is one
    template <class F> __device__ __forceinline__ void row_sums(F term, float *out, const float *add) const
    {
        float f[Elt<T>::EPC];
        if (held_all) {                          // (the exchanges of four loads' rows overlap)
            constexpr int BATCH = N < 4 ? N : 4;
            static_assert(N % BATCH == 0, "whole batches");
#pragma unroll
            for (int i0 = 0; i0 < N; i0 += BATCH) {
                if (i0 * rows_per_load() >= g) break;
                float a[BATCH];
#pragma unroll
                for (int i = 0; i < BATCH; ++i) {
                    unpack4<T>(held[i0 + i], f);
                    a[i] = c0 < chunks ? term(f, c0 * Elt<T>::EPC) : 0.f;
                }
                lanes::over_group(a, shift, lanes::Sum());
#pragma unroll
                for (int i = 0; i < BATCH; ++i) {
                    const int row = row0 + (i0 + i) * rows_per_load();
                    if (c0 == 0 && row < g) out[row] = add != nullptr ? add[row] + a[i] : a[i];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
        for (int r = 0; r < g; r += rows_per_load()) {
            const int row = r + row0;
            float a[1] = {0.f};
            for (int c = c0; c < chunks; c += WAVE) {
                unpack4<T>(fetch(row, c), f);
                a[0] += term(f, c * Elt<T>::EPC);
            }
            lanes::over_group(a, shift, lanes::Sum());
            if (c0 == 0 && row < g) out[row] = add != nullptr ? add[row] + a[0] : a[0];
        }
    }
    // out[row] = <row, q>, plus `add`[row] if there is one
    __device__ __forceinline__ void row_dots(const float *q, float *out, const float *add) const
    {
        constexpr int EPC = Elt<T>::EPC;
        if (!held_all) {
            row_sums([q](const float *f, int col) {
                float a = 0.f;
#pragma unroll
                for (int e = 0; e < EPC; ++e) a = fmaf(f[e], q[col + e], a);
                return a;
            }, out, add);
            return;
        }
        float mine[EPC], f[EPC];                 // this lane's piece of q is the same for every row (lanes without a piece hold zeros)
#pragma unroll
        for (int e = 0; e < EPC; ++e) mine[e] = 0.f;
        if (c0 < chunks) {                       // (one branch around all of them: a choice per element left 4-byte loads, eight for two; 128 + 32, eight sets, g = 4, L = 5634 20.9 / 12.7 us)
#pragma unroll
            for (int e = 0; e < EPC; ++e) mine[e] = q[c0 * EPC + e];
        }
        constexpr int BATCH = N < 4 ? N : 4;
#pragma unroll
        for (int i0 = 0; i0 < N; i0 += BATCH) {
            if (i0 * rows_per_load() >= g) break;
            float a[BATCH];
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                unpack4<T>(held[i0 + i], f);
                a[i] = 0.f;
#pragma unroll
                for (int e = 0; e < EPC; ++e) a[i] = fmaf(f[e], mine[e], a[i]);
            }
            lanes::over_group(a, shift, lanes::Sum());
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int row = row0 + (i0 + i) * rows_per_load();
                if (c0 == 0 && row < g) out[row] = add != nullptr ? add[row] + a[i] : a[i];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // out = sum of weight[row] * row (held: of rows past the group, which are zeros, whatever the weight as long as it is a number)
    __device__ __forceinline__ void weighted_sum(const float *weight, T *out) const
    {
        constexpr int EPC = Elt<T>::EPC;
        auto finish = [&](float (&acc)[EPC], int c) {
            if (g > 1) lanes::over_strided(acc, shift, lanes::Sum());          // (lanes without a row of the group add zeros)
            if (row0 == 0 && c < chunks) *reinterpret_cast<uintx4 *>(out + c * EPC) = pack4<T>(acc);
        };
        float f[EPC], acc[EPC];
        if (held_all) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
            constexpr int BATCH = N < 8 ? N : 8;
            static_assert(N % BATCH == 0, "whole batches");
#pragma unroll
            for (int i0 = 0; i0 < N; i0 += BATCH) {
                if (i0 * rows_per_load() >= g) break;
                float w[BATCH];                  // (the caller's weights are WAVE numbers, zeros from g on)
#pragma unroll
                for (int i = 0; i < BATCH; ++i) w[i] = weight[min(row0 + (i0 + i) * rows_per_load(), WAVE - 1)];
#pragma unroll
                for (int i = 0; i < BATCH; ++i) {
                    unpack4<T>(held[i0 + i], f);
#pragma unroll
                    for (int e = 0; e < EPC; ++e) acc[e] = fmaf(w[i], f[e], acc[e]);
                }
            }
            finish(acc, c0);
            return;
        }
        for (int cb = 0; cb < chunks; cb += WAVE) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
#pragma unroll 4
            for (int r = 0; r < g; r += rows_per_load()) {
                const int row = r + row0;
                const float w = row < g ? weight[row] : 0.f;
                unpack4<T>(fetch(row, cb + c0), f);
#pragma unroll
                for (int e = 0; e < EPC; ++e) acc[e] = row < g ? fmaf(w, f[e], acc[e]) : acc[e];
            }
            finish(acc, cb + c0);
        }
    }
    __device__ __forceinline__ void copy_row(int row, T *out, int lane) const      // bit for bit
    {
        if (requested) {
            const int at = row >> (6 - shift);
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (i == at && row0 == (row & (rows_per_load() - 1)) && c0 < chunks) *reinterpret_cast<uintx4 *>(out + c0 * Elt<T>::EPC) = held[i];
            return;
        }
        for (int c = lane; c < chunks; c += WAVE)
            *reinterpret_cast<uintx4 *>(out + c * Elt<T>::EPC) = *at(row, c);
    }
};

// Summary query: the mean of n_q hps query rows, hps neighbouring heads of each of n_q tokens.
// WAVES wavefronts take 16 chunks of 16 bytes (SQ_CHUNKS, block xb of them): a load covers 256 bytes of four rows, so the 64 row
// slots of 16 wavefronts take the 256 rows of 16 queries x 16 heads in four loads per lane, all in flight at once; the partial
// sums are merged in a fixed order (deterministic), the four rows of a wavefront by exchanges, the wavefronts through LDS.
constexpr int SQ_DEPTH = 8;
constexpr int SQ_CHUNKS = 16;
template <typename T, int WAVES> using SummaryPart = float[WAVES][SQ_CHUNKS][Elt<T>::EPC + 1];
// `rows`: the first token's first head; tokens are H rows apart.  `out`: the d_qk sums' means (memory or LDS).
template <int WAVES, typename T>
__device__ __forceinline__ void summary_columns(const T *rows, int H, int hps, int d_qk, int n_q, int xb, SummaryPart<T, WAVES> &part, float *out)
{
    constexpr int EPC = Elt<T>::EPC, SQ_SLOTS = WAVES * (WAVE / SQ_CHUNKS);
    static_assert(WAVES * WAVE >= SQ_CHUNKS * EPC, "a thread per component");
    const int n_chunks = d_qk / EPC;
    const int sub = threadIdx.x % SQ_CHUNKS, slot = threadIdx.x / SQ_CHUNKS, wave = threadIdx.x / WAVE;
    const int chunk = xb * SQ_CHUNKS + sub;
    const int n = n_q * hps;                       // row u is head u % hps of token u / hps
    float acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
    if (chunk < n_chunks) {
        const int step_t = SQ_SLOTS / hps, step_h = SQ_SLOTS % hps;
        int ut = slot / hps, uh = slot % hps;       // pair u = slot + 64 j  ->  (u / hps, u % hps), stepped with carry
        const T *const base = rows + chunk * EPC;
        for (int u0 = slot; u0 < n; u0 += SQ_SLOTS * SQ_DEPTH) {
            uint4 v[SQ_DEPTH];
#pragma unroll
            for (int i = 0; i < SQ_DEPTH; ++i) {
                const int u = u0 + i * SQ_SLOTS;
                v[i] = u < n ? *reinterpret_cast<const uint4 *>(base + ((size_t)ut * H + uh) * d_qk) : make_uint4(0, 0, 0, 0);
                ut += step_t; uh += step_h;
                if (uh >= hps) { uh -= hps; ++ut; }
            }
#pragma unroll
            for (int i = 0; i < SQ_DEPTH; ++i) {
                float f[EPC];
                Elt<T>::unpack(v[i], f);
#pragma unroll
                for (int e = 0; e < EPC; ++e) acc[e] += f[e];
            }
        }
    }
    static_assert(SQ_CHUNKS == 16, "the four rows of a wavefront are its four groups of 16 lanes");
    lanes::over_strided(acc, 4, lanes::Sum());
    if ((threadIdx.x & (WAVE - 1)) < SQ_CHUNKS) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) part[wave][sub][e] = acc[e];
    }
    __syncthreads();
    // thread x sums the wavefronts' partial values of component x % EPC of chunk x / EPC (wavefront order: the same sum on every run)
    const int ol = threadIdx.x / EPC, oe = threadIdx.x % EPC, ochunk = xb * SQ_CHUNKS + ol;
    if (ol < SQ_CHUNKS && ochunk < n_chunks) {
        float t = 0.f;
#pragma unroll
        for (int wv = 0; wv < WAVES; ++wv) t += part[wv][ol][oe];
        out[ochunk * EPC + oe] = t / (float)n;
    }
}

// One group by one wavefront: scores against the summary query `qb` (Eq. 6), both components reduced (Eq. 7, Eq. 8 or an ablation's
// strategy), the anchor's token index (first_token + row) and, if asked for, the weights.  row_val, row_norm: 64 floats of LDS each,
// the wavefront's own.
template <typename T, int NP, int NS>
__device__ __forceinline__ void condense_group(const Rows<T, NP> &pool, const Rows<T, NS> &sel, const float *qb, int mla, int d_pool, int g, float scale,
                                               int pool_reduce, int sel_reduce, T *pool_out, T *sel_out, int32_t *anchor, int first_token,
                                               float *alpha_out, float *row_val, float *row_norm, int lane)
{
    constexpr int EPC = Elt<T>::EPC;
    auto square = [](const float *f, int) {
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) a = fmaf(f[e], f[e], a);
        return a;
    };
    if (mla) pool.row_dots(qb, row_val, nullptr);
    __builtin_amdgcn_wave_barrier();
    sel.row_dots(qb + (mla ? d_pool : 0), row_val, mla ? row_val : nullptr);
    __builtin_amdgcn_wave_barrier();
    const float my_score = lane < g ? scale * row_val[lane] : -INFINITY;      // lane r holds the score of row r
    float bmax;
    const int brow = wave_argmax(my_score, g, &bmax);
    const float pmine = lane < g ? __expf(my_score - bmax) : 0.f;
    const float alpha = pmine / lanes::over_group<WAVE>(pmine, lanes::Sum());

    // one component: a weighted sum of the group's rows, or one of them
    auto reduce = [&](auto &rows, int strategy, T *out) {
        int pick = brow;
        if (strategy == LCA_REDUCE_MAXPOOL) {
            rows.row_sums(square, row_norm, nullptr);
            __builtin_amdgcn_wave_barrier();
            pick = wave_argmax(lane < g ? row_norm[lane] : -INFINITY, g, nullptr);
        }
        if (strategy == LCA_REDUCE_MAXSEL || strategy == LCA_REDUCE_MAXPOOL) {
            rows.copy_row(pick, out, lane);
            return;
        }
        __builtin_amdgcn_wave_barrier();
        row_val[lane] = lane >= g ? 0.f : strategy == LCA_REDUCE_MEAN ? 1.f / (float)g : alpha;
        __builtin_amdgcn_wave_barrier();
        rows.weighted_sum(row_val, out);
    };
    reduce(pool, pool_reduce, pool_out);
    reduce(sel, sel_reduce, sel_out);
    if (anchor != nullptr && lane == 0) *anchor = first_token + brow;
    if (alpha_out != nullptr && lane < g) alpha_out[lane] = alpha;
}

}  // namespace group_rows
}  // namespace lca

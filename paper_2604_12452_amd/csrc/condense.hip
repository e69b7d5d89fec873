// Latent-space condensation kernels (section 4.2 of the paper; Algorithm 1, first step and group loop).
//
//   summary_query_kernel   qbar = mean of the last n_q queries (and of the heads of a set)
//   condense_reg_kernel    one wavefront per group, the group's rows held in registers; scores by
//                          per-lane partial dots + a reduce-scatter butterfly, online softmax over
//                          sub-blocks of <= 8 rows, pooling in-lane, anchor by (score, index) max.
//                          HBM-bound: every C^KV / K^R byte is read once, as 16-byte coalesced loads.
//   condense_any_kernel    any sizes and reduce strategies.
//   condense_one_kernel    few groups: the summary query and the groups in one launch.
//
// gfx950 only (wave64).
#include "group_rows.h"

namespace lca {
namespace {

using namespace group_rows;

// ---------------------------------------------------------------------------------------------
// Summary query: qbar[b,s,x] = mean over t in [L-n_q, L), h in set s of Q[b,t,h,x].
// One workgroup per (b, s, 16 chunks of 16 bytes), see summary_columns.  Bound by the memory round trip: the lca_condense call of
// 29 groups at 512 + 64 took 11.2 us with 64 chunks per workgroup and one row per load, and takes 8.4 us.
// Sixteen wavefronts have 64 row slots.  Four are enough where there are no more than 16 rows, and where the workgroups alone fill the
// chip (SQ_MANY): there most of sixteen would be waiting for one load.  The cache update's call, fp32 128 + 128, 16 sets, 42 sequences,
// g = 2: 14.9 us with sixteen, 9.5 with four; fp32 960 + 64, 16 sets, 28 sequences, 64 queries 43.2 / 28.0; bf16 512 + 64, 128 sequences 13.7 / 12.7.
// ---------------------------------------------------------------------------------------------
constexpr int SQ_WAVES = 16, SQ_WAVES_FEW = 4, SQ_MANY = 512;
template <typename T, int WAVES>
__global__ __launch_bounds__(WAVES *WAVE) void summary_query_kernel(const T *__restrict__ Q, float *__restrict__ qbar, int L, int H, int S,
                                                                       int d_qk, int n_q)
{
    __shared__ SummaryPart<T, WAVES> part;
    const int n_chunks = d_qk / Elt<T>::EPC;
    const int xblocks = (n_chunks + SQ_CHUNKS - 1) / SQ_CHUNKS;
    const int bs = blockIdx.x / xblocks, xb = blockIdx.x % xblocks;
    const int b = bs / S, s = bs % S, hps = H / S;
    summary_columns<WAVES>(Q + (((size_t)b * L + (L - n_q)) * H + (size_t)s * hps) * d_qk, H, hps, d_qk, n_q, xb, part, qbar + (size_t)bs * d_qk);
}

// ---------------------------------------------------------------------------------------------
// wave helpers
// ---------------------------------------------------------------------------------------------
// Sum R (1, 2, 4 or 8) per-lane partial values across the wave so that lane l ends with the total of value
// (l >> (6 - log2 R)).  log2(R) halving exchanges, then an all-reduce over the remaining lane bits.
template <int R>
__device__ __forceinline__ float wave_reduce_scatter(float (&v)[R], int lane)
{
    static_assert(R == 1 || R == 2 || R == 4 || R == 8, "three halving exchanges are written out");
    // (the lanes whose bit is set keep the second half of the values: what a swap of one register's upper lanes against the other's lower ones leaves in place)
    if constexpr (R > 1) {
#pragma unroll
        for (int i = 0; i < R / 2; ++i) { lanes::swap32(v[i], v[i + R / 2]); v[i] += v[i + R / 2]; }
    }
    if constexpr (R > 2) {
#pragma unroll
        for (int i = 0; i < R / 4; ++i) { lanes::swap16(v[i], v[i + R / 4]); v[i] += v[i + R / 4]; }
    }
    if constexpr (R > 4) {
        const bool hi = (lane & 8) != 0;
        const float lo_half = v[0], hi_half = v[1];      // (values first: a choice between two array elements would become an indexed access to the array)
        v[0] = (hi ? hi_half : lo_half) + lanes::dpp<lanes::ROR + 8>(hi ? lo_half : hi_half);
    }
    return lanes::over_group<WAVE / R>(v[0], lanes::Sum());
}

// ---------------------------------------------------------------------------------------------
// Register-resident condensation: one wave per (sequence, KV source, group).
//   pool part : lane l owns 16-byte chunk l of every row of the sub-block (R <= 8 rows in registers)
//   sel part  : lane l owns row (l >> SH) and every (64/R)-th chunk of it, so its partial dot already
//               sits with the lane that receives that row's score from the reduce-scatter
// ---------------------------------------------------------------------------------------------
template <typename T, int DP, int DS, int G, bool MLA, bool HOLD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HOLD ? 2 : 3, 8)))
void condense_reg_kernel(const T *__restrict__ POOL, const T *__restrict__ SEL, const float *__restrict__ qbar,
                         T *__restrict__ pool_rep, T *__restrict__ sel_rep, int32_t *__restrict__ anchor,
                         float *__restrict__ alpha_dbg, int B, int L, int S, int m, float scale)
{
    constexpr int EPC = Elt<T>::EPC;
    constexpr int NCP = DP / EPC, NCS = DS / EPC;
    constexpr int R = G < 8 ? G : 8;            // rows per sub-block (8 keeps three wavefronts per SIMD resident)
    constexpr int NSB = G / R;
    constexpr int LOG2R = R == 8 ? 3 : R == 4 ? 2 : R == 2 ? 1 : 0;
    constexpr int SH = 6 - LOG2R;               // lane l holds the score of sub-block row l >> SH
    constexpr int LPR = 1 << SH;                // lanes per row for the sel part
    constexpr int SPL = (NCS + LPR - 1) / LPR;  // sel chunks per lane
    constexpr int DQK = MLA ? DP + DS : DS;
    static_assert(G % R == 0 && DP % EPC == 0 && DS % EPC == 0 && NCP <= WAVE, "shape");

    const int lane = threadIdx.x & (WAVE - 1);
    const long wave_id = (long)blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x / WAVE);
    const int P = MLA ? 1 : S;                  // KV sources per sequence
    const long n_units = (long)B * P * m;
    if (wave_id >= n_units) return;             // whole wave leaves together
    // the KV sources of a group are neighbours in the unit order: the P wavefronts that read the P interleaved parts of the
    // same g token rows run at the same time, and the rows are fetched from memory as whole contiguous pieces
    const int p = (int)(wave_id % P), j = (int)((wave_id / P) % m), b = (int)(wave_id / ((long)m * P));

    const T *pool_base = POOL + ((size_t)b * L * P + p) * DP;   // row i at + i * P * DP
    const T *sel_base = SEL + ((size_t)b * L * P + p) * DS;
    const bool has_pool = lane < NCP;
    const int pcol = (has_pool ? lane : 0) * EPC;
    const int my_row = lane >> SH, sub = lane & (LPR - 1);

    // the loads of sub-block sb: R whole pool rows (a chunk per lane) and this lane's chunks of its own sel row
    auto load_sub_block = [&](int sb, uint4 (&pdata)[R], uint4 (&sdata)[SPL]) {
        const int row0 = j * G + sb * R;
#pragma unroll
        for (int r = 0; r < R; ++r)
            pdata[r] = has_pool ? *reinterpret_cast<const uint4 *>(pool_base + (size_t)(row0 + r) * P * DP + pcol) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < SPL; ++i) {
            const int c = sub + i * LPR;
            sdata[i] = c < NCS ? *reinterpret_cast<const uint4 *>(sel_base + (size_t)(row0 + my_row) * P * DS + c * EPC) : make_uint4(0, 0, 0, 0);
        }
    };
    // HOLD (several sets over one latent sequence, at most two sub-blocks): the group is loaded once and stays in
    // registers for every set; otherwise a sub-block is loaded when its turn comes.
    constexpr int NHELD = HOLD ? NSB : 1;
    uint4 pheld[NHELD][R], sheld[NHELD][SPL];
    if constexpr (HOLD) {
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) load_sub_block(sb, pheld[sb], sheld[sb]);
    }

    const int s_begin = MLA ? 0 : p, s_end = MLA ? S : p + 1;
    for (int s = s_begin; s < s_end; ++s) {
        const float *qb = qbar + ((size_t)b * S + s) * DQK;
        float m_run = -INFINITY, l_run = 0.f;
        float acc[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
        float best_score = -INFINITY;
        int best_row = 0;
        const size_t unit = ((size_t)b * S + s) * m + j;

        auto sub_block = [&](int sb, const uint4 (&pdata)[R], const uint4 (&sdata)[SPL]) {
            // sel part of the score: this lane's chunks of its own row, summed over the row's lanes
            float ssum = 0.f;
#pragma unroll
            for (int i = 0; i < SPL; ++i) {
                const int c = sub + i * LPR;
                if (c < NCS) {
                    float f[EPC];
                    Elt<T>::unpack(sdata[i], f);
                    const float *qs = qb + (MLA ? DP : 0) + c * EPC;
#pragma unroll
                    for (int e = 0; e < EPC; ++e) ssum = fmaf(f[e], qs[e], ssum);
                }
            }
            float dot = lanes::over_group<LPR>(ssum, lanes::Sum());
            if (MLA) {   // pool part of the score: per-lane partial dots of all rows, reduce-scattered
                float qp[EPC];
#pragma unroll
                for (int e = 0; e < EPC; ++e) qp[e] = has_pool ? qb[pcol + e] : 0.f;
                float part[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float f[EPC];
                    Elt<T>::unpack(pdata[r], f);
                    float a = 0.f;
#pragma unroll
                    for (int e = 0; e < EPC; ++e) a = fmaf(f[e], qp[e], a);
                    part[r] = a;
                }
                dot += wave_reduce_scatter<R>(part, lane);
            }
            const float score = scale * dot;              // row my_row of this sub-block
            if (alpha_dbg != nullptr && sub == 0) alpha_dbg[unit * G + sb * R + my_row] = score;   // normalised below
            // sub-block maximum and its lowest row
            float bmax;
            const int brow = wave_argmax(score, WAVE, &bmax) >> SH;
            if (bmax > best_score) { best_score = bmax; best_row = sb * R + brow; }   // earlier sub-block wins ties
            // online softmax over sub-blocks (Eq. 6) and weighted pooling (Eq. 7)
            const float m_new = fmaxf(m_run, bmax);
            const float corr = __expf(m_run - m_new);      // 0 on the first sub-block
            const float pmine = __expf(score - m_new);
            l_run *= corr;
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] *= corr;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float pr = readlane_f(pmine, r << SH);
                l_run += pr;
                float f[EPC];
                Elt<T>::unpack(pdata[r], f);
#pragma unroll
                for (int e = 0; e < EPC; ++e) acc[e] = fmaf(pr, f[e], acc[e]);
            }
            m_run = m_new;
        };
        if constexpr (HOLD) {
#pragma unroll
            for (int sb = 0; sb < NSB; ++sb) sub_block(sb, pheld[sb], sheld[sb]);
        } else {
#pragma unroll 1
            for (int sb = 0; sb < NSB; ++sb) {
                uint4 pdata[R], sdata[SPL];
                load_sub_block(sb, pdata, sdata);            // every load of the sub-block is issued first
                sub_block(sb, pdata, sdata);
            }
        }

        const float inv_l = 1.f / l_run;
        if (has_pool) {
            float o[EPC];
#pragma unroll
            for (int e = 0; e < EPC; ++e) o[e] = acc[e] * inv_l;
            *reinterpret_cast<uint4 *>(pool_rep + unit * DP + pcol) = Elt<T>::pack(o);
        }
        const int a_tok = j * G + best_row;
        if (lane < NCS)
            *reinterpret_cast<uint4 *>(sel_rep + unit * DS + lane * EPC) =
                *reinterpret_cast<const uint4 *>(sel_base + (size_t)a_tok * P * DS + lane * EPC);
        if (lane == 0) anchor[unit] = a_tok;
        if (alpha_dbg != nullptr && sub == 0) {      // each lane turns the scores it wrote into weights
            for (int sb = 0; sb < NSB; ++sb) {
                float *ap = alpha_dbg + unit * G + sb * R + my_row;
                *ap = __expf(*ap - m_run) * inv_l;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Condensation at any widths (16-byte multiples, up to 1024 columns), any group size up to 64, any reduce strategy for either
// component (the ablation grid of section 5.4, Table 5): one wavefront per (sequence, set, group).
//
// A component's rows are read as 16-byte pieces, `lpr` lanes per row (the power of two that holds the row's pieces) and
// 64 / lpr rows per load; what a wavefront can hold in registers (HELD) is requested at once and used for scores, norms and
// pooling alike, the rest is read again when its turn comes (from the caches).  Bound by the latency of that round trip
// at small sizes and by memory at large ones.  The call at B = 1, L = 2500, four KV heads, 64 / 64: 18.0 -> 9.7 us; at L = 16384,
// 512 + 64, g = 24: 111 -> 33 us (scalar loads and a reduction per row before).
// ---------------------------------------------------------------------------------------------
constexpr int ANY_WAVES = 4;         // wavefronts (groups) per workgroup
struct AnyParams {
    const void *POOL, *SEL;
    const float *qbar;               // [B, S, d_qk]
    void *pool_rep, *sel_rep;
    int32_t *anchor;
    float *alpha_dbg;
    int L, S, m, g, d_pool, d_sel, mla, pool_reduce, sel_reduce;
    float scale;
};

// NP, NS: loads of the pooled / selected rows that a wavefront can hold.
template <typename T, int NP, int NS>
__global__ __launch_bounds__(ANY_WAVES *WAVE) void condense_any_kernel(const AnyParams kp)
{
    constexpr int EPC = Elt<T>::EPC;
    __shared__ float per_row[ANY_WAVES][2][WAVE];          // per wavefront and row of its group: score, then weight; norm
    const int lane = threadIdx.x & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int g = kp.g, m = kp.m, S = kp.S, mla = kp.mla, d_pool = kp.d_pool, d_sel = kp.d_sel;
    const int d_qk = mla ? d_pool + d_sel : d_sel;
    const int blocks = (m + ANY_WAVES - 1) / ANY_WAVES;    // workgroups per (sequence, set)
    const int bs = blockIdx.x / blocks, s = bs % S, b = bs / S, j = (int)(blockIdx.x % blocks) * ANY_WAVES + wave;
    if (j >= m) return;
    const int P = mla ? 1 : S, p = mla ? 0 : s;
    const T *const pool_base = (const T *)kp.POOL + (((size_t)b * kp.L + (size_t)j * g) * P + p) * d_pool;
    const T *const sel_base = (const T *)kp.SEL + (((size_t)b * kp.L + (size_t)j * g) * P + p) * d_sel;
    Rows<T, NP> pool;
    Rows<T, NS> sel;
    pool.init(pool_base, (size_t)P * d_pool, d_pool / EPC, g, lane);
    sel.init(sel_base, (size_t)P * d_sel, d_sel / EPC, g, lane);
    if (mla || kp.pool_reduce != LCA_REDUCE_MAXSEL) pool.request();      // (else the anchor's row is all that is read)
    sel.request();
    const float *const qb = kp.qbar + (size_t)bs * d_qk;

    const size_t unit = (size_t)bs * m + j;
    condense_group<T>(pool, sel, qb, mla, d_pool, g, kp.scale, kp.pool_reduce, kp.sel_reduce, (T *)kp.pool_rep + unit * d_pool,
                      (T *)kp.sel_rep + unit * d_sel, kp.anchor + unit, j * g, kp.alpha_dbg != nullptr ? kp.alpha_dbg + unit * g : nullptr,
                      per_row[wave][0], per_row[wave][1], lane);
}

// ---------------------------------------------------------------------------------------------
// Condensation of few groups in one launch: every workgroup averages the queries of its set for itself, in LDS, while the rows of its groups (one per
// wavefront, held in registers) are on their way.  Bound by that one round trip to memory and the chain behind it (100 MHz stamps, four KV heads, 64 / 64, g = 16: 1.7 us
// until the data is there, summary query 1.0, scores 0.5, softmax 0.2, pooled row 0.5), where two launches pay two starts and two round trips.
// ---------------------------------------------------------------------------------------------
constexpr int ONE_WAVES = 8, ONE_THREADS = ONE_WAVES * WAVE;
constexpr int ONE_DEPTH = 8;         // query loads in flight per lane
constexpr int ONE_COLUMNS = 576;     // widest summary query
struct OneParams {
    AnyParams a;
    const void *Q;
    int H, n_q, hps;
    int pieces, slots;               // 16-byte pieces of a query; queries that the workgroup's threads take at a time, a piece each
    int step_t, step_h;              // slots = step_t hps + step_h
    unsigned pieces_magic, hps_magic;        // 2^32 / divisor + 1 (0 for a divisor of 1)
};
__device__ __forceinline__ int udiv_magic(unsigned x, unsigned magic) { return magic == 0 ? x : __umulhi(x, magic); }

template <typename T, int NP, int NS>
__global__ __launch_bounds__(ONE_THREADS) void condense_one_kernel(const OneParams op)
{
    constexpr int EPC = Elt<T>::EPC;
    const AnyParams &kp = op.a;
    __shared__ float per_row[ONE_WAVES][2][WAVE];          // per wavefront and row of its group: score, then weight; norm
    __shared__ float part[ONE_THREADS][EPC + 1];
    __shared__ __attribute__((aligned(16))) float qbar[ONE_COLUMNS];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int g = kp.g, m = kp.m, S = kp.S, mla = kp.mla, d_pool = kp.d_pool, d_sel = kp.d_sel;
    const int d_qk = mla ? d_pool + d_sel : d_sel;
    const int s = blockIdx.y, b = blockIdx.z, j = blockIdx.x * ONE_WAVES + wave;
    const int P = mla ? 1 : S, p = mla ? 0 : s;
    Rows<T, NP> pool;
    Rows<T, NS> sel;
    pool.init((const T *)kp.POOL + (((size_t)b * kp.L + (size_t)j * g) * P + p) * d_pool, (size_t)P * d_pool, d_pool / EPC, g, lane);
    sel.init((const T *)kp.SEL + (((size_t)b * kp.L + (size_t)j * g) * P + p) * d_sel, (size_t)P * d_sel, d_sel / EPC, g, lane);

    // queries: thread t takes piece t % pieces of queries t / pieces, t / pieces + slots, .. (query u: token u / hps, head u % hps)
    const int pieces = op.pieces, slots = op.slots, hps = op.hps, n = op.n_q * hps;
    const int slot = udiv_magic(tid, op.pieces_magic), piece = tid - slot * pieces;
    float acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
    int ut = udiv_magic(slot, op.hps_magic), uh = slot - ut * hps;
    const T *const base = (const T *)op.Q + (((size_t)b * kp.L + (kp.L - op.n_q)) * op.H + (size_t)s * hps) * d_qk + piece * EPC;
    for (int u0 = 0; u0 < n; u0 += slots * ONE_DEPTH) {
        uint4 v[ONE_DEPTH];
#pragma unroll
        for (int i = 0; i < ONE_DEPTH; ++i) {
            v[i] = u0 + i * slots + slot < n && slot < slots ? *reinterpret_cast<const uint4 *>(base + ((size_t)ut * op.H + uh) * d_qk) : make_uint4(0, 0, 0, 0);
            ut += op.step_t; uh += op.step_h;
            if (uh >= hps) { uh -= hps; ++ut; }
        }
        if (u0 == 0 && j < m) {                  // (the group's rows behind the first of them)
            if (mla || kp.pool_reduce != LCA_REDUCE_MAXSEL) pool.request();
            sel.request();
        }
#pragma unroll
        for (int i = 0; i < ONE_DEPTH; ++i) {
            float f[EPC];
            Elt<T>::unpack(v[i], f);
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] += f[e];
        }
    }
    // ... added up over the slots in a fixed order: inside a wavefront where its lanes are whole slots, then through LDS
    const bool whole = (WAVE & (pieces - 1)) == 0 && (pieces & (pieces - 1)) == 0 && pieces <= WAVE;
    if (whole) lanes::over_strided(acc, 31 - __builtin_clz(pieces), lanes::Sum());
    const int parts = whole ? ONE_WAVES : slots;
    if (!whole || lane < pieces) {
        float *const mine = part[whole ? wave * pieces + lane : tid];
#pragma unroll
        for (int e = 0; e < EPC; ++e) mine[e] = acc[e];
    }
    __syncthreads();
    for (int x = tid; x < d_qk; x += ONE_THREADS) {
        const float *const from = part[x / EPC] + x % EPC;
        float t = 0.f;
        for (int i0 = 0; i0 < parts; i0 += 8) {
            float y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) y[i] = from[min(i0 + i, parts - 1) * pieces * (EPC + 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) t += i0 + i < parts ? y[i] : 0.f;
        }
        qbar[x] = t / (float)n;
    }
    __syncthreads();
    if (j >= m) return;
    const size_t unit = ((size_t)b * S + s) * m + j;
    condense_group<T>(pool, sel, qbar, mla, d_pool, g, kp.scale, kp.pool_reduce, kp.sel_reduce, (T *)kp.pool_rep + unit * d_pool,
                      (T *)kp.sel_rep + unit * d_sel, kp.anchor + unit, j * g, kp.alpha_dbg != nullptr ? kp.alpha_dbg + unit * g : nullptr,
                      per_row[wave][0], per_row[wave][1], lane);
}
template <typename T> hipError_t run_one(const CondenseArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    constexpr int EPC = Elt<T>::EPC;
    auto magic = [](int dv) { return dv > 1 ? (unsigned)((1ull << 32) / (unsigned)dv + 1) : 0u; };
    OneParams op;
    op.a = AnyParams{a.POOL, a.SEL, nullptr, a.pool_rep, a.sel_rep, a.anchor, a.alpha_dbg, d.L, d.S, d.m, d.g,
                     d.d_pool, d.d_sel, d.mode == LCA_MODE_MLA, d.pool_reduce, d.sel_reduce, d.scale};
    op.Q = a.Q; op.H = d.H; op.n_q = d.n_q; op.hps = d.H / d.S;
    op.pieces = d.d_qk / EPC; op.slots = ONE_THREADS / op.pieces;
    op.step_t = op.slots / op.hps; op.step_h = op.slots % op.hps;
    op.pieces_magic = magic(op.pieces); op.hps_magic = magic(op.hps);
    const dim3 grid((d.m + ONE_WAVES - 1) / ONE_WAVES, d.S, d.B);
    const int pool = Rows<T, 1>::loads(d.d_pool / EPC, d.g), sel = Rows<T, 1>::loads(d.d_sel / EPC, d.g);
    if (pool <= 4 && sel <= 4) condense_one_kernel<T, 4, 4><<<grid, ONE_THREADS, 0, st>>>(op);
    else if (pool <= 8 && sel <= 8) condense_one_kernel<T, 8, 8><<<grid, ONE_THREADS, 0, st>>>(op);
    else if (pool <= 16) condense_one_kernel<T, 16, 4><<<grid, ONE_THREADS, 0, st>>>(op);
    // (36 held pieces and the query loads do not fit in 256 registers: 84 to 92 bytes a lane are spilled.  Still the faster form: 16 sets of 512 + 64, g = 32, L = 1200 15.7 us, two launches 18.4)
    else condense_one_kernel<T, 32, 4><<<grid, ONE_THREADS, 0, st>>>(op);
    return hipGetLastError();
}

template <typename T, int DP, int DS, int G, bool MLA>
hipError_t run_reg(const CondenseArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    const long units = (long)d.B * (MLA ? 1 : d.S) * d.m;
    const int blocks = (int)((units + 3) / 4);
    if constexpr (MLA && G <= 16) {
        if (d.S > 1) {       // every set reads the same group: it is kept in registers across the sets
            condense_reg_kernel<T, DP, DS, G, MLA, true><<<blocks, 256, 0, st>>>(
                (const T *)a.POOL, (const T *)a.SEL, a.qbar, (T *)a.pool_rep, (T *)a.sel_rep, a.anchor, a.alpha_dbg, d.B, d.L, d.S, d.m, d.scale);
            return hipGetLastError();
        }
    }
    condense_reg_kernel<T, DP, DS, G, MLA, false><<<blocks, 256, 0, st>>>(
        (const T *)a.POOL, (const T *)a.SEL, a.qbar, (T *)a.pool_rep, (T *)a.sel_rep, a.anchor, a.alpha_dbg, d.B, d.L, d.S, d.m, d.scale);
    return hipGetLastError();
}

template <typename T>
hipError_t run_any(const CondenseArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    const AnyParams kp{a.POOL, a.SEL, a.qbar, a.pool_rep, a.sel_rep, a.anchor, a.alpha_dbg, d.L, d.S, d.m, d.g,
                       d.d_pool, d.d_sel, d.mode == LCA_MODE_MLA, d.pool_reduce, d.sel_reduce, d.scale};
    const unsigned grid = (d.m + ANY_WAVES - 1) / ANY_WAVES * d.S * d.B;
    // Small groups of narrow rows are many and short, bound by the instructions of a wavefront: the smallest form that holds the rows.
    // One form for all (<16, 4>) / this rule, bf16: 16 sets of 64 + 64, L = 42872, g = 1 1015 / 397 us; 16 sets of 32 + 32, L = 20000, g = 2
    // 229 / 97; 8 KV heads 64 / 64, L = 60000, g = 4 162 / 78; four, L = 2500, g = 16 9.6 / 9.2.
    constexpr int EPC = Elt<T>::EPC;
    const int pool = Rows<T, 1>::loads(d.d_pool / EPC, d.g), sel = Rows<T, 1>::loads(d.d_sel / EPC, d.g);
    if (pool <= 1 && sel <= 1) condense_any_kernel<T, 1, 1><<<grid, ANY_WAVES * WAVE, 0, st>>>(kp);
    else if (pool <= 4 && sel <= 4) condense_any_kernel<T, 4, 4><<<grid, ANY_WAVES * WAVE, 0, st>>>(kp);
    else condense_any_kernel<T, 16, 4><<<grid, ANY_WAVES * WAVE, 0, st>>>(kp);
    return hipGetLastError();
}

template <typename T, int DP, int DS, bool MLA>
bool try_reg(const CondenseArgs &a, hipStream_t st, hipError_t &err)
{
    switch (a.d.g) {
    case 1: err = run_reg<T, DP, DS, 1, MLA>(a, st); return true;
    case 2: err = run_reg<T, DP, DS, 2, MLA>(a, st); return true;
    case 4: err = run_reg<T, DP, DS, 4, MLA>(a, st); return true;
    case 8: err = run_reg<T, DP, DS, 8, MLA>(a, st); return true;
    case 16: err = run_reg<T, DP, DS, 16, MLA>(a, st); return true;
    case 32: err = run_reg<T, DP, DS, 32, MLA>(a, st); return true;
    default: return false;
    }
}

}  // namespace

// qbar [B,S,d_qk] = mean of the last n_q of the L queries in Q [B,L,H,d_qk] (and of each set's heads)
template <typename T>
static void run_summary_query(const Dims &d, const void *Q, int L, float *qbar, hipStream_t st)
{
    const int blocks = d.B * d.S * ((d.d_qk / Elt<T>::EPC + SQ_CHUNKS - 1) / SQ_CHUNKS);
    if ((long)d.n_q * (d.H / d.S) <= SQ_WAVES_FEW * (WAVE / SQ_CHUNKS) || blocks >= SQ_MANY)
        summary_query_kernel<T, SQ_WAVES_FEW><<<blocks, SQ_WAVES_FEW * WAVE, 0, st>>>((const T *)Q, qbar, L, d.H, d.S, d.d_qk, d.n_q);
    else
        summary_query_kernel<T, SQ_WAVES><<<blocks, SQ_WAVES * WAVE, 0, st>>>((const T *)Q, qbar, L, d.H, d.S, d.d_qk, d.n_q);
}
hipError_t launch_summary_query(const Dims &d, const void *Q, int L, float *qbar, hipStream_t st)
{
    if (d.dtype == LCA_BF16) run_summary_query<uint16_t>(d, Q, L, qbar, st);
    else if (d.dtype == LCA_F16) run_summary_query<f16_t>(d, Q, L, qbar, st);
    else run_summary_query<float>(d, Q, L, qbar, st);
    return hipGetLastError();
}

// Whether a call takes condense_one_kernel: few groups (a workgroup and a half per CU), whose sets' queries a workgroup reads in about a microsecond.
// Two launches / one, us: 28 heads over 4 KV heads, g = 32 (57 KB of queries), L = 1500 9.8 / 7.5, L = 16000 (236 workgroups) 12.2 / 9.4, 24000 (360) 15.3 / 16.9;
// g = 16, L = 8192 9.3 / 6.9; 32 over 8, L = 6000 (312) 10.8 / 8.5, 10000 (568) 12.8 / 13.3; 64 / 64, four KV heads, L = 2500 8.4 / 6.1; fp32 128 + 32, g = 16, 4 heads (41 KB)
// 7.5 / 6.8, 8 heads (82 KB) 7.5 / 7.4, 16 heads 7.6 / 8.1; 256 + 32, 8 heads (74 KB) 10.5 / 9.0, g = 32 11.8 / 11.7.
// Groups of one load per component leave a workgroup little beside the queries: one workgroup per CU (128 / 128, one KV head, g = 4, twice L = 4283, 268 workgroups 6.8 / 7.4;
// 96 / 96, two, L = 6084, 350 workgroups 7.3 / 8.0; 128 / 128, one, L = 5452, 167 workgroups 7.1 / 5.8).
// Rows of 64 pieces are at home in condense_reg_kernel (512 + 64, one set of 2 heads 6.9 / 10.0); with three sets or more the kernel before would be the
// matrix-core one, whose start-up is long: 16 sets, L = 1200 15.2 / 9.8, 3000 (256 workgroups) 15.5 / 10.9, 5000 (512) 16.3 / 22.6, g = 32, L = 1200 18.4 / 15.7.
// One to three sets of narrow rows have few workgroups of little work: two launches / one over 340 random calls of groups of 8 and more 1.097 to 1.26 by the group size (64 / 64,
// one KV head, g = 32, L = 2574 7.4 / 5.7), but smaller groups, whose summary query is short too, are even (g = 2 1.025, g = 4 1.065) and some slower (96 / 80, g = 4, L = 194
// 5.9 / 6.2; g = 2, L = 108 5.9 / 6.3): two launches.
// condense_reg_kernel's own widths leave less to gain than the any-width kernel's where groups are small and the summary query is short: 16 bits, 128 / 128, groups of up to four
// rows and under 24 queries per set 1.04 times as long in one launch over 80 random calls (bf16, one KV head of four heads, g = 4, L = 88 5.0 / 5.8 us), from 28 queries on 0.90 to 1.01, g = 8 1.01 with 8 and 16
// queries and 0.91 with 24, g = 16 0.89 with 16; fp32 128 + 32, one set 1.03 (L = 202, g = 2, four heads 5.3 / 5.6).  With three sets and more that kernel takes the sets of a group in turn, which takes
// longer than a second workgroup on a CU: groups of one load, 264 workgroups, eight sets 12.8 / 7.2, four sets 0.80, two 1.04 (and 0.99 to 1.26 at the other widths).
static bool condense_in_one(const Dims &d)
{
    const int epc = 16 / d.elt, pool = d.d_pool / epc, sel = d.d_sel / epc, hps = d.H / d.S;
    // condense_reg_kernel would take the groups
    const bool own = d.g <= 32 && (d.g & (d.g - 1)) == 0 && d.pool_reduce == LCA_REDUCE_WEIGHTED && d.sel_reduce == LCA_REDUCE_MAXSEL;
    const bool gqa16 = own && d.mode == LCA_MODE_GQA && d.dtype != LCA_F32 && d.d_pool == 128 && d.d_sel == 128;
    const bool mla32 = own && d.mode == LCA_MODE_MLA && d.dtype == LCA_F32 && d.d_pool == 128 && d.d_sel == 32;
    const int pool_loads = Rows<float, 1>::loads(pool, d.g), sel_loads = Rows<float, 1>::loads(sel, d.g);
    const long wgs = (long)((d.m + ONE_WAVES - 1) / ONE_WAVES) * d.S * d.B, most = d.g <= 16 && pool <= 32 && (pool_loads + sel_loads > 2 || (mla32 && d.S >= 3)) ? 384 : 256;
    return wgs <= most && (long)d.n_q * hps * d.d_qk * d.elt <= 80 << 10 && d.d_qk <= ONE_COLUMNS && pool <= WAVE && sel <= WAVE && pool_loads <= 32 &&
           sel_loads <= (pool_loads <= 8 ? 8 : 4) && (pool <= 32 || d.S >= 3) && (pool + sel >= 24 || (long)d.B * d.S >= 4 || d.g >= 8) &&
           !((gqa16 || (mla32 && d.S == 1)) && d.g <= 4 && d.n_q * hps < 24);
}

hipError_t launch_condense(const CondenseArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    if (d.m == 0) return hipSuccess;        // nothing to condense, and nobody to read a summary query
    auto any = [&]() {
        return d.dtype == LCA_BF16 ? run_any<uint16_t>(a, st) : d.dtype == LCA_F16 ? run_any<f16_t>(a, st) : run_any<float>(a, st);
    };
    if (condense_in_one(d)) return d.dtype == LCA_BF16 ? run_one<uint16_t>(a, st) : d.dtype == LCA_F16 ? run_one<f16_t>(a, st) : run_one<float>(a, st);
    // 1. summary query (Algorithm 1, first step)
    hipError_t err = launch_summary_query(d, a.Q, d.L, a.qbar, st);
    if (err != hipSuccess) return err;
    // MLA widths, several sets, groups of whole 16-row tiles: scores and pooling on the matrix cores.  (Measured at 128K, g = 16,
    // this kernel / the register kernel below, summary query included: 52 / 40 us with one set, 52 / 51 with two, 55 / 72 with
    // four, 60 / 111 with eight, 72 / 190 with sixteen.)
    if (condense_mla_mfma_supported(d) && d.S >= 3) return launch_condense_mla_mfma(a, st);
    // 2. groups
    const bool mla = d.mode == LCA_MODE_MLA;
    // the register kernels implement the method's own strategies (weighted pooling, max selection); the ablation's others run any-width
    if (d.pool_reduce != LCA_REDUCE_WEIGHTED || d.sel_reduce != LCA_REDUCE_MAXSEL) return any();
    if (d.dtype == LCA_F16 && mla && d.d_pool == 512 && d.d_sel == 64 && try_reg<f16_t, 512, 64, true>(a, st, err)) return err;
    if (d.dtype == LCA_F16 && !mla && d.d_pool == 128 && d.d_sel == 128 && try_reg<f16_t, 128, 128, false>(a, st, err)) return err;
    if (d.dtype == LCA_BF16 && mla && d.d_pool == 512 && d.d_sel == 64 && try_reg<uint16_t, 512, 64, true>(a, st, err)) return err;
    if (d.dtype == LCA_BF16 && !mla && d.d_pool == 128 && d.d_sel == 128 && try_reg<uint16_t, 128, 128, false>(a, st, err)) return err;
    if (d.dtype == LCA_F32 && mla && d.d_pool == 128 && d.d_sel == 32 && try_reg<float, 128, 32, true>(a, st, err)) return err;
    return any();
}

}  // namespace lca

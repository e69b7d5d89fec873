// Decode step over a condensed cache at the MLA widths (d_c = 512, d_R = 64, bf16 or fp16; section 4.3 of the paper,
// decoding paragraph; absorbed form of section 3): the new token's query attends the m representatives and the
// k raw tail rows, and the (up to 16) heads of a condensed set share every cache row.
//
// One cache row of 1152 bytes feeds 16 heads x (576 + 512) multiply-adds, about 30 flops per byte: at HBM speed
// that is beyond the vector ALU, so the products run on the matrix cores with the heads as the 16 columns of
// 16x16x32 MFMAs:
//   S^T[key, head]  = K Q^T       A = 16 key rows from LDS (16-byte reads), B = Q^T in registers (18 k-steps)
//   O^T[dv, head]  += V^T P^T     A = V^T through LDS transpose reads,       B = P^T = exp2(S^T - ref)
// With long ranges every WAVEFRONT works alone on its own entries (no barriers in the loop; short ranges: see SHARED) with two 18 KB LDS buffers of its
// own: a tile is 16 entries (16 latent rows of 1 KB at a 1040-byte stride, the RoPE parts XOR-swizzled), copied with
// direct-to-LDS loads; the copy of tile t+1 is in flight while tile t is used -- twice: all 576 columns as keys, the
// first 512 as values.  S^T row m of the tile comes from LDS row 4(m%4) + m/4, so that the S^T accumulators already
// are the B fragments of the second product (16x16x16 MFMAs) when the transpose reads of a 16-lane block take rows 4
// apart (conflict-free on the 1040-byte stride).  Softmax keeps one fixed reference per head (taken at the first
// tile), so the 128 accumulation registers are never rescaled; if a row sum ends beyond 2^100 (or, in fp16, an
// exponential left the type's range and the sum is infinite) the wavefront collects the exact maximum of its range
// and runs it again.  The four wavefronts' results (reference, sum, unnormalised output per head) are merged in LDS
// into one partial result per workgroup; the workgroups' partial results are merged by decode_merge_kernel.
#include "lanes.h"
#include "lca_internal.h"
#include "mla_tile16.h"

namespace lca {
namespace {

using namespace tile16;

// A row sum beyond this (or not finite) makes the wavefront run its range again from the exact maxima.  The sum adds the
// ROUNDED exponentials, so one that left fp16's range (65504) arrives here as an infinity.
constexpr float SUM_LIMIT = 0x1p100f;

constexpr int NKS = DQK / 32;                   // 18 k-steps of S^T
constexpr int PV_GROUP = 8;                     // value tiles (of 16 columns) whose V^T fragments are requested together
constexpr int MROW = DP + 4;                    // floats per head of a wavefront's output in LDS (merge at the end)
static_assert(16 * MROW * 4 <= 2 * BUF_BYTES, "the output of 16 heads fits a wavefront's two tile buffers");
constexpr float NEG_BIG = -1.0e30f;
constexpr float LN2 = 0.6931471805599453f;

struct DmParams {
    const uint16_t *q, *pool_rep, *sel_rep, *pool_tail, *sel_tail;
    const uint8_t *pool_q8, *sel_q8;       // 8-bit representatives (E4M3 codes) and their row scales [.., m_cap, 2], or NULL
    const float *scales;
    float *part;
    void *O;                               // not NULL: one workgroup per (sequence, set), which then writes the final output itself
    int S, hps, m, k, n_parts, m_cap, k_cap, k_start;
    int wgs, tiles_per_part;               // workgroups of a (sequence, set); tiles of a wavefront
    unsigned wgs_magic;                    // 2^32 / wgs + 1: blockIdx / wgs in one multiplication
    float scale_log2, bias_log2;
};

// Two E4M3 codes (the low or the high half of w) times a power-of-two scale, as two elements of type E: exact.
template <typename E> __device__ __forceinline__ unsigned cvt2_fp8(unsigned w, float scale, bool high);
template <> __device__ __forceinline__ unsigned cvt2_fp8<__bf16>(unsigned w, float scale, bool high)
{
    return high ? __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, scale, true))
                : __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, scale, false));
}
template <> __device__ __forceinline__ unsigned cvt2_fp8<_Float16>(unsigned w, float scale, bool high)
{
    return high ? __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, scale, true))
                : __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, scale, false));
}
// 16 codes -> 16 elements (two 16-byte pieces)
template <typename E> __device__ __forceinline__ void cvt16_fp8(const uint4 &c, float scale, uint4 &lo, uint4 &hi)
{
    lo = make_uint4(cvt2_fp8<E>(c.x, scale, false), cvt2_fp8<E>(c.x, scale, true), cvt2_fp8<E>(c.y, scale, false), cvt2_fp8<E>(c.y, scale, true));
    hi = make_uint4(cvt2_fp8<E>(c.z, scale, false), cvt2_fp8<E>(c.z, scale, true), cvt2_fp8<E>(c.w, scale, false), cvt2_fp8<E>(c.w, scale, true));
}

// Q8: the representatives come as E4M3 codes with a power-of-two scale per row and component.  A tile then holds
// entries of one kind only (the list of tiles is the representatives' tiles followed by the tail's), and a tile of
// representatives is fetched into registers (its 8 KB + 1 KB of codes are contiguous) while the tile before it is used,
// converted -- one instruction per two codes, the row's scale riding along -- and written into the same LDS layout
// the 16-bit tiles use; from there on nothing differs.
//
// SHARED: the wavefronts of a workgroup take neighbouring tiles, a tile each per step, exchange P^T through LDS and every one works on a quarter of the
// value columns over all four tiles.  Nothing is left to merge over the wavefronts (2.9 of the 8.5 us that a workgroup of two steps takes), the
// accumulators are a quarter, and the first two tiles are requested at once; but two barriers per step keep the wavefronts' requests together, which
// long ranges pay for (see launch_decode_mla).
template <typename E, bool Q8, bool SHARED>
__global__ __launch_bounds__(256, 1) void decode_mla_kernel(const DmParams kp)
{
    constexpr int NDT = DP / 16 / (SHARED ? 4 : 1), STRIDE = SHARED ? 4 : 1;     // value tiles of a wavefront; from one of its tiles to the next
    typedef E ex8 __attribute__((ext_vector_type(8)));
    typedef E ex4 __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(1024))) char bufs[4][2][BUF_BYTES];
    __shared__ ex4 p_s[SHARED ? 4 : 1][64];                                 // P^T of a step: one tile per wavefront
    __shared__ float max_s[4][16], sum_s[4][16];                            // per wavefront and head

    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, q4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg_per_bs = kp.wgs, bs = wg_per_bs == 1 ? blockIdx.x : __umulhi(blockIdx.x, kp.wgs_magic), wg = blockIdx.x - bs * wg_per_bs;
    const int b = kp.S == 1 ? bs : bs / kp.S;
    const int m = kp.m, n = kp.m + kp.k;
    const int rep_tiles = Q8 ? (m + BN - 1) / BN : 0;                       // Q8: tiles [0, rep_tiles) hold representatives only
    const int tiles_total = Q8 ? rep_tiles + (kp.k + BN - 1) / BN : (n + BN - 1) / BN;
    const int tiles_per_part = kp.tiles_per_part;
    // tiles [t_lo, t_hi) of the workgroup (SHARED) or of the wavefront, which takes first, first + STRIDE, ..: `mine` of them
    const int t_lo = min((4 * wg + (SHARED ? 0 : wave)) * tiles_per_part, tiles_total), t_hi = min(t_lo + (SHARED ? 4 : 1) * tiles_per_part, tiles_total);
    const int steps = (t_hi - t_lo + STRIDE - 1) / STRIDE, first = t_lo + (SHARED ? wave : 0), mine = (t_hi - first + STRIDE - 1) / STRIDE;
    const int e_hi = Q8 ? n : min(n, t_hi * BN);
    const unsigned buf_lds = lds_address(bufs[wave][0]);

    // source rows: entry e < m is representative e, else tail token e - m in ring row (k_start + e - m) mod k_cap
    const uint16_t *prep = kp.pool_rep + (size_t)bs * kp.m_cap * DP, *srep = kp.sel_rep + (size_t)bs * kp.m_cap * DS;
    const uint16_t *ptail = kp.pool_tail + (size_t)b * kp.k_cap * DP, *stail = kp.sel_tail + (size_t)b * kp.k_cap * DS;
    auto ring_row = [&](int e) { const int t = kp.k_start + e - m; return t >= kp.k_cap ? t - kp.k_cap : t; };
    // first entry of tile tl and the end of the entries it may show (Q8: the end of its kind)
    auto is_q8 = [&](int tl) { return Q8 && tl < rep_tiles; };
    auto first_entry = [&](int tl) { return !Q8 ? tl * BN : tl < rep_tiles ? tl * BN : m + (tl - rep_tiles) * BN; };
    auto segment_end = [&](int tl) { return !Q8 ? e_hi : tl < rep_tiles ? m : n; };

    // per-lane LDS offsets inside a tile buffer
    const int krow = 4 * (col & 3) + (col >> 2);                            // LDS row behind S^T row `col` of the tile's 16 entries
    const int k_off = krow * RSB + 16 * q4;                                 // + 64*ks
    const int ksel_row = SEL_OFF + krow * (DS * 2);                         // chunk c at slot c ^ (row & 7)
    const int v_off = (4 * (col >> 2) + q4) * RSB + 8 * (col & 3) + (SHARED ? 32 * NDT * wave : 0);   // + 32*t: transpose read of 4 keys (rows 4 apart) x 4 columns

    ex8 qf[NKS];        // Q^T fragments
    floatx4 acc[NDT];
    float m_ref = NEG_BIG, l_run = 0.f, m_seen = NEG_BIG;
    const float c = kp.scale_log2;
    typedef __attribute__((address_space(3))) ex4 *lds_b64_ptr;

    // Q8: the codes of one tile of representatives in registers.  Load i brings rows 2i, 2i+1 of the latent part (lane l:
    // 16 codes at column 16 (l & 31) of row 2i + (l >> 5)), one more the RoPE part (lane l: 16 codes at column 16 (l & 3)
    // of row l >> 2); lane r < 16 holds the two scales of row r.  Rows past the end repeat the last one.
    uint4 q8_pool[BN / 2], q8_sel;
    float2 q8_scale = float2{1.f, 1.f};
    auto fetch_q8 = [&](int tl) {
        const uint8_t *pq = kp.pool_q8 + (size_t)bs * kp.m_cap * DP, *sq = kp.sel_q8 + (size_t)bs * kp.m_cap * DS;
        const int e0 = tl * BN;
#pragma unroll
        for (int i = 0; i < BN / 2; ++i) {
            const int e = min(e0 + 2 * i + (lane >> 5), m - 1);
            q8_pool[i] = *reinterpret_cast<const uint4 *>(pq + (size_t)e * DP + 16 * (lane & 31));
        }
        q8_sel = *reinterpret_cast<const uint4 *>(sq + (size_t)min(e0 + (lane >> 2), m - 1) * DS + 16 * (lane & 3));
        q8_scale = *reinterpret_cast<const float2 *>(kp.scales + ((size_t)bs * kp.m_cap + min(e0 + (lane & 15), m - 1)) * 2);
    };
    // ... converted (one instruction per two codes, the row's scale riding along) and written in the 16-bit layout
    auto convert_q8 = [&](char *buf) {
#pragma unroll
        for (int i = 0; i < BN / 2; ++i) {
            const float s0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, q8_scale.x), 2 * i));
            const float s1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, q8_scale.x), 2 * i + 1));
            uint4 lo, hi;
            cvt16_fp8<E>(q8_pool[i], lane < 32 ? s0 : s1, lo, hi);
            char *dst = buf + (2 * i + (lane >> 5)) * RSB + 32 * (lane & 31);
            *reinterpret_cast<uint4 *>(dst) = lo;
            *reinterpret_cast<uint4 *>(dst + 16) = hi;
        }
        const int r = lane >> 2, c0 = 2 * (lane & 3);                       // chunk c of row r sits at slot c ^ (r & 7)
        uint4 lo, hi;
        cvt16_fp8<E>(q8_sel, __shfl(q8_scale.y, r, 64), lo, hi);
        char *dst = buf + SEL_OFF + r * (DS * 2);
        *reinterpret_cast<uint4 *>(dst + ((c0 ^ (r & 7)) << 4)) = lo;
        *reinterpret_cast<uint4 *>(dst + (((c0 + 1) ^ (r & 7)) << 4)) = hi;
    };
    // 16-bit tiles: COPIES direct-to-LDS loads into tile buffer `bi` -- 16 latent rows (one load each) and the RoPE parts
    // of 8 rows per load; rows past the range repeat its last row
    auto issue_dma = [&](int tl, int bi) {
        const int e0 = first_entry(tl), seg_end = segment_end(tl), e_last = e0 + BN - 1;
        const unsigned dst = buf_lds + bi * BUF_BYTES;
        // the usual tile: 16 consecutive rows of one buffer (no end of range, no rep/tail seam, no wrap of the ring)
        const bool in_rep = e_last < m, in_tail = e0 >= m && ring_row(e0) + BN <= kp.k_cap;
        if (e_last < seg_end && (in_rep || in_tail)) {
            const size_t row0 = in_rep ? e0 : ring_row(e0);
            const char *pb0 = (const char *)((in_rep ? prep : ptail) + row0 * DP);
            const char *sb0 = (const char *)((in_rep ? srep : stail) + row0 * DS);
#pragma unroll
            for (int r = 0; r < BN; ++r) dma_row(lane * 16, pb0 + r * (DP * 2), dst + r * RSB);
#pragma unroll
            for (int j = 0; j < BN / 8; ++j) {
                const int r = 8 * j + (lane >> 3);
                dma_row(r * (DS * 2) + (((lane & 7) ^ (r & 7)) << 4), sb0, dst + SEL_OFF + 8 * j * (DS * 2));
            }
        } else {
#pragma unroll 4
            for (int r = 0; r < BN; ++r) {
                const int e = min(e0 + r, seg_end - 1);
                const uint16_t *src = e < m ? prep + (size_t)e * DP : ptail + (size_t)ring_row(e) * DP;
                dma_row(lane * 16, src, dst + r * RSB);
            }
#pragma unroll
            for (int j = 0; j < BN / 8; ++j) {
                const int r = 8 * j + (lane >> 3);
                const int e = min(e0 + r, seg_end - 1);
                const uint16_t *src = (e < m ? srep + (size_t)e * DS : stail + (size_t)ring_row(e) * DS) + (((lane & 7) ^ (r & 7)) << 3);
                dma_lanes(src, dst + SEL_OFF + 8 * j * (DS * 2));
            }
        }
    };
    auto issue = [&](int tl, int bi) {
        if (is_q8(tl)) fetch_q8(tl);
        else issue_dma(tl, bi);
    };
    // Q^T fragments: lane (col = head of the set, q4) holds q[head, 32 ks + 8 q4 .. +7]; columns past the set's heads are zero
    auto load_q = [&]() {
        const uint16_t *qp = kp.q + ((size_t)bs * kp.hps + min(col, kp.hps - 1)) * DQK + 8 * q4;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            qf[ks] = *reinterpret_cast<const ex8 *>(qp + 32 * ks);
            if (col >= kp.hps) qf[ks] = ex8{0, 0, 0, 0, 0, 0, 0, 0};
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[ks]));   // here, before the waits that count copies
    };
    // One sweep over the tiles, one per wavefront and step.  The tile of step `st` sits in buffer st & 1; the next one is on its way -- by
    // direct-to-LDS copy into the other buffer, or into the registers -- while `body` uses it.  (A tile of codes is never
    // followed by one before it in kind, so behind the copies of a 16-bit tile only copies of a 16-bit tile can be in flight.)
    // The queries travel together with the first tile: their latency is paid once.
    bool q_loaded = false;
    auto sweep = [&](auto &&body) {
        if constexpr (SHARED) {
            // The first two tiles are requested together (codes, whose registers hold one tile: in a step before the first), by the
            // same instructions as the others: code of their own would run once, and cold.
            int asked = 0;                                                  // tiles requested so far
            for (int st = Q8 ? -1 : 0; st < steps; ++st) {
                const int tl = first + STRIDE * st;
                char *buf = bufs[wave][st & 1];
                if (Q8 && st >= 0 && st < mine && is_q8(tl)) convert_q8(buf);
#pragma nounroll
                for (; asked < mine && asked <= st + 1; ++asked) issue(first + STRIDE * asked, asked & 1);
                if (!q_loaded) {
                    load_q();
                    q_loaded = true;
                }
                if (Q8 && st < 0) continue;
                if (st < mine && !is_q8(tl)) {
                    if (st + 1 < mine) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES) : "memory");   // this tile has landed, the next may still travel
                    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                }
                body(st, tl, buf);
            }
        } else {
            if (steps > 0) issue(first, 0);
            if (!q_loaded) load_q();
            q_loaded = true;
            for (int st = 0; st < steps; ++st) {
                const int tl = first + st;
                char *buf = bufs[wave][st & 1];
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // this wavefront's reads of the tiles before are done
                if (is_q8(tl)) {
                    convert_q8(buf);
                    if (st + 1 < steps) issue(tl + 1, (st & 1) ^ 1);
                } else if (st + 1 < steps) {
                    issue_dma(tl + 1, (st & 1) ^ 1);
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES) : "memory");
                } else {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                }
                body(st, tl, buf);
            }
        }
    };
    // S^T = K Q^T for the tile's 16 entries, and the logits in base 2 (scale, bias of the representatives, entries past the
    // range hidden): accumulator register r of this lane is entry 4 r + q4 of the tile
    auto tile_logits = [&](int tl, const char *buf, float (&lg)[4]) {
        const int e0 = first_entry(tl), seg_end = segment_end(tl);
        ex8 kf[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            const char *p = ks < DP / 32 ? buf + k_off + 64 * ks : buf + ksel_row + (((4 * (ks - DP / 32) + q4) ^ (krow & 7)) << 4);
            kf[ks] = *reinterpret_cast<const ex8 *>(p);
        }
        __builtin_amdgcn_sched_barrier(0);
        floatx4 sacc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) sacc = mfma_16x16x32(kf[ks], qf[ks], sacc);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = e0 + 4 * r + q4;                                  // accumulator row 4 q4 + r sits in LDS row 4 r + q4
            lg[r] = e < seg_end ? fmaf(sacc[r], c, e < m ? kp.bias_log2 : 0.f) : -INFINITY;
        }
    };
    auto head_max = [&](const float (&lg)[4]) {
        float mx = fmaxf(fmaxf(fmaxf(lg[0], lg[1]), fmaxf(lg[2], lg[3])), NEG_BIG);
        return lanes::across32(lanes::across16(mx, lanes::Max()), lanes::Max());
    };

    if constexpr (SHARED) {
        // The largest of a value over the wavefronts, per head (lane: head `col`); a barrier of the whole workgroup.
        auto across_max = [&](float v) {
            if (q4 == 0) max_s[wave][col] = v;
            __syncthreads();
            return fmaxf(fmaxf(max_s[0][col], max_s[1][col]), fmaxf(max_s[2][col], max_s[3][col]));
        };

        float l_all = 0.f;
        for (bool again = false;;) {                                            // normally one pass; a second one from the exact maxima
#pragma unroll
            for (int t = 0; t < NDT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
            l_run = 0.f;
            m_ref = again ? m_seen : NEG_BIG;
            bool ref_missing = !again;                                          // (the same in every wavefront)

            sweep([&](int st, int tl, const char *buf) {
                const int n_tiles = min(4, t_hi - t_lo - 4 * st);               // of this step
                float lg[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
                if (wave < n_tiles) tile_logits(tl, buf, lg);
                if (ref_missing) {                                              // the first step fixes the reference
                    const float mx = across_max(head_max(lg));
                    m_ref = (m_ref == NEG_BIG) ? mx : m_ref;
                    ref_missing = __builtin_amdgcn_ballot_w64(m_ref == NEG_BIG) != 0;
                }
                // P^T in the element type (B fragment of a 16x16x16 product: k-slot r of this lane is the key of register r) and
                // its sum (of the rounded values, the ones the second product sees)
                ex4 pb;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pb[r] = (E)__builtin_amdgcn_exp2f(lg[r] - m_ref);
                    l_run += (float)pb[r];
                }
                p_s[wave][lane] = pb;
                __syncthreads();                                                // every wavefront's P^T and tile are in LDS
                // O^T += V^T P^T: this wavefront's value columns over every tile of the step
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if (w < n_tiles) {
                        const ex4 pw = p_s[w][lane];
                        const char *const vals = bufs[w][st & 1] + v_off;
                        ex4 vf[NDT];
#pragma unroll
                        for (int t = 0; t < NDT; ++t) vf[t] = lds_read_tr16((lds_b64_ptr)(vals + 32 * t));
#pragma unroll
                        for (int t = 0; t < NDT; ++t) acc[t] = mfma_16x16x16(vf[t], pw, acc[t]);
                    }
                __syncthreads();                                                // the step's tiles and P^T may be overwritten
            });

            float l_tot = lanes::across32(lanes::across16(l_run, lanes::Sum()), lanes::Sum());
            if (q4 == 0) sum_s[wave][col] = l_tot;
            __syncthreads();
            l_all = (sum_s[0][col] + sum_s[1][col]) + (sum_s[2][col] + sum_s[3][col]);
            if (again || __builtin_amdgcn_ballot_w64(!(l_all <= SUM_LIMIT)) == 0) break;
            // (the same in every wavefront) a head ran out of exponent headroom: exact maxima of the workgroup's entries, then the pass again
            m_seen = NEG_BIG;
            sweep([&](int, int tl, const char *buf) {
                if (tl >= t_hi) return;
                float lg[4];
                tile_logits(tl, buf, lg);
                m_seen = fmaxf(m_seen, head_max(lg));
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // (nobody else reads this tile: no barrier before its buffer is filled again)
            });
            m_seen = across_max(m_seen);
            again = true;
        }

        // Every wavefront has the whole sums of its value columns, scaled to the reference all of them share: the final output where the
        // workgroup has the (sequence, set) to itself, else this workgroup's partial result (natural-log units).
        if (col >= kp.hps) return;
        const int x = 16 * NDT * wave + 4 * q4;
        if (kp.O != nullptr) {
            const float inv = 1.f / l_all;
            E *const dst = reinterpret_cast<E *>(kp.O) + ((size_t)bs * kp.hps + col) * DP + x;
#pragma unroll
            for (int t = 0; t < NDT; ++t) *reinterpret_cast<ex4 *>(dst + 16 * t) = ex4{(E)(acc[t][0] * inv), (E)(acc[t][1] * inv), (E)(acc[t][2] * inv), (E)(acc[t][3] * inv)};
            return;
        }
        float *const dst = kp.part + (((size_t)bs * wg_per_bs + wg) * kp.hps + col) * (DP + 2);
#pragma unroll
        for (int t = 0; t < NDT; ++t) {
            *reinterpret_cast<float2 *>(dst + 2 + x + 16 * t) = float2{acc[t][0], acc[t][1]};
            *reinterpret_cast<float2 *>(dst + 2 + x + 16 * t + 2) = float2{acc[t][2], acc[t][3]};
        }
        if (wave == 0 && q4 == 0) {
            dst[0] = steps <= 0 ? -INFINITY : m_ref * LN2;
            dst[1] = l_all;
        }
    } else {
        float l_tot = 0.f;
        for (bool again = false;;) {                                            // normally one pass; a second one from the exact maxima
#pragma unroll
            for (int t = 0; t < NDT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
            l_run = 0.f;
            m_ref = again ? m_seen : NEG_BIG;
            bool ref_missing = !again;

            sweep([&](int, int tl, const char *buf) {
                float lg[4];
                tile_logits(tl, buf, lg);
                if (ref_missing) {                                              // the first tile fixes the reference
                    const float mx = head_max(lg);
                    m_ref = (m_ref == NEG_BIG) ? mx : m_ref;
                    ref_missing = __builtin_amdgcn_ballot_w64(m_ref == NEG_BIG) != 0;
                }
                // P^T in the element type (B fragment of a 16x16x16 product: k-slot r of this lane is the key of register r) and
                // its sum (of the rounded values, the ones the second product sees)
                ex4 pb;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pb[r] = (E)__builtin_amdgcn_exp2f(lg[r] - m_ref);
                    l_run += (float)pb[r];
                }
                // O^T += V^T P^T: fragments of PV_GROUP value tiles requested together, one group ahead
                ex4 vf[2][PV_GROUP];
                auto request = [&](int grp, int bsel) {
#pragma unroll
                    for (int i = 0; i < PV_GROUP; ++i) vf[bsel][i] = lds_read_tr16((lds_b64_ptr)(buf + v_off + 32 * (grp * PV_GROUP + i)));
                };
                request(0, 0);
#pragma unroll
                for (int grp = 0; grp < NDT / PV_GROUP; ++grp) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (grp + 1 < NDT / PV_GROUP) request(grp + 1, (grp + 1) & 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < PV_GROUP; ++i) acc[grp * PV_GROUP + i] = mfma_16x16x16(vf[grp & 1][i], pb, acc[grp * PV_GROUP + i]);
                }
            });

            l_tot = lanes::across32(lanes::across16(l_run, lanes::Sum()), lanes::Sum());
            if (again || __builtin_amdgcn_ballot_w64(!(l_tot <= SUM_LIMIT)) == 0) break;
            // (wave-uniform) a head ran out of exponent headroom: exact maxima of the range, then the pass again
            m_seen = NEG_BIG;
            sweep([&](int, int tl, const char *buf) {
                float lg[4];
                tile_logits(tl, buf, lg);
                m_seen = fmaxf(m_seen, head_max(lg));
            });
            again = true;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                      // the last tile's reads are done before the buffers are reused

        // The four wavefronts' results (reference, sum, unnormalised output per head) are merged here, through LDS, so that
        // one partial result per workgroup goes to memory: each wavefront publishes its references and sums and leaves its
        // accumulators as they are in its own (now idle) tile buffer; then wavefront w adds up value columns
        // [128 w, 128 w + 128) of every head over the four buffers, scaled to the common reference on the way, and writes
        // them: as this workgroup's partial result (natural-log units), or -- when the workgroup has the whole (sequence, set)
        // to itself -- normalised, as the final output.  Four heads' sixteen reads are in flight together: one head after another, with the
        // accumulators rescaled before they were written, the merge took 7 500 of the 19 400 cycles of a two-tile step.
        const bool any = t_lo < t_hi;
        {
            float *mine = reinterpret_cast<float *>(bufs[wave][0]) + col * MROW + 4 * q4;   // [head][MROW] floats, 33 KB of the two buffers' 36.5 KB
#pragma unroll
            for (int t = 0; t < NDT; ++t) *reinterpret_cast<floatx4 *>(mine + 16 * t) = acc[t];
        }
        if (q4 == 0) {
            max_s[wave][col] = any ? m_ref : -INFINITY;
            sum_s[wave][col] = any ? l_tot : 0.f;
        }
        __syncthreads();
        float m_all = -INFINITY, l_all = 0.f, factor[4];                        // of head `col`
#pragma unroll
        for (int w = 0; w < 4; ++w) m_all = fmaxf(m_all, max_s[w][col]);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = max_s[w][col];
            factor[w] = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - m_all);
            l_all += sum_s[w][col] * factor[w];
        }
        const float inv = 1.f / l_all;
        float *dst0 = kp.part + ((size_t)bs * wg_per_bs + wg) * kp.hps * (DP + 2);
        const int x = 128 * wave + 2 * lane;
        auto of_head = [](float v, int h) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), h)); };   // (lane h: head h)
        for (int h0 = 0; h0 < kp.hps; h0 += 4) {
            float2 v[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int w = 0; w < 4; ++w) v[i][w] = *reinterpret_cast<const float2 *>(reinterpret_cast<const float *>(bufs[w][0]) + (h0 + i) * MROW + x);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int h = h0 + i;
                if (h >= kp.hps) break;
                float2 sum = float2{0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float f = of_head(factor[w], h);
                    sum.x = fmaf(v[i][w].x, f, sum.x);
                    sum.y = fmaf(v[i][w].y, f, sum.y);
                }
                if (kp.O != nullptr) {
                    typedef E ex2 __attribute__((ext_vector_type(2)));
                    const float n = of_head(inv, h);
                    *reinterpret_cast<ex2 *>(reinterpret_cast<E *>(kp.O) + ((size_t)bs * kp.hps + h) * DP + x) = ex2{(E)(sum.x * n), (E)(sum.y * n)};
                } else {
                    *reinterpret_cast<float2 *>(dst0 + (size_t)h * (DP + 2) + 2 + x) = sum;
                }
            }
        }
        if (kp.O != nullptr) return;
        if (wave == 0 && q4 == 0 && col < kp.hps) {
            float *dst = dst0 + (size_t)col * (DP + 2);
            dst[0] = m_all == -INFINITY ? -INFINITY : m_all * LN2;
            dst[1] = l_all;
        }
    }
}

}  // namespace

bool decode_mla_supported(const Dims &d)
{
    const int hps = d.H / d.S;
    return (d.dtype == LCA_BF16 || d.dtype == LCA_F16) && d.mode == LCA_MODE_MLA && d.d_pool == DP && d.d_sel == DS && hps <= 16 && d.scale > 0.f;
}

// Wavefronts per (sequence, set), a multiple of 4 (a workgroup's, which leave one partial result): four tiles for each, where
// the cache is long enough to fill the chip that way, never more workgroups than CUs (a second round costs as much as the
// first).  A short or lonely cache is bound by the chain of tiles a wavefront works through: two tiles for each while the
// workgroups stay below 160, one while they stay below 200 and the merge has few results to add: 16 of a full set of heads (33 KB each), or 48 where there are
// fewer than 92 workgroups or fewer than eight heads.  (Two / one tile each at 17 to 48 results: 1 to 7 heads, up to 200 workgroups, 91 random calls 1.01 to 1.16, H = 4, B = 1, 20 results
// 9.8 / 8.7 us, B = 8, 20 9.4 / 8.9, B = 4, 48 10.3 / 9.9; beyond 48 the gain ends, 7 heads, B = 2, 64 1.01, B = 3 1.00.  8 to 12 heads up to 92 workgroups 1.02 to 1.11, beyond from
// 1.07 to 0.95; 16 heads, B = 1, 36 1.08, 48 1.02, 56 1.00, B = 2, 40 (80 workgroups) 1.02, B = 4, 24 (96) 0.98, B = 8, 24 0.92.)  Measured with the wavefronts of a workgroup sharing its tiles (step with merge, 16 heads, 16 bits; four / two / one tile each): B = 1, L = 700 13.8 /
// 10.7 / 9.7 us, L = 4001 14.3 / 11.1 / 10.4, L = 16000 14.1 / 11.5 / 11.1, L = 131072 16.1 / 14.9 / 17.1; two / one: B = 2, L = 8000 11.7 / 10.8 (46 workgroups), B = 4,
// L = 4001 11.7 / 11.4 (76), L = 8000 11.8 / 11.7 (92), but B = 3, L = 16000 11.9 / 12.0 (93), B = 6, L = 4001 11.9 / 11.9 (114), B = 8, L = 4001 12.5 / 12.8 (152); B = 16,
// L = 4001 15.9 / 14.1 / 15.7; B = 32, L = 700 15.9 / 14.4 / 18.1 (96, 192, 352 workgroups), L = 1500 17.3 / 20.7 / 20.6; B = 150, L = 20000 96 us with two workgroups
// per sequence (300 on 256 CUs), 71.5 us with one.
// Up to 16 tiles one workgroup takes them all: it writes the output itself, and the merge's launch costs more than a chain of up to
// four tiles is long (one workgroup / two tiles / one tile each: B = 1, L = 80 7.6 / 7.6 / 9.0, 160 9.2 / 10.5 / 9.2; B = 60, L = 160 9.6 / 12.4 / 12.5; not any more at
// the end of that range, 250 11.5 / 10.6 / 9.3).
int decode_mla_parts(const Dims &d)
{
    const int tiles = (d.m + BN - 1) / BN + (d.k + BN - 1) / BN;      // (an upper bound when the two kinds share tiles)
    const long pairs = (long)d.B * d.S;
    auto wgs_for = [&](int per_wave) { return (tiles + 4 * per_wave - 1) / (4 * per_wave); };
    int wgs = wgs_for(4);
    if (wgs == 1) return 4;
    if (wgs_for(1) <= 48 && pairs * wgs_for(1) <= (wgs_for(1) <= 16 || d.H / d.S < 8 ? 200 : 92)) wgs = wgs_for(1);
    else if (pairs * wgs_for(2) <= 160) wgs = wgs_for(2);
    const long most = pairs >= 256 ? 1 : 256 / pairs;
    if (wgs > most) wgs = (int)most;
    if (wgs < 1) wgs = 1;
    return 4 * wgs;
}

// Tiles per wavefront up to which the wavefronts of a workgroup share them: two, or four where the workgroup has the (sequence, set) to itself (nothing
// else of a chip-filling grid then waits at its barriers).  Alone / shared, 16 heads: one tile B = 1, L = 700 11.2 / 9.6 us; two B = 1, L = 4001 12.2 / 10.9,
// L = 131072 15.8 / 14.7, B = 8, L = 20000 14.9 / 13.8, 8-bit B = 1, L = 6000 13.0 / 11.6; three B = 16, L = 30000 18.6 / 19.4, but B = 60, L = 160, one workgroup
// each, 10.3 / 9.3; four B = 32, L = 1000 16.5 / 17.8, B = 10, L = 250, one workgroup each, 11.6 / 11.5; eighteen B = 32, L = 131072 66.4 / 69.5.
constexpr int SHARED_STEPS = 2, SHARED_STEPS_ONE = 4;
template <typename E, bool Q8> static void run(const DmParams &kp, unsigned grid, int steps, hipStream_t st)
{
    if (steps <= (kp.n_parts == 4 ? SHARED_STEPS_ONE : SHARED_STEPS)) decode_mla_kernel<E, Q8, true><<<grid, 256, 0, st>>>(kp);
    else decode_mla_kernel<E, Q8, false><<<grid, 256, 0, st>>>(kp);
}

hipError_t launch_decode_mla(const DecodeArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    DmParams kp;
    kp.q = (const uint16_t *)a.q; kp.pool_rep = (const uint16_t *)a.pool_rep; kp.sel_rep = (const uint16_t *)a.sel_rep;
    kp.pool_tail = (const uint16_t *)a.pool_tail; kp.sel_tail = (const uint16_t *)a.sel_tail; kp.part = a.part;
    kp.S = d.S; kp.hps = d.H / d.S; kp.m = d.m; kp.k = d.k; kp.n_parts = a.splits;
    kp.m_cap = a.m_cap; kp.k_cap = a.k_cap; kp.k_start = a.k_start;
    kp.scale_log2 = d.scale * 1.4426950408889634f;
    kp.bias_log2 = d.rep_logit_bias * 1.4426950408889634f;
    kp.pool_q8 = a.pool_q8; kp.sel_q8 = a.sel_q8; kp.scales = a.scales;
    kp.O = a.splits == 4 ? a.O : nullptr;
    const unsigned grid = d.B * d.S * (a.splits / 4);
    const bool q8 = a.pool_q8 != nullptr;
    const int tiles = q8 ? (d.m + BN - 1) / BN + (d.k + BN - 1) / BN : (d.m + d.k + BN - 1) / BN, steps = (tiles + a.splits - 1) / a.splits;
    kp.wgs = a.splits / 4;
    kp.wgs_magic = kp.wgs > 1 ? (unsigned)((1ull << 32) / (unsigned)kp.wgs + 1) : 0u;      // (exact: several workgroups share a pair only in grids of up to 256)
    kp.tiles_per_part = steps;
    if (d.dtype == LCA_F16) {
        if (q8) run<_Float16, true>(kp, grid, steps, st);
        else run<_Float16, false>(kp, grid, steps, st);
    } else {
        if (q8) run<__bf16, true>(kp, grid, steps, st);
        else run<__bf16, false>(kp, grid, steps, st);
    }
    return hipGetLastError();
}

}  // namespace lca

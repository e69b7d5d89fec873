// Tiled attention kernel on the matrix cores for the shapes that have no kernel of their own: fp32, heads narrower or wider
// than the two layer widths, any scale.  Prefill over the condensed context (section 4.3, Eq. 10; per-query partition of
// appendix A.2) and, with dense = 1, plain causal attention (section 3, Eq. 5).
//
// What these shapes need is parallelism and reuse, not the last MFMA: one wavefront per query row, every key element a
// scalar load of its own, took 128 us for 0.36 GFLOP in fp32 (L = 1024, 4 heads, 128 + 32) and 1.44 ms for 5.3 GFLOP in bf16
// (L = 2500, 16 heads over 4 KV heads, 64 / 64).  With the condensation before it the first takes 20.4 us now (launches, memory latency, a chain of
// fp32 products per tile), the second 32.0 us (vector ALU: exponentials and the splitting of the probabilities).  Two things the compiler does
// are kept from it below, each of which had every tile wait for the next one's loads (21.9 and 38.5 us; fp32, 8 heads, L = 4096 153 us, now 128;
// bf16 256 + 32, 8 heads, two times L = 4000 182, now 156): the queries' arrival left open until the loop, and load offsets computed in the
// registers that loads fill.  Here
//   * a workgroup owns 16 QB query rows of one condensed set, numbered (token, head of the set): the heads of a set see the
//     same keys, so the rows of a workgroup span few tokens;
//   * its wavefronts split the KEY tiles among them, each with a softmax (a reference that follows the maximum) of its own, and are merged through
//     LDS at the end: small problems, where a row sees a few hundred entries, still fill the chip, and nothing in the loop
//     waits for another wavefront;
//   * a tile (16 NB entries) travels memory -> registers -> the wavefront's own LDS area one tile ahead of its use, as
//     16-byte pieces; rows are an odd number of 16-byte pieces apart, which spreads the key reads (16 rows, one piece
//     each) and the value reads (rows 4 apart) over all banks;
//   * products are computed transposed as in the other kernels: S^T[key, row] = K Q^T and O^T[dv, row] += V^T P^T with 16x16
//     MFMAs, a lane's accumulator registers being one row's logits and, as they are, the operand of the second product.
//
// Precision is that of fp32 arithmetic throughout.  fp32 data uses the fp32 matrix instructions.  16-bit data is exact as an
// operand; the fp32 probabilities are not, so the second product takes them in three parts that add up to all their 24 bits: bf16
// 8 + 8 + 8, fp16 11 + 11 + 2.  (fp16 parts are of 2^15 p: whole down to p = 2^-16, below that cut off at 2^-40, the last bit
// of 2^-16.  Two fp16 parts, and the 2^15 put into the exponential's argument, whose last bit that costs four binades, left an error of
// 2^-21.4 of p where it is 2^-24 now, as in bf16 and fp32; the attention at B = 1, L = 2500, 16 heads over 4 KV heads, 64 / 64: 27.7 us so, 29.5 us
// with all the bits.)
//
// The matrix product multiplies entries a row does not see by a zero probability; an infinity or a NaN in such an entry
// would reach the row.  So if any result of the workgroup is not finite its rows are redone one by one (attn_row.h), each
// touching only the entries it sees.
#include "attn_row.h"
#include "mla_tile16.h"

namespace lca {
namespace {

using attn_row::RowParams;
using tile16::bf16x4;
using tile16::bf16x8;
using tile16::f16x4;
using tile16::f16x8;
using tile16::floatx4;
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// Wavefronts per workgroup at most: eight in fp32 where two of them fit a SIMD's registers (its tiles are long chains of small products).
template <typename T> constexpr int max_waves(int ndt) { return sizeof(T) == 4 && ndt <= 8 ? 8 : 4; }
// fp32 at 512 columns: queries, accumulators and the next tile are 416 of a lane's 512 registers, and with the rest some are kept in memory.
template <typename T> constexpr bool full_class(int ndt) { return sizeof(T) == 4 && ndt >= 32; }
constexpr int RSRC_WORD3 = 0x00020000;   // raw buffer of dwords, gfx9 layout
constexpr size_t LDS_BYTES = 160 * 1024;      // of a CU

// Per element type: columns of one fragment chunk (a 16-byte piece per lane, four lanes deep), and the two products.
template <typename T> struct Mma;
template <typename E8, typename E4, typename E, int NPARTS> struct Mma16 {
    static constexpr int EPC = 8, CHUNK = 32, PARTS = NPARTS;
    // LDS row behind S^T row m of a block of 16, and the entry that accumulator register r of lane group q4 stands for: the
    // transpose reads of the value operand take rows 4 apart
    __device__ static int row_of_m(int m) { return 4 * (m & 3) + (m >> 2); }
    __device__ static int entry(int r, int q4) { return 4 * r + q4; }
    __device__ static floatx4 score(const uintx4 &k, const uintx4 &q, floatx4 c)
    {
        return tile16::mfma_16x16x32(__builtin_bit_cast(E8, k), __builtin_bit_cast(E8, q), c);
    }
    template <int NB> struct Parts { E4 v[NPARTS][NB]; };
    template <int NB> struct Frag { E4 v[NB]; };
    // `base`: the tile's first value row; V^T fragment of value columns 16 t .. 16 t + 15
    template <int NB> __device__ static Frag<NB> value(const char *base, int rs, int t, int col, int q4)
    {
        typedef __attribute__((address_space(3))) E4 *lds_ptr;
        Frag<NB> f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            f.v[b] = tile16::lds_read_tr16((lds_ptr)(base + (16 * b + 4 * (col >> 2) + q4) * rs + 8 * (col & 3) + 32 * t));
        return f;
    }
    template <int NB> __device__ static floatx4 accumulate(const Frag<NB> &v, const Parts<NB> &p, int part, floatx4 c)
    {
        if constexpr (NB == 2) {
            return tile16::mfma_16x16x32(__builtin_shufflevector(v.v[0], v.v[1], 0, 1, 2, 3, 4, 5, 6, 7),
                                         __builtin_shufflevector(p.v[part][0], p.v[part][1], 0, 1, 2, 3, 4, 5, 6, 7), c);
        } else {
            return tile16::mfma_16x16x16(v.v[0], p.v[part][0], c);
        }
    }
};
template <> struct Mma<uint16_t> : Mma16<bf16x8, bf16x4, __bf16, 3> {
    static constexpr float P_SCALE = 1.f;          // what the probabilities are multiplied by on their way into the second product
    static constexpr float REF_SLACK = 8.f;        // binades a row's maximum may be above the reference of its exponentials
    // p = its leading 8 bits + the next 8 + the last 8 (cut off, not rounded: a subtraction each and one byte
    // permutation per pair)
    template <int NB> __device__ static void split(const float (&p)[NB][4], Parts<NB> &o)
    {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            unsigned x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = __float_as_uint(p[b][r]);
#pragma unroll
            for (int i = 0; i < PARTS; ++i) {
                typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
                o.v[i][b] = __builtin_bit_cast(bf16x4, uintx2{__builtin_amdgcn_perm(x[1], x[0], 0x07060302u), __builtin_amdgcn_perm(x[3], x[2], 0x07060302u)});
                if (i + 1 < PARTS) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = __float_as_uint(__uint_as_float(x[r]) - __uint_as_float(x[r] & 0xffff0000u));
                }
            }
        }
    }
    __device__ static void store4(uint16_t *p, const floatx4 &v)
    {
        *reinterpret_cast<bf16x4 *>(p) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    }
};
template <> struct Mma<f16_t> : Mma16<f16x8, f16x4, _Float16, 3> {
    static constexpr float P_SCALE = 32768.f;      // (an exact product; the results are divided by it with the row's sum)
    static constexpr float REF_SLACK = 0.f;        // (2^15 p may not pass 65504)
    // 2^15 p = its leading 11 bits + the next 11 + the last 2 (cut off, not rounded: one conversion per pair)
    template <int NB> __device__ static void split(const float (&p)[NB][4], Parts<NB> &o)
    {
        typedef __fp16 half2 __attribute__((ext_vector_type(2)));
        typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                float x = p[b][r] * P_SCALE, y = p[b][r + 1] * P_SCALE;
#pragma unroll
                for (int i = 0; i < PARTS; ++i) {
                    const half2 cut = __builtin_amdgcn_cvt_pkrtz(x, y);
                    const f16x2 h = __builtin_bit_cast(f16x2, cut);
                    o.v[i][b][r] = h[0];
                    o.v[i][b][r + 1] = h[1];
                    x -= (float)h[0];
                    y -= (float)h[1];
                }
            }
    }
    __device__ static void store4(f16_t *p, const floatx4 &v)
    {
        *reinterpret_cast<f16x4 *>(p) = f16x4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
    }
};
template <> struct Mma<float> {
    static constexpr int EPC = 4, CHUNK = 16, PARTS = 1;
    static constexpr float P_SCALE = 1.f, REF_SLACK = 8.f;
    __device__ static int row_of_m(int m) { return m; }
    __device__ static int entry(int r, int q4) { return 4 * q4 + r; }
    __device__ static floatx4 score(const uintx4 &k, const uintx4 &q, floatx4 c)
    {
        const floatx4 a = __builtin_bit_cast(floatx4, k), b = __builtin_bit_cast(floatx4, q);
#pragma unroll
        for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
        return c;
    }
    template <int NB> struct Parts { float v[NB][4]; };
    template <int NB> __device__ static void split(const float (&p)[NB][4], Parts<NB> &o)
    {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) o.v[b][r] = p[b][r];
    }
    template <int NB> struct Frag { float v[NB][4]; };
    template <int NB> __device__ static Frag<NB> value(const char *base, int rs, int t, int col, int q4)
    {
        Frag<NB> f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) f.v[b][r] = *reinterpret_cast<const float *>(base + (16 * b + 4 * q4 + r) * rs + 4 * (16 * t + col));
        return f;
    }
    template <int NB> __device__ static floatx4 accumulate(const Frag<NB> &v, const Parts<NB> &p, int, floatx4 c)
    {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f32_16x16x4f32(v.v[b][r], p.v[b][r], c, 0, 0, 0);
        return c;
    }
    __device__ static void store4(float *p, const floatx4 &v) { *reinterpret_cast<floatx4 *>(p) = v; }
};

// Division by a number known on the host: two multiplications by 2^64 / d + 1, exact for every 32-bit x, where a division is thirty-odd
// instructions, of which a workgroup would issue a dozen before its first load.
struct Div {
    unsigned lo, hi, one;                // the 64-bit factor; all ones for d = 1, whose factor has 65 bits
    template <bool PLAIN> __device__ int of(unsigned x, unsigned d) const      // (PLAIN: an ordinary division by d all the same)
    {
        if constexpr (PLAIN) return (int)(x / d);
        else return (int)((x & one) | ((unsigned)(((unsigned long long)x * hi + __umulhi(x, lo)) >> 32) & ~one));
    }
};
static Div make_div(unsigned d)
{
    const unsigned long long f = ~0ull / d + 1;           // (d = 1: not used; a power of two: exactly 2^64 / d)
    return Div{(unsigned)f, (unsigned)(f >> 32), d == 1 ? ~0u : 0u};
}

template <typename T> struct TileParams {
    RowParams<T> r;
    int n_blocks;                        // workgroups per (sequence, set)
    Div by_blocks, by_s, by_hps, by_g;
};

// Byte layout of one wavefront's LDS area, the same on both sides of the launch.
template <typename T, int NDT, int NKC, int QB, int NB> struct Layout {
    int rsk, rsv, v_off, sel_off, cp, nc;      // row strides, start of the value rows, of the selected part in a key row; 16-byte pieces per row
    int stage, area;                           // bytes of a tile; of the area (the merge and the row-by-row path use it too)
    __host__ __device__ Layout(int d_pool, int d_sel, int mla)
    {
        constexpr int ELT = (int)sizeof(T), MERGE = 16 * QB * (16 * NDT + 4) * 4;
        cp = d_pool * ELT / 16;
        nc = cp + d_sel * ELT / 16;
        rsk = NKC * 64 + 16;                                    // an odd number of 16-byte pieces
        rsv = mla ? rsk : (d_pool * ELT + 63) / 64 * 64 + 16;
        v_off = mla ? 0 : 16 * NB * rsk;
        sel_off = mla ? cp * 16 : 0;
        stage = 16 * NB * (rsk + (mla ? 0 : rsv)) + NDT * 16 * ELT;      // (value reads of a partial last column block may pass the last row's end)
        const int row = ((mla ? d_pool + d_sel : d_sel) + attn_row::WAVE) * 4;
        area = stage > MERGE ? stage : MERGE;
        area = area > row ? area : row;
        area = (area + 63) / 64 * 64;
    }
};

// Largest / sum over the four lanes (l, l ^ 16, l ^ 32, l ^ 48) that hold one query row, by swapping rows of sixteen lanes
// between two copies (no LDS traffic).
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float row_max4(float x)
{
    const uintx2 a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uintx2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float row_sum4(float x)
{
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

// NDT: value columns / 16, NKC: key columns / Mma::CHUNK (both upper bounds; what lies past the real widths is zero keys and
// results nobody stores), QB: blocks of 16 query rows, NB: blocks of 16 entries per tile, NIT: 16-byte pieces of a
// row / 16 (upper bound).  LATE: the 512-column fp32 class's second form (see late_form).
template <typename T, int NDT, int NKC, int QB, int NB, int NIT, bool LATE>
__global__ __launch_bounds__(64 * max_waves<T>(NDT)) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 && NDT <= 4 ? 3 : NDT <= 8 || (sizeof(T) == 2 && NDT <= 16) ? 2 : 1, 8)))
void attn_tile_kernel(const TileParams<T> tp)
{
    typedef Mma<T> M;
    const RowParams<T> &kp = tp.r;
    extern __shared__ __attribute__((aligned(64))) char smem[];
    constexpr int TK = 16 * NB, ROWS = 16 * QB, MROW = 16 * NDT + 4;
    constexpr bool FULL = full_class<T>(NDT);
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, q4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = blockDim.x >> 6;
    const Layout<T, NDT, NKC, QB, NB> lay(kp.d_pool, kp.d_sel, kp.mla);
    char *const area = smem + wave * lay.area;

    // which rows: the latest (heaviest) first
    const int hps = kp.H / kp.S, L = kp.L, g = kp.g;
    const int bs = tp.by_blocks.template of<LATE>(blockIdx.x, tp.n_blocks), blk = tp.n_blocks - 1 - (int)(blockIdx.x - bs * tp.n_blocks), b = tp.by_s.template of<LATE>(bs, kp.S), s = bs - b * kp.S;
    const int n_rows = L * hps, r0 = blk * ROWS, r_last = min(r0 + ROWS, n_rows) - 1;
    const int w_seen = kp.dense ? L : kp.w;                // raw tokens a row sees before it sees a representative
    auto visible = [&](int t) { return tp.by_g.template of<LATE>(max(t + 1 - w_seen, 0), g); };
    const int t_first = tp.by_hps.template of<LATE>(r0, hps), t_last = tp.by_hps.template of<LATE>(r_last, hps);
    const int mt_first = visible(t_first), n_rep = visible(t_last), raw0 = mt_first * g;
    const int rep_tiles = (n_rep + TK - 1) / TK, n_tiles = rep_tiles + (t_last + 1 - raw0 + TK - 1) / TK;
    const int d_qk = kp.mla ? kp.d_pool + kp.d_sel : kp.d_sel;
    const float c = kp.scale * 1.4426950408889634f, bias2 = kp.rep_bias * 1.4426950408889634f;

    int t_row[QB], mt_row[QB];
    size_t q_row[QB];                    // row index of the query in Q, O and lse: (b L + t) H + h
    bool live[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int r = r0 + 16 * qb + col, rc = min(r, n_rows - 1), t = tp.by_hps.template of<LATE>(rc, hps);
        live[qb] = r < n_rows;
        t_row[qb] = t;
        mt_row[qb] = visible(t);
        q_row[qb] = ((size_t)b * L + t) * kp.H + s * hps + (rc - t * hps);
    }

    // the pieces of one tile in registers: lane = (row of four, piece of sixteen of both components), or, where either component
    // has at most eight (NIT == 1), lane = (row of eight, piece of eight) for one component after the other: with both in one row of
    // lanes each needs a load of its own all the same (its descriptor), half of whose lanes are idle (condensation + attention at 64 / 64,
    // 16 heads over 4 KV heads, L = 2500: 40.8 us so, 38.9 us as it is).  Loads go through buffer descriptors: the
    // address of a load is a scalar plus an offset that the lane keeps, and rows past a segment's end read as zeros (hidden
    // below).  With 64-bit addresses per load a third of the loop's issue time was integer multiplication.
    const int sub = lane & 15, rr = lane >> 4, p = kp.mla ? 0 : s;
    constexpr int ELT = (int)sizeof(T);
    const int pool_bytes = kp.d_pool * ELT, sel_bytes = kp.d_sel * ELT;
    const T *const rep_p = kp.pool_rep + ((size_t)b * kp.S + s) * kp.m * kp.d_pool, *const rep_s = kp.sel_rep + ((size_t)b * kp.S + s) * kp.m * kp.d_sel;
    const T *const raw_p = kp.POOL + ((size_t)b * L * kp.P + p) * kp.d_pool, *const raw_s = kp.SEL + ((size_t)b * L * kp.P + p) * kp.d_sel;
    static_assert(NIT > 1 || (16 * NDT <= 8 * M::EPC && NKC * M::CHUNK <= 8 * M::EPC), "at most eight pieces per component");
    const int r8 = lane >> 3, x8 = lane & 7, ncs = lay.nc - lay.cp;
    uintx4 held[4 * NB][NIT];
    // The lane's offsets in a tile of the kind in hand, taken again only where the kind changes: computed beside the loads, they went into registers
    // of the previous tile's pieces, and the wait that needs covered the loads just issued -- a round trip to memory in every tile.
    int voff[NIT == 1 ? 2 : NIT], kind = -1;
    auto set_kind = [&](bool is_rep) {
        const int ps = (is_rep ? 1 : kp.P) * pool_bytes, ss = (is_rep ? 1 : kp.P) * sel_bytes;
        if constexpr (NIT == 1) {
            voff[0] = r8 * ps + x8 * 16;
            voff[1] = r8 * ss + x8 * 16;
        } else {
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int x = sub + 16 * it;
                voff[it] = x < lay.cp ? rr * ps + x * 16 : rr * ss + (x - lay.cp) * 16;
            }
        }
        kind = is_rep;
    };
    auto load_tile = [&](int tile) {
        const bool is_rep = tile < rep_tiles;
        if (kind != (int)is_rep) set_kind(is_rep);
#pragma unroll
        for (int &v : voff) asm volatile("" : "+v"(v));
        const unsigned e0 = is_rep ? tile * TK : raw0 + (tile - rep_tiles) * TK, step = is_rep ? 1 : kp.P, last = is_rep ? n_rep - 1 : t_last;
        const unsigned ps = step * pool_bytes, ss = step * sel_bytes;           // bytes between rows of the segment
        const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc((void *)(is_rep ? rep_p : raw_p), (short)0, last * ps + pool_bytes, RSRC_WORD3);
        const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc((void *)(is_rep ? rep_s : raw_s), (short)0, last * ss + sel_bytes, RSRC_WORD3);
        if constexpr (NIT == 1) {
            if (x8 < lay.cp) {
#pragma unroll
                for (int i = 0; i < 2 * NB; ++i) held[i][0] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(prs, voff[0], (e0 + 8 * i) * ps, 0));
            }
            if (x8 < ncs) {
#pragma unroll
                for (int i = 0; i < 2 * NB; ++i) held[2 * NB + i][0] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(srs, voff[1], (e0 + 8 * i) * ss, 0));
            }
            return;
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int x = sub + 16 * it;
            if (x < lay.cp) {
#pragma unroll
                for (int i = 0; i < 4 * NB; ++i) held[i][it] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(prs, voff[it], (e0 + 4 * i) * ps, 0));
                asm volatile("; pooled part");       // (keeps the two branches apart: merged into one load, the descriptor would be a per-lane choice)
            } else if (x < lay.nc) {
#pragma unroll
                for (int i = 0; i < 4 * NB; ++i) held[i][it] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(srs, voff[it], (e0 + 4 * i) * ss, 0));
                asm volatile("; selected part");
            }
        }
    };
    auto store_tile = [&]() {
        if constexpr (NIT == 1) {
            char *const vdst = area + lay.v_off + x8 * 16 + r8 * lay.rsv, *const kdst = area + lay.sel_off + x8 * 16 + r8 * lay.rsk;
            if (x8 < lay.cp) {
#pragma unroll
                for (int i = 0; i < 2 * NB; ++i) *reinterpret_cast<uintx4 *>(vdst + 8 * i * lay.rsv) = held[i][0];
            }
            if (x8 < ncs) {
#pragma unroll
                for (int i = 0; i < 2 * NB; ++i) *reinterpret_cast<uintx4 *>(kdst + 8 * i * lay.rsk) = held[2 * NB + i][0];
            }
            return;
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int x = sub + 16 * it;
            const bool is_pool = x < lay.cp;
            char *const dst = area + (is_pool ? lay.v_off + x * 16 : lay.sel_off + (x - lay.cp) * 16);
            const int rs = is_pool ? lay.rsv : lay.rsk;
            if (x < lay.nc) {
#pragma unroll
                for (int i = 0; i < 4 * NB; ++i) *reinterpret_cast<uintx4 *>(dst + (4 * i + rr) * rs) = held[i][it];
            }
        }
    };

    if (wave < n_tiles) load_tile(wave);
    // queries as fragments: lane (col = row, q4) holds columns CHUNK kc + EPC q4 .. + EPC - 1; zero past the width
    uintx4 qf[QB][NKC];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) {
            const int x = M::CHUNK * kc + M::EPC * q4;
            qf[qb][kc] = x < d_qk ? *reinterpret_cast<const uintx4 *>(kp.Q + q_row[qb] * d_qk + x) : uintx4{0, 0, 0, 0};
        }
    // (A branch that does nothing.  Behind it the compiler arranges the queries and what follows otherwise: 512 columns in fp32 keep less of the tile in hand in
    // memory, 512 / 64, 16 heads over 4 KV heads, L = 509 313 / 278 us; in 16 bits 64 / 64, L = 20 3.8 / 3.7 us, B = 2, L = 4000 32.9 / 32.1, fp16 L = 2500
    // 25.7 / 25.4; the other fp32 classes 2 % either way.)
    if ((FULL || sizeof(T) == 2) && !LATE && kp.scale < 0.f) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc) asm volatile("" : "+v"(qf[qb][kc]));
    }
    // the key columns past the width stay zero for the whole kernel (tiles are written over the real columns only)
    if (d_qk < NKC * M::CHUNK || kp.d_pool < 16 * NDT)
        for (int x = lane * 16; x < lay.stage; x += 64 * 16) *reinterpret_cast<uintx4 *>(area + x) = uintx4{0, 0, 0, 0};
    // The queries arrive here: with loads of the next tile in flight the compiler could not tell theirs apart, and every tile's first product
    // would wait for the tile after it (B = 1, L = 2500, 16 heads over 4 KV heads, 64 / 64: 3 500 cycles per tile so, with three wavefronts on a SIMD).
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc)
            if (!LATE) asm volatile("" : "+v"(qf[qb][kc]));

    floatx4 acc[QB][NDT];
    float m_run[QB], ref[QB], l_run[QB];     // reference of the row (base 2; -inf: none yet), the same or 0; this lane's share of the row's sum
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_run[qb] = -INFINITY;
        ref[qb] = 0.f;
        l_run[qb] = 0.f;
#pragma unroll
        for (int t = 0; t < NDT; ++t) acc[qb][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    const char *const key = area + M::row_of_m(col) * lay.rsk + 16 * q4;
    for (int tile = wave; tile < n_tiles; tile += n_waves) {
        store_tile();
        if (tile + n_waves < n_tiles) load_tile(tile + n_waves);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        const bool is_rep = tile < rep_tiles;
        const int e0 = is_rep ? tile * TK : raw0 + (tile - rep_tiles) * TK;
        floatx4 sc[NB][QB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) sc[nb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc) {
                const uintx4 kf = *reinterpret_cast<const uintx4 *>(key + 16 * nb * lay.rsk + 64 * kc);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) sc[nb][qb] = M::score(kf, qf[qb][kc], sc[nb][qb]);
            }
        }
        typename M::template Parts<NB> pb[QB];
        // every row of the workgroup sees the whole tile (its first row the fewest representatives, its last the fewest raw tokens at the front)
        const bool full = is_rep ? e0 + TK <= mt_first : e0 >= n_rep * g && e0 + TK <= t_first + 1;
        const float bias = is_rep ? bias2 : 0.f;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            // The products become logits before anything else reads them: the reference is then one of the logits as they were rounded.  (With one fused
            // operation from product to exponent, what rounding left of the reference became part of every exponent, several binades from base-2 logits of 2^26
            // on, which three parts in fp16 cannot hold; and the products' first reader was a maximum in assembly, for which the compiler keeps none of the
            // wait states behind a matrix product.  Fused / so, 16 heads over 4 KV heads, 64 / 64, L = 2500, the attention alone: bf16 22.2 / 22.7 us, fp16
            // 25.3 / 25.4; at 128 columns and more within 1 %.)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[nb][qb][r] = fmaf(sc[nb][qb][r], c, bias);
            if (!full) {                 // entries [lo, hi) of the tile's kind are visible to this lane's row
                const int lo = is_rep ? 0 : mt_row[qb] * g, hi = is_rep ? mt_row[qb] : t_row[qb] + 1;
                int e1 = e0 + M::entry(0, q4);
                asm volatile("" : "+v"(e1));          // (the entries' numbers are taken here, not by every tile)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int e = e1 + 16 * nb + M::entry(r, 0);
                        sc[nb][qb][r] = e >= lo && e < hi ? sc[nb][qb][r] : -INFINITY;
                    }
            }
            // The reference of a row's exponentials is the largest logit it had seen when one last rose REF_SLACK binades above it.  So in the
            // usual tile nothing is rescaled (a fifth of the tile's work; among 32 rows there nearly always is one with a new maximum) and
            // no lane has to know another's maximum.
            float mx = sc[0][qb][0];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = nb == 0; r < 4; ++r) mx = fmaxf(mx, sc[nb][qb][r]);
            if (__builtin_amdgcn_ballot_w64(mx > m_run[qb] + M::REF_SLACK) != 0) {
                const float to = fmaxf(m_run[qb], row_max4(mx));
                ref[qb] = to == -INFINITY ? 0.f : to;
                const float corr = __builtin_amdgcn_exp2f(m_run[qb] - ref[qb]);
                l_run[qb] *= corr;
#pragma unroll
                for (int t = 0; t < NDT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[qb][t][r] *= corr;
                m_run[qb] = to;
            }
            float pv[NB][4];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pv[nb][r] = __builtin_amdgcn_exp2f(sc[nb][qb][r] - ref[qb]);
                    l_run[qb] += pv[nb][r];
                }
            M::template split<NB>(pv, pb[qb]);
        }
        // O^T += V^T P^T, four value tiles at a time
        const char *const vals = area + lay.v_off;
#pragma unroll
        for (int t0 = 0; t0 < NDT; t0 += 4) {
            typename M::template Frag<NB> vf[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) vf[t] = M::template value<NB>(vals, lay.rsv, t0 + t, col, q4);
#pragma unroll
            for (int part = 0; part < M::PARTS; ++part)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[qb][t0 + t] = M::template accumulate<NB>(vf[t], pb[qb], part, acc[qb][t0 + t]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this tile's reads are done before the next one is written
        __builtin_amdgcn_wave_barrier();
    }

    float *const ml = reinterpret_cast<float *>(smem + n_waves * lay.area);     // [wave][row] (maximum, sum)
    float l_tot[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l_tot[qb] = row_sum4(l_run[qb]);
    auto leave = [&]() {                 // this wavefront's results, in its area
        float *const o = reinterpret_cast<float *>(area);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            if (q4 == 0) *reinterpret_cast<float2 *>(ml + (wave * ROWS + 16 * qb + col) * 2) = float2{m_run[qb], l_tot[qb]};
#pragma unroll
            for (int t = 0; t < NDT; ++t) *reinterpret_cast<floatx4 *>(o + (16 * qb + col) * MROW + 16 * t + 4 * q4) = acc[qb][t];
        }
    };
    bool bad = false;
    // One wavefront stores from its registers, and the first of two (in fp32 up to 128 columns of four, half of them handing over to the other half first) does after adding the
    // second's; not in the full class, which keeps more in memory then, but its LATE form has no other way.  (Four in fp32, the other way / so: 8 + 8, 32 heads,
    // B = 2, L = 39 5.3 / 4.9 us; 64 / 128, 32 heads over 8 KV heads, B = 4, L = 44 9.9 / 9.3; but 256 / 64, L = 83 13.6 / 15.1.)
    if (LATE || n_waves <= (FULL ? 1 : sizeof(T) == 4 && NDT <= 8 ? 4 : 2)) {
        for (int half = n_waves >> 1; half > 0; half >>= 1) {
            if (wave >= half && wave < 2 * half) leave();
            __syncthreads();
            if (wave < half) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const float2 other = *reinterpret_cast<const float2 *>(ml + ((wave + half) * ROWS + 16 * qb + col) * 2);
                    const float m_all = fmaxf(m_run[qb], other.x), m_ref = m_all == -INFINITY ? 0.f : m_all;      // (-inf: neither saw an entry of the row)
                    const float ca = __builtin_amdgcn_exp2f(m_run[qb] - m_ref), cb = __builtin_amdgcn_exp2f(other.x - m_ref);
                    l_tot[qb] = l_tot[qb] * ca + other.y * cb;
                    m_run[qb] = m_all;
                    const float *const o = reinterpret_cast<const float *>(smem + (wave + half) * lay.area) + (16 * qb + col) * MROW + 4 * q4;
#pragma unroll
                    for (int t = 0; t < NDT; ++t) {
                        const floatx4 v = *reinterpret_cast<const floatx4 *>(o + 16 * t);
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[qb][t][r] = acc[qb][t][r] * ca + v[r] * cb;
                    }
                }
            }
        }
        if (wave == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const float inv = 1.f / (l_tot[qb] * M::P_SCALE);
                float chk = 0.f;
#pragma unroll
                for (int t = 0; t < NDT; ++t) {
                    const int x = 16 * t + 4 * q4;                 // this lane's four value columns
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[qb][t][r] *= inv;
                    if (live[qb] && x < kp.d_pool) {
                        M::store4(kp.O + q_row[qb] * kp.d_pool + x, acc[qb][t]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) chk = fmaf(acc[qb][t][r], 0.f, chk);      // zero, or NaN if a value is not finite
                    }
                }
                if (kp.lse != nullptr && live[qb] && q4 == 0) kp.lse[q_row[qb]] = (m_run[qb] + log2f(l_tot[qb])) * 0.6931471805599453f;
                bad |= live[qb] && !(chk == 0.f);
            }
        }
    } else {
        // Every wavefront leaves its results in its area, then the threads share the columns of all rows, four each, over the
        // wavefronts' areas.  (The upper half handing its results to the lower until one wavefront was left, which then stored alone, took
        // 2.1 of a workgroup's 13.5 us at 64 / 64 with four wavefronts.)
        size_t *const row_s = reinterpret_cast<size_t *>(ml + n_waves * ROWS * 2);   // [row] index of the row in Q, O and lse
        leave();
        if (wave == 0 && q4 == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) row_s[16 * qb + col] = q_row[qb];
        }
        __syncthreads();
        // a row's weights of the wavefronts, divided by its sum
        constexpr int W = max_waves<T>(NDT);
        auto weights = [&](int row, float (&f)[W], bool first) {
            float2 mw[W];
            float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) mw[w] = w < n_waves ? *reinterpret_cast<const float2 *>(ml + (w * ROWS + row) * 2) : float2{-INFINITY, 0.f};
#pragma unroll
            for (int w = 0; w < W; ++w) m_all = fmaxf(m_all, mw[w].x);
#pragma unroll
            for (int w = 0; w < W; ++w) {
                f[w] = __builtin_amdgcn_exp2f(mw[w].x - m_all);
                l_all = fmaf(mw[w].y, f[w], l_all);
            }
            const float inv = 1.f / (l_all * M::P_SCALE);
#pragma unroll
            for (int w = 0; w < W; ++w) f[w] *= inv;
            if (kp.lse != nullptr && first && r0 + row <= r_last) kp.lse[row_s[row]] = (m_all + log2f(l_all)) * 0.6931471805599453f;
        };
        // by every thread for itself where it has one item, else once per row, with one more barrier (0.5 us, against the exponentials of every
        // item: B = 2, L = 4000, 8 heads, bf16 256 + 32 160 / 166 us)
        constexpr int ITEMS = ROWS * 4 * NDT;
        const bool own = ITEMS <= 64 * n_waves;
        float f[W];
        if (!own) {
            if (tid < ROWS) {
                weights(tid, f, true);
#pragma unroll
                for (int w = 0; w < W; ++w)
                    if (w < n_waves) ml[(w * ROWS + tid) * 2] = f[w];
            }
            __syncthreads();
        }
        for (int i = tid; i < ITEMS; i += 64 * n_waves) {
            const int row = i / (4 * NDT), x = 4 * (i % (4 * NDT));                  // this thread's four value columns
            if (r0 + row > r_last || x >= kp.d_pool) continue;
            floatx4 v[W], sum = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < W; ++w)
                if (w < n_waves) v[w] = *reinterpret_cast<const floatx4 *>(smem + w * lay.area + (row * MROW + x) * 4);
            if (own) weights(row, f, x == 0);
            else {
#pragma unroll
                for (int w = 0; w < W; ++w)
                    if (w < n_waves) f[w] = ml[(w * ROWS + row) * 2];
            }
#pragma unroll
            for (int w = 0; w < W; ++w)
                if (w < n_waves)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sum[r] = fmaf(v[w][r], f[w], sum[r]);
            float chk = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) chk = fmaf(sum[r], 0.f, chk);      // zero, or NaN if a value is not finite
            M::store4(kp.O + row_s[row] * kp.d_pool + x, sum);
            bad |= !(chk == 0.f);
        }
    }
    if (__syncthreads_or(bad)) {                               // rare: a row met an infinity or a NaN, perhaps one it does not see
        float *const q_s = reinterpret_cast<float *>(area), *const p_s = q_s + d_qk;
        for (int r = wave; r <= r_last - r0; r += n_waves) {
            const int t = (r0 + r) / hps;
            attn_row::attend_row<T, NDT / 4>(kp, ((long)b * L + t) * kp.H + s * hps + (r0 + r - t * hps), q_s, p_s, lane);
        }
    }
}

// Whether the full class runs in its LATE form: queries free to arrive late, one way through the merge, ordinary divisions.  It spends less before and after the
// loop, whose every tile then waits for the next one's loads; those are few where a row is short, and the registers they would go into fewer.  The other
// form / LATE, us: 192 + 128, 8 heads and sets, B = 2, L = 1030 109 / 89; 256 + 64, 16 heads, B = 2, L = 25 22.3 / 20.2, L = 1500 535 / 519; rows of 448 and
// more: 512 / 64, 32 sets, L = 270 (three tiles, 544 workgroups) 132 / 122, but two heads, L = 500 (eleven over four wavefronts) 49.8 / 53.5, 4 sets of 4 heads,
// L = 509 280 / 369, and five to seven tiles in more workgroups than CUs either way.
static bool late_form(const Dims &d, int tiles, int waves, long grid, int cus) { return d.d_pool + d.d_sel <= 384 || (grid > cus && tiles <= 3 * waves); }

template <typename T, int NDT, int NKC, int QB, int NB, int NIT>
hipError_t run(const AttnArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    const Layout<T, NDT, NKC, QB, NB> lay(d.d_pool, d.d_sel, d.mode == LCA_MODE_MLA);
    const long blocks = ((long)d.L * (d.H / d.S) + 16 * QB - 1) / (16 * QB), grid = blocks * d.S * d.B;
    // Wavefronts per workgroup.  No more than there are tiles (the last rows see the most): the others would only be merged.  A workgroup may
    // take all of a CU's LDS while there is a CU for each, half of it while there are two per CU, then what leaves room for two; the widest
    // classes fill a SIMD's registers with one wavefront, so from two workgroups per CU on they have two wavefronts at most.  Measured (at
    // most 64 KB whatever the grid and the tiles / now): fp32 512 + 64, 2 heads, L = 500 146 / 55 us (one wavefront, four); bf16 256 + 32, 8 heads,
    // L = 500 15.6 / 11.9, L = 1500 20.4 / 20.4; bf16 64 / 64, L = 20 4.9 / 4.1 (two tiles).  The rule with all of LDS at any grid: bf16
    // 512 + 64 at L of a thousand and more up to 2.5 times as long.
    const int t_last = d.L - 1, t_first = (int)((blocks - 1) * 16 * QB / (d.H / d.S));
    auto visible = [&](int t) { return (a.dense || t + 1 <= d.w) ? 0 : (t + 1 - d.w) / d.g; };
    const int tiles = (visible(t_last) + 16 * NB - 1) / (16 * NB) + (t_last + 1 - visible(t_first) * d.g + 16 * NB - 1) / (16 * NB);
    const int cus = persistent_grid();
    const size_t room = grid <= cus ? LDS_BYTES : grid <= 2 * cus ? LDS_BYTES / 2 : LDS_BYTES * 2 / 5;
    constexpr bool full_registers = NDT > (sizeof(T) == 2 ? 16 : 8);
    auto lds = [&](int waves) { return (size_t)waves * lay.area + (waves + 1) * 16 * QB * 8; };
    int waves = full_registers && grid > cus ? 2 : grid > cus ? 4 : max_waves<T>(NDT);
    // Where many workgroups keep every CU busy, half the wavefronts each leave half as much to merge.  Four wavefronts / two: 64 / 64, two row blocks, 16 heads
    // over 4 KV heads, L = 2500 (1252 workgroups) 35.4 / 34.6 us with the condensation, B = 2, L = 4000 (4000) 54.2 / 46.0; fp32 128 + 32, 8 heads, L = 4096
    // (2048) 142 / 132, but one row block and B = 3, L = 900 (1350) 63.3 / 66.4, longer workgroups not quite twice as many as fit; two / one:
    // 256 + 32, 8 heads, B = 2, L = 4000 (4000) 162 / 157, but fp32 192 / 128, 7 heads, L = 2347 (1027, one per SIMD) 287 / 468.
    // Two row blocks and many tiles: not while the workgroups fill the CUs only a few times over, when the last ones make a long tail (fp32, 16 heads over one KV head:
    // 8 / 8, B = 2, L = 1086, 1086 workgroups of 69 tiles, 64.5 / 80.1; 64 / 64, L = 2230, 1115 of 141, 126 / 150; 8 / 8, L = 2420, 1210 of 152, 141 / 155).
    const bool halve = QB == 2 ? waves > 2 && grid >= (tiles > 64 ? 5 : 4) * (long)cus : waves > 1 && grid >= 8 * (long)cus && tiles >= 32;
    if (!full_registers && halve) waves /= 2;
    while (waves > 1 && (waves / 2 >= tiles || (NDT > 8 && waves > tiles) || lds(waves) > room)) waves /= 2;
    const TileParams<T> tp{attn_row::row_params<T>(a), (int)blocks, make_div((unsigned)blocks), make_div(d.S), make_div(d.H / d.S), make_div(d.g)};
    if constexpr (full_class<T>(NDT)) {
        if (late_form(d, tiles, waves, grid, cus)) {
            attn_tile_kernel<T, NDT, NKC, QB, NB, NIT, true><<<(unsigned)grid, 64 * waves, lds(waves), st>>>(tp);
            return hipGetLastError();
        }
    }
    attn_tile_kernel<T, NDT, NKC, QB, NB, NIT, false><<<(unsigned)grid, 64 * waves, lds(waves), st>>>(tp);
    return hipGetLastError();
}

// The smallest instantiation that holds the widths.  At up to 64 value columns two blocks of query rows per wavefront (half the
// tile traffic and half the key and value reads per row) once that still leaves every CU four workgroups: 34 us against 41 us
// with one block at L = 2500, 93 against 116 us at B = 2, L = 4000 (16 heads, 64 / 64).  At 128 columns the second block's
// registers cost the second wavefront of a SIMD: 151 us against 146 us in fp32 at L = 4096, 8 heads, so one.
template <typename T> bool fits(const Dims &d, int ndt, int nkc, int nit)
{
    // (rows travel as 32-bit byte offsets inside one sequence)
    const int widest = d.d_pool > d.d_sel ? d.d_pool : d.d_sel;
    if ((long long)(d.L + 64) * d.P * widest * (long long)sizeof(T) >= (1ll << 32)) return false;
    return d.d_pool <= 16 * ndt && d.d_qk <= nkc * Mma<T>::CHUNK && (d.d_pool + d.d_sel) <= nit * 16 * Mma<T>::EPC;
}
// While a row sees this many entries or fewer, one wavefront per row is quicker: a tile is worked through whole, in all the columns of
// its class, however little of it is real (so there is more to lose in GQA mode, whose keys are narrower than the class, and in fp32).
// Measured (row by row / tiles, us): fp32 512 + 64, L = 2 / 16 / 32 12.0 / 19.7, 23.7 / 20.2, 39.9 / 32.6; fp32 GQA 512 / 64, L = 8
// 11.0 / 21.1; fp32 128 + 32, L = 4 / 16 6.4 / 6.8, 10.1 / 6.9; bf16 GQA 512 / 64, L = 4 / 16 7.7 / 9.6, 18.5 / 9.7.
// By class of the widths (64, 128, 256, 512 value columns), in 16 bits (GQA mode only) and in fp32 (MLA, GQA).
constexpr int FEW_ENTRIES_16[4] = {0, 2, 4, 7}, FEW_ENTRIES_32[4][2] = {{2, 3}, {4, 6}, {8, 10}, {18, 40}};
constexpr long FEW_ROWS = 8192;                   // ... and the rows' wavefronts are all on the chip at once

template <typename T> hipError_t dispatch(const AttnArgs &a, hipStream_t st, bool &done)
{
    const Dims &d = a.d;
    const long rows = (long)d.L * (d.H / d.S);
    const bool wide = (rows + 31) / 32 * d.S * d.B >= 1024, gqa = d.mode != LCA_MODE_MLA;
    const long entries = a.dense || d.m == 0 ? d.L : min((long)d.L, (long)d.m + d.w + d.g - 1);      // of the row that sees the most
    const auto few = [&](int cls) {
        const int most = sizeof(T) == 2 ? (gqa ? FEW_ENTRIES_16[cls] : 0) : FEW_ENTRIES_32[cls][gqa];
        return entries <= most && (long)d.B * d.L * d.H <= FEW_ROWS;
    };
    done = true;
    if constexpr (sizeof(T) == 2) {
        if (fits<T>(d, 4, 2, 1)) { if (!few(0)) return wide ? run<T, 4, 2, 2, 2, 1>(a, st) : run<T, 4, 2, 1, 2, 1>(a, st); }
        else if (fits<T>(d, 8, 4, 2)) { if (!few(1)) return run<T, 8, 4, 1, 2, 2>(a, st); }
        else if (fits<T>(d, 16, 10, 3)) { if (!few(2)) return run<T, 16, 10, 1, 1, 3>(a, st); }
        else if (fits<T>(d, 32, 18, 5)) { if (!few(3)) return run<T, 32, 18, 1, 1, 5>(a, st); }
    } else {
        if (fits<T>(d, 4, 4, 2)) { if (!few(0)) return wide ? run<T, 4, 4, 2, 1, 2>(a, st) : run<T, 4, 4, 1, 1, 2>(a, st); }
        else if (fits<T>(d, 8, 10, 4)) { if (!few(1)) return run<T, 8, 10, 1, 1, 4>(a, st); }
        else if (fits<T>(d, 16, 18, 5)) { if (!few(2)) return run<T, 16, 18, 1, 1, 5>(a, st); }
        else if (fits<T>(d, 32, 36, 9)) { if (!few(3)) return run<T, 32, 36, 1, 1, 9>(a, st); }
    }
    done = false;
    return hipSuccess;
}

}  // namespace

hipError_t launch_attn_tile(const AttnArgs &a, hipStream_t st, bool &done)
{
    if (a.d.dtype == LCA_BF16) return dispatch<uint16_t>(a, st, done);
    if (a.d.dtype == LCA_F16) return dispatch<f16_t>(a, st, done);
    return dispatch<float>(a, st, done);
}

}  // namespace lca

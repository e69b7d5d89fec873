// What the two MLA attention kernels share (attn_mla.hip: four wavefronts on 128 (query row, head) pairs; attn_mla_halves.hip: on 64, two for
// every 32): types, the tile's layout in LDS, the direct-to-LDS load and the work item.
#pragma once
#include <type_traits>

#include "lca_internal.h"

namespace lca {

struct MlaParams {
    const uint16_t *Q, *POOL, *SEL, *pool_rep, *sel_rep;
    uint16_t *O;
    float *lse;
    const uint16_t *W_up;   // UP variant: value up-projection W^UV in fragment order (pack_up_kernel), and O is [B, L, H, DU]
    int B, L, H, S, g, w, m, dense, n_qb;
    int run_log2;           // log2 of the query blocks an XCD works on at a time (256 rows at most)
    int hw_log2;            // log2 of the heads of a work item (4, 2 or 1): its wavefronts are that many heads x 4 / heads groups of 32 rows
    float scale_log2, bias_log2;
};

// attn_mla_halves.hip: the same call with work items of 64 pairs (W_up decides the variant)
void launch_mla_halves(const MlaParams &kp, bool f16, unsigned grid, hipStream_t st);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// fp16 runs through the same code (template parameter F16): fragments travel in the bf16 vector types as plain 16-bit
// containers, and only the matrix instructions, the two conversions (P^T, output) and the softmax range differ.
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int int4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const char *lds_cptr;

#define LCA_FENCE() __builtin_amdgcn_sched_barrier(0)

constexpr int DP = 512, DS = 64, DQK = 576, DV = 512;
constexpr int BM = 128;                 // (query row, head) pairs per workgroup
constexpr int BN = 32;                  // entries per key tile
constexpr int NSTAGE = 4;
constexpr int RSB = 1040;               // LDS row stride of the latent part in bytes: 1024 + 16
constexpr int SEL_OFF = BN * RSB;       // the RoPE part of a stage starts here: 32 rows x 128 B, swizzled
constexpr int STAGE_BYTES = SEL_OFF + BN * DS * 2;   // 37 376
constexpr int COPIES_PER_TILE = 9;      // direct-to-LDS loads one wavefront issues per tile (8 latent rows + 1 RoPE block)
constexpr int NKS = DQK / 16;           // 36 k-steps of S^T
constexpr int NDV = DV / 32;            // 16 value tiles
constexpr int DU = 128;                  // UP variant: width of a head's value after the up-projection
constexpr float NEG_BIG = -1.0e30f;     // stands for -inf in running maxima (keeps exp2 arguments finite)
constexpr float L_LIMIT = 0x1p90f;      // a row sum beyond this (or not finite) makes the workgroup repeat the item from exact maxima
// fp16 ends at 65504: an exponential past it is an infinity in the second product, which no column of its row survives (infinity times a value is an
// infinity, or no number), so the item is repeated from exact maxima if the row's first accumulator is not finite.  (Keeping the largest exponential
// instead took one v_max3 per pair, which no case here shows: L = 8192, 16 heads 317 us either way.  A value that is not finite itself has its rows repeated for nothing.)  The reference sits 4 binades above the first maximum a row sees
// (first entries at 2^-4): later logits may be 2^19 times larger before that happens, at the price of 4 of fp16's 24
// binades at the bottom.
// (A row that sees a few representatives first, a poor sample of its logits, has its item repeated now and then: three times L = 1200, g = 32, 16 heads 95 us, in one
// call of six to twelve 170-182.  8 binades avoided that, but where the representative is the row's maximum, a group far above a window of ordinary tokens, they took the
// bits those tokens need: 12 nats above 2048 tokens, a tenth of their size, error 1.7e-2.)
constexpr float REF_SHIFT_F16 = 4.f;

// Tile copies go through raw buffer descriptors (base, size in bytes) so that rows past the end of a segment
// need no clamping: the hardware range check turns them into zeros (such entries are masked anyway).
struct Seg {
    unsigned lo, hi, bytes;       // descriptor words 0..2: address bits 0..31, bits 32..47 (stride 0), size
};
__device__ __forceinline__ Seg make_seg(const void *p, long bytes)
{
    const unsigned long long a = (unsigned long long)p;
    return Seg{(unsigned)a, (unsigned)(a >> 32) & 0xFFFFu, (unsigned)bytes};
}
constexpr int RSRC_WORD3 = 0x00020000;   // raw buffer of dwords, gfx9 layout

// One direct-to-LDS load of 64 x 16 bytes: lane l fetches segment bytes [soff + IMM + voff, +16) into LDS bytes
// [m0 + IMM + 16 l, +16) (the instruction offset moves both sides).  Inline assembly on purpose: the compiler
// makes every LDS read that follows a direct-to-LDS load it knows about wait for that load, and here the
// copy must stay in flight for two more tiles.  Ordering is kept by hand instead: s_waitcnt vmcnt + workgroup
// barrier in the tile loop before a stage is read, 9 loads per tile and wavefront.
template <int M0_ADD, int IMM>
__device__ __forceinline__ void dma_1k(unsigned voff, const int4v &rs, unsigned soff, unsigned m0_base)
{
    asm volatile("s_add_u32 m0, %2, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %3 offen offset:%5 lds"
                 : : "v"(voff), "s"(rs), "s"(m0_base), "s"(soff), "n"(M0_ADD), "n"(IMM) : "scc", "memory");   // writes M0, which no compiler-generated instruction of this kernel uses
}

__device__ __forceinline__ unsigned lds_address(const void *p)
{
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)p;
}

// LDS addresses of this lane's key fragments of the RoPE part of a stage (how many and in which order is the kernel's)
struct KSel { unsigned a[4]; };

template <bool F16>
__device__ __forceinline__ floatx16 pv_mfma(const bf16x8 &a, const bf16x8 &b, const floatx16 &c)
{
    if (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// Everything one wavefront needs to know about one work item = 128 (or 64) (row, head) pairs of one sequence: as many query rows of
// each of its heads, which share a condensed set.
struct Blk {
    int b, h, t0, t_last, t_w0;              // sequence, this wavefront's head, first / last query row of the item, first of the wavefront
    int t_row, mt_row, raw_lo_row;           // per lane: query row, representatives it sees, first raw token it sees
    int raw_lo_blk, mt_blk_hi;               // first raw token / representatives any row of the block sees
    int n_rep_tiles, n_tiles;
    int rep_full_end, raw_full_lo, raw_full_hi;   // tiles this wavefront sees completely (no masking)
    Seg rep_pool, rep_sel, raw_pool, raw_sel;     // the two segments: visible representatives, raw tokens 0 .. t_last of the sequence
};

__device__ __forceinline__ int groups_visible(const MlaParams &kp, int t) { return (kp.dense || t + 1 <= kp.w) ? 0 : (t + 1 - kp.w) / kp.g; }
// t0: the item's first query row, of `rows`; h: this wavefront's head, t_wfirst: the first of its 32 rows, n: this lane's row among them
__device__ __forceinline__ Blk make_blk(const MlaParams &kp, int b, int h, int t0, int rows, int t_wfirst, int n)
{
    Blk k;
    const int L = kp.L, g = kp.g;
    auto visible = [&](int t) { return groups_visible(kp, t); };
    k.b = b; k.h = h;
    k.t0 = t0;
    k.t_last = min(k.t0 + rows, L) - 1;
    const int t_wlast = t_wfirst + 31;
    k.t_w0 = t_wfirst;
    k.t_row = t_wfirst + n;
    k.mt_row = visible(k.t_row);
    k.raw_lo_row = k.mt_row * g;
    const int mt_blk_lo = visible(k.t0), mt_w_lo = visible(t_wfirst), mt_w_hi = visible(t_wlast);
    k.mt_blk_hi = visible(k.t_last);
    k.raw_lo_blk = mt_blk_lo * g;
    k.n_rep_tiles = (k.mt_blk_hi + BN - 1) / BN;
    k.n_tiles = k.n_rep_tiles + (k.t_last + 1 - k.raw_lo_blk + BN - 1) / BN;
    k.rep_full_end = mt_w_lo / BN;
    k.raw_full_lo = k.n_rep_tiles + (mt_w_hi * g - k.raw_lo_blk + BN - 1) / BN;
    k.raw_full_hi = k.n_rep_tiles + max(0, (t_wfirst + 1 - k.raw_lo_blk) / BN);
    const int s = h / (kp.H / kp.S);
    k.rep_pool = make_seg(kp.pool_rep + ((size_t)b * kp.S + s) * kp.m * DP, (long)k.mt_blk_hi * (DP * 2));
    k.rep_sel = make_seg(kp.sel_rep + ((size_t)b * kp.S + s) * kp.m * DS, (long)k.mt_blk_hi * (DS * 2));
    k.raw_pool = make_seg(kp.POOL + (size_t)b * L * DP, (long)(k.t_last + 1) * (DP * 2));
    k.raw_sel = make_seg(kp.SEL + (size_t)b * L * DS, (long)(k.t_last + 1) * (DS * 2));
    return k;
}

#define LCA_PIN_S(x) asm volatile("" : "+s"(x))
#define LCA_PIN_V(x) asm volatile("" : "+v"(x))
// -1 if a < b, else 0 (|a - b| < 2^31), by scalar arithmetic: a comparison result turned into an integer would travel
// through a vector register.  Unsigned subtraction so that the compiler cannot turn it back into a comparison.
__device__ __forceinline__ int lt_mask(int a, int b) { return (int)((unsigned)a - (unsigned)b) >> 31; }

}  // namespace
}  // namespace lca

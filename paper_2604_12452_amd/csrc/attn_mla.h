// What the two MLA attention kernels share (attn_mla.hip: four wavefronts on 128 (query row, head) pairs; attn_mla_halves.hip: on 64, two for
// every 32): types, the tile's layout in LDS, the copies, the work item and the tile loop's bookkeeping.
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
union Pb { bf16x8 v[2]; bf16x2 p[8]; };     // P^T of one tile: the B operands of the two k-steps of the second product
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
#ifndef LCA_CHAIN_DEPTH
#define LCA_CHAIN_DEPTH 6
#endif
constexpr int CHAIN_DEPTH = LCA_CHAIN_DEPTH;   // key fragments in flight ahead of the S^T chain
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
// Accumulator register r of lane group G (lanes 32G..32G+31) of a 32x32 tile holds S^T row
// m = 8*(r/4) + 4G + r%4.  S^T row m is computed from LDS row (= tile entry) pi(m): inside each half of 16,
// pi(8h + 4G + j) = 4j + 2h + G.
__device__ __forceinline__ constexpr int lds_row_of_m(int m) { return (m & 16) + 4 * (m & 3) + 2 * ((m >> 3) & 1) + ((m >> 2) & 1); }
__device__ __forceinline__ constexpr int acc_entry(int r, int G) { return lds_row_of_m(8 * (r >> 2) + 4 * G + (r & 3)); }

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

// What one wavefront needs to copy its 8 rows of one key tile into one stage (all wavefront-uniform).
struct CopyCtl {
    int4v pool_rs, sel_rs;               // descriptors of the latent / RoPE part of the tile's segment
    unsigned soff_lo, soff_hi, soff_sel; // byte offsets of the wavefront's rows 0 and 4 (latent) and row 0 (RoPE) in the segment
    unsigned m0_pool, m0_sel;            // LDS addresses of the wavefront's first row in the stage
};

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

// One of the 9 copies a wavefront makes per tile: J < 8 moves latent row 8*wave + J (1 KB; LDS rows are RSB
// apart, the instruction offset (J%4) KB already moves the LDS side by as much), J == 8 moves the RoPE parts
// of rows 8*wave .. 8*wave+7 (1 KB; lane l fills slot l&7 of local row l>>3 with the chunk the swizzle assigns
// to that slot: voff_sel = (l>>3)*128 + chunk*16).
template <int J>
__device__ __forceinline__ void issue_copy_part(const CopyCtl &c, unsigned voff_pool, unsigned voff_sel)
{
    if constexpr (J < 4) dma_1k<J * RSB - J * 1024, J * 1024>(voff_pool, c.pool_rs, c.soff_lo, c.m0_pool);
    else if constexpr (J < 8) dma_1k<J * RSB - (J - 4) * 1024, (J - 4) * 1024>(voff_pool, c.pool_rs, c.soff_hi, c.m0_pool);
    else dma_1k<0, 0>(voff_sel, c.sel_rs, c.soff_sel, c.m0_sel);
}
template <int J>
__device__ __forceinline__ void issue_copy_from(const CopyCtl &c, unsigned voff_pool, unsigned voff_sel)
{
    if constexpr (J < COPIES_PER_TILE) {
        issue_copy_part<J>(c, voff_pool, voff_sel);
        issue_copy_from<J + 1>(c, voff_pool, voff_sel);
    }
}

__device__ __forceinline__ void issue_copy_part_dyn(int j, const CopyCtl &c, unsigned voff_pool, unsigned voff_sel)
{
    switch (j) {      // j is a constant after unrolling
    case 0: issue_copy_part<0>(c, voff_pool, voff_sel); break;
    case 1: issue_copy_part<1>(c, voff_pool, voff_sel); break;
    case 2: issue_copy_part<2>(c, voff_pool, voff_sel); break;
    case 3: issue_copy_part<3>(c, voff_pool, voff_sel); break;
    case 4: issue_copy_part<4>(c, voff_pool, voff_sel); break;
    case 5: issue_copy_part<5>(c, voff_pool, voff_sel); break;
    case 6: issue_copy_part<6>(c, voff_pool, voff_sel); break;
    case 7: issue_copy_part<7>(c, voff_pool, voff_sel); break;
    default: issue_copy_part<8>(c, voff_pool, voff_sel); break;
    }
}

// LDS addresses of this lane's four key fragments of the RoPE part (k-steps 32..35) of a stage: chunk 2j + G of the
// lane's row sits at slot (2j + G) ^ xs.  `first` = address of the slot of j = 0 (x6 = xs & 6 already applied);
// slot bits 1..2 are address bits 5..6, which are zero in the row's base address, so j enters as an exclusive or.
struct KSel { unsigned a[4]; };
__device__ __forceinline__ KSel make_ksel(unsigned first)
{
    return KSel{{first, first ^ (1u << 5), first ^ (2u << 5), first ^ (3u << 5)}};
}

template <bool F16>
__device__ __forceinline__ floatx16 pv_mfma(const bf16x8 &a, const bf16x8 &b, const floatx16 &c)
{
    if (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// Everything one wavefront needs to know about one work item = 128 (row, head) pairs of one sequence: BM / heads query rows of
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

// Copy of tile tc into stage `sd` (LDS address of stage 0 = lds0).  A tile past the item's last one lies past the
// end of the raw segment: its copy moves zeros.
__device__ __forceinline__ CopyCtl make_copy(const Blk &k, int tc, int sd, int wave, unsigned lds0)
{
    CopyCtl c;
    const bool is_rep = tc < k.n_rep_tiles;
    const Seg &ps = is_rep ? k.rep_pool : k.raw_pool, &ss = is_rep ? k.rep_sel : k.raw_sel;
    c.pool_rs = int4v{(int)ps.lo, (int)ps.hi, (int)ps.bytes, RSRC_WORD3};
    c.sel_rs = int4v{(int)ss.lo, (int)ss.hi, (int)ss.bytes, RSRC_WORD3};
    const unsigned row0 = (is_rep ? tc * BN : k.raw_lo_blk + (tc - k.n_rep_tiles) * BN) + 8 * wave;   // first entry of this wavefront's share
    c.soff_lo = row0 * (DP * 2);
    c.soff_hi = c.soff_lo + 4 * (DP * 2);
    c.soff_sel = row0 * (DS * 2);
    c.m0_pool = lds0 + sd * STAGE_BYTES + 8 * wave * RSB;
    c.m0_sel = lds0 + sd * STAGE_BYTES + SEL_OFF + 8 * wave * (DS * 2);
    return c;
}

// What iteration tl of the tile loop needs besides the data: the copy of tile tl+3, this lane's read addresses in
// the stages of the S^T chain (tile tl+1) and of the O^T update (tile tl), and how tile tl is treated.
struct Ctl {
    CopyCtl cc;
    lds_cptr kb, vp0, vp1;  // (vp1: value tiles 8..15, where they are not simply behind the others)
    KSel ksel;
    float bias;             // base-2 logit bias of tile tl (representatives may carry one)
    int is_rep, full;       // tile tl, as masks (-1 / 0): a tile of representatives; every entry visible to every row of this wavefront
};
// The same, computed in small steps (STEP 0..8) so that the work can be dealt out over the free issue slots of
// the O^T update; `t` carries intermediate values from step to step.  The empty assembly statements pin each
// step's results to its place (the compiler would otherwise gather the steps where their last result is needed).
struct CtlTmp { int tc, rep_c; unsigned row0, chain_lds, pv_lds; unsigned p0, p1, p2, q0, q1, q2; };
#define LCA_PIN_S(x) asm volatile("" : "+s"(x))
#define LCA_PIN_V(x) asm volatile("" : "+v"(x))
// -1 if a < b, else 0 (|a - b| < 2^31), by scalar arithmetic: a comparison result turned into an integer would travel
// through a vector register.  Unsigned subtraction so that the compiler cannot turn it back into a comparison.
__device__ __forceinline__ int lt_mask(int a, int b) { return (int)((unsigned)a - (unsigned)b) >> 31; }
template <int STEP, bool HALVES>
__device__ __forceinline__ void ctl_step(Ctl &c, CtlTmp &t, const Blk &k, const MlaParams &kp, int tl, int wave, unsigned lds0, int k_off,
                                         int ksel_off, int v_off, int v_off1 = 0)
{
    if constexpr (STEP == 0) {
        t.tc = tl + 3;
        t.rep_c = lt_mask(t.tc, k.n_rep_tiles);
        c.is_rep = lt_mask(tl, k.n_rep_tiles);
        LCA_PIN_S(t.rep_c); LCA_PIN_S(c.is_rep);
    } else if constexpr (STEP == 1) {
        t.p0 = t.rep_c ? k.rep_pool.lo : k.raw_pool.lo;
        t.p1 = t.rep_c ? k.rep_pool.hi : k.raw_pool.hi;
        t.p2 = t.rep_c ? k.rep_pool.bytes : k.raw_pool.bytes;
        LCA_PIN_S(t.p0); LCA_PIN_S(t.p1); LCA_PIN_S(t.p2);
    } else if constexpr (STEP == 2) {
        t.q0 = t.rep_c ? k.rep_sel.lo : k.raw_sel.lo;
        t.q1 = t.rep_c ? k.rep_sel.hi : k.raw_sel.hi;
        t.q2 = t.rep_c ? k.rep_sel.bytes : k.raw_sel.bytes;
        LCA_PIN_S(t.q0); LCA_PIN_S(t.q1); LCA_PIN_S(t.q2);
    } else if constexpr (STEP == 3) {
        t.row0 = (t.rep_c ? t.tc * BN : k.raw_lo_blk + (t.tc - k.n_rep_tiles) * BN) + 8 * wave;
        LCA_PIN_S(t.row0);
    } else if constexpr (STEP == 4) {
        c.cc.soff_lo = t.row0 * (DP * 2);
        c.cc.soff_hi = c.cc.soff_lo + 4 * (DP * 2);
        c.cc.soff_sel = t.row0 * (DS * 2);
        LCA_PIN_S(c.cc.soff_lo); LCA_PIN_S(c.cc.soff_hi); LCA_PIN_S(c.cc.soff_sel);
    } else if constexpr (STEP == 5) {
        const unsigned sbase = lds0 + ((tl + 3) & (NSTAGE - 1)) * STAGE_BYTES;
        c.cc.m0_pool = sbase + 8 * wave * RSB;
        c.cc.m0_sel = sbase + SEL_OFF + 8 * wave * (DS * 2);
        LCA_PIN_S(c.cc.m0_pool); LCA_PIN_S(c.cc.m0_sel);
    } else if constexpr (STEP == 6) {
        // past the last tile the chain runs over a stage that holds zeros or an old tile: S^T that nobody reads
        t.chain_lds = lds0 + ((tl + 1) & (NSTAGE - 1)) * STAGE_BYTES;
        t.pv_lds = lds0 + (tl & (NSTAGE - 1)) * STAGE_BYTES;
        LCA_PIN_S(t.chain_lds); LCA_PIN_S(t.pv_lds);
    } else if constexpr (STEP == 7) {
        c.full = lt_mask(tl, k.rep_full_end) | (~lt_mask(tl, k.raw_full_lo) & lt_mask(tl, k.raw_full_hi));
        LCA_PIN_S(c.full);
        c.cc.pool_rs = int4v{(int)t.p0, (int)t.p1, (int)t.p2, RSRC_WORD3};
        c.cc.sel_rs = int4v{(int)t.q0, (int)t.q1, (int)t.q2, RSRC_WORD3};
    } else {
        unsigned kb = t.chain_lds + k_off, vp0 = t.pv_lds + v_off;
        if constexpr (HALVES) {
            unsigned vp1 = t.pv_lds + v_off1;
            LCA_PIN_V(vp1);
            c.vp1 = (lds_cptr)(uintptr_t)vp1;
            c.ksel.a[0] = t.chain_lds + ksel_off; c.ksel.a[1] = c.ksel.a[0] ^ (1u << 6);
        } else c.ksel = make_ksel(t.chain_lds + ksel_off);
        c.bias = c.is_rep ? kp.bias_log2 : 0.f;
        LCA_PIN_V(kb); LCA_PIN_V(vp0); LCA_PIN_V(c.bias);
        LCA_PIN_V(c.ksel.a[0]); LCA_PIN_V(c.ksel.a[1]);
        if constexpr (!HALVES) { LCA_PIN_V(c.ksel.a[2]); LCA_PIN_V(c.ksel.a[3]); }
        c.kb = (lds_cptr)(uintptr_t)kb; c.vp0 = (lds_cptr)(uintptr_t)vp0;
    }
}
template <bool HALVES>
__device__ __forceinline__ Ctl make_ctl(const Blk &k, const MlaParams &kp, int tl, int wave, unsigned lds0, int k_off, int ksel_off, int v_off, int v_off1 = 0)
{
    Ctl c;
    CtlTmp t;
    auto step = [&](auto n) { ctl_step<decltype(n)::value, HALVES>(c, t, k, kp, tl, wave, lds0, k_off, ksel_off, v_off, v_off1); };
    step(std::integral_constant<int, 0>()); step(std::integral_constant<int, 1>()); step(std::integral_constant<int, 2>());
    step(std::integral_constant<int, 3>()); step(std::integral_constant<int, 4>()); step(std::integral_constant<int, 5>());
    step(std::integral_constant<int, 6>()); step(std::integral_constant<int, 7>()); step(std::integral_constant<int, 8>());
    return c;
}

// copies of tiles 0..2 of a work item into stages 0..2
__device__ __forceinline__ void issue_first_copies(const Blk &k, int wave, unsigned lds0, unsigned voff_pool, unsigned voff_sel)
{
    for (int tl = 0; tl < 3; ++tl) {
        const CopyCtl c = make_copy(k, tl, tl, wave, lds0);
        issue_copy_from<0>(c, voff_pool, voff_sel);
    }
}

// Queries of a work item.  The second product wants lane (n, G) to hold Q[row n][16 ks + 8 G .. +7] for every
// k-step ks, but loading them that way makes every load instruction touch 32 rows = 32 cache lines for 16 bytes
// each.  So the loads are issued row-wise -- load i = 4c + q: lane l fetches the 16-byte piece l%8 of the 128-byte
// column block c of row 8q + l/8, eight whole cache lines per instruction -- and q_to_fragments turns the
// registers into fragments through a private 4 KB LDS buffer, one column block (four k-steps) at a time.
__device__ __forceinline__ void load_q(const MlaParams &kp, const Blk &k, int wave, int lane, bf16x8 (&qf)[NKS])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int t = min(k.t_w0 + 8 * q + (lane >> 3), kp.L - 1);
        const uint16_t *qp = kp.Q + (((size_t)k.b * kp.L + t) * kp.H + k.h) * DQK + (lane & 7) * 8;
#pragma unroll
        for (int c = 0; c < NKS / 4; ++c) qf[4 * c + q] = *reinterpret_cast<const bf16x8 *>(qp + c * 64);
    }
}

}  // namespace
}  // namespace lca

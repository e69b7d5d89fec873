// MLA prefill attention for calls with few work items (short prompts): the kernel of attn_mla.hip with a work item of half the size, whose key
// tiles are shared out over two wavefronts.
//
// A wavefront there owns 32 query rows and takes every key tile alone: an item lasts its number of tiles times 2 670 cycles, whatever else the
// chip has to do, and up to a few thousand tokens the chip has little (16 heads, L = 1500: 188 items on 256 CUs, the longest 36 tiles).  Here a
// workgroup has 64 (query row, head) pairs, and wavefronts w and w + 2 own the same 32 rows: of every tile of 32 entries the first takes the
// entries 0..15, the second 16..31, each with a softmax reference and an O^T (512 x 32, 256 accumulation registers) of its own, which they add
// up through LDS at the end of the item, half of the value columns each.  A tile costs a wavefront
//   S^T  36 MFMAs 16x16x32 (two query blocks of 16 per key fragment; 16 cycles each)   instead of 36 of 32x32x16
//   O^T  16 MFMAs 32x32x16 (one k-step)                                                 instead of 32
// and the tile itself and its copies stay as they are: 0.70 us a tile instead of 1.07 with half the CUs at work (230 instructions of about five cycles; without
// the copies 0.60, without LDS reads and exponentials as well 0.56).  Items are twice as many and half as long, and every tile is copied for 64 pairs instead of
// 128: where the chip is full anyway this is the slower form (the rule and its figures are at mla_halves in attn_mla.hip).
//
// Around the tile loop (100 MHz stamps, L = 300, 16 heads; the whole call 21.2 us undivided, 16.1 here): a pair loads its queries once, half the rows each, and
// shares them through LDS (each wavefront for itself: 288 KB through LDS, 1.06 us; fragments straight from memory, 64 bytes of 16 rows per load, 0.5 us slower
// still), and the two O^T are added up on the way to the output, 128 columns at a time (added up in registers first 18.5 us).  Without the first two tiles
// requested until the output is written an item change shows its round trip; few workgroups have one.
//
// S^T with 16x16x32: lane (q = l % 16, kg = l / 16) holds rows m = 4 kg + i (i = 0..3) of both query blocks, its queries q and 16 + q.
// The second product wants query l % 32 in lane l with eight keys: one v_permlane16_swap per register pair exchanges block 1 of the even
// lane groups with block 0 of the odd ones, after which k-slot (G = l / 32, 4 h + i) is row m = 8 G + 4 h + i.  Row m is computed from LDS
// row 16 half + pi(m), pi(8 G + 4 h + i) = 4 i + 2 h + G: 16 lanes read 16 rows that differ mod 16 (key reads) and rows 4 apart
// (transpose reads), as in attn_mla.hip.
#include "attn_mla.h"

namespace lca {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int HK = 16;                  // entries of a tile that a wavefront takes
constexpr int NCH = DQK / 32;           // 18 k-steps of S^T
constexpr int DEPTH = 4;                // key fragments in flight ahead of the S^T chain
constexpr int PG = 4;                   // V^T fragments in flight; the last PG steps of an O^T update run after the next barrier
constexpr int ORS = 128 * 2 + 16;       // row stride of the staging of the output in LDS (bytes)
constexpr int OWN = NDV / 2;            // value tiles of O^T a wavefront keeps at the end

union Pfrag { bf16x8 v; unsigned u[4]; };
struct Frags { bf16x4 lo[2][PG], hi[2][PG]; };
// per-lane softmax state of the two query blocks (base-2 logits)
struct State { float m_ref[2], l_run[2]; };

__device__ __forceinline__ constexpr int row_of_m(int m) { return 4 * (m & 3) + 2 * ((m >> 2) & 1) + (m >> 3); }

// V^T fragment of value tile j: step j of the O^T update.  The second wavefront of a pair has its value tiles in the order 8..15, 0..7, so that
// both keep their first eight (vp0: of this lane's tile 0 in that order, vp1 + 512: of its tile 8).
__device__ __forceinline__ void v_load(Frags &f, lds_cptr vp0, lds_cptr vp1, int j)
{
    typedef __attribute__((address_space(3))) bf16x4 *lds_b64_ptr;
    lds_cptr vp = (j < OWN ? vp0 : vp1) + j * 64;
    f.lo[(j / PG) & 1][j % PG] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64_ptr)(vp));
    f.hi[(j / PG) & 1][j % PG] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64_ptr)(vp + 2 * RSB));
}
template <bool F16>
__device__ __forceinline__ void pv_step(const Frags &f, const Pfrag &pb, floatx16 (&acc)[NDV], int j)
{
    const bf16x8 a = __builtin_shufflevector(f.lo[(j / PG) & 1][j % PG], f.hi[(j / PG) & 1][j % PG], 0, 1, 2, 3, 4, 5, 6, 7);
    acc[j] = pv_mfma<F16>(a, pb.v, acc[j]);
}

__device__ __forceinline__ bf16x8 key_frag(lds_cptr kb, const KSel &ksel, int ks)
{
    lds_cptr p = ks < DP / 32 ? kb + ks * 64 : (lds_cptr)(uintptr_t)ksel.a[ks - DP / 32];
    return *reinterpret_cast<__attribute__((address_space(3))) const bf16x8 *>(p);
}

// The copies of one tile after the other: what a wavefront's share (8 rows) of the next one needs.  Only the stage and the row advance from tile to
// tile; the segment changes once per item, in front of the tile loop's body.
struct Copies {
    int4v pool_rs, sel_rs;
    unsigned row_pool, row_sel;                  // byte offsets of the wavefront's first row in the segment
    unsigned m0;                                 // LDS address of its first row in the stage
    unsigned sel_delta, voff_pool, voff_pool4, voff_sel;    // (constants: RoPE part behind the latent part; per-lane offsets, of rows 0..3 and 4..7)
    __device__ __forceinline__ void start(const Blk &k, int tc, int wave)        // segment and row of tile tc
    {
        const bool is_rep = tc < k.n_rep_tiles;
        const Seg &ps = is_rep ? k.rep_pool : k.raw_pool, &ss = is_rep ? k.rep_sel : k.raw_sel;
        pool_rs = int4v{(int)ps.lo, (int)ps.hi, (int)ps.bytes, RSRC_WORD3};
        sel_rs = int4v{(int)ss.lo, (int)ss.hi, (int)ss.bytes, RSRC_WORD3};
        const unsigned row0 = (is_rep ? tc * BN : k.raw_lo_blk + (tc - k.n_rep_tiles) * BN) + 8 * wave;
        row_pool = row0 * (DP * 2);
        row_sel = row0 * (DS * 2);
    }
    __device__ __forceinline__ void issue(int j) const        // j: 0..8, a constant after unrolling
    {
        switch (j) {
        case 0: dma_1k<0 * RSB, 0>(voff_pool, pool_rs, row_pool, m0); break;
        case 1: dma_1k<1 * RSB - 1024, 1024>(voff_pool, pool_rs, row_pool, m0); break;
        case 2: dma_1k<2 * RSB - 2048, 2048>(voff_pool, pool_rs, row_pool, m0); break;
        case 3: dma_1k<3 * RSB - 3072, 3072>(voff_pool, pool_rs, row_pool, m0); break;
        case 4: dma_1k<4 * RSB, 0>(voff_pool4, pool_rs, row_pool, m0); break;
        case 5: dma_1k<5 * RSB - 1024, 1024>(voff_pool4, pool_rs, row_pool, m0); break;
        case 6: dma_1k<6 * RSB - 2048, 2048>(voff_pool4, pool_rs, row_pool, m0); break;
        case 7: dma_1k<7 * RSB - 3072, 3072>(voff_pool4, pool_rs, row_pool, m0); break;
        default: dma_1k<0, 0>(voff_sel, sel_rs, row_sel, m0 + sel_delta); break;
        }
    }
};

// S^T chain of this wavefront's half tile into `snext` (36 MFMAs, a key fragment feeds both query blocks) and, when LOOP, between its MFMAs the
// softmax of the half tile before it (`scur` into pb), the copy of the tile three steps ahead and the first V^T requests of the update that follows.
// (assembly, so that the accumulators are vector registers; the caller of the LOOP form keeps every reader of snext behind MFMAs of the update)
template <bool LOOP, bool F16>
__device__ __forceinline__ void chain(bf16x8 (&fr)[DEPTH], lds_cptr kb, const KSel &ksel, const bf16x8 (&qf)[NKS], floatx4 (&snext)[2], const floatx4 (&scur)[2],
                                      Pfrag &pb, State &st, float c, float bias, Frags &vf, lds_cptr vp0, lds_cptr vp1, const Copies &cp)
{
    float nb[2] = {0.f, 0.f}, p[2] = {0.f, 0.f};
    unsigned bits[4] = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < NCH; ++ks) {
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            LCA_FENCE();
            if (ks == 0) {
                if (F16) asm("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=&v"(snext[blk]) : "v"(fr[0]), "v"(qf[blk]));
                else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(snext[blk]) : "v"(fr[0]), "v"(qf[blk]));
            } else {
                if (F16) asm("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(snext[blk]) : "v"(fr[ks % DEPTH]), "v"(qf[2 * ks + blk]));
                else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(snext[blk]) : "v"(fr[ks % DEPTH]), "v"(qf[2 * ks + blk]));
            }
            LCA_FENCE();
            if (blk == 1) {
                if (ks + DEPTH < NCH) fr[ks % DEPTH] = key_frag(kb, ksel, ks + DEPTH);
                if (LOOP && ks >= NCH - COPIES_PER_TILE) cp.issue(ks - (NCH - COPIES_PER_TILE));
            } else if (LOOP) {
                // P^T = exp2(S^T c + bias - reference), a pair of registers per three steps; then the exchange between the lane groups
                if (ks == 0) { nb[0] = bias - st.m_ref[0]; nb[1] = bias - st.m_ref[1]; }
                if (ks < 12) {
                    const int k = ks / 3, sub = ks % 3, b = k >> 1;
                    if (sub < 2) p[sub] = __builtin_amdgcn_exp2f(fmaf(scur[b][2 * (k & 1) + sub], c, nb[b]));
                    else {
                        if (F16) bits[k] = __builtin_bit_cast(unsigned, f16x2{(_Float16)p[0], (_Float16)p[1]});
                        else bits[k] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)p[0], (__bf16)p[1]});
                        asm volatile("" : "+v"(bits[k]));       // (pins the conversion to this step)
                        st.l_run[b] += p[0];
                        st.l_run[b] += p[1];
                    }
                } else if (ks < 14) {
                    const int i = ks - 12;
                    const uintx2 sw = __builtin_amdgcn_permlane16_swap(bits[i], bits[2 + i], false, false);
                    pb.u[i] = sw[0]; pb.u[2 + i] = sw[1];
                    asm volatile("" : "+v"(pb.u[i]), "+v"(pb.u[2 + i]));
                } else v_load(vf, vp0, vp1, ks - 14);
            }
        }
    }
    LCA_FENCE();
    if (!LOOP) asm("s_nop 15\n\ts_nop 7" : "+v"(snext[0]), "+v"(snext[1]));
}

// Queries: the two wavefronts of a pair load 16 of their 32 rows each, row-wise (load 2 c + q: the 16-byte piece l % 8 of the 128-byte column block c of
// row 16 half + 8 q + l / 8, eight whole cache lines), and exchange them through LDS (36 KB per pair) on the way to the fragments of the first
// product: qf[2 ks + blk] = lane (q, kg) holds Q[row 16 blk + q][32 ks + 8 kg .. +7].  Piece p of row r of a block sits at r*128 + ((p ^ (r>>1)) & 7)*16: no
// bank conflicts either way.
__device__ __forceinline__ void load_q_rows(const MlaParams &kp, const Blk &k, int half, int lane, bf16x8 (&qr)[NKS])
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int t = min(k.t_w0 + 16 * half + 8 * q + (lane >> 3), kp.L - 1);
        const uint16_t *qp = kp.Q + (((size_t)k.b * kp.L + t) * kp.H + k.h) * DQK + (lane & 7) * 8;
#pragma unroll
        for (int c = 0; c < NKS / 4; ++c) qr[2 * c + q] = *reinterpret_cast<const bf16x8 *>(qp + c * 64);
    }
}
__device__ __forceinline__ void q_rows_to_lds(char *buf, int half, int lane, const bf16x8 (&qr)[NKS])
{
#pragma unroll
    for (int i = 0; i < NKS / 2; ++i) {
        const int r = 16 * half + 8 * (i & 1) + (lane >> 3);
        *reinterpret_cast<bf16x8 *>(buf + (i >> 1) * 4096 + r * 128 + (((lane & 7) ^ (r >> 1)) & 7) * 16) = qr[i];
    }
}
__device__ __forceinline__ void q_frags_from_lds(const char *buf, int lane, bf16x8 (&qf)[NKS])
{
#pragma unroll
    for (int i = 0; i < NKS; ++i) {
        const int r = 16 * (i & 1) + (lane & 15), piece = 4 * ((i >> 1) & 1) + (lane >> 4);
        qf[i] = *reinterpret_cast<const bf16x8 *>(buf + (i >> 2) * 4096 + r * 128 + ((piece ^ (r >> 1)) & 7) * 16);
    }
}

// Hide what a query row must not see in a boundary tile: register i holds entry e0 + 4 i, the row sees the `end - lo` entries from lo on.
__device__ __forceinline__ void mask4(floatx4 &sv, int e0, int lo, int end)
{
    const unsigned count = (unsigned)(end - lo);
#pragma unroll
    for (int i = 0; i < 4; ++i) sv[i] = (unsigned)(e0 + 4 * i - lo) < count ? sv[i] : -INFINITY;
}
// Over the lanes of a query (l % 16 alike)
__device__ __forceinline__ float over_groups_max(float t)
{
    const uintx2 a = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    t = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uintx2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float over_groups_sum(float t)
{
    const uintx2 a = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    t = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const uintx2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float row_max4(const floatx4 &sv, float c, float bias)
{
    return over_groups_max(fmaxf(fmaf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), c, bias), NEG_BIG));
}

// The pair's value up-projection (attn_mla.hip, up_project): this wavefront's value tiles are half of the contraction, `up` its part of all four
// output tiles, in the order that starts with the two it will store (W_mine: this head's matrix in fragment order, from the wavefront's k-steps on).
template <bool F16>
__device__ __forceinline__ void up_project_half(const floatx16 (&acc)[NDV], const uint16_t *W_mine, int half, int lane, floatx16 (&up)[DU / 32])
{
    const char *wl = reinterpret_cast<const char *>(W_mine) + lane * 16;
    constexpr int NMT = DU / 32, NF = 2 * OWN * NMT, AHEAD = 8;
    const int first = half * 2 * 1024, second = 2 * 1024 - first;        // output tiles 2 half, 2 half + 1, then the other two
    auto w = [&](int f) { return *reinterpret_cast<const bf16x8 *>(wl + (f / NMT) * NMT * 1024 + ((f & 2) ? second : first) + (f & 1) * 1024); };
    bf16x8 wf[AHEAD];
#pragma unroll
    for (int f = 0; f < AHEAD; ++f) wf[f] = w(f);
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) up[mt][r] = 0.f;
#pragma unroll
    for (int s = 0; s < 2 * OWN; ++s) {
        const int i = s >> 1, hh = s & 1;
        union { bf16x8 v; bf16x2 b[4]; f16x2 h[4]; } of;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float x0 = acc[i][8 * hh + 2 * j], x1 = acc[i][8 * hh + 2 * j + 1];
            if (F16) of.h[j] = f16x2{(_Float16)x0, (_Float16)x1};
            else of.b[j] = bf16x2{(__bf16)x0, (__bf16)x1};
        }
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt) {
            const int f = s * NMT + mt;
            up[mt] = pv_mfma<F16>(wf[f % AHEAD], of.v, up[mt]);
            if (f + AHEAD < NF) wf[f % AHEAD] = w(f + AHEAD);
        }
        LCA_FENCE();
    }
}

// Items, their order and the parameter block are those of attn_mla_kernel, an item of its 128 pairs being two here (two of four heads, one of two, or
// 64 of 128 rows); so is the tile loop's pipeline.
template <bool F16, bool UP>
__global__ __launch_bounds__(256) void attn_mla_kernel_halves(const MlaParams kp)
{
    __shared__ __attribute__((aligned(1024))) char stages[NSTAGE][STAGE_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave >> 1;
    const int L = kp.L, H = kp.H;
    const unsigned lds0 = lds_address(&stages[0][0]);

    const int hw = kp.hw_log2, rows = hw > 0 ? BM >> hw : BM / 2;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, n_slots = gridDim.x >> 3;
    const int n_units = kp.n_qb * kp.B, n_hg = 2 * (H >> hw), run = kp.run_log2;
    const int items_per_xcd = (((n_units - 1) >> (run + 3)) + 1) * (n_hg << run);
    auto item = [&](int kidx, int &b, int &h, int &t0, int &t_wfirst) {        // sequence, this wavefront's head, first row of the item and of the wavefront
        const int j = kidx / n_hg, hg = kidx - j * n_hg, deal = j >> run, pos = (xcd << run) + (j & ((1 << run) - 1)), last = (8 << run) - 1;
        const int ord = (deal << (run + 3)) + ((deal & 1) ? last - pos : pos);
        b = ord % kp.B;
        const int qb = kp.n_qb - 1 - ord / kp.B, r = wave & 1;
        t0 = qb * (BM >> hw) + (hw > 0 ? 0 : (1 - (hg & 1)) * (BM / 2));       // (the later rows first)
        h = hw > 1 ? hg * 2 + r : hw == 1 ? hg : hg >> 1;
        t_wfirst = t0 + (hw > 1 ? 0 : 32 * r);
        return ord < n_units && t0 < L;
    };

    const int q16 = lane & 15, kg = lane >> 4;
    const int krow = HK * half + row_of_m(q16);                                      // LDS row behind S^T row l % 16
    const int k_off = krow * RSB + kg * 16;
    const int ksel_off = SEL_OFF + krow * (DS * 2) + (((kg ^ (krow >> 1)) & 7) << 4);
    const int v_off0 = (HK * half + 4 * (q16 >> 2) + (lane >> 5)) * RSB + (16 * (kg & 1) + 4 * (lane & 3)) * 2;
    const int v_off = v_off0 + half * OWN * 64, v_off1 = v_off0 - half * OWN * 64;   // value tiles 8..15 first for the second half
    const int entry = HK * half + 2 * (kg & 1) + (kg >> 1);                          // register i of S^T is entry 4 i + this of the tile
    Copies cp;
    cp.voff_pool = lane * 16;
    cp.voff_pool4 = lane * 16 + 4 * (DP * 2);
    cp.voff_sel = (lane >> 3) * (DS * 2) + (((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) << 4);
    cp.sel_delta = SEL_OFF + 8 * wave * (DS * 2) - 8 * wave * RSB;
    const unsigned m0_first = lds0 + 8 * wave * RSB;
    const float c = kp.scale_log2;
    auto copy_tile = [&](const Blk &k, int tc, int stage) {          // the whole of one tile at once
        cp.start(k, tc, wave);
        cp.m0 = m0_first + stage * STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < COPIES_PER_TILE; ++j) cp.issue(j);
    };

    // A slot's items: one of every n_slots neighbours of the list, every other time counted from the other end, so that whoever has the longest of
    // one round has the shortest of the next.
    auto in_round = [&](int r) { return r * n_slots + ((r & 1) ? n_slots - 1 - slot : slot); };
    int round = 0, kidx = slot, ib, ih, it0, iw0;
    while (kidx < items_per_xcd && !item(kidx, ib, ih, it0, iw0)) kidx = in_round(++round);
    if (kidx >= items_per_xcd) return;
    Blk cur = make_blk(kp, ib, ih, it0, rows, iw0, q16);
    // representatives that the query row of block 1 sees (no branch: with one here the compiler takes the copies' scalars for per-lane values)
    auto visible_of_block1 = [&](const Blk &k) { return kp.dense ? 0 : max(k.t_row + 17 - kp.w, 0) / kp.g; };
    int mt_row1 = visible_of_block1(cur);

    bf16x8 qf[NKS];
    floatx16 acc[NDV];
    State st;
    copy_tile(cur, 0, 0);
    copy_tile(cur, 1, 1);
    load_q_rows(kp, cur, half, lane, qf);
    // stages 2 and 3 hold the queries until they are in registers: tile 2 is copied after that
    char *const qbuf = &stages[2][0] + (wave & 1) * (NKS / 4 * 4096);
    static_assert(2 * (NKS / 4) * 4096 <= 2 * STAGE_BYTES, "the queries must fit in two stages");

    while (true) {
        int pass = 0;
        float m_exact[2] = {NEG_BIG, NEG_BIG};
        while (true) {       // passes over this item: 0 = normal; 2 = again, from exact maxima
            {
                bf16x8 zf = {0, 0, 0, 0, 0, 0, 0, 0};
                asm volatile("" : "+v"(zf));
#pragma unroll
                for (int i = 0; i < NDV; ++i) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %1, 0" : "=a"(acc[i]) : "v"(zf));
            }
            st.m_ref[0] = m_exact[0]; st.m_ref[1] = m_exact[1]; st.l_run[0] = 0.f; st.l_run[1] = 0.f;
            bool need_ref = pass == 0;

            floatx4 snext[2], scur[2];
            Pfrag pb;
            Frags vf;
            bf16x8 fr[DEPTH];
            // there is no tile -1: its held-back MFMAs add V^T = 0 times P^T = 0
#pragma unroll
            for (int i = 0; i < PG; ++i) { vf.lo[1][i] = bf16x4{0, 0, 0, 0}; vf.hi[1][i] = bf16x4{0, 0, 0, 0}; }
            pb.v = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (pass == 0) {
                q_rows_to_lds(qbuf, half, lane, qf);
                __syncthreads();
                q_frags_from_lds(qbuf, lane, qf);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __syncthreads();                  // every wavefront has its queries
                copy_tile(cur, 2, 2);
            } else __syncthreads();
            {
                lds_cptr s0 = (lds_cptr)(uintptr_t)lds0;
                KSel ks0 = {{lds0 + ksel_off, (lds0 + ksel_off) ^ (1u << 6), 0, 0}};
#pragma unroll
                for (int i = 0; i < DEPTH; ++i) fr[i] = key_frag(s0 + k_off, ks0, i);
                chain<false, F16>(fr, s0 + k_off, ks0, qf, snext, snext, pb, st, c, 0.f, vf, s0, s0, cp);
            }
            scur[0] = snext[0]; scur[1] = snext[1];
            // What an iteration needs besides the data, carried on from tile to tile: the copy of tile tl+3, the stages of the S^T chain (tile tl+1) and of the O^T
            // update (tile tl) as this lane's read addresses, and whether the next tile has entries to hide.
            cp.start(cur, 3, wave);
            unsigned st_pv = lds0, st_chain = lds0 + STAGE_BYTES, st_copy = lds0 + 3 * STAGE_BYTES;
            cp.m0 = st_copy + 8 * wave * RSB;
            unsigned a_k = st_chain + k_off, a_v0 = st_pv + v_off, a_v1 = st_pv + v_off1;
            KSel a_s = {{st_chain + ksel_off, (st_chain + ksel_off) ^ (1u << 6), 0, 0}};
            float bias = cur.n_rep_tiles > 0 ? kp.bias_log2 : 0.f;
            int tl0 = 0;
            asm volatile("" : "+s"(tl0));
            auto tile_is_full = [&](int tl) { return lt_mask(tl, cur.rep_full_end) | (~lt_mask(tl, cur.raw_full_lo) & lt_mask(tl, cur.raw_full_hi)); };
            int full = tile_is_full(tl0);

            for (int tl = tl0; tl < cur.n_tiles; ++tl) {
                if (__builtin_expect((full == 0) | need_ref | (tl == cur.n_rep_tiles) | (tl + 3 == cur.n_rep_tiles), 0)) {
                    if (tl + 3 == cur.n_rep_tiles) cp.start(cur, tl + 3, wave);      // the raw tokens' segment from here on
                    if (tl == cur.n_rep_tiles) bias = 0.f;
                    if (full == 0) {
                        const bool is_rep = tl < cur.n_rep_tiles;
                        const int e0 = (is_rep ? tl * BN : cur.raw_lo_blk + (tl - cur.n_rep_tiles) * BN) + entry;
                        mask4(scur[0], e0, is_rep ? -(1 << 30) : cur.raw_lo_row, is_rep ? cur.mt_row : cur.t_row + 1);
                        mask4(scur[1], e0, is_rep ? -(1 << 30) : mt_row1 * kp.g, is_rep ? mt_row1 : cur.t_row + 17);
                    }
                    if (need_ref) {
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            const float mx = row_max4(scur[b], c, bias);
                            st.m_ref[b] = (st.m_ref[b] == NEG_BIG) ? (F16 ? mx + REF_SHIFT_F16 : mx) : st.m_ref[b];
                        }
                        need_ref = __builtin_amdgcn_ballot_w64((st.m_ref[0] == NEG_BIG) | (st.m_ref[1] == NEG_BIG)) != 0;
                    }
                }
                asm volatile("s_waitcnt vmcnt(9) lgkmcnt(0)" ::: "memory");
                __syncthreads();
                LCA_FENCE();
                lds_cptr kb = (lds_cptr)(uintptr_t)a_k, vp0 = (lds_cptr)(uintptr_t)a_v0, vp1 = (lds_cptr)(uintptr_t)a_v1;
#pragma unroll
                for (int i = 0; i < DEPTH; ++i) fr[i] = key_frag(kb, a_s, i);
#pragma unroll
                for (int j = NDV - PG; j < NDV; ++j) {          // the held-back steps of the tile before
                    LCA_FENCE();
                    pv_step<F16>(vf, pb, acc, j);
                }
                chain<true, F16>(fr, kb, a_s, qf, snext, scur, pb, st, c, bias, vf, vp0, vp1, cp);
                unsigned nk = 0, nv0 = 0, nv1 = 0, ns0 = 0, ns1 = 0, next = 0;
                int nfull = 0;
#pragma unroll
                for (int j = 0; j < NDV - PG; ++j) {
                    LCA_FENCE();
                    pv_step<F16>(vf, pb, acc, j);
                    LCA_FENCE();
                    v_load(vf, vp0, vp1, j + PG);
                    LCA_FENCE();
                    // (nothing reads the chain's result before four MFMAs of the update have run)
                    if (j >= 4) asm volatile("v_mov_b32 %0, %1" : "=v"(scur[(j - 4) >> 2][(j - 4) & 3]) : "v"(snext[(j - 4) >> 2][(j - 4) & 3]));
                    // the bookkeeping of iteration tl+1, a few instructions per MFMA
                    switch (j) {
                    case 0: cp.row_pool += BN * DP * 2; cp.row_sel += BN * DS * 2; LCA_PIN_S(cp.row_pool); LCA_PIN_S(cp.row_sel); break;
                    case 1: cp.m0 = st_pv + 8 * wave * RSB; LCA_PIN_S(cp.m0); break;
                    case 2: next = st_chain + STAGE_BYTES; next = next == lds0 + NSTAGE * STAGE_BYTES ? lds0 : next; LCA_PIN_S(next); break;
                    case 3: nfull = lt_mask(tl + 1, cur.rep_full_end); LCA_PIN_S(nfull); break;
                    case 4: nfull |= ~lt_mask(tl + 1, cur.raw_full_lo) & lt_mask(tl + 1, cur.raw_full_hi); LCA_PIN_S(nfull); break;
                    case 5: nk = next + k_off; LCA_PIN_V(nk); break;
                    case 6: ns0 = next + ksel_off; LCA_PIN_V(ns0); break;
                    case 7: ns1 = ns0 ^ (1u << 6); LCA_PIN_V(ns1); break;
                    case 9: nv0 = st_chain + v_off; LCA_PIN_V(nv0); break;
                    case 10: nv1 = st_chain + v_off1; LCA_PIN_V(nv1); break;
                    default: break;
                    }
                }
                LCA_FENCE();
                st_pv = st_chain; st_chain = next; full = nfull;
                a_k = nk; a_v0 = nv0; a_v1 = nv1; a_s.a[0] = ns0; a_s.a[1] = ns1;
            }
#pragma unroll
            for (int j = NDV - PG; j < NDV; ++j) pv_step<F16>(vf, pb, acc, j);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the trailing copies have landed before the stages are reused
            {
                const float l0 = over_groups_sum(st.l_run[0]), l1 = over_groups_sum(st.l_run[1]);
                const bool redo = pass == 0 && (!(l0 <= L_LIMIT) | !(l1 <= L_LIMIT) | (F16 && !(acc[0][0] * 0.f == 0.f)));
                if (!__syncthreads_or(redo)) break;
                // exact row maxima, one tile at a time: tile tl goes into stage tl % 2 after the barrier of tile tl-1
                m_exact[0] = NEG_BIG; m_exact[1] = NEG_BIG;
                for (int tl = 0; tl < cur.n_tiles; ++tl) {
                    copy_tile(cur, tl, tl & 1);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                    const unsigned stage = lds0 + (tl & 1) * STAGE_BYTES;
                    lds_cptr sp = (lds_cptr)(uintptr_t)stage;
                    const KSel ksp = {{stage + ksel_off, (stage + ksel_off) ^ (1u << 6), 0, 0}};
                    floatx4 sv[2];
#pragma unroll
                    for (int i = 0; i < DEPTH; ++i) fr[i] = key_frag(sp + k_off, ksp, i);
                    chain<false, F16>(fr, sp + k_off, ksp, qf, sv, sv, pb, st, c, 0.f, vf, sp, sp, cp);
                    const bool is_rep = tl < cur.n_rep_tiles;
                    const int e0 = (is_rep ? tl * BN : cur.raw_lo_blk + (tl - cur.n_rep_tiles) * BN) + entry;
                    mask4(sv[0], e0, is_rep ? -(1 << 30) : cur.raw_lo_row, is_rep ? cur.mt_row : cur.t_row + 1);
                    mask4(sv[1], e0, is_rep ? -(1 << 30) : mt_row1 * kp.g, is_rep ? mt_row1 : cur.t_row + 17);
#pragma unroll
                    for (int b = 0; b < 2; ++b) m_exact[b] = fmaxf(m_exact[b], row_max4(sv[b], c, is_rep ? kp.bias_log2 : 0.f));
                }
                __syncthreads();
                pass = 2;
                for (int tl = 0; tl < 3; ++tl) copy_tile(cur, tl, tl);
            }
        }

        // ---- the pair's results into one: this wavefront's value tiles 8..15 (in its order) are the partner's 0..7 ----
        int nb, nh, nt0, nw0;
        do kidx = in_round(++round);
        while (kidx < items_per_xcd && !item(kidx, nb, nh, nt0, nw0));
        const bool has_next = kidx < items_per_xcd;
        const int out_b = cur.b, out_h = cur.h, t_wfirst = cur.t_w0;
        const int lane_here = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));   // (afresh: see attn_mla.hip)
        const int n_here = lane_here & 31, G_here = lane_here >> 5;
        const bool odd = (lane_here & 16) != 0;                    // query row l % 32 is one of block 1
        const float m_two[2] = {st.m_ref[0], st.m_ref[1]}, l_two[2] = {over_groups_sum(st.l_run[0]), over_groups_sum(st.l_run[1])};
        const float m_mine = odd ? m_two[1] : m_two[0], l_mine = odd ? l_two[1] : l_two[0];
        if (has_next) {
            cur = make_blk(kp, nb, nh, nt0, rows, nw0, lane_here & 15);
            mt_row1 = visible_of_block1(cur);
            if (!UP) load_q_rows(kp, cur, half, lane_here, qf);
        }
        char *const xch = &stages[0][0];
        constexpr int XW = OWN * 16 * 256;                         // 32 KB per wavefront; then (reference, sum) of its 32 rows
        static_assert(4 * XW + 4 * 256 <= NSTAGE * STAGE_BYTES, "the exchange must fit");
#pragma unroll
        for (int i = 0; i < OWN; ++i)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *reinterpret_cast<floatx4 *>(xch + wave * XW + (i * 4 + r4) * 1024 + lane_here * 16) =
                    floatx4{acc[OWN + i][4 * r4], acc[OWN + i][4 * r4 + 1], acc[OWN + i][4 * r4 + 2], acc[OWN + i][4 * r4 + 3]};
        float2 *const rows_ml = reinterpret_cast<float2 *>(xch + 4 * XW);
        if (G_here == 0) rows_ml[wave * 32 + n_here] = make_float2(m_mine, l_mine);
        __syncthreads();
        const float2 other = rows_ml[(wave ^ 2) * 32 + n_here];
        const float m_ref = fmaxf(m_mine, other.x);
        const float f_mine = __builtin_amdgcn_exp2f(m_mine - m_ref), f_other = __builtin_amdgcn_exp2f(other.x - m_ref);   // (0 for a half that saw nothing)
        const float l_tot = l_mine * f_mine + other.y * f_other;
        const float inv = 1.f / l_tot, w_mine = f_mine * inv, w_other = f_other * inv;
        char *const from = xch + (wave ^ 2) * XW;                  // (nobody else reads it)
        auto partner4 = [&](int i, int r4) { return *reinterpret_cast<const floatx4 *>(from + (i * 4 + r4) * 1024 + lane_here * 16); };

        // ---- epilogue: this wavefront's half of the columns, transposed through LDS, stored coalesced ----
        const int rows_valid = min(max(L - t_wfirst, 0), 32);
        constexpr int DO = UP ? DU : DV;                     // width of an output row
        const __amdgpu_buffer_rsrc_t o_rs = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(kp.O + (((size_t)out_b * L + t_wfirst) * H + out_h) * DO), (short)0,
            rows_valid > 0 ? ((rows_valid - 1) * H * DO + DO) * 2 : 0, RSRC_WORD3);
        constexpr int CW = UP ? 64 : 128;                    // columns per pass
        const int o_voff = ((lane_here * 8 / CW) * H * DO + half * (DO / 2) + lane_here * 8 % CW) * 2;
        auto store_columns = [&](char *obuf, int col, auto value) {      // value(d4, r4): four neighbouring columns of this lane's row
#pragma unroll
            for (int d4 = 0; d4 < CW / 32; ++d4)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const floatx4 x = value(d4, r4);
                    union { bf16x4 h; f16x4 hf; uint2 u; } o;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (F16) o.hf[i] = (_Float16)x[i];
                        else o.h[i] = (__bf16)x[i];
                    }
                    *reinterpret_cast<uint2 *>(obuf + n_here * ORS + (d4 * 32 + 8 * r4 + 4 * G_here) * 2) = o.u;
                }
            __builtin_amdgcn_wave_barrier();
            constexpr int RPS = 512 / CW;                    // rows of one wave-wide store
#pragma unroll
            for (int r0 = 0; r0 < 32; r0 += RPS) {
                const uintx4 v = *reinterpret_cast<const uintx4 *>(obuf + (r0 + lane_here * 8 / CW) * ORS + (lane_here * 8 % CW) * 2);
                __builtin_amdgcn_raw_buffer_store_b128(v, o_rs, o_voff, (r0 * H * DO + col) * 2, 0);
            }
            __builtin_amdgcn_wave_barrier();
        };
        if constexpr (UP) {
            floatx16 up[DU / 32];
#pragma unroll
            for (int i = 0; i < OWN; ++i)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const floatx4 o = partner4(i, r4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][4 * r4 + j] = acc[i][4 * r4 + j] * w_mine + o[j] * w_other;
                }
            __syncthreads();     // every wavefront has read: the stages are free
            if (has_next) { copy_tile(cur, 0, 0); copy_tile(cur, 1, 1); }
            up_project_half<F16>(acc, kp.W_up + (size_t)out_h * DU * DV + half * (OWN * 2 * (DU / 32) * 512), half, lane_here, up);
            if (has_next) load_q_rows(kp, cur, half, lane_here, qf);
            char *const xu = &stages[3][0];                        // 8 KB per wavefront: the two output tiles the partner stores
            static_assert(4 * 8192 <= STAGE_BYTES, "the exchange must fit");
#pragma unroll
            for (int k = 0; k < 8; ++k)
                *reinterpret_cast<floatx4 *>(xu + wave * 8192 + k * 1024 + lane_here * 16) =
                    floatx4{up[2 + (k >> 2)][4 * (k & 3)], up[2 + (k >> 2)][4 * (k & 3) + 1], up[2 + (k >> 2)][4 * (k & 3) + 2], up[2 + (k >> 2)][4 * (k & 3) + 3]};
            __syncthreads();
            store_columns(&stages[2][0] + wave * 32 * ORS, 0, [&](int d4, int r4) {
                const floatx4 o = *reinterpret_cast<const floatx4 *>(xu + (wave ^ 2) * 8192 + (d4 * 4 + r4) * 1024 + lane_here * 16);
                return floatx4{up[d4][4 * r4] + o[0], up[d4][4 * r4 + 1] + o[1], up[d4][4 * r4 + 2] + o[2], up[d4][4 * r4 + 3] + o[3]};
            });
        } else {
            // 128 columns at a time: what the partner left of them is read first, then the same part of LDS takes the output
            static_assert(32 * ORS <= 4 * 4096, "output staging must fit where four value tiles were");
#pragma unroll
            for (int ps = 0; ps < OWN / 4; ++ps) {
                floatx4 o[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) o[k] = partner4(ps * 4 + (k >> 2), k & 3);
                store_columns(from + ps * 4 * 4096, ps * 128, [&](int d4, int r4) {
                    floatx4 x;
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = acc[ps * 4 + d4][4 * r4 + j] * w_mine + o[d4 * 4 + r4][j] * w_other;
                    return x;
                });
            }
        }
        if (kp.lse != nullptr) {
            const int t_row_here = t_wfirst + n_here;
            if (half == 0 && G_here == 0 && t_row_here < L)
                kp.lse[((size_t)out_b * L + t_row_here) * H + out_h] = (m_ref + log2f(l_tot)) * 0.6931471805599453f;
        }
        if (!has_next) break;
        __syncthreads();         // every wavefront is done with the stages
        if (!UP) { copy_tile(cur, 0, 0); copy_tile(cur, 1, 1); }
    }
}

}  // namespace

void launch_mla_halves(const MlaParams &kp, bool f16, unsigned grid, hipStream_t st)
{
    if (kp.W_up != nullptr) {
        if (f16) attn_mla_kernel_halves<true, true><<<grid, 256, 0, st>>>(kp);
        else attn_mla_kernel_halves<false, true><<<grid, 256, 0, st>>>(kp);
    } else {
        if (f16) attn_mla_kernel_halves<true, false><<<grid, 256, 0, st>>>(kp);
        else attn_mla_kernel_halves<false, false><<<grid, 256, 0, st>>>(kp);
    }
}

}  // namespace lca

// Exchanges between the lanes of a wavefront by the vector ALU: DPP inside 16 lanes, v_permlane16_swap / v_permlane32_swap across them.  A shuffle through
// LDS (ds_bpermute) takes about 130 cycles from issue to use, and the kernels that reduce over lanes (condensation, cache update, decode merge) are chains of
// a dozen and more of them; one of these takes 10 to 20.  Calls back to back in a graph, by shuffles / so: condensation 512 + 64, L = 1500 8.57 / 7.83 us, 64 / 64,
// L = 2500 9.29 / 8.35, fp32 128 + 32, L = 1024 8.25 / 7.53; cache update, 28 heads over 4 KV heads, g = 16 6.29 / 5.17, g = 32 8.41 / 6.69; decode step with merge, 16
// heads, 512 + 64, B = 1, L = 4001 10.4 / 10.0, 28 over 4, B = 5, L = 4001 7.80 / 7.40.
// Every lane adds the same numbers in the same tree whatever its place in the group, so equal rows keep equal bits.
#pragma once
#include <hip/hip_runtime.h>

namespace lca {
namespace lanes {

typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

struct Sum { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct Max { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

constexpr int XOR1 = 0xB1, XOR2 = 0x4E, HALF_MIRROR = 0x141, MIRROR = 0x140, ROR = 0x120;      // DPP controls; ROR + n: rotated by n inside 16 lanes
template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// The odd 16-lane rows of a against the even ones of b; the upper half of a against the lower one of b.
__device__ __forceinline__ void swap16(float &a, float &b)
{
    const uintx2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float &a, float &b)
{
    const uintx2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
template <class Op> __device__ __forceinline__ float across16(float v, Op op) { float w = v; swap16(v, w); return op(v, w); }     // lane l with lane l ^ 16
template <class Op> __device__ __forceinline__ float across32(float v, Op op) { float w = v; swap32(v, w); return op(v, w); }     // lane l with lane l ^ 32

// Over aligned groups of LANES lanes (a power of two), the result in all of them.  (The mirrors reach the other half of a group: all its lanes
// hold the half's result by then.)
template <int LANES, class Op> __device__ __forceinline__ float over_group(float v, Op op)
{
    if (LANES >= 2) v = op(v, dpp<XOR1>(v));
    if (LANES >= 4) v = op(v, dpp<XOR2>(v));
    if (LANES >= 8) v = op(v, dpp<HALF_MIRROR>(v));
    if (LANES >= 16) v = op(v, dpp<MIRROR>(v));
    if (LANES >= 32) v = across16(v, op);
    if (LANES >= 64) v = across32(v, op);
    return v;
}
// The same for N values and groups of 2^shift lanes, shift wave-uniform.
template <int N, class Op> __device__ __forceinline__ void over_group(float (&v)[N], int shift, Op op)
{
    auto each = [&](auto step) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = step(v[i]);
    };
    if (shift >= 1) each([&](float x) { return op(x, dpp<XOR1>(x)); });
    if (shift >= 2) each([&](float x) { return op(x, dpp<XOR2>(x)); });
    if (shift >= 3) each([&](float x) { return op(x, dpp<HALF_MIRROR>(x)); });
    if (shift >= 4) each([&](float x) { return op(x, dpp<MIRROR>(x)); });
    if (shift >= 5) each([&](float x) { return across16(x, op); });
    if (shift >= 6) each([&](float x) { return across32(x, op); });
}
// Over the lanes that share l mod 2^shift (the other lane bits), shift wave-uniform.
template <int N, class Op> __device__ __forceinline__ void over_strided(float (&v)[N], int shift, Op op)
{
    auto each = [&](auto step) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = step(v[i]);
    };
    if (shift <= 3) each([&](float x) { return op(x, dpp<ROR + 8>(x)); });
    if (shift <= 2) each([&](float x) { return op(x, dpp<ROR + 4>(x)); });
    if (shift <= 1) each([&](float x) { return op(x, dpp<ROR + 2>(x)); });
    if (shift <= 0) each([&](float x) { return op(x, dpp<ROR + 1>(x)); });
    if (shift <= 4) each([&](float x) { return across16(x, op); });
    if (shift <= 5) each([&](float x) { return across32(x, op); });
}

}  // namespace lanes
}  // namespace lca

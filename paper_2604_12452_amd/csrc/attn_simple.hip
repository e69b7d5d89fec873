// Straightforward attention kernel for any sizes and all element types: one wavefront per (sequence, token, head) row
// (attn_row.h).  Serves what the tiled kernels do not take (attn_tile.hip): a pooled component above 512 columns, keys above 576,
// both components together beyond the widest class's pieces, sequences of 4 GB and more, and rows that see a few entries only.
#include "attn_row.h"

namespace lca {
namespace {

using namespace attn_row;

template <typename T>
__global__ __launch_bounds__(WAVE) void attn_simple_kernel(const RowParams<T> kp)
{
    __shared__ float q_s[MAXD];
    __shared__ float p_s[WAVE];
    attend_row<T, MAXD / WAVE>(kp, blockIdx.x, q_s, p_s, threadIdx.x);
}

template <typename T> void run(const AttnArgs &a, hipStream_t st)
{
    const long rows = (long)a.d.B * a.d.L * a.d.H;
    attn_simple_kernel<T><<<(unsigned)rows, WAVE, 0, st>>>(row_params<T>(a));
}

}  // namespace

hipError_t launch_attn_simple(const AttnArgs &a, hipStream_t st)
{
    if (a.d.dtype == LCA_BF16) run<uint16_t>(a, st);
    else if (a.d.dtype == LCA_F16) run<f16_t>(a, st);
    else run<float>(a, st);
    return hipGetLastError();
}

}  // namespace lca

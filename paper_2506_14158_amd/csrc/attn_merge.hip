// The merge kernel of a divided attention launch (attn_merge.h), as a launch of its own.
#include "attn_merge.h"

namespace s4c {

namespace {

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a, int passes) {
    merge::merge_rows<T, D>(a, blockIdx.x, blockIdx.y, passes);
}

template <typename T>
hipError_t launch(const AttnArgs& a, hipStream_t st) {
    const merge::Grid g = merge::grid_of(a);
    const dim3 grid((unsigned)g.units, (unsigned)g.chunks), block(256);
    if (a.D == 64) hipLaunchKernelGGL((attn_merge_kernel<T, 64>), grid, block, 0, st, a, g.passes);
    else hipLaunchKernelGGL((attn_merge_kernel<T, 128>), grid, block, 0, st, a, g.passes);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_merge(const AttnArgs& a, int dtype, hipStream_t st) {
    return dtype == S4C_F32 ? launch<float>(a, st) : dtype == S4C_F16 ? launch<f16_t>(a, st) : launch<bf16_t>(a, st);
}

}  // namespace s4c

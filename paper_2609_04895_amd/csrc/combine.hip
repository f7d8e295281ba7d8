// combine.hip - the gated combine of the expert outputs of a batch of layers
// (the device function is in combine.h).
#include "combine.h"

namespace cmoe {

namespace {

// grid: x = workgroups of one layer, y = layers of the batch
__global__ __launch_bounds__(kCombineThreads) void combine_kernel(Layout lo, int l0, float* __restrict__ y) {
    combine_quad(lo, l0 + blockIdx.y, blockIdx.y, y, (int64_t)blockIdx.x * kCombineThreads + threadIdx.x);
}

}  // namespace

hipError_t launch_combine(const Layout& lo, int l0, int nl, float* y, hipStream_t st, const Timing& tm) {
    launch_kernel(combine_kernel, dim3((unsigned)combine_groups(lo), nl), dim3(kCombineThreads), st, tm, lo, l0, y);
    return hipGetLastError();
}

}  // namespace cmoe

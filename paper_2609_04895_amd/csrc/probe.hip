// probe.hip - a streaming read of a device buffer with the access pattern of
// the FFN kernels' expert weight loads: 16-byte nontemporal loads, 64 lanes
// covering one contiguous kilobyte per instruction, sixteen kilobytes in flight
// per wavefront, each wavefront, a workgroup of its own, walking one contiguous
// block.  Its rate is the practical ceiling that the weight stream of a token
// can reach on this device, measured in the caller's process.
//
// Blocks of 64 KB, handed out as wavefronts end, so that the slowest ones do not
// set the time.  Best of eight launches over 1 and 4 GiB, TB/s: 7.06 and 7.11;
// blocks of 128 to 512 KB 6.91 to 7.01 and 7.03 to 7.09; eight kilobytes in
// flight 6.99 and 7.07; four wavefronts per workgroup 6.87 and 6.92, and with
// eight kilobytes in flight and 4096 blocks in all (no block waits for another
// to end) 6.58 and 6.97, which the gate/up kernel exceeds.
#include "cmoe_internal.h"

namespace cmoe {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Where the xor of everything read is stored if it equals a value that it
// never takes in practice: the loads are kept, and nothing is written.  (The
// variable has external linkage, so the compiler cannot drop the store, and
// with it the loads.)
__device__ u32x4 g_probe_sink;

namespace {

constexpr int kProbeDepth = 16;                 // 1 KB loads in flight per wavefront
constexpr int64_t kProbeBlockBytes = 64 << 10;  // one wavefront's block
static_assert(kProbeBlockBytes % (1024 * kProbeDepth) == 0, "whole rounds of loads");

__global__ __launch_bounds__(64) void read_probe_kernel(const u32x4* __restrict__ src) {
    constexpr int64_t n = kProbeBlockBytes / 16;  // 16-byte units
    const u32x4* p = src + blockIdx.x * n + threadIdx.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int64_t i = 0; i < n; i += 64 * kProbeDepth) {
        u32x4 v[kProbeDepth];
#pragma unroll
        for (int u = 0; u < kProbeDepth; ++u) v[u] = __builtin_nontemporal_load(p + i + 64 * u);
#pragma unroll
        for (int u = 0; u < kProbeDepth; ++u) acc ^= v[u];
    }
    if (acc.x == 0x9E3779B9u && acc.y == 0x7F4A7C15u && acc.z == 0x85EBCA6Bu && acc.w == 0xC2B2AE35u) g_probe_sink = acc;
}

}  // namespace

int64_t read_probe_bytes(int64_t bytes) { return bytes / kProbeBlockBytes * kProbeBlockBytes; }

hipError_t launch_read_probe(const void* src, int64_t bytes, hipStream_t st, const Timing& tm) {
    launch_kernel(read_probe_kernel, dim3((unsigned)(bytes / kProbeBlockBytes)), dim3(64), st, tm,
                  static_cast<const u32x4*>(src));
    return hipGetLastError();
}

}  // namespace cmoe

// ANS decode (Non-Parallel: 64 interleaved coders per chunk).
#include "kernels.hpp"

namespace zf {
// One chunk per wave; each wave's model, ring and output staging are dynamic
// LDS.
__global__ __launch_bounds__(1024) void k_decode_ans(LaunchArgs A) {
    const uint32_t waves = blockDim.x / 64;
    const uint32_t u = A.kind_begin[K_ANS] + blockIdx.x * waves + first32(threadIdx.x / 64);
    if (u >= A.kind_begin[K_ANS + 1]) return;
    extern __shared__ __attribute__((aligned(16))) uint32_t ans_smem[];
    unit_ans_t<false>(A, A.chunks[A.tiles[u].chunk], ans_smem + (threadIdx.x / 64) * kAnsLdsWords);
}
// The fused model: one wave per workgroup, so that its LDS addresses are
// constants.
__global__ __launch_bounds__(64) void k_decode_ans_fused(LaunchArgs A) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kAnsLdsWordsFused];
    const uint32_t u = A.kind_begin[K_ANS] + blockIdx.x;
    unit_ans_t<true>(A, A.chunks[A.tiles[u].chunk], lds);
}

void launch_ans(const LaunchArgs &A, uint32_t waves, hipStream_t st) {
    const uint32_t n = A.kind_begin[K_ANS + 1] - A.kind_begin[K_ANS];
    if (!n) return;
    // Work of as many whole chunks as fit the chip with the fused model at
    // once (eight per compute unit) waits for the step's latency, where that
    // model wins; with more, the other's 19 waves a CU do, or are about even.
    // 64 KiB of flags each: 1,024 chunks 84 us fused, 143 us not; 2,048 97 and
    // 146 us; 2,304 160 and 154 us; 4,096 189 and 176 us; 16,384 729 and 703 us.
    // Workgroups of a size that the caller set run the other.
    if (A.ans_alone && A.ans_load <= 8 * cu_count()) {
        hipLaunchKernelGGL(k_decode_ans_fused, dim3(n), dim3(64), 0, st, A);
        return;
    }
    waves = waves > 16 ? 16 : waves;
    const size_t lds = size_t(waves) * kAnsLdsWords * sizeof(uint32_t);  // at most 130 KiB
    if (lds > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_decode_ans),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    hipLaunchKernelGGL(k_decode_ans, dim3((n + waves - 1) / waves), dim3(64 * waves), lds, st, A);
}
}  // namespace zf

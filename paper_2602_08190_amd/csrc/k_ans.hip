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
    unit_ans_t<Ans::kTwo>(A, A.chunks[A.tiles[u].chunk], ans_smem + (threadIdx.x / 64) * kAnsLdsWords);
}
// The fused model: one wave per workgroup, so that its LDS addresses are
// constants.
__global__ __launch_bounds__(64) void k_decode_ans_fused(LaunchArgs A) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kAnsLdsWordsFused];
    const uint32_t u = A.kind_begin[K_ANS] + blockIdx.x;
    unit_ans_t<Ans::kFused>(A, A.chunks[A.tiles[u].chunk], lds);
}

// The small layout, likewise.
__global__ __launch_bounds__(64) void k_decode_ans_small(LaunchArgs A) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kAnsLdsWordsSmall];
    const uint32_t u = A.kind_begin[K_ANS] + blockIdx.x;
    unit_ans_t<Ans::kSmall>(A, A.chunks[A.tiles[u].chunk], lds);
}

void launch_ans(const LaunchArgs &A, uint32_t waves, hipStream_t st) {
    const uint32_t n = A.kind_begin[K_ANS + 1] - A.kind_begin[K_ANS];
    if (!n) return;
    // Work of as many whole chunks as fit the chip with the fused model at
    // once (eight per compute unit) waits for the step's latency, where that
    // model wins; with more, the other's 18 waves a CU do, or are about even.
    // 64 KiB of flags each: 1,024 chunks 79 us fused, 136 us not; 2,048 89 and
    // 136 us; 2,304 160 and 143 us; 4,096 189 and 158 us; 16,384 729 and 613 us.
    // Workgroups of a size that the caller set run the other.
    if (A.ans_alone && A.ans_load <= 8 * cu_count()) {
        hipLaunchKernelGGL(k_decode_ans_fused, dim3(n), dim3(64), 0, st, A);
        return;
    }
    // With 25 waves a compute unit instead of 18 the small layout may need a round
    // less.  Flags in chunks of 64 KiB, kTwo and kSmall: 18 chunks a compute unit 171
    // and 199 us, 19 268 and 202, 24 290 and 226, 26 294 and 344, 34 359 and 382, 38 418
    // and 387, 46 459 and 435; of 16 KiB 18 51 and 53, 19 76 and 53, 26 82 and 82, 38
    // 114 and 94, 64 170 and 158; of 4 KiB 18 19.3 and 19.4, 19 27 and 19, 64 57 and 48.
    // Past three rounds chunks of 64 KiB gain or lose by what they hold (64 a compute
    // unit, flags 613 and 603, text 643 and 684; the fact table's indices 585 and 632).
    const uint32_t cus = cu_count(), rounds = rounds_of(A.ans_load, kAnsWavesCu * cus);
    if (A.ans_alone && rounds_of(A.ans_load, kAnsWavesCuSmall * cus) < rounds &&
        (rounds <= 3 || A.ans_bytes <= 32768)) {
        hipLaunchKernelGGL(k_decode_ans_small, dim3(n), dim3(64), 0, st, A);
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

// LZ77 decode (Non-Parallel) and plain copies.
#include "kernels.hpp"

namespace zf {
// One chunk per workgroup, its output in dynamic LDS.
constexpr uint32_t kLzWaves = 8;
__global__ __launch_bounds__(64 * kLzWaves) void k_decode_lz_chunk(LaunchArgs A) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lz_lds[];
    chunk_lz<kLzWaves>(A, A.chunks[A.tiles[A.kind_begin[K_LZ] + blockIdx.x].chunk], lz_lds);
}
// blk: output bytes per block (4, 8 or 16; other values select 16).
void launch_lz(const LaunchArgs &A, uint32_t waves, uint32_t blk, hipStream_t st) {
    const uint32_t n = A.kind_begin[K_LZ + 1] - A.kind_begin[K_LZ];
    if (!n) return;
    // The chunk kernel while its workgroups, two per compute unit for chunks of
    // 64 KiB, come in few enough rounds: what a round takes is a chunk's latency,
    // and the other kernel's 32 waves a compute unit make up for theirs, three
    // and a half times that, from about four and a half rounds on.  Full 64 KiB
    // chunks of text: 16 chunks 81 us (283 the other), 512 96 (352), 2,048 386
    // (442), 3,072 568 (535); chunks of 16 to 64 KiB, 128 MiB 437 (416): hence
    // the mean of the chunks and of their work in whole chunks.
    const uint32_t out_lds = lz_head<kLzWaves>() + ((A.lz_bytes + 15) & ~15u) + 32;  // at most 73.9 KiB
    const uint32_t slots = cu_count() * min(4u, 163840u / out_lds);
    if (A.lz_whole && uint64_t(n) + A.lz_load <= 9ull * slots) {
        if (out_lds > 65536)
            (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_decode_lz_chunk),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(out_lds));
        hipLaunchKernelGGL(k_decode_lz_chunk, dim3(n), dim3(64 * kLzWaves), out_lds, st, A);
        return;
    }
    blk = (blk == 4 || blk == 8) ? blk : 16;
    const dim3 grid((n + waves - 1) / waves), block(64 * waves);
    const size_t lds = size_t(waves) * 64 * blk * sizeof(uint32_t);  // at most 64 KiB
    if (blk == 4) hipLaunchKernelGGL(k_decode_lz<4>, grid, block, lds, st, A);
    else if (blk == 8) hipLaunchKernelGGL(k_decode_lz<8>, grid, block, lds, st, A);
    else hipLaunchKernelGGL(k_decode_lz<16>, grid, block, lds, st, A);
}
ZF_DEFINE_LAUNCHER(K_PLAIN, launch_plain)
}  // namespace zf

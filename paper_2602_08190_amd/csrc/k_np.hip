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
    // The chunk kernel while its workgroups, at most three per compute unit, come
    // in few enough rounds: a round takes a chunk's latency, and the other kernel's
    // 32 waves a compute unit make up for theirs, which is as long below 4.5 KiB and
    // up to four times that at 64 KiB.  Text, the other kernel and this: one chunk
    // of 4,000, 5,000, 16,000 and 65,536 bytes 14.3 and 16.8, 19.1 and 17.7, 61 and
    // 27, 279 and 75 us; 768 of 5,000 24.2 and 23.6, 1,024 of 7,000 33.5 and 41, of
    // 12,000 60 and 52; 1,536 of 16,000 93 and 75, 2,048 95 and 106; of 65,536 512 352
    // and 93, 2,048 437 and 376, 2,304 472 and 441, 3,072 522 and 568.  Hence a
    // limit of three to nine chunks per compute unit by the largest one's bytes, for
    // the mean of the chunks and of their work in whole ones (16 to 64 KiB, 128
    // MiB: 416 and 437 us).
    const uint32_t out_lds = lz_head<kLzWaves>() + ((A.lz_bytes + 15) & ~15u) + 32;  // at most 72.1 KiB
    const uint64_t per_cu = min(9u, max(3u, A.lz_bytes / 2560));
    if (A.lz_whole && A.lz_bytes > 4608 && A.lz_bytes <= kLzMaxChunk &&
        n + uint64_t(A.lz_load) <= 2 * per_cu * cu_count()) {
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

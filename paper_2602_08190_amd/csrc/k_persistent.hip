// The persistent multi-codec kernel, the small helper kernels and the host
// entry that enqueues a launch's decode.
#define ZF_UNIT_LOOP
#include "kernels.hpp"
#include "plan.hpp"

namespace zf {

// Persistent: waves pull units of [ub, ue) from eight queues, one per XCD,
// until all are empty.  Units are ordered by kind, the costliest kinds first;
// the range is dealt to the queues in blocks of kPersistBlock consecutive
// units, round robin, so every XCD works through the kinds in that order and
// neighbouring tiles of a chunk stay on one XCD (and its L2).  A workgroup
// starts on the queue of its own XCD (workgroups are dealt to the XCDs in
// turn) and moves on to the others' when it is empty.  ctr: the eight
// counters, 32 dwords apart.
constexpr uint32_t kPersistBlock = 16;
// Its register budget is the union of every kind's routine (about 140 VGPRs
// unconstrained, 2 to 3 waves per SIMD); it is held to 128 (4 waves per SIMD,
// a few spills), the fastest of 2, 4 and 6 waves per SIMD on the fact table.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_decode_persistent(
    LaunchArgs A, uint32_t ub, uint32_t ue, uint32_t *ctr) {
    __shared__ __attribute__((aligned(16))) uint32_t lz_rows[4][kAnsLdsWords > kSdBufAlloc ? kAnsLdsWords : kSdBufAlloc];
    uint32_t *mine = lz_rows[threadIdx.x / 64];
    const uint32_t n = ue - ub, nblk = (n + kPersistBlock - 1) / kPersistBlock;
    const uint32_t x0 = blockIdx.x % 8;
    for (uint32_t k = 0; k < 8; k++) {
        const uint32_t x = (x0 + k) % 8;
        // queue x holds blocks x, x + 8, x + 16, ... of the range
        const uint32_t qlen = x < nblk ? ((nblk - x + 7) / 8) * kPersistBlock : 0u;
        for (;;) {
            uint32_t i = 0;
            if (lane_id() == 0) i = atomicAdd(ctr + 32 * x, 1u);
            i = first32(i);
            if (i >= qlen) break;
            const uint32_t u = ub + ((i / kPersistBlock) * 8 + x) * kPersistBlock + i % kPersistBlock;
            if (u >= ue) continue;  // the last block's tail
            uint32_t kind = 0;
            while (kind + 1 < K_COUNT && u >= A.kind_begin[kind + 1]) kind++;
            run_unit<0>(A, kind, u, mine);
        }
    }
}

__global__ void k_zero_counters(uint32_t *c) {
    if (threadIdx.x < 16) c[32 * threadIdx.x] = 0;
}

struct OutTable {
    uint8_t *p[kMaxCols];
};
__global__ void k_set_out_tab(uint8_t **tab, OutTable t, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) tab[i] = t.p[i];
}

// A batch's transfer, read from pinned host memory over the link by a few
// workgroups, a piece each at a time, 16 KiB in flight per workgroup.  Against
// a copy command per column range, each of which costs the host and the copy
// engine about 10 us: a staged 16-column table of 500,009 rows in three batches
// 666 -> 491 us (host 960 -> 130 us), 20,011 rows in one 298 -> 140 us.  16
// workgroups carry what the link does (1 MiB 21.5 us, a copy command 27; 8 MiB
// 150 and 156; 256 MiB both 57 GB/s).  Each asks for a compute unit's whole
// LDS, to share it with no workgroup that uses LDS, as those of the kernels do
// whose waves wait for memory in step with others (FOR and plain copies use
// none): loads of one compute unit return in order, and those of a decode
// beside the copy would wait for the link's (the ANS stage 97 us alone, 150 to
// 207 us beside the copy without this; the table 582 us).
constexpr uint32_t kCopyBlocks = 16, kCopyLds = 160 * 1024;
__global__ __launch_bounds__(256) void k_copy(const CopyPiece *tab, uint32_t n) {
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const CopyPiece p = tab[i];
        const ZF_GLOBAL uint8_t *src = gp(uniform_ptr(p.src));
        ZF_GLOBAL uint8_t *dst = gp(uniform_ptr(p.dst));
        uint64_t done = 0;
        if (((reinterpret_cast<uintptr_t>(p.src) | reinterpret_cast<uintptr_t>(p.dst)) & 15u) == 0) {
            const ZF_GLOBAL u32x4 *s4 = reinterpret_cast<const ZF_GLOBAL u32x4 *>(src);
            ZF_GLOBAL u32x4 *d4 = reinterpret_cast<ZF_GLOBAL u32x4 *>(dst);
            const uint32_t nv = uint32_t(p.len / 16);
            for (uint32_t k = threadIdx.x; k < nv; k += 4 * 256) {
                u32x4 v[4];
#pragma unroll
                for (uint32_t u = 0; u < 4; u++)
                    if (k + 256 * u < nv) v[u] = __builtin_nontemporal_load(s4 + k + 256 * u);
#pragma unroll
                for (uint32_t u = 0; u < 4; u++)
                    if (k + 256 * u < nv) d4[k + 256 * u] = v[u];
            }
            done = 16ull * nv;
        }
        for (uint64_t k = done + threadIdx.x; k < p.len; k += 256) dst[k] = src[k];
    }
}

// ============================================================ host side
hipError_t launch_copy(const CopyPiece *tab, uint32_t n, hipStream_t st) {
    if (!n) return hipSuccess;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_copy), hipFuncAttributeMaxDynamicSharedMemorySize,
                              int(kCopyLds));
    hipLaunchKernelGGL(k_copy, dim3(n < kCopyBlocks ? n : kCopyBlocks), dim3(256), kCopyLds, st, tab, n);
    return hipGetLastError();
}

hipError_t launch_set_out_tab(uint8_t **d_tab, uint8_t *const *ptrs, uint32_t n, hipStream_t st) {
    OutTable t{};
    for (uint32_t i = 0; i < n && i < kScratchCol; i++) t.p[i] = ptrs[i];
    hipLaunchKernelGGL(k_set_out_tab, dim3(1), dim3(kMaxCols), 0, st, d_tab, t, kMaxCols);
    return hipGetLastError();
}

bool decode_forks(const LaunchArgs &A) {
    auto count = [&](uint32_t k) { return A.kind_begin[k + 1] - A.kind_begin[k]; };
    const uint32_t chain = count(K_LZ) + count(K_ANS), rest = A.kind_begin[K_COUNT] - chain - count(K_SDICT);
    return chain && rest && A.ans_load <= 8 * cu_count() && A.lz_load <= 2 * cu_count();
}

// Enqueue the decode of one launch's units.  persistent_waves > 0 selects
// the persistent kernel with that many waves in flight.  With `ev`, an event
// is recorded on `st` before and after each kind's launch (slot K_COUNT: the
// persistent kernel), and ev->used says which were recorded.  With `side`, the
// kinds that depend on none of LZ77, ANS and String-dictionary may be launched
// on its stream beside those: a chain of whole-chunk units that leaves most of
// the GPU idle takes about 100 us whatever else there is.  (With more such
// units the kinds compete instead.)  16 columns, one of them text, 1,500,007
// rows: 226 us one after the other, 202 us beside; 20,011 rows: 123 and 118 us.
hipError_t launch_decode(const LaunchArgs &A, uint32_t persistent_waves, const uint32_t *wpb,
                         uint32_t lz_blk, hipStream_t st, KindEvents *ev, const SideStream *side) {
    if (ev)
        for (uint32_t k = 0; k <= K_COUNT; k++) ev->used[k] = false;
    if (A.kind_begin[K_COUNT] == 0) return hipSuccess;
    auto mark = [&](uint32_t k, bool end) -> hipError_t {
        if (!ev) return hipSuccess;
        if (!end) ev->used[k] = true;
        return hipEventRecord(end ? ev->e1[k] : ev->e0[k], st);
    };
    hipError_t e = hipSuccess;
    if (persistent_waves) {
        // two-stage chunks: the kinds up to RLE (LZ77, ANS, RLE) write the
        // scratch area that String-dictionary and TREE units read, so they
        // get a launch of their own first; otherwise one launch takes all
        if ((e = mark(K_COUNT, false)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_zero_counters, dim3(1), dim3(64), 0, st, A.counter);
        const uint32_t blocks = (persistent_waves + 3) / 4, all = A.kind_begin[K_COUNT];
        const uint32_t cut = A.two_stage ? A.kind_begin[K_SDICT] : all;
        if (cut > 0)
            hipLaunchKernelGGL(k_decode_persistent, dim3(blocks), dim3(256), 0, st, A, 0u, cut, A.counter);
        if (all > cut)
            hipLaunchKernelGGL(k_decode_persistent, dim3(blocks), dim3(256), 0, st, A, cut, all,
                               A.counter + 8 * 32);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        return mark(K_COUNT, true);
    }
    // launch order: the slow serial kinds first
    // (TREE after the RLE kinds, which write its chunks' run starts; SDICT
    // after ANS, which writes its chunks' entry indices)
    static const uint32_t order[K_COUNT] = {K_LZ,     K_ANS,    K_SDICT,  K_RLE32,  K_RLE64, K_TREE, K_DICT128,
                                            K_DICT64, K_DICT32, K_FOR64, K_FOR32, K_F2I,   K_PLAIN};
    const hipStream_t main = st;
    const bool fork = side && side->stream && !ev && decode_forks(A);
    if (fork) {
        if ((e = hipEventRecord(side->fork, main)) != hipSuccess) return e;
        if ((e = hipStreamWaitEvent(side->stream, side->fork, 0)) != hipSuccess) return e;
    }
    for (uint32_t i = 0; i < K_COUNT; i++) {
        const uint32_t k = order[i];
        if (A.kind_begin[k + 1] == A.kind_begin[k]) continue;
        st = fork && k != K_LZ && k != K_ANS && k != K_SDICT ? side->stream : main;
        if ((e = mark(k, false)) != hipSuccess) return e;
        switch (k) {
        case K_LZ: launch_lz(A, wpb[K_LZ], lz_blk, st); break;
        case K_ANS: launch_ans(A, wpb[K_ANS], st); break;
        case K_RLE32: launch_rle32(A, wpb[K_RLE32], st); break;
        case K_RLE64: launch_rle64(A, wpb[K_RLE64], st); break;
        case K_TREE: launch_tree(A, wpb[K_TREE], st); break;
        case K_SDICT: launch_sdict(A, wpb[K_SDICT], st); break;
        case K_DICT128: launch_dict128(A, wpb[K_DICT128], st); break;
        case K_DICT64: launch_dict64(A, wpb[K_DICT64], st); break;
        case K_DICT32: launch_dict32(A, wpb[K_DICT32], st); break;
        case K_FOR64: launch_for64(A, wpb[K_FOR64], st); break;
        case K_FOR32: launch_for32(A, wpb[K_FOR32], st); break;
        case K_F2I: launch_f2i(A, wpb[K_F2I], st); break;
        case K_PLAIN: launch_plain(A, wpb[K_PLAIN], st); break;
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = mark(k, true)) != hipSuccess) return e;
    }
    if (fork) {
        if ((e = hipEventRecord(side->join, side->stream)) != hipSuccess) return e;
        if ((e = hipStreamWaitEvent(main, side->join, 0)) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace zf

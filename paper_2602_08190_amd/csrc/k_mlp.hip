// Cost-model network on the GPU: forward, backward and Adam, in FP32.
//
//   h1 = relu(W1 x + b1)   (64 x 32)      x: 32 chunk statistics
//   h2 = relu(W2 h1 + b2)  (64 x 64)
//   y  = W3 h2 + b3        (24 x 64)      y: predicted log time per (codec, schedule)
//
// Loss over n samples: (1/n) sum_i (y_i[k_i] - t_i)^2, only the measured
// output k_i of each sample counts.  Every product but the one-hot last
// layer's gradient is a 16 x 16 x 4 FP32 matrix instruction (operands and
// sums in FP32).  The per-workgroup partial gradients are summed over
// workgroups in a fixed order, so a training run is bit-reproducible.
#include <hip/hip_runtime.h>

#include <cstdint>

#include <mutex>
#include <string>

#include "zf.h"

namespace zf {
void set_last_error(const std::string &m);

static zf_status fail_with(zf_status st, const char *msg) {
    set_last_error(msg);
    return st;
}
static zf_status launched() {
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return ZF_OK;
    set_last_error(std::string("kernel launch failed: ") + hipGetErrorString(e));
    return ZF_E_HIP;
}

constexpr int NI = 32, NH = 64, NO = 24, TS = 64;  // inputs, hidden, outputs, samples per block
constexpr int OW1 = 0, OB1 = OW1 + NH * NI, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NO * NH, NP = OB3 + NO;
static_assert(NP == 7832, "parameter count");

typedef float f32x4 __attribute__((ext_vector_type(4)));

// v_mfma_f32_16x16x4_f32: lane l gives A[l % 16][k] and B[k][l % 16] for
// k = l / 16 and holds D[4 (l / 16) + r][l % 16] in register r.
__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Four floats at p (4-byte aligned).
__device__ __forceinline__ f32x4 ld4(const float *p) {
    f32x4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
// acc += sum over t of a[t] b[t]: four k steps of a 16 x 16 tile, where lane
// group g holds k = 4 g + t of the 16 (any order of k serves, as long as a
// and b agree).  Two chains: half the rounding steps one after another.
__device__ __forceinline__ void mfma4(f32x4 a, f32x4 b, f32x4 (&acc)[2]) {
    acc[0] = mfma(a[0], b[0], acc[0]);
    acc[1] = mfma(a[1], b[1], acc[1]);
    acc[0] = mfma(a[2], b[2], acc[0]);
    acc[1] = mfma(a[3], b[3], acc[1]);
}
__device__ __forceinline__ float relu(float a) { return a > 0.f ? a : 0.f; }

// Scores of 16 samples per workgroup, wave w computing neurons [16 w, 16 w +
// 16) of each layer: the weights are read straight from memory, 16 rows of 64
// bytes per load, all of them asked for before the first product; only the
// activations cross the waves, through LDS.  The call is bound by its launch
// and two memory round trips: 2,048 samples 176 us when one workgroup held 64
// samples and every product read two LDS operands with all lanes of a weight
// read in one bank, 4.2 us so.
constexpr int FS = 16;
__global__ __launch_bounds__(256) void k_mlp_forward(const float *P, const float *X, uint32_t n, float *Y) {
    __shared__ __attribute__((aligned(16))) float h1[FS][68], h2[FS][68];
    const uint32_t s0 = blockIdx.x * FS, lane = threadIdx.x % 64, w = threadIdx.x / 64;
    const uint32_t r = lane % 16, g = lane / 16, j = 16 * w + r;
    const bool out = w < 2 && j < uint32_t(NO);  // this lane's neuron of the last layer
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 x[2], w1[2], w2[4], w3[4];
#pragma unroll
    for (uint32_t q = 0; q < 2; q++) {
        x[q] = s0 + r < n ? ld4(X + uint64_t(s0 + r) * NI + 16 * q + 4 * g) : zero;
        w1[q] = ld4(P + OW1 + j * NI + 16 * q + 4 * g);
    }
#pragma unroll
    for (uint32_t q = 0; q < 4; q++) {
        w2[q] = ld4(P + OW2 + j * NH + 16 * q + 4 * g);
        w3[q] = out ? ld4(P + OW3 + j * NH + 16 * q + 4 * g) : zero;
    }
    const float b1 = P[OB1 + j], b2 = P[OB2 + j], b3 = out ? P[OB3 + j] : 0.f;
    f32x4 acc[2] = {zero, zero};
#pragma unroll
    for (uint32_t q = 0; q < 2; q++) mfma4(x[q], w1[q], acc);
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) h1[4 * g + i][j] = relu((acc[0][i] + acc[1][i]) + b1);
    __syncthreads();
    acc[0] = acc[1] = zero;
#pragma unroll
    for (uint32_t q = 0; q < 4; q++) mfma4(*reinterpret_cast<const f32x4 *>(&h1[r][16 * q + 4 * g]), w2[q], acc);
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) h2[4 * g + i][j] = relu((acc[0][i] + acc[1][i]) + b2);
    __syncthreads();
    if (w >= 2) return;
    acc[0] = acc[1] = zero;
#pragma unroll
    for (uint32_t q = 0; q < 4; q++) mfma4(*reinterpret_cast<const f32x4 *>(&h2[r][16 * q + 4 * g]), w3[q], acc);
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) {
        const uint32_t s = s0 + 4 * g + i;
        if (out && s < n) Y[uint64_t(s) * NO + j] = (acc[0][i] + acc[1][i]) + b3;
    }
}

// Row strides: 80 (and 48) floats put the four rows a matrix operand takes
// down a column in four different quarters of the banks; rows read along
// their length stay 16-byte aligned.
struct MlpShared {
    float w1[NH][36];
    float w2[NH][80];
    float w3[NO][68];
    float x[TS][48];
    float h1[TS][80];
    float h2[TS][80];
    float d2[TS][80];   // dL/dz2 (masked by relu')
    float d1[TS][80];   // dL/dz1
    float red[2][8][NH];
    float b1[NH], b2[NH];
    float dy[TS];       // dL/dy[k] per sample
    int k[TS];          // -1: out of range, or past the batch
};

// Partial gradient of the block's 64 samples -> work[block][NP + 1] (last =
// loss).  Eight waves, two per SIMD, share the block's matrix products (128
// matrix instructions a wave, 3.4 us of the matrix units); one workgroup per
// 64 samples because that is the partial the workspace holds.  2,048 samples:
// 180 us with one neuron per thread and every operand from LDS,
// 10.7 us so.
constexpr int GT = 512;
__global__ __launch_bounds__(GT) void k_mlp_grad(const float *P, const float *X, const int32_t *K,
                                                 const float *T, uint32_t n, float *work) {
    __shared__ __attribute__((aligned(16))) MlpShared S;
    const uint32_t s0 = blockIdx.x * TS;
    const uint32_t t = threadIdx.x, lane = t % 64, w = t / 64, r = lane % 16, g = lane / 16;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (uint32_t i = 4 * t; i < uint32_t(NH * NI); i += 4 * GT)
        *reinterpret_cast<f32x4 *>(&S.w1[i / NI][i % NI]) = ld4(P + OW1 + i);
    for (uint32_t i = 4 * t; i < uint32_t(NH * NH); i += 4 * GT)
        *reinterpret_cast<f32x4 *>(&S.w2[i / NH][i % NH]) = ld4(P + OW2 + i);
    for (uint32_t i = 4 * t; i < uint32_t(NO * NH); i += 4 * GT)
        *reinterpret_cast<f32x4 *>(&S.w3[i / NH][i % NH]) = ld4(P + OW3 + i);
    for (uint32_t i = 4 * t; i < uint32_t(TS * NI); i += 4 * GT) {
        const uint32_t s = s0 + i / NI;
        *reinterpret_cast<f32x4 *>(&S.x[i / NI][i % NI]) = s < n ? ld4(X + uint64_t(s) * NI + i % NI) : zero;
    }
    if (t < NH) {
        S.b1[t] = P[OB1 + t];
        S.b2[t] = P[OB2 + t];
    }
    __syncthreads();
    // 64 x 64 results: 16 tiles, wave w takes columns [16 (w % 4), ...) of
    // rows [16 (w / 4), ...) and [32 + 16 (w / 4), ...)
    const uint32_t c0 = 16 * (w % 4), c = c0 + r;
#pragma unroll
    for (uint32_t h = 0; h < 2; h++) {
        const uint32_t r0 = 32 * h + 16 * (w / 4);
        f32x4 acc[2] = {zero, zero};
#pragma unroll
        for (uint32_t q = 0; q < NI; q += 16)
            mfma4(*reinterpret_cast<const f32x4 *>(&S.x[r0 + r][q + 4 * g]),
                  *reinterpret_cast<const f32x4 *>(&S.w1[c][q + 4 * g]), acc);
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) S.h1[r0 + 4 * g + i][c] = relu((acc[0][i] + acc[1][i]) + S.b1[c]);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t h = 0; h < 2; h++) {
        const uint32_t r0 = 32 * h + 16 * (w / 4);
        f32x4 acc[2] = {zero, zero};
#pragma unroll
        for (uint32_t q = 0; q < NH; q += 16)
            mfma4(*reinterpret_cast<const f32x4 *>(&S.h1[r0 + r][q + 4 * g]),
                  *reinterpret_cast<const f32x4 *>(&S.w2[c][q + 4 * g]), acc);
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) S.h2[r0 + 4 * g + i][c] = relu((acc[0][i] + acc[1][i]) + S.b2[c]);
    }
    __syncthreads();
    // eight threads per sample: y[k], the error, and dz2[j] = dy W3[k][j]
    // relu'(z2) for their eight neurons j
    const float inv_n = 1.f / float(n);
    float l = 0.f;  // this thread's share of the loss (one thread per sample)
    {
        const uint32_t s = t / 8, p = 8 * (t % 8);
        int k = s0 + s < n ? K[s0 + s] : -1;
        const bool ok = k >= 0 && k < NO;
        f32x4 h[2], v[2];
#pragma unroll
        for (uint32_t q = 0; q < 2; q++) {
            h[q] = *reinterpret_cast<const f32x4 *>(&S.h2[s][p + 4 * q]);
            v[q] = ok ? *reinterpret_cast<const f32x4 *>(&S.w3[k][p + 4 * q]) : zero;
        }
        float y = 0.f;
#pragma unroll
        for (uint32_t q = 0; q < 8; q++) y = fmaf(v[q / 4][q % 4], h[q / 4][q % 4], y);
        y += __shfl_xor(y, 1, 64);
        y += __shfl_xor(y, 2, 64);
        y += __shfl_xor(y, 4, 64);
        float e = 0.f;
        if (s0 + s < n) e = ok ? (y + P[OB3 + k]) - T[s0 + s] : __builtin_nanf("");
        const float dy = 2.f * e * inv_n;
#pragma unroll
        for (uint32_t q = 0; q < 2; q++) {
            f32x4 d;
#pragma unroll
            for (uint32_t i = 0; i < 4; i++) d[i] = ok && h[q][i] > 0.f ? dy * v[q][i] : 0.f;
            *reinterpret_cast<f32x4 *>(&S.d2[s][p + 4 * q]) = d;
        }
        if (p == 0) {
            S.dy[s] = dy;
            S.k[s] = ok ? k : -1;
            l = (e * inv_n) * e;
        }
    }
    // loss: over the wave's eight samples here, over the waves at the end
    l += __shfl_xor(l, 8, 64);
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    __syncthreads();
    float *G = work + uint64_t(blockIdx.x) * (NP + 1);
    {
        // layer 3: dW3[o][j] = sum_s [k_s == o] dy_s h2[s][j]; db3[o] = sum_s
        // [k_s == o] dy_s.  Wave w takes outputs w, w + 8, w + 16, lane j
        // neuron j, over the samples of those outputs only.
        float a[3] = {0.f, 0.f, 0.f}, b[3] = {0.f, 0.f, 0.f};
        const int ks = S.k[lane];
        const float dys = S.dy[lane];
        for (uint64_t m = __ballot(ks >= 0 && uint32_t(ks) % 8 == w); m; m &= m - 1) {
            const int s = __builtin_ctzll(m);
            const int o = __builtin_amdgcn_readlane(ks, s) >> 3;
            const float d = __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(__float_as_uint(dys)), s)));
            const float v = S.h2[s][lane];
#pragma unroll
            for (int q = 0; q < 3; q++)
                if (o == q) {
                    a[q] = fmaf(d, v, a[q]);
                    b[q] += d;
                }
        }
#pragma unroll
        for (uint32_t q = 0; q < 3; q++) {
            G[OW3 + (w + 8 * q) * NH + lane] = a[q];
            if (lane == 0) G[OB3 + w + 8 * q] = b[q];
        }
    }
    // layer 2: dW2[j][i] = sum_s dz2[s][j] h1[s][i], and dz1[s][i] = (sum_j
    // dz2[s][j] W2[j][i]) relu'(z1)
#pragma unroll
    for (uint32_t h = 0; h < 2; h++) {
        const uint32_t r0 = 32 * h + 16 * (w / 4);
        f32x4 acc[2] = {zero, zero};
#pragma unroll
        for (uint32_t s = 0; s < TS; s += 4)
            acc[(s / 4) % 2] = mfma(S.d2[s + g][r0 + r], S.h1[s + g][c], acc[(s / 4) % 2]);
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) G[OW2 + (r0 + 4 * g + i) * NH + c] = acc[0][i] + acc[1][i];
        acc[0] = acc[1] = zero;
#pragma unroll
        for (uint32_t q = 0; q < NH; q += 16) {
            const uint32_t j = q + 4 * g;
            const f32x4 b = {S.w2[j][c], S.w2[j + 1][c], S.w2[j + 2][c], S.w2[j + 3][c]};
            mfma4(*reinterpret_cast<const f32x4 *>(&S.d2[r0 + r][j]), b, acc);
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; i++)
            S.d1[r0 + 4 * g + i][c] = S.h1[r0 + 4 * g + i][c] > 0.f ? acc[0][i] + acc[1][i] : 0.f;
    }
    {
        float a = 0.f;
#pragma unroll
        for (uint32_t s = 0; s < 8; s++) a += S.d2[8 * w + s][lane];
        S.red[0][w][lane] = a;
    }
    __syncthreads();
    {
        // layer 1: dW1[i][q] = sum_s dz1[s][i] x[s][q], one tile a wave
        const uint32_t r0 = 16 * (w / 2), q = 16 * (w % 2) + r;
        f32x4 acc[2] = {zero, zero};
#pragma unroll
        for (uint32_t s = 0; s < TS; s += 4)
            acc[(s / 4) % 2] = mfma(S.d1[s + g][r0 + r], S.x[s + g][q], acc[(s / 4) % 2]);
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) G[OW1 + (r0 + 4 * g + i) * NI + q] = acc[0][i] + acc[1][i];
        float a = 0.f;
#pragma unroll
        for (uint32_t s = 0; s < 8; s++) a += S.d1[8 * w + s][lane];
        S.red[1][w][lane] = a;
        if (lane == 0) S.b1[w] = l;  // (the biases are no longer read)
    }
    __syncthreads();
    if (w < 2) {  // db2, db1
        float a = 0.f;
#pragma unroll
        for (uint32_t q = 0; q < 8; q++) a += S.red[w][q][lane];
        G[(w ? OB1 : OB2) + lane] = a;
    } else if (t == 2 * 64) {
        float a = 0.f;
#pragma unroll
        for (uint32_t q = 0; q < 8; q++) a += S.b1[q];
        G[NP] = a;
    }
}

// grad[p] = sum over blocks of the partials: RG running sums per parameter
// (block b in sum b % RG), then those in order.  Eight times as many loads in
// flight as one sum per parameter (32 partials: 8.7 -> 2.4 us).
constexpr uint32_t RG = 8, RP = 32;
__global__ __launch_bounds__(RG * RP) void k_mlp_reduce(const float *work, uint32_t nblocks, float *grad,
                                                        float *loss) {
    __shared__ float sum[RG][RP];
    const uint32_t q = threadIdx.x % RP, g = threadIdx.x / RP, p = blockIdx.x * RP + q;
    float a = 0.f;
    if (p <= uint32_t(NP)) {
#pragma unroll 4
        for (uint32_t b = g; b < nblocks; b += RG) a += work[uint64_t(b) * (NP + 1) + p];
    }
    sum[g][q] = a;
    __syncthreads();
    if (g != 0 || p > uint32_t(NP)) return;
#pragma unroll
    for (uint32_t i = 1; i < RG; i++) a += sum[i][q];
    if (p < uint32_t(NP)) grad[p] = a;
    else *loss = a;
}

__global__ void k_mlp_adam(float *P, const float *G, float *M, float *V, float lr, float b1, float b2,
                           float eps, float c1, float c2) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= uint32_t(NP)) return;
    const float g = G[p];
    const float m = b1 * M[p] + (1.f - b1) * g;
    const float v = b2 * V[p] + (1.f - b2) * g * g;
    M[p] = m;
    V[p] = v;
    P[p] -= lr * (m * c1) / (sqrtf(v * c2) + eps);
}

// Allocation-free gradient (zf_mlp_grad_noalloc): the per-workgroup partials
// live in this file-scope device array instead of a caller workspace.  Every
// partial a launch reads is written by the same launch first, so nothing has
// to be cleared between calls.  In host code `scratch` only names the symbol;
// its device address comes from hipGetSymbolAddress, once per device.
constexpr uint32_t kStaticBlocks = (ZF_MLP_STATIC_MAX_N + TS - 1) / TS;
static __device__ __align__(256) float scratch[uint64_t(kStaticBlocks) * (NP + 1)];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static float *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first
// call per device).
static zf_status static_scratch(float **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_with(ZF_E_HIP, "hipGetDevice failed");
    if (dev < 0 || dev >= kMaxDevices) return fail_with(ZF_E_UNSUPPORTED, "device index above 63");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_last_error(std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
            return ZF_E_HIP;
        }
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return ZF_OK;
}

}  // namespace zf

using namespace zf;

extern "C" {

zf_status zf_mlp_forward(const float *d_params, const float *d_x, uint32_t n, float *d_y,
                         zf_stream_t stream) {
    if (!n) return ZF_OK;
    if (!d_params || !d_x || !d_y) return fail_with(ZF_E_INVALID, "null pointer");
    hipLaunchKernelGGL(k_mlp_forward, dim3(uint32_t((uint64_t(n) + FS - 1) / FS)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), d_params, d_x, n, d_y);
    return launched();
}

uint64_t zf_mlp_grad_work_bytes(uint32_t n) {
    return uint64_t((n + TS - 1) / TS) * (NP + 1) * sizeof(float);
}

zf_status zf_mlp_grad(const float *d_params, const float *d_x, const int32_t *d_k, const float *d_t,
                      uint32_t n, float *d_grad, float *d_loss, void *d_work, uint64_t work_bytes,
                      zf_stream_t stream) {
    if (!n || !d_params || !d_x || !d_k || !d_t || !d_grad || !d_loss || !d_work)
        return fail_with(ZF_E_INVALID, "null pointer or empty batch");
    if (work_bytes < zf_mlp_grad_work_bytes(n)) return fail_with(ZF_E_TOO_SMALL, "workspace too small");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t nb = (n + TS - 1) / TS;
    float *work = static_cast<float *>(d_work);
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(GT), 0, st, d_params, d_x, d_k, d_t, n, work);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NP + RP) / RP), dim3(RG * RP), 0, st, work, nb, d_grad,
                       d_loss);
    return launched();
}

zf_status zf_mlp_grad_noalloc(const float *d_params, const float *d_x, const int32_t *d_k,
                              const float *d_t, uint32_t n, float *d_grad, float *d_loss,
                              zf_stream_t stream) {
    if (!n || !d_params || !d_x || !d_k || !d_t || !d_grad || !d_loss)
        return fail_with(ZF_E_INVALID, "null pointer or empty batch");
    if (n > ZF_MLP_STATIC_MAX_N) {
        set_last_error("zf_mlp_grad_noalloc: " + std::to_string(n) + " samples exceed the static scratch "
                       "limit of " + std::to_string(ZF_MLP_STATIC_MAX_N) + " (use zf_mlp_grad with a workspace)");
        return ZF_E_UNSUPPORTED;
    }
    float *work = nullptr;
    const zf_status st0 = static_scratch(&work);
    if (st0 != ZF_OK) return st0;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t nb = (n + TS - 1) / TS;
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(GT), 0, st, d_params, d_x, d_k, d_t, n, work);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NP + RP) / RP), dim3(RG * RP), 0, st, work, nb, d_grad,
                       d_loss);
    return launched();
}

zf_status zf_mlp_adam(float *d_params, const float *d_grad, float *d_m, float *d_v, uint32_t step,
                      float lr, float beta1, float beta2, float eps, zf_stream_t stream) {
    if (!d_params || !d_grad || !d_m || !d_v || step == 0)
        return fail_with(ZF_E_INVALID, "null pointer or step 0");
    const double c1 = 1.0 / (1.0 - __builtin_pow(double(beta1), double(step)));
    const double c2 = 1.0 / (1.0 - __builtin_pow(double(beta2), double(step)));
    hipLaunchKernelGGL(k_mlp_adam, dim3((NP + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), d_params, d_grad, d_m, d_v, lr, beta1, beta2,
                       eps, float(c1), float(c2));
    return launched();
}

}  // extern "C"

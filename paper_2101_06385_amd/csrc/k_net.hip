// Kernels of the differentiable generalized-SP2 network (Eq. general SP2 as matrix layers)
//
//     X_{k+1} = W_k X_k^2 + B_k X_k + c_k I,   k = 0 .. K-1
//
// The forward layers reuse the squaring kernels (alpha, beta, gamma) = (W_k, B_k, c_k).
// This file holds what the network adds:
//   k_pack_coef   : (W, B, c) device arrays -> per-layer coefficient triples
//   k_copy_pad    : n x n (leading dimension ld) <-> zero-padded n_p x n_p
// The reverse layers are in k_adjoint.hip.
#include "sp2_internal.h"

namespace sp2 {
namespace {

constexpr int kThreads = 256;

__global__ void k_pack_coef(const float* __restrict__ w, const float* __restrict__ b, const float* __restrict__ c,
                            int K, float* __restrict__ out) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x) {
        out[3 * k + 0] = w[k];
        out[3 * k + 1] = b[k];
        out[3 * k + 2] = c[k];
    }
}

// to_pad = 1: dst (np x np, zero padding) <- src (n x n, ld);  0: dst (n x n, ld) <- src (np x np)
__global__ void k_copy_pad(const float* __restrict__ src, float* __restrict__ dst, int n, int ld, int np,
                           int to_pad) {
    const size_t total = to_pad ? (size_t)np * np : (size_t)n * n;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        if (to_pad) {
            const int i = (int)(idx / np), j = (int)(idx % np);
            dst[idx] = (i < n && j < n) ? src[(size_t)i * ld + j] : 0.f;
        } else {
            const int i = (int)(idx / n), j = (int)(idx % n);
            dst[(size_t)i * ld + j] = src[(size_t)i * np + j];
        }
    }
}

// dst (np x np, zero padding) <- (src + src^T)/2 for the n x n matrix src (leading dimension
// ld): the part of a loss gradient that acts on a symmetric layer output.  One 32 x 32 output
// tile per block; the mirrored input tile goes through LDS so that both reads are row
// segments.  a + b == b + a in IEEE arithmetic, so the result is exactly symmetric.
constexpr int kSymT = 32;
__global__ __launch_bounds__(kThreads) void k_sym_pad(const float* __restrict__ src, float* __restrict__ dst,
                                                      int n, int ld, int np) {
    __shared__ float tr[kSymT][kSymT + 1];
    const int bi = blockIdx.y * kSymT, bj = blockIdx.x * kSymT;
    const int c = threadIdx.x % kSymT, r0 = threadIdx.x / kSymT;   // 8 rows per pass
    for (int r = r0; r < kSymT; r += kThreads / kSymT) {
        const int i = bj + r, j = bi + c;   // mirrored tile: rows of bj, columns of bi
        tr[r][c] = (i < n && j < n) ? src[(size_t)i * ld + j] : 0.f;
    }
    __syncthreads();
    for (int r = r0; r < kSymT; r += kThreads / kSymT) {
        const int i = bi + r, j = bj + c;
        const float a = (i < n && j < n) ? src[(size_t)i * ld + j] : 0.f;
        dst[(size_t)i * np + j] = 0.5f * (a + tr[c][r]);
    }
}

inline int grid_for(size_t total) {
    size_t g = (total + kThreads - 1) / kThreads;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (int)g;
}

}  // namespace

hipError_t launch_pack_coef(const float* w, const float* b, const float* c, int K, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_coef, dim3(1), dim3(kThreads), 0, s, w, b, c, K, out);
    return hipGetLastError();
}

hipError_t launch_copy_pad(const float* src, float* dst, int n, int ld, int np, int to_pad, hipStream_t s) {
    const size_t total = to_pad ? (size_t)np * np : (size_t)n * n;
    hipLaunchKernelGGL(k_copy_pad, dim3(grid_for(total)), dim3(kThreads), 0, s, src, dst, n, ld, np, to_pad);
    return hipGetLastError();
}

hipError_t launch_sym_pad(const float* src, float* dst, int n, int ld, int np, hipStream_t s) {
    if (np % kSymT) return hipErrorInvalidValue;
    const dim3 grid(np / kSymT, np / kSymT);
    hipLaunchKernelGGL(k_sym_pad, grid, dim3(kThreads), 0, s, src, dst, n, ld, np);
    return hipGetLastError();
}

}  // namespace sp2

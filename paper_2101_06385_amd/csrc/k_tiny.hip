// The whole solve of a problem with n <= 64 in one workgroup (gfx950): spectral bounds, input
// layer, every layer of Alg. 1, the FP64 refinement and the final checks in one launch.
//
// At this size a layer is 12 products per wave; as a launch of its own it takes 6.9 us of memory
// trips and the launch itself (n = 10, 20 layers and 10 other launches: 325 us per call).  Here
// the planes and the FP64 matrices live in LDS, S in the accumulator layout in registers, and
// each layer costs two barriers.  4 waves, wave (bi, bj) on the 32 x 32 block (bi, bj) of the
// upper triangle (wave (1, 0) only keeps step), the layers bounded by the latency of their
// chain: products, epilogue, wave sums, control.  The chains of products and sums per element
// are those of the 64-tile and FP64 kernels, so D is bit-identical to theirs; every thread runs
// the control on the same sums.
#include "sp2_control.h"
#include "sp2_internal.h"

#include <type_traits>

namespace sp2 {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kN = kTinyMax;
constexpr int kThreads = 256;
constexpr int kPitch = kN + 2;   // doubles per row of an FP64 matrix in LDS: 16-byte aligned, odd in 16 bytes

template <typename T16>
struct TinyOps;
template <>
struct TinyOps<_Float16> {
    typedef _Float16 vec8 __attribute__((ext_vector_type(8)));
    __device__ static inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
template <>
struct TinyOps<__bf16> {
    typedef __bf16 vec8 __attribute__((ext_vector_type(8)));
    __device__ static inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

struct TinyLds {
    double x[2][kN * kPitch];          // FP64 matrices (the input layer's H, S and Y of the FP64 layers)
    unsigned char planes[2][2][4][1024];   // [plane][32-row block][16-wide unit of K], lane order of the MFMA
    double red[3][kThreads];
    double sums[4][2];
    StateHot hot;
};

// Sum over the 256 threads in the order of a halving tree (as the input layer's partial sums),
// in every thread.
__device__ __forceinline__ double block_sum(double v, double* sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    if (t < 64) {
        const double r = wave_sum0((sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]));
        if (t == 0) sh[0] = r;   // wave 0 alone read sh, in order
    }
    __syncthreads();
    const double r = sh[0];
    __syncthreads();
    return r;
}
__device__ __forceinline__ double block_max(double v, double* sh) {
    const int t = threadIdx.x;
#pragma unroll 1
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    const double r = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    __syncthreads();
    return r;
}

// One FP64 layer Y = alpha X^2 + beta X + gamma I on LDS matrices, upper triangle and mirror;
// returns this wave's sums of Tr Y and ||Y||_F^2 in lane 0 (unless tr_out is null).  `out` takes Y too (n x n, ldo).
__device__ __forceinline__ void layer64(const double* __restrict__ x, double* __restrict__ y, int n, double alpha,
                                        double beta, double gamma, double* __restrict__ out, int ldo, double* tr_out,
                                        double* fr_out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
    double ts = 0.0, fs = 0.0;   // summed per 16 x 16 block, blocks in row-major order, as a 32-tile's
    if (wm <= wn) {
        f64x4 acc[2][2];
        for (int m = 0; m < 2; ++m)
            for (int q = 0; q < 2; ++q) acc[m][q] = f64x4{0.0, 0.0, 0.0, 0.0};
        const int r16 = lane & 15, j2 = 2 * (lane >> 4);
        for (int st = 0; st < (n + 15) / 16; ++st) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {   // K 16 st + 8 h + 2 (lane / 16) + s, as in k_square_f64
                f64x2 fa[2], fb[2];
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    fa[m] = *(const f64x2*)(x + (wm * 32 + m * 16 + r16) * kPitch + 16 * st + 8 * h + j2);
                    fb[m] = *(const f64x2*)(x + (wn * 32 + m * 16 + r16) * kPitch + 16 * st + 8 * h + j2);
                }
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            acc[m][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[m][s], fb[q][s], acc[m][q], 0, 0, 0);
            }
        }
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int col = wn * 32 + q * 16 + (lane & 15);
                double tr = 0.0, fr = 0.0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = wm * 32 + m * 16 + 4 * r + (lane >> 4);
                    if (row > col) continue;
                    const double xv = acc[m][q][r];
                    double v = (beta != 0.0) ? fma(alpha, xv, beta * x[row * kPitch + col]) : alpha * xv;
                    if (row == col && col < n) v += gamma;
                    y[row * kPitch + col] = v;
                    y[col * kPitch + row] = v;
                    if (out && col < n) {
                        out[(size_t)row * ldo + col] = v;
                        out[(size_t)col * ldo + row] = v;
                    }
                    if (row == col) {
                        tr += v;
                        fr += v * v;
                    } else {
                        fr += 2.0 * v * v;
                    }
                }
                if (tr_out) {
                    ts += wave_sum0(tr);
                    fs += wave_sum0(fr);
                }
            }
    }
    if (tr_out) {
        *tr_out = ts;
        *fr_out = fs;
    }
}

// kSplit: T16 planes with FP32 S; otherwise FP64 S.  kTimed: the same solve, which also records its
// phases in `ticks` by the wall clock of the device (one kernel that asks for `ticks` at each phase takes
// 1 us longer at n = 10: 85.0 against 83.9 us per call).
template <typename T16, bool kSplit, bool kTimed>
__global__ __launch_bounds__(kThreads) void k_tiny(const double* __restrict__ h, int ldh, double* __restrict__ d,
                                                   int ldd, DevState* st, StateParams p, float in_scale,
                                                   float out_scale, int refine, DevState* __restrict__ host_state,
                                                   TinyTicks* __restrict__ ticks) {
    typedef typename TinyOps<T16>::vec8 vec8;
    __shared__ __attribute__((aligned(16))) TinyLds L;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int n = p.n;
    if (kTimed && t == 0) ticks->start = wall_clock64();
    init_state(st, p);
    StateHot hot;
    init_hot(&hot, p);

    // H, zero padded
    double* hx = L.x[0];
#pragma unroll 4
    for (int i = t; i < kN * kN; i += kThreads) {
        const int r = i / kN, c = i % kN;
        hx[r * kPitch + c] = (r < n && c < n) ? h[(size_t)r * ldh + c] : 0.0;
    }
    __syncthreads();
    // ------------------------------------------------------------- spectral bounds
    if (!p.have_bounds) {
        double lo = INFINITY, hi = -INFINITY, bad = 0.0;
#pragma unroll 1
        for (int row = wave; row < n; row += 4) {
            double s = lane < n ? fabs(hx[row * kPitch + lane]) : 0.0;
            s = wave_sum(s);
            const double dd = hx[row * kPitch + row];
            const double slack = (2.0 * n + 4.0) * 2.220446049250313e-16;
            const double r = (s - fabs(dd)) * (1.0 + slack) + slack * fabs(dd);
            lo = fmin(lo, dd - r);
            hi = fmax(hi, dd + r);
            if (!isfinite(s) || !isfinite(dd)) bad = 1.0;
        }
        lo = -block_max(-lo, L.red[0]);
        hi = block_max(hi, L.red[0]);
        bad = block_max(bad, L.red[0]);
        if (bad != 0.0 || !isfinite(lo) || !isfinite(hi)) {
            hot.status = SP2_ENONFINITE;
            lo = 0.0;
            hi = 1.0;
        }
        hot.emin = lo;
        hot.emax = hi;
    }
    // ------------------------------------------------------------- input layer
    double span = hot.emax - hot.emin;
    if (!(span > 0.0)) span = 1.0;   // degenerate spectrum: every eigenvalue maps to ~1
    const double w0 = -1.0 / span, b0 = hot.emax / span;
    double* s0 = L.x[1];
    double tr = 0.0, fr = 0.0, as = 0.0;
#pragma unroll 2
    for (int i = t; i < kN * kN; i += kThreads) {
        const int r = i / kN, c = i % kN;
        const double x = hx[r * kPitch + c], y = hx[c * kPitch + r];
        const double hs = 0.5 * (x + y);
        as = fmax(as, fabs(x - y));
        double v = 0.0;
        if (r < n && c < n) v = w0 * hs + (r == c ? b0 : 0.0);
        const double vd = kSplit ? (double)(float)v : v;
        if (r == c) tr += vd;
        fr += 1.0 * vd * vd;
        s0[r * kPitch + c] = vd;
    }
    double n_s = block_sum(tr, L.red[0]), n_x = block_sum(fr, L.red[1]);   // (barriers: S_0 is complete)
    const double asym = block_max(as, L.red[2]);

    // ------------------------------------------------------------- layers of Alg. 1
    const int bi = wave >> 1, bj = wave & 1, c = lane & 31, hi32 = lane >> 5;
    const bool active = bi <= bj && 32 * bj < n;
    float s[16];          // split: this wave's block of S, row 8 (k / 4) + 4 (lane / 32) + k % 4, column lane % 32
    int cur = 1;          // FP64: L.x[cur] holds S
    auto put_planes = [&](int k, float y) {   // element k of this wave's block and its mirror
        const int r = 8 * (k >> 2) + 4 * hi32 + (k & 3);
        if (bi == bj && r > c) return;
        const float ys = y * in_scale;
        const T16 h0 = (T16)ys, h1 = (T16)(ys - (float)h0);
        T16* a = (T16*)(L.planes[0][bi][2 * bj + (c >> 4)] + (r + 32 * ((c >> 3) & 1)) * 16) + (c & 7);
        T16* b = (T16*)(L.planes[0][bj][2 * bi + (r >> 4)] + (c + 32 * ((r >> 3) & 1)) * 16) + (r & 7);
        constexpr int P = sizeof(L.planes[0]) / sizeof(T16);
        a[0] = h0;
        a[P] = h1;
        b[0] = h0;
        b[P] = h1;
    };
    if constexpr (kSplit) {
        for (int i = t; i < (int)(sizeof(L.planes) / 4); i += kThreads) ((unsigned*)L.planes)[i] = 0;
        __syncthreads();
        for (int k = 0; k < 16; ++k) {
            const int r = 8 * (k >> 2) + 4 * hi32 + (k & 3);
            s[k] = (float)s0[(32 * bi + r) * kPitch + 32 * bj + c];
            if (active) put_planes(k, s[k]);
        }
    }
    __syncthreads();
    if (kTimed && t == 0) ticks->prep = wall_clock64();
    for (int layer = 1;; ++layer) {
        StepOut o;
        control_step(&hot, layer, n_s, n_x, &o);
        if (t == 0) {
            st->ns[layer] = n_s;
            st->nx[layer] = n_x;
            st->iderr[layer] = n_s - n_x;
            if (o.chosen) {
                st->sigma[layer] = (signed char)o.sigma;
                st->sigma_c[layer] = o.sigma_c;
            }
        }
        if (hot.stopped) break;   // the same in every thread
        if (kTimed && t == 0) ticks->layer[layer - 1][0] = wall_clock64();
        double s0w = 0.0, s1w = 0.0;
        if constexpr (kSplit) {
            f32x16 acc;
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            if (active) {
                for (int u = 0; u < (n + 15) / 16; ++u) {
                    const vec8 a0 = *(const vec8*)(L.planes[0][bi][u] + 16 * lane);
                    const vec8 a1 = *(const vec8*)(L.planes[1][bi][u] + 16 * lane);
                    const vec8 b0v = *(const vec8*)(L.planes[0][bj][u] + 16 * lane);
                    const vec8 b1v = *(const vec8*)(L.planes[1][bj][u] + 16 * lane);
                    acc = TinyOps<T16>::mfma(a0, b0v, acc);
                    acc = TinyOps<T16>::mfma(a0, b1v, acc);
                    acc = TinyOps<T16>::mfma(a1, b0v, acc);
                }
            }
            __syncthreads();   // every wave has read the planes
            if (active) {
                const float alpha = (float)o.coef64[0], beta = (float)o.coef64[1], gamma = (float)o.coef64[2];
                double tw = 0.0, fw = 0.0;
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int r = 8 * (k >> 2) + 4 * hi32 + (k & 3);
                    const float x = acc[k] * out_scale;
                    float y = (beta != 0.f) ? fmaf(alpha, x, beta * s[k]) : alpha * x;
                    if (bi == bj && r == c && 32 * bj + c < n) y += gamma;
                    s[k] = y;
                    if (32 * bi + 8 * (k >> 2) >= n) continue;   // padding rows stay zero
                    put_planes(k, y);
                    if (bi != bj || r < c) {
                        fw += 2.0 * (double)y * (double)y;
                    } else if (r == c) {
                        tw += (double)y;
                        fw += (double)y * (double)y;
                    }
                }
                s0w = wave_sum0(tw);
                s1w = wave_sum0(fw);
            }
        } else {
            layer64(L.x[cur], L.x[cur ^ 1], n, o.coef64[0], o.coef64[1], o.coef64[2], nullptr, 0, &s0w, &s1w);
            cur ^= 1;
        }
        if (lane == 0) {
            L.sums[wave][0] = s0w;
            L.sums[wave][1] = s1w;
        }
        __syncthreads();
        if (kSplit) {   // one 64-tile: blocks in order
            n_s = ((L.sums[0][0] + L.sums[1][0]) + L.sums[2][0]) + L.sums[3][0];
            n_x = ((L.sums[0][1] + L.sums[1][1]) + L.sums[2][1]) + L.sums[3][1];
        } else {        // four 32-tiles: the control's tree
            n_s = (L.sums[0][0] + L.sums[2][0]) + (L.sums[1][0] + L.sums[3][0]);
            n_x = (L.sums[0][1] + L.sums[2][1]) + (L.sums[1][1] + L.sums[3][1]);
        }
        if (!kSplit) __syncthreads();   // the sums are read before the next layer writes them
        if (kTimed && t == 0) ticks->layer[layer - 1][1] = wall_clock64();
    }
    if (kTimed && t == 0) ticks->loop_end = wall_clock64();
    // ------------------------------------------------------------- refinement of S_{m-1}
    if constexpr (kSplit) {
        double* x = L.x[0];
        cur = 0;
        for (int i = t; i < kN * kPitch; i += kThreads) x[i] = 0.0;
        __syncthreads();
        if (active)
            for (int k = 0; k < 16; ++k) {
                const int r = 32 * bi + 8 * (k >> 2) + 4 * hi32 + (k & 3), q = 32 * bj + c;
                if (r > q) continue;
                x[r * kPitch + q] = (double)s[k];
                x[q * kPitch + r] = (double)s[k];
            }
    }
    __syncthreads();
    if (refine) {
        if (kTimed && t == 0) ticks->ref[0] = wall_clock64();
        for (int step = 0; step < 2; ++step) {
            layer64(L.x[cur], L.x[cur ^ 1], n, hot.rcoef[step][0], hot.rcoef[step][1], hot.rcoef[step][2],
                    step ? d : nullptr, ldd, nullptr, nullptr);
            cur ^= 1;
            __syncthreads();
            if (kTimed && t == 0) ticks->ref[step + 1] = wall_clock64();
        }
    } else {
        for (int i = t; i < n * n; i += kThreads) d[(size_t)(i / n) * ldd + i % n] = L.x[cur][(i / n) * kPitch + i % n];
        if (kTimed && t == 0) ticks->ref[0] = ticks->ref[1] = ticks->ref[2] = wall_clock64();
    }
    // ------------------------------------------------------------- final checks
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int i = t; i < n * n; i += kThreads) {
        const int r = i / n, q = i % n;
        const double x = L.x[cur][r * kPitch + q];
        if (r == q) v[0] += x;
        v[1] += x * x;
        if (p.want_energy) v[2] += x * h[(size_t)r * ldh + q];
    }
    for (int k = 0; k < 3; ++k) v[k] = block_sum(v[k], L.red[k]);
    if (t == 0) {
        finish_state(&hot, v[0], v[1], v[2], asym);
        L.hot = hot;
    }
    __syncthreads();
    if (t < 64) ((unsigned*)st)[t] = ((const unsigned*)&L.hot)[t];
    __syncthreads();
    if (host_state) copy_state(host_state, st);
    if (kTimed && t == 0) ticks->end = wall_clock64();
}

}  // namespace

hipError_t launch_tiny(const double* h, int ldh, double* d, int ldd, DevState* st, const DevState& init, int scale_log2,
                       int refine, DevState* host_state, TinyTicks* ticks, hipStream_t s) {
    if (init.n < 1 || init.n > kTinyMax) return hipErrorInvalidValue;
    const float isc = ldexpf(1.f, scale_log2), osc = ldexpf(1.f, -2 * scale_log2);
#define SP2_K(T16, SPLIT, TIMED)                                                                                 \
    hipLaunchKernelGGL((k_tiny<T16, SPLIT, TIMED>), dim3(1), dim3(kThreads), 0, s, h, ldh, d, ldd, st,           \
                       state_params(init), isc, osc, refine, host_state, ticks)
#define SP2_L(T16, SPLIT)                  \
    do {                                   \
        if (ticks) SP2_K(T16, SPLIT, true); \
        else SP2_K(T16, SPLIT, false);     \
    } while (0)
    if (init.precision == SP2_FP16X2) SP2_L(_Float16, true);
    else if (init.precision == SP2_BF16X2) SP2_L(__bf16, true);
    else if (init.precision == SP2_FP64) SP2_L(_Float16, false);
    else return hipErrorInvalidValue;
#undef SP2_L
#undef SP2_K
    return hipGetLastError();
}

}  // namespace sp2

// Preparation, control and reduction kernels of libsp2 (gfx950).
//
//   k_state_init  : per-call device state
//   k_gershgorin  : FP64 Gershgorin row intervals, one wavefront per row
//   k_bounds      : min/max of the row intervals -> spectral bounds of Alg. 1
//   k_init        : input layer S_0 = W_0 H + B_0 of Alg. 1 (reversed rescale into [0,1]),
//                   symmetrized, stored in the state precision and split into planes
//   k_control     : one layer of Alg. 1's scalar logic: IdErr_n, sigma_n, stopping tests
//   k_select_f64  : widen the state matrix that is refined to FP64
//   k_dstats      : FP64 partial sums of Tr D, ||D||_F^2 and Tr[D H]
//   k_finalize    : final occupation / idempotency acceptance test
//
// All reductions use a fixed order (strided per-thread sums, then a fixed tree), so a
// given input reproduces bit-identical traces, histories and statuses.
#include "lds_stage.h"
#include "sp2_internal.h"
#include "sp2_control.h"

#include <math.h>

namespace sp2 {

namespace {

constexpr int kThreads = 256;

// Fixed-order block sum of `count` doubles per thread (count <= 3), result in out[] of thread 0.
template <int C>
__device__ inline void block_sum(double (&v)[C], double* sh /* C * kThreads */) {
    const int t = threadIdx.x;
    for (int c = 0; c < C; ++c) sh[c * kThreads + t] = v[c];
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (t < w)
            for (int c = 0; c < C; ++c) sh[c * kThreads + t] += sh[c * kThreads + t + w];
        __syncthreads();
    }
    for (int c = 0; c < C; ++c) v[c] = sh[c * kThreads];
}

__global__ void k_state_init(DevState* st, StateParams p) { init_state(st, p); }

// One wavefront per row i: r_i = sum_{j != i} |H_ij| in FP64; the row interval
// [H_ii - r_i, H_ii + r_i] widened by (2n + 4) ulp-units for the summation error.
constexpr int kGershRowsPerBlock = kThreads / 64;

__device__ __forceinline__ void gershgorin_body(const double* __restrict__ h, int ldh, int n,
                                                         double* __restrict__ blk, int bid) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = bid * kGershRowsPerBlock + wave;
    __shared__ double sh[3][kGershRowsPerBlock];
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    if (row < n) {
        const double* hr = h + (size_t)row * ldh;
        double s = 0.0;
        for (int j = lane; j < n; j += 64) s += fabs(hr[j]);
        s = wave_sum(s);
        const double d = hr[row];
        const double slack = (2.0 * n + 4.0) * 2.220446049250313e-16;
        const double r = (s - fabs(d)) * (1.0 + slack) + slack * fabs(d);
        lo = d - r;
        hi = d + r;
        if (!isfinite(s) || !isfinite(d)) bad = 1.0;
    }
    if (lane == 0) {
        sh[0][wave] = lo;
        sh[1][wave] = hi;
        sh[2][wave] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kGershRowsPerBlock; ++w) {
            lo = fmin(lo, sh[0][w]);
            hi = fmax(hi, sh[1][w]);
            bad = fmax(bad, sh[2][w]);
        }
        blk[3 * bid + 0] = lo;
        blk[3 * bid + 1] = hi;
        blk[3 * bid + 2] = bad;
    }
}

__device__ __forceinline__ void bounds_body(DevState* st, const double* __restrict__ blk, int nblk) {
    __shared__ double sh[3][kThreads];
    const int t = threadIdx.x;
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    for (int i = t; i < nblk; i += kThreads) {
        lo = fmin(lo, blk[3 * i]);
        hi = fmax(hi, blk[3 * i + 1]);
        bad = fmax(bad, blk[3 * i + 2]);
    }
    sh[0][t] = lo;
    sh[1][t] = hi;
    sh[2][t] = bad;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (t < w) {
            sh[0][t] = fmin(sh[0][t], sh[0][t + w]);
            sh[1][t] = fmax(sh[1][t], sh[1][t + w]);
            sh[2][t] = fmax(sh[2][t], sh[2][t + w]);
        }
        __syncthreads();
    }
    if (t == 0) {
        lo = sh[0][0];
        hi = sh[1][0];
        if (sh[2][0] != 0.0 || !isfinite(lo) || !isfinite(hi)) {
            st->status = SP2_ENONFINITE;
            lo = 0.0;
            hi = 1.0;
        }
        st->emin = lo;
        st->emax = hi;
    }
}

// ---------------------------------------------------------------------------------
// Input layer.  64 x 64 tiles over the upper triangle of the padded matrix; each tile
// reads H(I,J) and H(J,I) so that the state is built from (H + H^T)/2 and is exactly
// symmetric.  Writes both the tile and its mirror; padding rows/cols are zero.
// parts: per tile [Tr part, ||.||_F^2 part, max |H_ij - H_ji|].
// ---------------------------------------------------------------------------------
constexpr int kInitTile = 64;

// kFm: the split planes in the fragment-major layout and S as 32 x 32 blocks of the upper
// triangle in accumulator order (k_square_fm.h).
template <typename St, typename T16, bool kSplit, bool kFm = false>
__device__ __forceinline__ void init_body(const double* __restrict__ h, int ldh,
                                                   const DevState* __restrict__ st, St* __restrict__ s_out,
                                                   T16* __restrict__ p0, T16* __restrict__ p1, float in_scale,
                                                   double* __restrict__ parts, int bid) {
    __shared__ double a[kInitTile][kInitTile + 1];
    __shared__ double b[kInitTile][kInitTile + 1];
    __shared__ double red[3][kThreads];
    const int n = st->n, np = st->n_padded;
    const int T = np / kInitTile;
    int I, J;
    tile_of(bid, T, T, &I, &J);   // plain column-strip order
    const int t = threadIdx.x;
    const int r0 = I * kInitTile, c0 = J * kInitTile;
    for (int idx = t; idx < kInitTile * kInitTile; idx += kThreads) {
        const int r = idx / kInitTile, c = idx % kInitTile;
        const int gi = r0 + r, gj = c0 + c;
        a[r][c] = (gi < n && gj < n) ? h[(size_t)gi * ldh + gj] : 0.0;
        const int hi_ = c0 + r, hj = r0 + c;
        b[r][c] = (hi_ < n && hj < n) ? h[(size_t)hi_ * ldh + hj] : 0.0;
    }
    __syncthreads();
    const double emin = st->emin, emax = st->emax;
    double span = emax - emin;
    if (!(span > 0.0)) span = 1.0;   // degenerate spectrum: every eigenvalue maps to ~1
    const double w0 = -1.0 / span, b0 = emax / span;
    const bool diag = (I == J);
    double tr = 0.0, fr = 0.0, as = 0.0;
    // pass 1: the tile itself, row-major (coalesced); the value is kept in `a`
    for (int idx = t; idx < kInitTile * kInitTile; idx += kThreads) {
        const int r = idx / kInitTile, c = idx % kInitTile;
        const int gi = r0 + r, gj = c0 + c;
        const double x = a[r][c], y = b[c][r];
        const double hs = 0.5 * (x + y);
        as = fmax(as, fabs(x - y));
        double v = 0.0;
        if (gi < n && gj < n) v = w0 * hs + (gi == gj ? b0 : 0.0);
        const St vs = (St)v;
        if (!kFm) s_out[(size_t)gi * np + gj] = vs;
        if (kSplit && !kFm) {
            const float xs = (float)vs * in_scale;
            const T16 h0 = (T16)xs;
            const T16 h1 = (T16)(xs - (float)h0);
            p0[(size_t)gi * plane_ld(np) + gj] = h0;
            p1[(size_t)gi * plane_ld(np) + gj] = h1;
        }
        const double vd = (double)vs;
        if (gi == gj) tr += vd;
        fr += (diag ? 1.0 : 2.0) * vd * vd;
        a[r][c] = vd;
    }
    __syncthreads();
    if constexpr (kFm) {
        typedef T16 vec8 __attribute__((ext_vector_type(8)));
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const size_t ps = (size_t)fm_pstride(np) * 512;
        for (int side = 0; side < (diag ? 1 : 2); ++side) {   // the tile, then its mirror
            const int br = side ? c0 : r0, bc = side ? r0 : c0;
            for (int item = t; item < kInitTile * kInitTile / 8; item += kThreads) {
                const int r = item % kInitTile, ch = item / kInitTile;   // row, chunk of 8 columns
                vec8 h0, h1;
                for (int e = 0; e < 8; ++e) {
                    const float xs = (float)(side ? a[8 * ch + e][r] : a[r][8 * ch + e]) * in_scale;
                    const T16 hh = (T16)xs;
                    h0[e] = hh;
                    h1[e] = (T16)(xs - (float)hh);
                }
                const size_t o = (size_t)((br + r) / 32) * ps + (size_t)((bc + 8 * ch) / 16) * 512 +
                                 ((r & 31) + 32 * (ch & 1)) * 8;
                *(vec8*)(p0 + o) = h0;
                *(vec8*)(p1 + o) = h1;
            }
        }
        for (int item = t; item < 4 * 256; item += kThreads) {   // S: 4 blocks of 256 x 4 values
            const int bi = item >> 9, bj = (item >> 8) & 1, g = (item >> 6) & 3, lane = item & 63;
            if (diag && bi > bj) continue;
            f32x4 v;
            for (int e = 0; e < 4; ++e) v[e] = (float)a[32 * bi + 8 * g + 4 * (lane >> 5) + e][32 * bj + (lane & 31)];
            *(f32x4*)((float*)s_out + ((size_t)(r0 / 32 + bi) * (np / 32) + c0 / 32 + bj) * 1024 + 256 * g + 4 * lane) = v;
        }
    }
    // pass 2: the mirror tile (J, I), row-major over its rows (coalesced)
    if (!diag && !kFm) {
        for (int idx = t; idx < kInitTile * kInitTile; idx += kThreads) {
            const int r = idx / kInitTile, c = idx % kInitTile;   // mirror element (c0 + r, r0 + c)
            const St vs = (St)a[c][r];
            const size_t off = (size_t)(c0 + r) * np + (r0 + c);
            s_out[off] = vs;
            if (kSplit) {
                const float xs = (float)vs * in_scale;
                const T16 h0 = (T16)xs;
                const T16 h1 = (T16)(xs - (float)h0);
                const size_t poff = (size_t)(c0 + r) * plane_ld(np) + (r0 + c);
                p0[poff] = h0;
                p1[poff] = h1;
            }
        }
    }
    double v2[2] = {tr, fr};
    block_sum<2>(v2, &red[0][0]);
    // max-reduction of the asymmetry (order independent)
    __syncthreads();
    red[2][t] = as;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (t < w) red[2][t] = fmax(red[2][t], red[2][t + w]);
        __syncthreads();
    }
    if (t == 0) {
        parts[3 * bid + 0] = v2[0];
        parts[3 * bid + 1] = v2[1];
        parts[3 * bid + 2] = red[2][0];
    }
}

template <typename Src>
__device__ __forceinline__ void select_body(const DevState* __restrict__ st, const Src* __restrict__ s0,
                                                         const Src* __restrict__ s1, double* __restrict__ out,
                                                         int ld_out, int n_valid, int np, int bid, int nbid) {
    const Src* src = st->refine_src ? s1 : s0;
    const size_t total = (size_t)n_valid * n_valid;
    for (size_t idx = (size_t)bid * kThreads + threadIdx.x; idx < total;
         idx += (size_t)nbid * kThreads) {
        const int i = (int)(idx / n_valid), j = (int)(idx % n_valid);
        out[(size_t)i * ld_out + j] = (double)src[(size_t)i * np + j];
    }
}

// Rows per block of the final reductions.
constexpr int kStatRows = 4;

__device__ __forceinline__ void dstats_body(const double* __restrict__ d, int ldd,
                                                     const double* __restrict__ h, int ldh, int n,
                                                     double* __restrict__ parts, int bid) {
    __shared__ double sh[3 * kThreads];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double v[3] = {0.0, 0.0, 0.0};
    for (int rr = wave; rr < kStatRows; rr += kThreads / 64) {
        const int i = bid * kStatRows + rr;
        if (i >= n) break;
        const double* dr = d + (size_t)i * ldd;
        const double* hr = h ? h + (size_t)i * ldh : nullptr;
        for (int j = lane; j < n; j += 64) {
            const double x = dr[j];
            if (j == i) v[0] += x;
            v[1] += x * x;
            if (hr) v[2] += x * hr[j];
        }
    }
    block_sum<3>(v, sh);
    if (threadIdx.x == 0) {
        parts[3 * bid + 0] = v[0];
        parts[3 * bid + 1] = v[1];
        parts[3 * bid + 2] = v[2];
    }
}

__device__ __forceinline__ void finalize_body(DevState* st, const double* __restrict__ dparts, int nd,
                                                       const double* __restrict__ iparts, int ni) {
    __shared__ double sh[3 * kThreads];
    __shared__ double mx[kThreads];
    double v[3] = {0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < nd; i += kThreads) {
        v[0] += dparts[3 * i];
        v[1] += dparts[3 * i + 1];
        v[2] += dparts[3 * i + 2];
    }
    block_sum<3>(v, sh);
    double a = 0.0;
    for (int i = threadIdx.x; i < ni; i += kThreads) a = fmax(a, iparts[3 * i + 2]);
    mx[threadIdx.x] = a;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) mx[threadIdx.x] = fmax(mx[threadIdx.x], mx[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    finish_state(st, v[0], v[1], v[2], mx[0]);
}

__global__ __launch_bounds__(kThreads) void k_fill(double* __restrict__ d, int ldd, int n, double diag) {
    const size_t total = (size_t)n * n;
    for (size_t idx = (size_t)blockIdx.x * kThreads + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * kThreads) {
        const int i = (int)(idx / n), j = (int)(idx % n);
        d[(size_t)i * ldd + j] = (i == j) ? diag : 0.0;
    }
}

template <typename T16>
__global__ __launch_bounds__(kThreads) void k_split(const float* __restrict__ x, T16* __restrict__ p0,
                                                    T16* __restrict__ p1, int np, float in_scale) {
    // x: np x np (row stride np); planes: row stride plane_ld(np)
    const size_t total = (size_t)np * np, pld = (size_t)plane_ld(np);
    for (size_t idx = (size_t)blockIdx.x * kThreads + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * kThreads) {
        const float xs = x[idx] * in_scale;
        const T16 h0 = (T16)xs;
        const size_t o = (idx / np) * pld + idx % np;
        p0[o] = h0;
        p1[o] = (T16)(xs - (float)h0);
    }
}

// planes of x (np x np) in the fragment order of k_square_fm.h, one 32 x 16 block per wave (the
// stores whole, the loads 256 bytes of a row per four waves), eight columns of a row per lane
template <typename T16>
__global__ __launch_bounds__(kThreads) void k_split_fm(const float* __restrict__ x, T16* __restrict__ p0,
                                                       T16* __restrict__ p1, int np, float in_scale) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef T16 vec8 __attribute__((ext_vector_type(8)));
    const size_t total = (size_t)np * (np / 8), ps = (size_t)fm_pstride(np) * 512;
    for (size_t idx = (size_t)blockIdx.x * kThreads + threadIdx.x; idx < total; idx += (size_t)gridDim.x * kThreads) {
        const size_t block = idx / 64;
        const int lane = (int)(idx % 64), r = 32 * (int)(block / (np / 16)) + (lane & 31);
        const int c = 2 * (int)(block % (np / 16)) + (lane >> 5);   // chunk of 8 columns
        const f32x4* src = (const f32x4*)(x + (size_t)r * np + 8 * c);
        const f32x4 v[2] = {src[0], src[1]};
        vec8 h0, h1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float xs = v[e >> 2][e & 3] * in_scale;
            const T16 a = (T16)xs;
            h0[e] = a;
            h1[e] = (T16)(xs - (float)a);
        }
        const size_t o = (size_t)(r >> 5) * ps + (size_t)(c >> 1) * 512 + ((r & 31) + 32 * (c & 1)) * 8;
        *(vec8*)(p0 + o) = h0;
        *(vec8*)(p1 + o) = h1;
    }
}

__global__ __launch_bounds__(kThreads) void k_sum_parts(const double* __restrict__ parts, int nparts,
                                                        double* __restrict__ out2) {
    __shared__ double sh[2 * kThreads];
    double v[2] = {0.0, 0.0};
    for (int i = threadIdx.x; i < nparts; i += kThreads) {
        v[0] += parts[2 * i];
        v[1] += parts[2 * i + 1];
    }
    block_sum<2>(v, sh);
    if (threadIdx.x == 0) {
        out2[0] = v[0];
        out2[1] = v[1];
    }
}

__global__ void k_set3(float* dst, float a, float b, float c) {
    if (threadIdx.x == 0) {
        dst[0] = a;
        dst[1] = b;
        dst[2] = c;
    }
}

__global__ void k_zero_ints(int* p, int count) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) p[i] = 0;
}

// Finite-temperature read-out D = (1 - c_0) I + c_0 S_0 - sum_{k>=1} c_k X_k, R matrices at a
// time into D in FP64: first = D starts as a_0 X_0 + diag I, otherwise the sum goes on from D;
// one term after the other for each element, so R changes no bit.  A pass with parts also
// takes the sums of D that k_dstats takes.  The blocks go through the matrices side by side
// (rows apart, one wavefront per row, a pass took 776 us at n = 8192).
//  * Bound: HBM.  n = 8192 with 12 terms: two passes of six (each X read once, D written twice
//    and read once) and the sums 1.19 ms (4.5 TB/s), against 3.46 ms with one pass per term into a
//    padded accumulator, a copy of it into D and a separate pass for the sums.
struct ReadoutArgs {
    const void* x[kReadoutMax];
    double a[kReadoutMax];
    double diag;
    double* d;
    const double* h;   // with parts: Tr[D H] too, or null
    double* parts;     // or null
    int ldd, ldh, n, np, first;
    int vec;   // rows of D and H start on 16 bytes
};
typedef double f64v2 __attribute__((ext_vector_type(2)));
template <typename St, int R>
__global__ __launch_bounds__(kThreads) void k_readout(ReadoutArgs q) {
    typedef St StV __attribute__((ext_vector_type(16 / sizeof(St))));
    constexpr int V = 16 / sizeof(St);
    __shared__ double sh[3 * kThreads];
    const int per_row = (q.n + V * kThreads - 1) / (V * kThreads);
    const long long units = (long long)q.n * per_row;
    double v[3] = {0.0, 0.0, 0.0};
    for (long long unit = blockIdx.x; unit < units; unit += gridDim.x) {
        const int i = (int)(unit / per_row), j0 = ((int)(unit % per_row) * kThreads + (int)threadIdx.x) * V;
        if (j0 >= q.n) continue;
        double* dr = q.d + (size_t)i * q.ldd + j0;
        const double* hr = q.parts && q.h ? q.h + (size_t)i * q.ldh + j0 : nullptr;
        StV x[R];
        double d[V], e[V];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = *(const StV*)((const St*)q.x[r] + (size_t)i * q.np + j0);
        const bool whole = j0 + V <= q.n;
        if (whole && q.vec) {
#pragma unroll
            for (int u = 0; u < V; u += 2) {
                const f64v2 t = q.first ? f64v2{0.0, 0.0} : *(const f64v2*)(dr + u);
                const f64v2 w = hr ? *(const f64v2*)(hr + u) : f64v2{0.0, 0.0};
                d[u] = t[0];
                d[u + 1] = t[1];
                e[u] = w[0];
                e[u + 1] = w[1];
            }
        } else {
#pragma unroll
            for (int u = 0; u < V; ++u) {
                d[u] = j0 + u < q.n && !q.first ? dr[u] : 0.0;
                e[u] = j0 + u < q.n && hr ? hr[u] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const bool diag = i == j0 + u;
            double y = q.first ? q.a[0] * (double)x[0][u] + (diag ? q.diag : 0.0) : d[u] + q.a[0] * (double)x[0][u];
#pragma unroll
            for (int r = 1; r < R; ++r) y += q.a[r] * (double)x[r][u];
            d[u] = y;
            if (j0 + u < q.n) {
                if (diag) v[0] += y;
                v[1] += y * y;
                if (hr) v[2] += y * e[u];
            }
        }
        if (whole && q.vec) {
#pragma unroll
            for (int u = 0; u < V; u += 2) *(f64v2*)(dr + u) = f64v2{d[u], d[u + 1]};
        } else {
#pragma unroll
            for (int u = 0; u < V; ++u)
                if (j0 + u < q.n) dr[u] = d[u];
        }
    }
    if (!q.parts) return;
    block_sum<3>(v, sh);
    if (threadIdx.x == 0)
        for (int c = 0; c < 3; ++c) q.parts[3 * blockIdx.x + c] = v[c];
}

// Up to kMaxCoefs floats passed by value into device memory (kernel arguments are part of
// the launch, so this works inside a captured stream as well).
constexpr int kMaxCoefs = 3 * SP2_MAX_LAYERS;
template <typename T>
struct CoefBlock {
    T v[kMaxCoefs];
};
template <typename T>
__global__ void k_store_coefs(T* __restrict__ dst, CoefBlock<T> b, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) dst[i] = b.v[i];
}

// Fixed-order sum of per-block triples (Tr part, ||.||_F^2 part, Tr[DH] part).
__global__ __launch_bounds__(kThreads) void k_sum3(const double* __restrict__ parts, int nparts,
                                                   double* __restrict__ out3) {
    __shared__ double sh[3 * kThreads];
    double v[3] = {0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < nparts; i += kThreads) {
        v[0] += parts[3 * i];
        v[1] += parts[3 * i + 1];
        v[2] += parts[3 * i + 2];
    }
    block_sum<3>(v, sh);
    if (threadIdx.x == 0) {
        out3[0] = v[0];
        out3[1] = v[1];
        out3[2] = v[2];
    }
}

// Occupation 0 or n: no recursion is run; the state records a converged call of 0 layers.
__global__ void k_mark_trivial(DevState* st) {
    if (threadIdx.x == 0) {
        st->stopped = 1;
        st->converged = 1;
        st->layers = 0;
        st->skip = 1;
    }
}

__global__ __launch_bounds__(kThreads) void k_gershgorin(const double* __restrict__ h, int ldh, int n,
                                                         double* __restrict__ blk) {
    gershgorin_body(h, ldh, n, blk, blockIdx.x);
}
__global__ __launch_bounds__(kThreads) void k_bounds(DevState* st, const double* __restrict__ blk, int nblk) {
    bounds_body(st, blk, nblk);
}
__global__ __launch_bounds__(kThreads) void k_control(DevState* st, const double* __restrict__ parts, int nparts,
                                                      int stride, int layer, volatile int* __restrict__ host_flag) {
    __shared__ double sh[kControlLds];
    control_body<kThreads>(st, parts, nparts, stride, layer, host_flag, sh);
}
// host_state: null, or the mapped host copy of the state that a waiting host reads
__global__ __launch_bounds__(kThreads) void k_finalize(DevState* st, const double* __restrict__ dparts, int nd,
                                                       const double* __restrict__ iparts, int ni,
                                                       DevState* __restrict__ host_state) {
    finalize_body(st, dparts, nd, iparts, ni);
    __syncthreads();
    if (host_state) copy_state(host_state, st);
}
template <typename St, typename T16, bool kSplit>
__global__ __launch_bounds__(kThreads) void k_init(const double* __restrict__ h, int ldh,
                                                   const DevState* __restrict__ st, St* __restrict__ s_out,
                                                   T16* __restrict__ p0, T16* __restrict__ p1, float in_scale,
                                                   double* __restrict__ parts) {
    init_body<St, T16, kSplit>(h, ldh, st, s_out, p0, p1, in_scale, parts, blockIdx.x);
}
// fragment-major input layer; also clears the partial-sum buffers of the layers
template <typename T16>
__global__ __launch_bounds__(kThreads) void k_init_fm(const double* __restrict__ h, int ldh,
                                                      const DevState* __restrict__ st, float* __restrict__ s_out,
                                                      T16* __restrict__ p0, T16* __restrict__ p1, float in_scale,
                                                      double* __restrict__ parts, double* __restrict__ zero, int nzero) {
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < nzero; i += gridDim.x * kThreads) zero[i] = 0.0;
    init_body<float, T16, true, true>(h, ldh, st, s_out, p0, p1, in_scale, parts, blockIdx.x);
}
// S_{m-1} from its 32 x 32 upper blocks (accumulator order) to FP64 rows, one block and its
// mirror per workgroup; rows and columns from 32 ceil(n / 32) on are zero, those from n_valid
// on are not written.
__global__ __launch_bounds__(kThreads) void k_select_fm(const DevState* __restrict__ st, const float* __restrict__ s0,
                                                        const float* __restrict__ s1, double* __restrict__ out,
                                                        int ld_out, int n, int n_valid, int sb) {
    __shared__ float b[32][33];
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int bi = blockIdx.y, bj = blockIdx.x, t = threadIdx.x;
    if (bi > bj) return;
    const float* src = (st->refine_src ? s1 : s0) + ((size_t)bi * sb + bj) * 1024;
    const int g = t >> 6, lane = t & 63, r0 = 8 * g + 4 * (lane >> 5), c = lane & 31;
    const f32x4 v = 32 * bj < n ? ((const f32x4*)src)[t] : f32x4{0.f, 0.f, 0.f, 0.f};
    for (int e = 0; e < 4; ++e) {
        if (bi == bj && r0 + e > c) continue;
        b[r0 + e][c] = v[e];
        if (bi == bj) b[c][r0 + e] = v[e];
    }
    __syncthreads();
    for (int i = t; i < 1024; i += kThreads) {
        const int r = i >> 5, q = i & 31;
        const int gr = 32 * bi + r, gc = 32 * bj + q;
        if (gr < n_valid && gc < n_valid) out[(size_t)gr * ld_out + gc] = (double)b[r][q];
        const int mr = 32 * bj + r, mc = 32 * bi + q;
        if (bi != bj && mr < n_valid && mc < n_valid) out[(size_t)mr * ld_out + mc] = (double)b[q][r];
    }
}
// the control after the last layer launched: leaves the state in its first hot block
__global__ __launch_bounds__(64) void k_lead_finish(LeadArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lead[];
    lead_load(a, lds_addr(lead));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    Coefs cf;
    (void)lead_finish(a, lead, true, &cf);
}
template <typename Src>
__global__ __launch_bounds__(kThreads) void k_select_f64(const DevState* __restrict__ st, const Src* __restrict__ s0,
                                                         const Src* __restrict__ s1, double* __restrict__ out,
                                                         int ld_out, int n_valid, int np) {
    select_body<Src>(st, s0, s1, out, ld_out, n_valid, np, blockIdx.x, gridDim.x);
}
__global__ __launch_bounds__(kThreads) void k_dstats(const double* __restrict__ d, int ldd,
                                                     const double* __restrict__ h, int ldh, int n,
                                                     double* __restrict__ parts) {
    dstats_body(d, ldd, h, ldh, n, parts, blockIdx.x);
}

// ---------------------------------------------------------------------------------
// Batched versions: one launch covers all problems; blocks are split between problems
// by the prefix offsets `offs`, single-block steps use one block per problem.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_gershgorin_g(const BatchProblem* __restrict__ pr,
                                                           const int* __restrict__ offs, int np_) {
    const int p = find_group(offs, np_, blockIdx.x);
    gershgorin_body(pr[p].h, pr[p].ldh, pr[p].n, pr[p].gersh, blockIdx.x - offs[p]);
}
__global__ __launch_bounds__(kThreads) void k_bounds_g(const BatchProblem* __restrict__ pr) {
    const BatchProblem& q = pr[blockIdx.x];
    if (q.st->have_bounds) return;
    bounds_body(q.st, q.gersh, q.gersh_blocks);
}
template <typename T16, bool kSplit>
__global__ __launch_bounds__(kThreads) void k_init_g(const BatchProblem* __restrict__ pr,
                                                     const int* __restrict__ offs, int np_) {
    const int p = find_group(offs, np_, blockIdx.x);
    const BatchProblem& q = pr[p];
    init_body<float, T16, kSplit>(q.h, q.ldh, q.st, (float*)q.s[0], (T16*)q.pl[0][0], (T16*)q.pl[0][1],
                                  q.in_scale, q.init_parts, blockIdx.x - offs[p]);
}
// the first layer's control (those behind it run in the squaring launches)
__global__ __launch_bounds__(kThreads) void k_control_g(const BatchProblem* __restrict__ pr) {
    __shared__ double sh[kControlLds];
    const BatchProblem& q = pr[blockIdx.x];
    control_body<kThreads>(q.st, q.init_parts, q.init_tiles, 3, 1, nullptr, sh);
}
__global__ __launch_bounds__(kThreads) void k_select_g(const BatchProblem* __restrict__ pr, int per_problem) {
    const int p = blockIdx.x / per_problem;
    const BatchProblem& q = pr[p];
    select_body<float>(q.st, (const float*)q.s[0], (const float*)q.s[1], q.s64, q.np, q.np, q.np,
                       blockIdx.x - p * per_problem, per_problem);
}
__global__ __launch_bounds__(kThreads) void k_dstats_g(const BatchProblem* __restrict__ pr,
                                                       const int* __restrict__ offs, int np_) {
    const int p = find_group(offs, np_, blockIdx.x);
    const BatchProblem& q = pr[p];
    dstats_body(q.d, q.ldd, q.want_energy ? q.h : nullptr, q.ldh, q.n, q.dstats, blockIdx.x - offs[p]);
}
__global__ __launch_bounds__(kThreads) void k_finalize_g(const BatchProblem* __restrict__ pr) {
    const BatchProblem& q = pr[blockIdx.x];
    finalize_body(q.st, q.dstats, q.dstats_blocks, q.init_parts, q.init_tiles);
}

// Device state of problem blockIdx.x between its region and slot blockIdx.x of a
// contiguous staging array (to_regions: staging -> region), so that a batched call moves
// all the states with one host transfer each way.
static_assert(sizeof(DevState) % 4 == 0, "states move as 32-bit words");
__global__ __launch_bounds__(64) void k_state_copy_g(const BatchProblem* __restrict__ pr, DevState* stage,
                                                     int to_regions) {
    unsigned* r = (unsigned*)pr[blockIdx.x].st;
    unsigned* g = (unsigned*)(stage + blockIdx.x);
    for (int i = threadIdx.x; i < (int)(sizeof(DevState) / 4); i += 64) {
        if (to_regions) r[i] = g[i];
        else g[i] = r[i];
    }
    if (to_regions)
        for (int i = threadIdx.x; i < kDoneInts; i += 64) done_counters(pr[blockIdx.x].st)[i] = 0;
}

inline int grid_for(size_t total) {
    size_t g = (total + kThreads - 1) / kThreads;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (int)g;
}

}  // namespace

// ------------------------------------------------------------------------------ launchers
hipError_t launch_state_init(DevState* st, const DevState& in, hipStream_t s) {
    hipLaunchKernelGGL(k_state_init, dim3(1), dim3(kThreads), 0, s, st, state_params(in));
    return hipGetLastError();
}

int gershgorin_blocks(int n) { return (n + kGershRowsPerBlock - 1) / kGershRowsPerBlock; }

hipError_t launch_gershgorin(const double* h, int ldh, int n, double* blk, int* nblk, hipStream_t s) {
    *nblk = gershgorin_blocks(n);
    hipLaunchKernelGGL(k_gershgorin, dim3(*nblk), dim3(kThreads), 0, s, h, ldh, n, blk);
    return hipGetLastError();
}

hipError_t launch_bounds(DevState* st, const double* blk, int nblk, hipStream_t s) {
    hipLaunchKernelGGL(k_bounds, dim3(1), dim3(kThreads), 0, s, st, blk, nblk);
    return hipGetLastError();
}

int init_tiles(int np) {
    const int T = np / kInitTile;
    return ntiles_upper(T);
}

hipError_t launch_init_np(const double* h, int ldh, DevState* st, int np, int precision, void* s_out, void* p0,
                          void* p1, int scale_log2, double* parts, hipStream_t s) {
    const int nt = init_tiles(np);
    const float in_scale = ldexpf(1.f, scale_log2);
    switch (precision) {
        case SP2_FP64:
            hipLaunchKernelGGL((k_init<double, _Float16, false>), dim3(nt), dim3(kThreads), 0, s, h, ldh, st,
                               (double*)s_out, (_Float16*)nullptr, (_Float16*)nullptr, 1.f, parts);
            break;
        case SP2_FP32:
            hipLaunchKernelGGL((k_init<float, _Float16, false>), dim3(nt), dim3(kThreads), 0, s, h, ldh, st,
                               (float*)s_out, (_Float16*)nullptr, (_Float16*)nullptr, 1.f, parts);
            break;
        case SP2_FP16X2:
            hipLaunchKernelGGL((k_init<float, _Float16, true>), dim3(nt), dim3(kThreads), 0, s, h, ldh, st,
                               (float*)s_out, (_Float16*)p0, (_Float16*)p1, in_scale, parts);
            break;
        case SP2_BF16X2:
            hipLaunchKernelGGL((k_init<float, __bf16, true>), dim3(nt), dim3(kThreads), 0, s, h, ldh, st,
                               (float*)s_out, (__bf16*)p0, (__bf16*)p1, in_scale, parts);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_init_fm(const double* h, int ldh, DevState* st, int np, int precision, float* s_out, void* p0,
                          void* p1, int scale_log2, double* parts, double* zero, int nzero, hipStream_t s) {
    const int nt = init_tiles(np);
    const float in_scale = ldexpf(1.f, scale_log2);
    if (precision == SP2_FP16X2)
        hipLaunchKernelGGL((k_init_fm<_Float16>), dim3(nt), dim3(kThreads), 0, s, h, ldh, st, s_out, (_Float16*)p0,
                           (_Float16*)p1, in_scale, parts, zero, nzero);
    else if (precision == SP2_BF16X2)
        hipLaunchKernelGGL((k_init_fm<__bf16>), dim3(nt), dim3(kThreads), 0, s, h, ldh, st, s_out, (__bf16*)p0,
                           (__bf16*)p1, in_scale, parts, zero, nzero);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_select_fm(const DevState* st, const float* s0, const float* s1, double* out, int ld_out, int n,
                            int n_valid, int np, hipStream_t s) {
    const int blocks = (n_valid + 31) / 32;
    hipLaunchKernelGGL(k_select_fm, dim3(blocks, blocks), dim3(kThreads), 0, s, st, s0, s1, out, ld_out, n, n_valid,
                       np / 32);
    return hipGetLastError();
}

hipError_t launch_lead_finish(const LeadArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_lead_finish, dim3(1), dim3(64), lead_bytes(a), s, a);
    return hipGetLastError();
}

hipError_t launch_control_stride(DevState* st, const double* parts, int nparts, int stride, int layer,
                                 int* host_flag, hipStream_t s) {
    hipLaunchKernelGGL(k_control, dim3(1), dim3(kThreads), 0, s, st, parts, nparts, stride, layer,
                       (volatile int*)host_flag);
    return hipGetLastError();
}

hipError_t launch_select_f64(const DevState* st, const void* s0, const void* s1, int state_f64, double* out,
                             int ld_out, int n_valid, int np, hipStream_t s) {
    const int g = grid_for((size_t)n_valid * n_valid);
    if (state_f64)
        hipLaunchKernelGGL((k_select_f64<double>), dim3(g), dim3(kThreads), 0, s, st, (const double*)s0,
                           (const double*)s1, out, ld_out, n_valid, np);
    else
        hipLaunchKernelGGL((k_select_f64<float>), dim3(g), dim3(kThreads), 0, s, st, (const float*)s0,
                           (const float*)s1, out, ld_out, n_valid, np);
    return hipGetLastError();
}

int dstats_blocks(int n) { return (n + kStatRows - 1) / kStatRows; }

hipError_t launch_dstats(const double* d, int ldd, const double* h, int ldh, int n, double* parts, int* nparts,
                         hipStream_t s) {
    *nparts = dstats_blocks(n);
    hipLaunchKernelGGL(k_dstats, dim3(*nparts), dim3(kThreads), 0, s, d, ldd, h, ldh, n, parts);
    return hipGetLastError();
}

hipError_t launch_finalize(DevState* st, const double* dparts, int nd, const double* iparts, int ni,
                           DevState* host_state, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kThreads), 0, s, st, dparts, nd, iparts, ni, host_state);
    return hipGetLastError();
}

hipError_t launch_fill(double* d, int ldd, int n, double diag, hipStream_t s) {
    hipLaunchKernelGGL(k_fill, dim3(grid_for((size_t)n * n)), dim3(kThreads), 0, s, d, ldd, n, diag);
    return hipGetLastError();
}

hipError_t launch_split(const float* x, void* p0, void* p1, int np, int precision, int scale_log2,
                        hipStream_t s) {
    const size_t total = (size_t)np * np;
    const float sc = ldexpf(1.f, scale_log2);
    if (precision == SP2_FP16X2)
        hipLaunchKernelGGL((k_split<_Float16>), dim3(grid_for(total)), dim3(kThreads), 0, s, x, (_Float16*)p0,
                           (_Float16*)p1, np, sc);
    else if (precision == SP2_BF16X2)
        hipLaunchKernelGGL((k_split<__bf16>), dim3(grid_for(total)), dim3(kThreads), 0, s, x, (__bf16*)p0,
                           (__bf16*)p1, np, sc);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_split_fm(const float* x, void* p0, void* p1, int np, int precision, int scale_log2, hipStream_t s) {
    const dim3 grid(grid_for((size_t)np * (np / 8)));
    const float sc = ldexpf(1.f, scale_log2);
    if (precision == SP2_FP16X2)
        hipLaunchKernelGGL((k_split_fm<_Float16>), grid, dim3(kThreads), 0, s, x, (_Float16*)p0, (_Float16*)p1, np, sc);
    else if (precision == SP2_BF16X2)
        hipLaunchKernelGGL((k_split_fm<__bf16>), grid, dim3(kThreads), 0, s, x, (__bf16*)p0, (__bf16*)p1, np, sc);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_sum_parts(const double* parts, int nparts, double* out2, hipStream_t s) {
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(kThreads), 0, s, parts, nparts, out2);
    return hipGetLastError();
}

}  // namespace sp2

namespace sp2 {
hipError_t launch_set3(float* dst, float a, float b, float c, hipStream_t s) {
    hipLaunchKernelGGL(k_set3, dim3(1), dim3(64), 0, s, dst, a, b, c);
    return hipGetLastError();
}
hipError_t launch_readout(int precision, const void* const* x, const double* a, int count, int first, double diag,
                          int np, double* d, int ldd, int n, const double* h, int ldh, double* parts, hipStream_t s) {
    if (count < 1 || count > kReadoutMax) return hipErrorInvalidValue;
    ReadoutArgs q;
    for (int r = 0; r < kReadoutMax; ++r) {
        q.x[r] = r < count ? x[r] : nullptr;
        q.a[r] = r < count ? a[r] : 0.0;
    }
    q.diag = diag;
    q.d = d;
    q.h = h;
    q.parts = parts;
    q.ldd = ldd;
    q.ldh = ldh;
    q.n = n;
    q.np = np;
    q.first = first;
    q.vec = (uintptr_t)d % 16 == 0 && ldd % 2 == 0 && (!parts || !h || ((uintptr_t)h % 16 == 0 && ldh % 2 == 0));
#define SP2_L(R)                                                                                                \
    if (precision == SP2_FP64)                                                                                  \
        hipLaunchKernelGGL((k_readout<double, R>), dim3(dstats_blocks(n)), dim3(kThreads), 0, s, q);            \
    else                                                                                                        \
        hipLaunchKernelGGL((k_readout<float, R>), dim3(dstats_blocks(n)), dim3(kThreads), 0, s, q);             \
    break;
    switch (count) {
        case 1: SP2_L(1)
        case 2: SP2_L(2)
        case 3: SP2_L(3)
        case 4: SP2_L(4)
        case 5: SP2_L(5)
        default: SP2_L(6)
    }
#undef SP2_L
    return hipGetLastError();
}
hipError_t launch_store_coefs(float* dst, const double* vals, int count, hipStream_t s) {
    if (count < 0 || count > kMaxCoefs) return hipErrorInvalidValue;
    CoefBlock<float> b;
    for (int i = 0; i < kMaxCoefs; ++i) b.v[i] = i < count ? (float)vals[i] : 0.f;
    hipLaunchKernelGGL(k_store_coefs<float>, dim3(1), dim3(128), 0, s, dst, b, count);
    return hipGetLastError();
}
hipError_t launch_store_coefs64(double* dst, const double* vals, int count, hipStream_t s) {
    if (count < 0 || count > kMaxCoefs) return hipErrorInvalidValue;
    CoefBlock<double> b;
    for (int i = 0; i < kMaxCoefs; ++i) b.v[i] = i < count ? vals[i] : 0.0;
    hipLaunchKernelGGL(k_store_coefs<double>, dim3(1), dim3(128), 0, s, dst, b, count);
    return hipGetLastError();
}
hipError_t launch_sum3(const double* parts, int nparts, double* out3, hipStream_t s) {
    hipLaunchKernelGGL(k_sum3, dim3(1), dim3(kThreads), 0, s, parts, nparts, out3);
    return hipGetLastError();
}
hipError_t launch_zero_ints(int* p, int count, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_ints, dim3(4), dim3(256), 0, s, p, count);
    return hipGetLastError();
}
hipError_t launch_mark_trivial(DevState* st, hipStream_t s) {
    hipLaunchKernelGGL(k_mark_trivial, dim3(1), dim3(64), 0, s, st);
    return hipGetLastError();
}
}  // namespace sp2

namespace sp2 {
hipError_t launch_batch_gershgorin(const BatchProblem* pr, const int* offs, int nprob, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_gershgorin_g, dim3(blocks), dim3(kThreads), 0, s, pr, offs, nprob);
    return hipGetLastError();
}
hipError_t launch_batch_bounds(const BatchProblem* pr, int nprob, hipStream_t s) {
    hipLaunchKernelGGL(k_bounds_g, dim3(nprob), dim3(kThreads), 0, s, pr);
    return hipGetLastError();
}
hipError_t launch_batch_init(int precision, const BatchProblem* pr, const int* offs, int nprob, int blocks,
                             hipStream_t s) {
    if (precision == SP2_FP16X2)
        hipLaunchKernelGGL((k_init_g<_Float16, true>), dim3(blocks), dim3(kThreads), 0, s, pr, offs, nprob);
    else if (precision == SP2_BF16X2)
        hipLaunchKernelGGL((k_init_g<__bf16, true>), dim3(blocks), dim3(kThreads), 0, s, pr, offs, nprob);
    else if (precision == SP2_FP32)
        hipLaunchKernelGGL((k_init_g<_Float16, false>), dim3(blocks), dim3(kThreads), 0, s, pr, offs, nprob);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}
hipError_t launch_batch_control(const BatchProblem* pr, int nprob, hipStream_t s) {
    hipLaunchKernelGGL(k_control_g, dim3(nprob), dim3(kThreads), 0, s, pr);
    return hipGetLastError();
}
hipError_t launch_batch_select(const BatchProblem* pr, int nprob, int per_problem, hipStream_t s) {
    hipLaunchKernelGGL(k_select_g, dim3(nprob * per_problem), dim3(kThreads), 0, s, pr, per_problem);
    return hipGetLastError();
}
hipError_t launch_batch_dstats(const BatchProblem* pr, const int* offs, int nprob, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_dstats_g, dim3(blocks), dim3(kThreads), 0, s, pr, offs, nprob);
    return hipGetLastError();
}
hipError_t launch_batch_finalize(const BatchProblem* pr, int nprob, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize_g, dim3(nprob), dim3(kThreads), 0, s, pr);
    return hipGetLastError();
}
hipError_t launch_batch_states(const BatchProblem* pr, DevState* stage, int nprob, int to_regions, hipStream_t s) {
    hipLaunchKernelGGL(k_state_copy_g, dim3(nprob), dim3(64), 0, s, pr, stage, to_regions);
    return hipGetLastError();
}
}  // namespace sp2

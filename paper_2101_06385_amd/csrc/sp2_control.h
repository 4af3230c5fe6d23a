// Device-side control of Alg. 1 (sigma_n, IdErr_n, the stopping tests, accelerated layers),
// shared by the stand-alone control kernels and by the squaring kernels, whose last finished
// tile runs the control of the next layer.
#pragma once

#include "sp2_internal.h"

#include <math.h>

namespace sp2 {
namespace {

// ---------------------------------------------------------------------------------
// Alg. 1 control for layer `layer` (n).  The partial sums describe S_{n-1}:
//   N_S = Tr S_{n-1}           (measured, FP64 sum of the stored diagonal)
//   N_X = Tr S_{n-1}^2 = ||S_{n-1}||_F^2   (S symmetric; FP64 sum of exact squares)
// so IdErr_n = Tr[S_{n-1} - S_{n-1}^2] is known before X_n is formed, and layer n's
// kernels receive sigma_n as coefficients (or a skip flag once a test has held).
// ---------------------------------------------------------------------------------
// Accelerated layers stop once both tracked bounds are this close to their fixed points.
constexpr double kAccSwitch = 0.01;

// One accelerated layer (Sec. Accelerated Deep-NN SP2) from the bounds l < h of the
// unoccupied / occupied eigenvalues of S_{n-1} in [0, 1].  The x^2 side applies
// ((x - v)/(1 - v))^2: the images of [0, l] and [h, 1] are [0, (l - v)^2/(1 - v)^2] and
// [(h - v)^2/(1 - v)^2, 1] for 0 <= v <= l/2, and their separation peaks at
// v = h + l - 1, hence v = clamp(h + l - 1, 0, l/2).  The 2x - x^2 side is its mirror image
// 1 - ((1 - w - x)/(1 - w))^2 with w = clamp(1 - h - l, 0, (1 - h)/2).  The wider
// separation wins (the x^2 side on a tie).  Writes Y = a X^2 + b X + c I, the real
// weight sigma_n = +-1/(1 - 2v) and the bounds after the layer.
__device__ inline void accelerated_choice(double l, double h, int* sgn, double* a, double* b, double* c,
                                          double* sigma, double* l1, double* h1) {
    const double v = fmin(fmax(h + l - 1.0, 0.0), 0.5 * l);
    const double dv = 1.0 - v;
    const double ld = (l - v) * (l - v) / (dv * dv), hd = (h - v) * (h - v) / (dv * dv);
    const double w = fmin(fmax(1.0 - h - l, 0.0), 0.5 * (1.0 - h));
    const double dw = 1.0 - w;
    const double lu = 1.0 - (dw - l) * (dw - l) / (dw * dw), hu = 1.0 - (dw - h) * (dw - h) / (dw * dw);
    if (hd - ld >= hu - lu) {
        *sgn = 1;
        *a = 1.0 / (dv * dv);
        *b = -2.0 * v / (dv * dv);
        *c = v * v / (dv * dv);
        *sigma = 1.0 / (1.0 - 2.0 * v);
        *l1 = ld;
        *h1 = hd;
    } else {
        *sgn = -1;
        *a = -1.0 / (dw * dw);
        *b = 2.0 / dw;
        *c = 0.0;
        *sigma = -1.0 / (1.0 - 2.0 * w);
        *l1 = lu;
        *h1 = hu;
    }
}

// Runs on one workgroup of at least kControlThreads threads (every thread of the workgroup
// calls it); sh: kControlLds doubles of LDS.  The partial sums are read with agent-scope
// loads, because the workgroups of the same launch may have written them on other XCDs.
// Fixed order: strided sums per thread, then a tree (across waves through LDS, the last six
// levels inside wave 0), the same on every path, so the histories are bit-identical.
constexpr int kControlThreads = 256;
constexpr int kControlLds = 2 * kControlThreads;
__device__ __forceinline__ double ld_agent(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void control_body(DevState* st, const double* parts, int nparts, int stride, int layer,
                                             volatile int* host_flag, double* sh) {
    if (st->stopped) {
        if (threadIdx.x == 0) {
            st->skip = 1;
            if (host_flag) *host_flag = 1;
        }
        return;
    }
    const int t = threadIdx.x;
    double v[2] = {0.0, 0.0};
    if (t < kControlThreads) {
        for (int i = t; i < nparts; i += kControlThreads) {
            v[0] += ld_agent(parts + (size_t)stride * i);
            v[1] += ld_agent(parts + (size_t)stride * i + 1);
        }
        sh[t] = v[0];
        sh[kControlThreads + t] = v[1];
    }
    __syncthreads();
    if (t >= 64) return;
    // wave 0: element t + 64 + (t + 128 + ...) in the order of a halving tree over 256
    for (int c = 0; c < 2; ++c) {
        const double* q = sh + c * kControlThreads + t;
        double x = (q[0] + q[128]) + (q[64] + q[192]);
        for (int w = 32; w > 0; w >>= 1) x += __shfl_down(x, w, 64);
        v[c] = x;
    }
    if (t != 0) return;
    const int n = layer;
    const double n_s = v[0], n_x = v[1];
    const double e = n_s - n_x;
    const int sp = st->sigma[n - 1];
    st->ns[n] = n_s;
    st->nx[n] = n_x;
    st->iderr[n] = e;
    bool stop = false, conv = false;
    if (!isfinite(n_s) || !isfinite(n_x)) {
        st->status = SP2_ENONFINITE;
        stop = true;
    } else if (n > st->max_layers) {
        stop = true;   // S_{max_layers} is refined; status set by the final check
    } else {
        if (n == 1 && st->accel) {
            // rescaled bounds of S_0 = (emax I - H)/(emax - emin): the order is reversed
            const double span = st->emax - st->emin;
            const double l0 = (st->emax - st->lumo) / span, h0 = (st->emax - st->homo) / span;
            if (0.0 <= l0 && l0 < h0 && h0 <= 1.0) {
                st->acc_l = l0;
                st->acc_h = h0;
            } else {
                st->accel = 0;
            }
        }
        // Interval consistency: inside the gap, exactly n_occ eigenvalues start in [h, 1] and
        // every layer maps the tracked intervals onto the next ones, so Tr S_{n-1} lies within
        // (N - n_occ) l + n_occ (1 - h) of n_occ; a larger distance (beyond rounding) means the
        // interval was not inside the gap.
        if (st->accel && st->gap_violation == 0) {
            const double nn = (double)st->n, occ = (double)st->n_occ;
            const double noise = (st->precision == SP2_FP64 ? 1e-8 : 1e-3) * nn;
            if (fabs(n_s - occ) > (nn - occ) * st->acc_l + occ * (1.0 - st->acc_h) + noise) st->gap_violation = n;
        }
        int s;
        double ca, cb, cc, sc;
        if (st->accel && fmax(st->acc_l, 1.0 - st->acc_h) > kAccSwitch) {
            double l1, h1;
            accelerated_choice(st->acc_l, st->acc_h, &s, &ca, &cb, &cc, &sc, &l1, &h1);
            st->acc_l = l1;
            st->acc_h = h1;
            st->acc_layers = n;
        } else {
            const double occ = (double)st->n_occ;
            const double val = fabs(2.0 * n_s - n_x - occ) - fabs(n_x - occ) - sp * st->eps;
            s = val > 0.0 ? 1 : (val < 0.0 ? -1 : (sp != 0 ? -sp : 1));
            ca = s > 0 ? 1.0 : -1.0;
            cb = s > 0 ? 0.0 : 2.0;
            cc = 0.0;
            sc = (double)s;
            if (st->accel) {   // the tracked intervals follow the SP2 maps too
                const double l = st->acc_l, h = st->acc_h;
                st->acc_l = s > 0 ? l * l : 2.0 * l - l * l;
                st->acc_h = s > 0 ? h * h : 2.0 * h - h * h;
            }
        }
        st->sigma[n] = (signed char)s;
        st->sigma_c[n] = sc;
        // the alternation test bounds IdErr_n by the two layers before it; it is taken
        // only when both were layers of Alg. 1
        if (e <= 0.0) conv = true;
        else if (n > 2 && n >= st->acc_layers + 3 && st->sigma[n - 1] != st->sigma[n - 2] &&
                 e > 4.5 * st->iderr[n - 2] * st->iderr[n - 2])
            conv = true;
        if (!conv) {
            st->coef[0] = (float)ca;
            st->coef[1] = (float)cb;
            st->coef[2] = (float)cc;
            st->coef64[0] = ca;
            st->coef64[1] = cb;
            st->coef64[2] = cc;
            st->skip = 0;
            st->layers = n;
            st->ran = n;
            return;
        }
        stop = true;
    }
    // stopping: refine S_{n-1}
    st->stopped = 1;
    if (host_flag) *host_flag = 1;   // lets a host that polls stop enqueueing layers
    st->skip = 1;
    st->converged = conv ? 1 : 0;
    st->layers = (conv || !isfinite(n_s) || !isfinite(n_x)) ? n : n - 1;
    const int last = st->sigma[n - 1];
    const int fs = last != 0 ? -last : 1;
    st->first_sign = fs;
    st->refine_src = (n - 1) & 1;
    // first composed step, then the opposite one (Eq. Refinement)
    const float sq[3] = {1.f, 0.f, 0.f}, pr[3] = {-1.f, 2.f, 0.f};
    for (int i = 0; i < 3; ++i) {
        st->rcoef[0][i] = fs > 0 ? sq[i] : pr[i];
        st->rcoef[1][i] = fs > 0 ? pr[i] : sq[i];
    }
    (void)stop;
}

// A tile's partial sums are in parts[2 t], parts[2 t + 1] (written by thread 0 with
// st_agent): counts the tile as done, and when it is the launch's last one runs the control of
// the next layer, so that no separate control launch stands between two layers.  The launch
// adds exactly a.ntiles arrivals; the count starts at 0 with the call's device state.  Every
// thread of the workgroup calls it; sh: kControlLds doubles of LDS that no wave still reads.
// Measured (n = 777, 40 layers): a control launch took 4.0 us and its gap 2 us per layer.
__device__ __forceinline__ void tile_done(const SquareArgs& a, double* sh, int* s_done) {
    if (!a.ctl) return;
    DevState* st = (DevState*)a.ctl;
    if (threadIdx.x == 0) {
        wait_stores();   // the partial sums are coherent before the arrival is counted
        *s_done = atomicAdd(&st->tiles_done, 1);
    }
    __syncthreads();
    if ((*s_done + 1) % a.ntiles == 0)
        control_body(st, a.parts, a.ntiles, 2, st->ran + 1, (volatile int*)a.host_flag, sh);
}

}  // namespace
}  // namespace sp2

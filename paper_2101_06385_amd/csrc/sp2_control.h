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

// The device state at the start of a call (by one workgroup).
__device__ __forceinline__ void init_hot(StateHot* st, const StateParams& p) {
    st->n = p.n;
    st->n_occ = p.n_occ;
    st->n_padded = p.np;
    st->max_layers = p.max_layers;
    st->precision = p.precision;
    st->tile = p.tile;
    st->have_bounds = p.have_bounds;
    st->want_energy = p.want_energy;
    st->stopped = 0;
    st->converged = 0;
    st->layers = 0;
    st->status = SP2_OK;
    st->skip = 0;
    st->first_sign = 0;
    st->refine_src = 0;
    st->ran = 0;
    st->accel = p.accel;
    st->acc_layers = 0;
    st->gap_violation = 0;
    st->sig1 = st->sig2 = 0;
    st->pad0 = 0;
    for (int i = 0; i < 3; ++i) st->coef[i] = 0.f;
    for (int i = 0; i < 6; ++i) st->rcoef[i / 3][i % 3] = 0.f;
    st->pad1 = 0.f;
    st->eps = p.eps;
    st->tol_tr = p.tol_tr;
    st->tol_id = p.tol_id;
    st->emin = p.emin;
    st->emax = p.emax;
    st->homo = p.homo;
    st->lumo = p.lumo;
    st->acc_l = 0.0;
    st->acc_h = 1.0;
    st->ide1 = st->ide2 = 0.0;
    st->asym = 0.0;
    st->trace_d = 0.0;
    st->frob_d = 0.0;
    st->energy = 0.0;
    st->pad2 = 0.0;
}
__device__ __forceinline__ void init_state(DevState* st, const StateParams& p) {
    const int t = threadIdx.x;
    for (int i = t; i <= SP2_MAX_LAYERS; i += blockDim.x) {
        st->sigma[i] = 0;
        st->iderr[i] = 0.0;
        st->ns[i] = 0.0;
        st->nx[i] = 0.0;
        st->sigma_c[i] = 0.0;
    }
    for (int i = t; i < kDoneInts; i += blockDim.x) done_counters(st)[i] = 0;
    if (t == 0) {
        for (int i = 0; i < 3; ++i) st->coef64[i] = 0.0;
        st->pad3 = 0.0;
        init_hot(st, p);
    }
}
// Final occupation / idempotency acceptance test.
__device__ __forceinline__ void finish_state(StateHot* st, double trace, double frob, double energy, double asym) {
    st->trace_d = trace;
    st->frob_d = frob;
    st->energy = st->want_energy ? energy : 0.0;
    st->asym = asym;
    int status = st->status;
    const double scale = fmax(fmax(fabs(st->emin), fabs(st->emax)), 1.0);
    if (status == SP2_OK && !(asym <= 1e-12 * scale)) status = SP2_EINVAL;
    if (status == SP2_OK) {
        const double idem = trace - frob;
        if (!isfinite(trace) || !isfinite(frob)) status = SP2_ENONFINITE;
        else if (st->gap_violation) status = SP2_ENOTIDEMP;   // the interval was not inside the gap
        else if (!st->converged) status = SP2_ENOCONV;
        else if (!(fabs(trace - st->n_occ) <= st->tol_tr) || !(fabs(idem) <= st->tol_id)) status = SP2_ENOTIDEMP;
    }
    st->status = status;
}
// by one workgroup
__device__ __forceinline__ void copy_state(DevState* dst, const DevState* src) {
    for (int i = threadIdx.x; i < (int)(sizeof(DevState) / 4); i += blockDim.x)
        ((unsigned*)dst)[i] = ((const unsigned*)src)[i];
}

// Sum over the wave in the order of a halving tree (x[t] += x[t + w], w = 32 .. 1); lane 0 has
// it.  The last four levels stay inside rows of 16 lanes (DPP), without LDS round trips.
template <int N>
__device__ __forceinline__ double dpp_shl(double v) {
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    const i32x2 x = __builtin_bit_cast(i32x2, v);
    const i32x2 y = {__builtin_amdgcn_update_dpp(0, x[0], 0x100 + N, 0xf, 0xf, true),
                     __builtin_amdgcn_update_dpp(0, x[1], 0x100 + N, 0xf, 0xf, true)};
    return __builtin_bit_cast(double, y);
}
__device__ __forceinline__ double wave_sum0(double v) {
    v += __shfl_down(v, 32, 64);
    v += __shfl_down(v, 16, 64);
    v += dpp_shl<8>(v);
    v += dpp_shl<4>(v);
    v += dpp_shl<2>(v);
    v += dpp_shl<1>(v);
    return v;
}
__device__ __forceinline__ double first_lane(double v) {
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    const i32x2 x = __builtin_bit_cast(i32x2, v);
    const i32x2 y = {__builtin_amdgcn_readfirstlane(x[0]), __builtin_amdgcn_readfirstlane(x[1])};
    return __builtin_bit_cast(double, y);
}

// Scalar logic of Alg. 1's layer n on the state's hot block: N_S and N_X of S_{n-1} in, the
// layer's sigma and coefficients or the stop out.
struct StepOut {
    bool chosen;      // a sigma was chosen (false: non-finite or past max_layers)
    int sigma;
    double sigma_c, coef64[3];
};
__device__ __forceinline__ void control_step(StateHot* st, int n, double n_s, double n_x, StepOut* o) {
    const double e = n_s - n_x;
    const int sp = st->sig1;
    bool conv = false;
    o->chosen = false;
    if (!isfinite(n_s) || !isfinite(n_x)) {
        st->status = SP2_ENONFINITE;
    } else if (n > st->max_layers) {
        // S_{max_layers} is refined; status set by the final check
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
        o->chosen = true;
        o->sigma = s;
        o->sigma_c = sc;
        // the alternation test bounds IdErr_n by the two layers before it; it is taken
        // only when both were layers of Alg. 1
        if (e <= 0.0) conv = true;
        else if (n > 2 && n >= st->acc_layers + 3 && sp != st->sig2 && e > 4.5 * st->ide2 * st->ide2) conv = true;
        st->sig2 = sp;
        st->sig1 = s;
        st->ide2 = st->ide1;
        st->ide1 = e;
        if (!conv) {
            o->coef64[0] = ca;
            o->coef64[1] = cb;
            o->coef64[2] = cc;
            for (int i = 0; i < 3; ++i) st->coef[i] = (float)o->coef64[i];
            st->skip = 0;
            st->layers = n;
            st->ran = n;
            return;
        }
    }
    // stopping: refine S_{n-1}
    st->stopped = 1;
    st->skip = 1;
    st->converged = conv ? 1 : 0;
    st->layers = (conv || !isfinite(n_s) || !isfinite(n_x)) ? n : n - 1;
    const int fs = sp != 0 ? -sp : 1;
    st->first_sign = fs;
    st->refine_src = (n - 1) & 1;
    // first composed step, then the opposite one (Eq. Refinement)
    const float sq[3] = {1.f, 0.f, 0.f}, pr[3] = {-1.f, 2.f, 0.f};
    for (int i = 0; i < 3; ++i) {
        st->rcoef[0][i] = fs > 0 ? sq[i] : pr[i];
        st->rcoef[1][i] = fs > 0 ? pr[i] : sq[i];
    }
}

// Runs on one workgroup of NT threads (64, or at least 256; every thread of the workgroup
// calls it); sh: kControlLds doubles of LDS.  The partial sums (a pair per tile, `stride`
// doubles apart) are read with agent-scope loads, because the workgroups of the same
// launch may have written them on other XCDs; the state's hot block comes in with them, one
// dword per lane, so the whole control waits for memory once.  Fixed order: 256 strided sums,
// then a tree over them, the same on every path, so the histories are bit-identical.
constexpr int kControlThreads = 256;
constexpr int kControlLds = 2 * kControlThreads + 32;
__device__ __forceinline__ double ld_agent(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int NT>
__device__ __forceinline__ void control_body(DevState* st, const double* parts, int nparts, int stride, int layer, volatile int* host_flag, double* sh) {
    static_assert(NT == 64 || NT >= kControlThreads, "one wave, or all the strided sums at once");
    const int t = threadIdx.x;
    unsigned hot = 0;
    if (t < 64) hot = ((const unsigned*)st)[t];
    double v[2];
    // sum k of 256: four loads in flight at a time (an element past the end adds zero)
    auto strided = [&](int k, double (&x)[2]) {
        x[0] = x[1] = 0.0;
        for (int i = k; i < nparts; i += 4 * kControlThreads) {
            double p[4], r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = i + j * kControlThreads;
                const double* q = parts + (size_t)stride * (e < nparts ? e : i);
                p[j] = ld_agent(q);
                r[j] = ld_agent(q + 1);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i + j * kControlThreads < nparts) {
                    x[0] += p[j];
                    x[1] += r[j];
                }
        }
    };
    if constexpr (NT == 64) {
        double x[4][2];
        if (nparts <= 4 * kControlThreads) {   // every load of the wave in flight at once
            double p[4][4], r[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int e = t + 64 * k + j * kControlThreads;
                    const double* q = parts + (size_t)stride * (e < nparts ? e : 0);
                    p[k][j] = ld_agent(q);
                    r[k][j] = ld_agent(q + 1);
                }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k][0] = x[k][1] = 0.0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (t + 64 * k + j * kControlThreads < nparts) {
                        x[k][0] += p[k][j];
                        x[k][1] += r[k][j];
                    }
            }
        } else {
            for (int k = 0; k < 4; ++k) strided(t + 64 * k, x[k]);
        }
        for (int c = 0; c < 2; ++c) v[c] = (x[0][c] + x[2][c]) + (x[1][c] + x[3][c]);
    } else {
        if (t < kControlThreads) {
            strided(t, v);
            sh[t] = v[0];
            sh[kControlThreads + t] = v[1];
        }
        __syncthreads();
        if (t >= 64) return;
        for (int c = 0; c < 2; ++c) {
            const double* q = sh + c * kControlThreads + t;
            v[c] = (q[0] + q[128]) + (q[64] + q[192]);
        }
    }
    unsigned* hs = (unsigned*)(sh + 2 * kControlThreads);
    hs[t] = hot;
    for (int c = 0; c < 2; ++c) v[c] = wave_sum0(v[c]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // wave 0 alone from here: its LDS is in order
    if (t == 0) {
        StateHot* h = (StateHot*)hs;
        if (h->stopped) {
            h->skip = 1;
            if (host_flag) *host_flag = 1;
        } else {
            const int n = layer ? layer : h->ran + 1;
            StepOut o;
            control_step(h, n, v[0], v[1], &o);
            st->ns[n] = v[0];
            st->nx[n] = v[1];
            st->iderr[n] = v[0] - v[1];
            if (o.chosen) {
                st->sigma[n] = (signed char)o.sigma;
                st->sigma_c[n] = o.sigma_c;
                if (!h->stopped)
                    for (int i = 0; i < 3; ++i) st->coef64[i] = o.coef64[i];
            }
            if (h->stopped && host_flag) *host_flag = 1;   // lets a host that polls stop enqueueing layers
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    ((unsigned*)st)[t] = hs[t];
}

// Leading control (see LeadArgs).  lead_load, by one wave, copies the hot block (256 bytes) and
// the partial sums behind it into lead_bytes of LDS at `lds` (16-byte aligned; the last 256
// bytes in front of the sums are for the block that is recorded) with
// global_load_lds; lead_finish, by every wave that needs the result, runs once they have landed
// (vector-memory loads complete in order, so any wait for a load behind lead_load will do).
struct Coefs {
    float f[3];
    double d[3];
};
__host__ __device__ inline size_t lead_bytes(const LeadArgs& a) {
    return 512 + ((size_t)a.nparts * a.stride * sizeof(double) + 1023) / 1024 * 1024;
}
__device__ __forceinline__ void lead_load(const LeadArgs& a, unsigned lds) {
    const unsigned lane = threadIdx.x & 63;
    asm volatile(
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dword %0, %1"
        :
        : "v"(4 * lane), "s"(a.hot_in), "s"(lds)
        : "memory", "m0");
    // whole 16 bytes (the buffers are padded to 256); past the end: the last ones again
    const unsigned bytes = ((unsigned)a.nparts * a.stride * 8u + 15u) & ~15u;
    for (unsigned o = 0; o < bytes; o += 1024) {
        unsigned off = o + lane * 16;
        off = off < bytes ? off : bytes - 16;
        asm volatile(
            "s_mov_b32 m0, %2\n\t"
            "s_nop 0\n\t"
            "global_load_lds_dwordx4 %0, %1"
            :
            : "v"(off), "s"(a.parts), "s"(lds + 512 + o)
            : "memory", "m0");
    }
}
// The layer's coefficients, or false when Alg. 1 has stopped.  record: this workgroup writes
// the state (exactly one of the launch).  lead: the LDS that lead_load filled.
__device__ __forceinline__ bool lead_finish(const LeadArgs& a, unsigned char* lead, bool record, Coefs* cf) {
    const int t = threadIdx.x & 63;
    const unsigned* hs = (const unsigned*)lead;   // other waves may still read it: never written
    const double* parts = (const double*)(lead + 512);
    double x[4][2], v[2];
    for (int k = 0; k < 4; ++k) {   // strided sums t + 64 k of 256
        x[k][0] = x[k][1] = 0.0;
        for (int i = t + 64 * k; i < a.nparts; i += kControlThreads) {
            const double* q = parts + (size_t)a.stride * i;
            x[k][0] += q[0];
            x[k][1] += q[1];
        }
    }
    for (int c = 0; c < 2; ++c) v[c] = (x[0][c] + x[2][c]) + (x[1][c] + x[3][c]);
    for (int c = 0; c < 2; ++c) v[c] = first_lane(wave_sum0(v[c]));
    StateHot h = *(const StateHot*)hs;   // every lane takes the same decision
    const int n = a.layer;
    StepOut o;
    o.chosen = false;
    const bool was = h.stopped != 0;
    if (!was) control_step(&h, n, v[0], v[1], &o);
    else h.skip = 1;
    if (record) {
        unsigned* out = (unsigned*)(lead + 256);
        if (t == 0) {
            *(StateHot*)out = h;
            if (!was) {
                DevState* st = (DevState*)a.st;
                st->ns[n] = v[0];
                st->nx[n] = v[1];
                st->iderr[n] = v[0] - v[1];
                if (o.chosen) {
                    st->sigma[n] = (signed char)o.sigma;
                    st->sigma_c[n] = o.sigma_c;
                }
            }
            if (h.stopped && a.host_flag) *(volatile int*)a.host_flag = 1;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        ((unsigned*)a.hot_out)[t] = out[t];
    }
    if (h.stopped) return false;
    for (int i = 0; i < 3; ++i) {
        cf->d[i] = o.coef64[i];
        cf->f[i] = (float)o.coef64[i];
    }
    return true;
}

// A tile's pair of partial sums is in parts (written by thread 0 with st_agent); slot t of the
// `arrivals` that the launch counts is done.  When it is the last one, the control of the next
// layer runs, so that no separate control launch stands between two layers.  Arrivals are
// counted in kDoneGroups groups and then over the groups (one counter for few tiles); the
// counters start at 0 with the call's device state and go on by whole launches.  Every thread
// of the workgroup calls it; sh: kControlLds doubles of LDS that no wave still reads.
// Measured (n = 777, 40 layers): a control launch took 4.0 us and its gap 2 us per layer.
template <int NT>
__device__ __forceinline__ void tile_done(DevState* st, const double* parts, int arrivals, int t, int* host_flag,
                                          double* sh, int* s_done) {
    if (threadIdx.x == 0) {
        wait_stores();   // the partial sums are coherent before the arrival is counted
        int* cnt = done_counters(st);
        int last;
        if (arrivals <= 2 * kDoneGroups) {
            last = (atomicAdd(cnt, 1) + 1) % arrivals == 0;
        } else {
            const int g = t % kDoneGroups, members = (arrivals - g + kDoneGroups - 1) / kDoneGroups;
            last = (atomicAdd(cnt + (1 + g) * kDoneLineInts, 1) + 1) % members == 0;
            if (last) last = (atomicAdd(cnt, 1) + 1) % kDoneGroups == 0;
        }
        *s_done = last;
    }
    __syncthreads();
    if (*s_done) control_body<NT>(st, parts, arrivals, 2, 0, (volatile int*)host_flag, sh);
}
template <int NT>
__device__ __forceinline__ void tile_done(const SquareArgs& a, int t, double* sh, int* s_done) {
    if (a.ctl) tile_done<NT>((DevState*)a.ctl, a.parts, a.arrivals, t, a.host_flag, sh, s_done);
}

}  // namespace
}  // namespace sp2

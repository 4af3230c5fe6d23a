// Internal declarations shared by the HIP kernels and the host driver of libsp2.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/sp2.h"
#include "sp2_args.h"

namespace sp2 {

// Split-K partial tiles of the persistent kernels cross XCDs, whose L2 caches are not
// coherent with each other.  They are written with agent-coherent (write-through) stores
// and read with agent-scope atomic loads, so neither side needs a device-wide fence: such a
// fence writes back or invalidates the whole L2 of the XCD, which also holds the other
// workgroups' panels and output.  A writer waits for its stores (wait_stores) before its
// arrival is counted.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st16_agent(void* p, u32x4_t v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ u32x4_t ld16_agent(const void* p) {
    typedef unsigned long long u64x2_t __attribute__((ext_vector_type(2)));
    const unsigned long long* q = (const unsigned long long*)p;
    const u64x2_t ab = {__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                        __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
    return __builtin_bit_cast(u32x4_t, ab);
}
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------------------------
// Per-call device state: lives at the start of the caller's workspace.
// Written by the control kernels; read by the layer kernels (skip flag, layer
// coefficients) and copied back to the host for sp2_info.
// ---------------------------------------------------------------------------------
// Everything the control of a layer reads, in one 256-byte block (one load by one wave).
struct StateHot {
    int n, n_occ, n_padded, max_layers;
    int precision, tile, have_bounds, want_energy;
    int stopped;        // 1 once a stopping test held, a non-finite value appeared or the cap hit
    int converged;
    int layers;         // m
    int status;         // device-side sp2_status
    int skip;           // layer kernels of the current layer do nothing when set
    int first_sign;     // first composed step of the refinement
    int refine_src;     // ping-pong index of the state matrix that is refined
    int ran;            // squaring layers that ran (the last layer whose control let it run)
    // accelerated layers (Sec. Accelerated Deep-NN SP2)
    int accel;          // 1 when the caller's interval rescaled into 0 <= l < h <= 1
    int acc_layers;     // index of the last accelerated layer (0: none)
    int gap_violation;  // first layer whose interval consistency check failed (0: none)
    int sig1, sig2;     // sigma of the last layer and of the one before it
    int pad0;
    float coef[3];      // (alpha, beta, gamma) of the current layer: Y = alpha X^2 + beta X + gamma I
    float rcoef[2][3];  // the two refinement layers
    float pad1;
    double eps, tol_tr, tol_id;
    double emin, emax;
    double homo, lumo;    // caller's interval inside the gap (energies)
    double acc_l, acc_h;  // unoccupied eigenvalues of S_{n-1} in [0, acc_l], occupied in [acc_h, 1]
    double ide1, ide2;    // IdErr of the last layer and of the one before it
    double asym;
    double trace_d, frob_d, energy;
    double pad2;
};
static_assert(sizeof(StateHot) == 256, "one 64-lane load");
struct DevState : StateHot {
    signed char sigma[SP2_MAX_LAYERS + 1];  // index n = layer n (sigma[0] = 0)
    double iderr[SP2_MAX_LAYERS + 1];
    double ns[SP2_MAX_LAYERS + 1];
    double nx[SP2_MAX_LAYERS + 1];
    double sigma_c[SP2_MAX_LAYERS + 1];
    double coef64[3];   // the current layer's (alpha, beta, gamma) unrounded, for the FP64 layer kernels
    double pad3;
};

// Arrival counters of the call (tile_done in sp2_control.h), right behind the device state:
// one 128-byte line each, kDoneGroups group counters and one for the groups.  Atomics on one
// address take 11.5 ns each on MI355X (1400 arrivals: 17.5 us on one counter, 4.5 us on 8).
constexpr int kDoneGroups = 32;
constexpr int kDoneLineInts = 32;
constexpr int kDoneInts = (kDoneGroups + 1) * kDoneLineInts;
constexpr size_t kStateBytes = (sizeof(DevState) + 255) / 256 * 256;
constexpr size_t kHot2 = kStateBytes + sizeof(int) * kDoneInts;   // second hot block (leading control)
constexpr size_t kStateArea = kHot2 + sizeof(StateHot);           // state, counters, second hot block
__host__ __device__ inline void* hot_block(DevState* st, int i) { return i & 1 ? (char*)st + kHot2 : (char*)st; }
__host__ __device__ inline int* done_counters(DevState* st) { return (int*)((char*)st + kStateBytes); }

// What a call's device state starts from.
struct StateParams {
    int n, n_occ, np, max_layers, precision, tile, have_bounds, want_energy, accel;
    double eps, tol_tr, tol_id, emin, emax, homo, lumo;
};
inline StateParams state_params(const DevState& in) {
    StateParams p;
    p.n = in.n;
    p.n_occ = in.n_occ;
    p.np = in.n_padded;
    p.max_layers = in.max_layers;
    p.precision = in.precision;
    p.tile = in.tile;
    p.have_bounds = in.have_bounds;
    p.want_energy = in.want_energy;
    p.eps = in.eps;
    p.tol_tr = in.tol_tr;
    p.tol_id = in.tol_id;
    p.emin = in.emin;
    p.emax = in.emax;
    p.accel = in.accel;
    p.homo = in.homo;
    p.lumo = in.lumo;
    return p;
}

// Upper-triangle tile enumeration shared by every kernel that works on (I <= J) tiles.
// The T x T tile grid is cut into column strips of width G; strips are enumerated left
// to right, and inside a strip the tiles go row by row.  Consecutive indices therefore
// form compact G-wide blocks of rows, so workgroups that run at the same time on one
// XCD share their row and column panels in that XCD's L2.
__host__ __device__ inline void tile_of(int t, int T, int G, int* pi, int* pj) {
    int s = 0, off = 0;
    for (;;) {
        int w = T - s * G < G ? T - s * G : G;
        int cnt = s * G * w + w * (w + 1) / 2;
        if (t < off + cnt) {
            int u = t - off;
            int sg = s * G;
            if (u < sg * w) {
                *pi = u / w;
                *pj = sg + u % w;
            } else {
                u -= sg * w;
                int i = 0;
                while (u >= w - i) { u -= w - i; ++i; }
                *pi = sg + i;
                *pj = sg + i + u;
            }
            return;
        }
        off += cnt;
        ++s;
    }
}

// Workgroups are dispatched round-robin over the 8 XCDs of the MI355X; this maps the
// hardware block index so that XCD x receives the contiguous tile range
// [x*per, (x+1)*per).  Returns -1 for the (at most 7) surplus blocks.
__device__ inline int xcd_tile_index(int b, int per, int ntiles) {
    int t = (b & 7) * per + (b >> 3);
    return t < ntiles ? t : -1;
}

inline int ntiles_upper(int T) { return T * (T + 1) / 2; }

// Sum over the wave, in every lane.
__device__ inline double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Group of a block in a launch that covers several problems: offs[0..n] are the first
// block of each problem (offs[0] = 0, offs[n] = total); returns p with offs[p] <= b < offs[p+1].
__device__ inline int find_group(const int* offs, int n, int b) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Autotuner table (sp2_tune.hip): the fastest measured schedule per (device, kind,
// precision, key); kind single: key = n rounded up to 256; kind batched: key = hash of the
// sorted sizes.
constexpr int kTuneSingle = 0, kTuneBatched = 1;
unsigned long long tune_key_single(int n);
unsigned long long tune_key_batched(int batch, const int* n);
bool tune_lookup(int kind, int precision, unsigned long long key, int* tile, int* kernel);
void tune_store(int kind, int precision, unsigned long long key, int tile, int kernel, float ms);

// Arguments of the FP32 adjoint layer of the generalized-SP2 network.
struct AdjointArgs {
    const float* g;       // G = dL/dX_{k+1}, np x np, symmetric
    const float* x;       // X_k, np x np, symmetric
    float* g_out;         // G_k = W_k (G X_k + X_k G) + B_k G
    double* parts;        // 3 doubles per tile: Tr G, <G, X_k>, <G, X_k^2>
    const float* coef;    // (W_k, B_k, c_k)
    int np, n;            // G and X are zero beyond n
    int T, ntiles;        // square_mix_grid over the rows to compute
};
// One layer's partials and where their sums go; parts null = none.
struct AdjointSums {
    const double* parts;
    float *dw, *db, *dc;
};

hipError_t launch_pack_coef(const float* w, const float* b, const float* c, int K, float* out, hipStream_t s);
hipError_t launch_copy_pad(const float* src, float* dst, int n, int ld, int np, int to_pad, hipStream_t s);
// dst (np x np, zero padded) <- (src + src^T)/2 of the n x n src (ld); np a multiple of 32
hipError_t launch_sym_pad(const float* src, float* dst, int n, int ld, int np, hipStream_t s);
// one adjoint layer (k_adjoint.hip), and the sums of another layer's partials (same tiles) along
hipError_t launch_adjoint(const AdjointArgs& a, const AdjointSums& prev, hipStream_t s);
hipError_t launch_reduce3(const AdjointSums& p, int nparts, hipStream_t s);

// One problem of a batched call (device copy; pointers into the batch workspace).  The
// batched path uses the FP32 state of the split and FP32 modes.
struct BatchProblem {
    const double* h;
    double* d;
    DevState* st;
    void* s[2];           // FP32 states, ping-pong
    void* pl[2][2];       // half-precision planes (split modes), ping-pong
    double* s64;          // refinement input (FP64)
    double* y;            // refinement intermediate (FP64)
    double* init_parts;   // 3 per input-layer tile
    double* gersh;        // 3 per Gershgorin block
    double* dstats;       // 3 per final-check block
    int ldh, ldd, n, np, n_occ, want_energy;
    int init_tiles, gersh_blocks, dstats_blocks;
    float in_scale;
};

hipError_t launch_batch_gershgorin(const BatchProblem* pr, const int* offs, int nprob, int blocks, hipStream_t s);
hipError_t launch_batch_bounds(const BatchProblem* pr, int nprob, hipStream_t s);
hipError_t launch_batch_init(int precision, const BatchProblem* pr, const int* offs, int nprob, int blocks,
                             hipStream_t s);
hipError_t launch_batch_control(const BatchProblem* pr, int nprob, hipStream_t s);   // of layer 1
hipError_t launch_batch_select(const BatchProblem* pr, int nprob, int per_problem, hipStream_t s);
hipError_t launch_batch_dstats(const BatchProblem* pr, const int* offs, int nprob, int blocks, hipStream_t s);
hipError_t launch_batch_finalize(const BatchProblem* pr, int nprob, hipStream_t s);
hipError_t launch_batch_states(const BatchProblem* pr, DevState* stage, int nprob, int to_regions, hipStream_t s);

// Host-side launchers (defined next to their kernels).
hipError_t launch_square_split(int precision, int tile, const SquareArgs& a, hipStream_t s);
hipError_t launch_square_plain(int precision, int tile, const SquareArgs& a, hipStream_t s);
// FP64 layer with direct-to-LDS staging, 128 tiles (k_square_f64.hip); variants 0..2
hipError_t launch_square_f64(int variant, const SquareArgs& a, hipStream_t s);
// FP64 layer on 64-tiles with the leftover ones cut into 32-tiles: a.T, a.ntiles from
// square_mix_grid over the rows to compute
void square_mix_grid(int edge, int* T, int* nmain, int* ntiles);
hipError_t launch_square_f64_mix(const SquareArgs& a, hipStream_t s);
// the same with leading control, where every 64-tile is cut (a.parts: not the buffer that `lead` reads)
bool square_leads(int edge);
bool few_cut_tiles(int T);   // at most two workgroups per CU: stages in rows of 256 bytes
hipError_t launch_square_f64_lead(const SquareArgs& a, const LeadArgs& lead, hipStream_t s);
// grouped FP64 layer over a map of 64-tiles (see TileRef), grid 8 per
hipError_t launch_square_f64_g(const SquareArgs* descs, const TileRef* map, int per, hipStream_t s);
// FP32 layers with direct-to-LDS staging (k_square_f32.hip), tiles as the FP64 ones
hipError_t launch_square_f32_mix(const SquareArgs& a, hipStream_t s);
hipError_t launch_square_f32_lead(const SquareArgs& a, const LeadArgs& lead, hipStream_t s);
hipError_t launch_square_f32_g(const SquareArgs* descs, const TileRef* map, int per, hipStream_t s);
int square_split_grid(int tile, int np, int* T, int* ntiles, int* per);
int square_plain_grid(int tile, int np, int* T, int* ntiles, int* per);
// persistent split square: kSkVariants kernel variants per tile edge (128, 256)
bool square_sk_plan(int tile, int variant, int np, int cus, int* wg_per_cu, StreamK* sk, int* T, int* ntiles);
size_t square_sk_partial_bytes(int tile, int np);
hipError_t launch_square_sk(int precision, int tile, int variant, const SquareArgs& a, const StreamK& sk,
                            hipStream_t s);
// the same pipeline with one workgroup per tile (tiles 128, 256): one problem, or grouped
hipError_t launch_square_dp(int precision, int tile, int variant, const SquareArgs& a, hipStream_t s);
hipError_t launch_square_dp_g(int precision, int tile, int variant, const SquareArgs* descs, const TileRef* map, int per,
                              hipStream_t s);
hipError_t launch_zero_ints(int* p, int count, hipStream_t s);

// preparation / control kernels (k_prep.hip)
hipError_t launch_state_init(DevState* st, const DevState& init, hipStream_t s);
hipError_t launch_gershgorin(const double* h, int ldh, int n, double* blk, int* nblk, hipStream_t s);
int gershgorin_blocks(int n);
hipError_t launch_bounds(DevState* st, const double* blk, int nblk, hipStream_t s);
hipError_t launch_init_np(const double* h, int ldh, DevState* st, int np, int precision, void* s_out,
                          void* p0, void* p1, int scale_log2, double* parts, hipStream_t s);
int init_tiles(int np);
// fragment-major path (k_square_fm.h): input layer, FP64 expansion of S, last control
hipError_t launch_init_fm(const double* h, int ldh, DevState* st, int np, int precision, float* s_out, void* p0,
                          void* p1, int scale_log2, double* parts, double* zero, int nzero, hipStream_t s);
hipError_t launch_select_fm(const DevState* st, const float* s0, const float* s1, double* out, int ld_out, int n,
                            int n_valid, int np, hipStream_t s);
hipError_t launch_lead_finish(const LeadArgs& a, hipStream_t s);
bool fm_wanted(bool split, int tile, int kernel, int np);
int fm_variant(int tile, int ntiles64);
hipError_t launch_fm(int precision, int variant, const FmArgs& a, hipStream_t s);
hipError_t launch_control_stride(DevState* st, const double* parts, int nparts, int stride, int layer,
                                 int* host_flag, hipStream_t s);
hipError_t launch_select_f64(const DevState* st, const void* s0, const void* s1, int state_f64,
                             double* out, int ld_out, int n_valid, int np, hipStream_t s);
hipError_t launch_dstats(const double* d, int ldd, const double* h, int ldh, int n,
                         double* parts, int* nparts, hipStream_t s);
int dstats_blocks(int n);
hipError_t launch_finalize(DevState* st, const double* dparts, int ndparts, const double* init_parts,
                           int ninit, DevState* host_state, hipStream_t s);
// the whole solve of n <= kTinyMax in one workgroup (k_tiny.hip): split modes and FP64
constexpr int kTinyMax = 64;
// The phases of such a solve in ticks of the device's wall clock (timed calls).
struct TinyTicks {
    long long start, prep, loop_end, end;
    long long ref[3];                      // before, between and after the refinement layers
    long long layer[SP2_MAX_LAYERS][2];    // layer n at n - 1: begin, end
};
hipError_t launch_tiny(const double* h, int ldh, double* d, int ldd, DevState* st, const DevState& init, int scale_log2,
                       int refine, DevState* host_state, TinyTicks* ticks, hipStream_t s);
hipError_t launch_fill(double* d, int ldd, int n, double diag, hipStream_t s);
hipError_t launch_split(const float* x, void* p0, void* p1, int np, int precision, int scale_log2,
                        hipStream_t s);
// the same in fragment order (k_square_fm.h); np a multiple of 32
hipError_t launch_split_fm(const float* x, void* p0, void* p1, int np, int precision, int scale_log2, hipStream_t s);
hipError_t launch_sum_parts(const double* parts, int nparts, double* out2, hipStream_t s);
hipError_t launch_set3(float* dst, float a, float b, float c, hipStream_t s);
// finite-temperature read-out: D (n x n, FP64) = a_0 X_0 + diag I (first) or D + a_0 X_0, then
// + a_r X_r for r < count <= kReadoutMax; with parts also the sums of launch_dstats
constexpr int kReadoutMax = 6;
hipError_t launch_readout(int precision, const void* const* x, const double* a, int count, int first, double diag,
                          int np, double* d, int ldd, int n, const double* h, int ldh, double* parts, hipStream_t s);
hipError_t launch_store_coefs(float* dst, const double* vals, int count, hipStream_t s);   // rounded to FP32
hipError_t launch_store_coefs64(double* dst, const double* vals, int count, hipStream_t s);
hipError_t launch_sum3(const double* parts, int nparts, double* out3, hipStream_t s);
hipError_t launch_mark_trivial(DevState* st, hipStream_t s);

// The whole sp2_density path (sp2_api.hip); poll_flag = false never touches host memory
// beyond the final read-back of the state (no mapped flag).
int density_call(const double* dH, int ldh, double* dD, int ldd, int n, int n_occ, double tol,
                 const sp2_options* opt, sp2_info* info, void* dWork, size_t work_bytes, void* stream,
                 sp2_timing* timing, bool poll_flag);

}  // namespace sp2

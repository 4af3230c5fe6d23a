// FP64 squaring layer Y = alpha X^2 + beta X + gamma I on v_mfma_f64_16x16x4f64 (gfx950),
// for the refinement layer (Eq. Refinement, computed in double precision) and the FP64
// mode.  Upper-triangle output tiles, one workgroup per tile, mirrored on store.
//
//  * Bound: the matrix pipes (64 cycles per v_mfma_f64_16x16x4f64, 78.6 TFLOP/s).  Several
//    independent workgroups of 4 waves per CU keep them busy: one's prologue, barriers and
//    epilogue hide behind the others' products.  64 x 64 tiles with two 16 KB stages fit
//    five to a CU (by LDS and by registers); the tiles beyond the last whole round of one per CU are cut into 32 x 32
//    ones so that the end of the launch is spread over the chip (k_square_f64_mix).
//    One layer, against the 8-wave 128 x 128 workgroups with one per CU (and their
//    persistent form with a split-K tail) used before: n = 256 17 -> 7.3 us, 832 128 -> 25 us,
//    2112 290 -> 167 us, 4096 1265 -> 1030 us (67 TFLOP/s), 5120 2233 -> 2015 us; 8192
//    8.58 -> 8.28 ms per layer of an FP64 solve (66 TFLOP/s), 17.3 -> 16.5 ms for the two
//    refinement layers of a mixed one.
//  * K-stages of 16 doubles: each row of a stage is one 128-byte line.  The two row
//    panels (I and J: X is symmetric, so both operands are K-contiguous rows) go straight
//    from global memory into LDS with global_load_lds_dwordx4 (16 bytes per lane, a
//    wavefront instruction fills a 1 KB block of 8 rows), ST stages deep, issued from
//    inline asm with explicit s_waitcnt accounting (the compiler would otherwise wait for
//    every load before each LDS read).
//  * Rows are XOR-swizzled in 16-byte chunks (chunk c of row r at c ^ ((r >> 1) & 7)), so
//    the 16 lanes of each ds_read_b128 pass hit distinct bank groups.
//  * The K order inside a stage is permuted per lane: MFMA s (0, 1) of unit h (0, 1) takes,
//    in its K lane j = lane / 16, the K index 8 h + 2 j + s.  A and B use the same map, so
//    every product term appears once; one 16-byte read then feeds two MFMAs.  Every tile
//    edge runs the same chain of products per element, so the tiling changes no bit.
#include "lds_stage.h"
#include "sp2_control.h"
#include "sp2_internal.h"

namespace sp2 {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// BT x BT output tile, WM x WN waves, ST LDS stages of 2 BT rows (panels I and J)
// of ROW bytes.
template <int BT, int WM, int WN, int ST, int ROW = 128>
struct F64Cfg {
    static constexpr int BK = ROW / 8;                   // doubles per row per stage
    static constexpr int CH = ROW / 16;                  // 16-byte chunks per row
    static constexpr int RPB = 1024 / ROW;               // rows per 1 KB direct-load block
    static constexpr int NW = WM * WN, NT = 64 * NW;
    static constexpr int WTM = BT / WM, WTN = BT / WN;
    static constexpr int MB = WTM / 16, NB = WTN / 16;   // 16 x 16 blocks per wave
    static constexpr int ARR = BT * ROW;                 // bytes of one panel stage
    static constexpr int STAGE = 2 * ARR;
    static constexpr int BPR = BT / RPB;                 // 1 KB blocks per panel stage
    static constexpr int LPW = 2 * BPR / NW;             // direct loads per wave per stage
    static constexpr int LDS = ST * STAGE;
    // tile_of strip of 384 columns: the tiles that an XCD runs at a time drift apart in K, and narrow
    // blocks of rows keep more of their panels in its L2 (n = 8192: 8.29 ms per layer of an FP64
    // solve, 8.61 with strips of 1024 columns; 512 and 192 are 1 % slower than 384; equal within 1 % up
    // to n = 7000)
    static constexpr int STRIP = BT == 128 ? 8 : 384 / BT;
    static_assert(MB >= 1 && NB >= 1 && (2 * BPR) % NW == 0, "tile / wave mismatch");
    static_assert(ROW == 128 || ROW == 256, "a line of the cache, or two");
    // chunk c of row r is stored at c ^ swz(r)
    static __device__ __forceinline__ int swz(int r) { return (ROW == 128 ? r >> 1 : r) & (CH - 1); }
};

// Output tile (I, J) of edge BT over all of K; t is the tile's slot in a.parts.
// LEAD: the layer's control at its head (`lead`, lead_bytes of LDS at `dyn`) instead of the next
// layer's control by the last tile.
template <int BT, int WM, int WN, int ST, int ROW = 128, bool LEAD = false>
__device__ __forceinline__ void f64_body(const SquareArgs& a, int I, int J, int t, unsigned char* __restrict__ lds,
                                         const LeadArgs* lead = nullptr, unsigned char* __restrict__ dyn = nullptr) {
    typedef F64Cfg<BT, WM, WN, ST, ROW> C;
    constexpr int kRow = ROW, kBK = C::BK;
    constexpr int MB = C::MB, NB = C::NB, LPW = C::LPW, VM = LPW * (ST - 1);
    static_assert(ST >= 2 && ST <= 4, "stages");
    const int np = a.np;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const double* x = (const double*)a.x0;
    const unsigned char* src[2] = {(const unsigned char*)(x + (size_t)I * BT * np),
                                   (const unsigned char*)(x + (size_t)J * BT * np)};
    const int nsl = ((a.k_all ? np : a.n_real) + kBK - 1) / kBK;

    // direct load l of this wave: lane L fills bytes [16 L, 16 L + 16) of a 1 KB block:
    // panel row q * RPB + L / CH, physical chunk L % CH = logical chunk (L % CH) ^ swz(row)
    unsigned voff[LPW];
#pragma unroll
    for (int l = 0; l < LPW; ++l) {
        const int row = ((wave * LPW + l) % C::BPR) * C::RPB + lane / C::CH;
        voff[l] = (unsigned)row * (unsigned)np * 8u + (unsigned)(((lane & (C::CH - 1)) ^ C::swz(row)) << 4);
    }
    auto load_one = [&](int l, int buf, int ks) {
        const int j = wave * LPW + l;
        const int arr = j / C::BPR, qd = j % C::BPR;
        dma16s(voff[l], src[arr] + (size_t)ks * kRow, lds_addr(lds + buf * C::STAGE + arr * C::ARR + qd * 1024));
    };
    auto issue = [&](int buf, int ks) {
#pragma unroll
        for (int l = 0; l < LPW; ++l) load_one(l, buf, ks);
    };
    // A unit is HU runs of 8 K; a run is one 16-byte read per row and lane, the logical chunk
    // 4 run + lane / 16 of row (block base + lane % 16).  A wave's next unit is read from LDS behind
    // the products of this one; with one block per wave (32-tiles) it takes four products to cover
    // those reads.
    constexpr int HU = ROW / 128, UNITS = kBK / 8 / HU;
    struct Frag {
        f64x2 a[HU][MB], b[HU][NB];
    };
    auto frags = [&](int buf, int u, Frag& f) {
        const int r16 = lane & 15;
        const unsigned char* base = lds + buf * C::STAGE;
#pragma unroll
        for (int k = 0; k < HU; ++k) {
            const int ch = 4 * (HU * u + k) + (lane >> 4);
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int row = wm * C::WTM + m * 16 + r16;
                f.a[k][m] = *(const f64x2*)(base + row * kRow + ((ch ^ C::swz(row)) << 4));
            }
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const int row = wn * C::WTN + n * 16 + r16;
                f.b[k][n] = *(const f64x2*)(base + C::ARR + row * kRow + ((ch ^ C::swz(row)) << 4));
            }
        }
    };

    f64x4 acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = f64x4{0.0, 0.0, 0.0, 0.0};
    // the MFMAs of one unit; with doit the direct loads of stage ks (into buffer buf) are
    // spread between them, so that their issue overlaps the matrix cores (scheduling barriers
    // keep the compiler from regrouping them)
    auto mma = [&](const Frag& f, bool doit, int buf, int ks) {
        constexpr int NM = 2 * HU * MB * NB;
        constexpr int EVERY = NM / LPW;
        static_assert(EVERY >= 1 && NM % LPW == 0, "interleave");
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int k = i / (2 * MB * NB), s = (i / (MB * NB)) & 1, m = (i / NB) % MB, n = i % NB;
            acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[k][m][s], f.b[k][n][s], acc[m][n], 0, 0, 0);
            if (i % EVERY == EVERY - 1) {
                __builtin_amdgcn_sched_barrier(0);
                if (doit) load_one(i / EVERY, buf, ks);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // stage q is issued by advance(q - ST + 1); the prologue plays those of 0 .. ST - 1
    const int pro = nsl < ST ? nsl : ST;
    if (LEAD && wave == 0) lead_load(*lead, lds_addr(dyn));
    for (int q = 0; q < pro; ++q) issue(q, q);
    // read while the first loads are in flight
    const bool stop = LEAD ? ((const StateHot*)lead->hot_in)->stopped && blockIdx.x != 0 : a.skip && *a.skip;
    if (stop) {
        wait_vm<VM>(0);
        return;
    }
    wait_vm<VM>((pro - 1) * LPW);
    __syncthreads();
    Coefs cf;
    if (LEAD && !lead_finish(*lead, dyn, blockIdx.x == 0 && wave == 0, &cf)) {   // Alg. 1 has stopped
        wait_vm<VM>(0);
        return;
    }
    Frag p, q;
    frags(0, 0, p);
    // stage `next` readable: its loads landed (this wave's), every wave past the barrier
    auto arrive = [&](int next) {
        const int last = (next + ST - 2 < nsl - 1) ? next + ST - 2 : nsl - 1;
        wait_vm<VM>((last - next) * LPW);
        stage_barrier();
    };
    // units: two per stage; p holds a stage's first, q its second.  Stage st + ST refills the
    // buffer of stage st once every wave has read it (after arrive(st + 1)).
    static_assert(UNITS == 2, "two units per stage");
    int st = 0;
    for (; st + 1 < nsl; ++st) {
        frags(st % ST, 1, q);
        mma(p, false, 0, 0);
        arrive(st + 1);
        frags((st + 1) % ST, 0, p);
        mma(q, st + ST < nsl, st % ST, st + ST);
    }
    frags(st % ST, 1, q);
    mma(p, false, 0, 0);
    mma(q, false, 0, 0);

    // ------------------------------------------------------------------- epilogue
    if (!LEAD)
        for (int i = 0; i < 3; ++i) cf.d[i] = a.coef64 ? a.coef64[i] : (double)a.coef[i];
    const double alpha = cf.d[0], beta = cf.d[1], gamma = cf.d[2];
    double* so = (double*)a.s_out;
    const double* si = (const double*)a.s_in;
    const int ldo = a.ld_out, nv = a.n_valid;
    const bool diag = (I == J);
    double tr = 0.0, fr = 0.0;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int col = J * BT + wn * C::WTN + n * 16 + (lane & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = I * BT + wm * C::WTM + m * 16 + 4 * r + (lane >> 4);
                if (diag && row > col) continue;
                const double xv = acc[m][n][r];
                double y = (beta != 0.0) ? fma(alpha, xv, beta * si[(size_t)row * np + col]) : alpha * xv;
                if (row == col && col < a.n_real) y += gamma;
                if (row < nv && col < nv) {
                    so[(size_t)row * ldo + col] = y;
                    if (row != col) so[(size_t)col * ldo + row] = y;
                }
                if (row == col) {
                    tr += y;
                    fr += y * y;
                } else {
                    fr += 2.0 * y * y;
                }
            }
        }
    }
    if (a.parts) {
        // in the stages, which every wave has left: the LDS of a workgroup stays a fifth of a CU's
        double* red = (double*)(lds + C::LDS - 256);
        int* s_done = (int*)(lds + C::LDS - 64);
        tr = wave_sum(tr);
        fr = wave_sum(fr);
        __syncthreads();
        if (lane == 0) {
            red[2 * wave] = tr;
            red[2 * wave + 1] = fr;
        }
        __syncthreads();
        if (tid == 0) {
            double s0 = 0.0, s1 = 0.0;
            for (int w = 0; w < C::NW; ++w) {
                s0 += red[2 * w];
                s1 += red[2 * w + 1];
            }
            st_agent(a.parts + 2 * t, s0);
            st_agent(a.parts + 2 * t + 1, s1);
        }
        if (!LEAD) tile_done<C::NT>(a, t, (double*)lds, s_done);
    }
}

// One workgroup per BT x BT tile of one problem.
template <int BT, int WM, int WN, int ST>
__global__ __launch_bounds__(64 * WM * WN) void k_square_f64(SquareArgs a) {
    typedef F64Cfg<BT, WM, WN, ST> C;
    __shared__ __attribute__((aligned(16))) unsigned char lds[C::LDS];
    const int t = xcd_tile_index(blockIdx.x, a.per, a.ntiles);
    if (t < 0) return;
    int I, J;
    tile_of(t, a.T, C::STRIP, &I, &J);
    f64_body<BT, WM, WN, ST>(a, I, J, t, lds);
}

typedef F64Cfg<64, 2, 2, 2> F64Main;

// Cut tile u of those behind `nmain` whole 64-tiles (blocks from nmain on).
template <int ROW>
__device__ __forceinline__ void f64_cut(const SquareArgs& a, int nmain, unsigned char* lds) {
    const int nsub = a.ntiles - nmain;
    const int u = xcd_tile_index(blockIdx.x - nmain, (nsub + 7) >> 3, nsub);
    if (u < 0) return;
    int I, J;
    tile_of(nmain + (u >> 2), a.T, F64Main::STRIP, &I, &J);
    const int i = 2 * I + ((u >> 1) & 1), j = 2 * J + (u & 1), slot = nmain + u;
    if (i > j) {   // below the diagonal: its mirror computes it
        if (a.skip && *a.skip) return;
        if (!a.parts) return;
        if (threadIdx.x == 0) {
            st_agent(a.parts + 2 * slot, 0.0);
            st_agent(a.parts + 2 * slot + 1, 0.0);
        }
        tile_done<256>(a, slot, (double*)lds, (int*)(lds + 4096));
        return;
    }
    f64_body<32, 2, 2, 2, ROW>(a, i, j, slot, lds);
}

// 64-tiles [0, nmain) whole (nmain a multiple of 8), the others as four 32-tiles each.
__global__ __launch_bounds__(256) void k_square_f64_mix(SquareArgs a, int nmain) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F64Main::LDS];
    int I, J;
    if ((int)blockIdx.x < nmain) {
        const int t = (blockIdx.x & 7) * (nmain >> 3) + (blockIdx.x >> 3);
        tile_of(t, a.T, F64Main::STRIP, &I, &J);
        f64_body<64, 2, 2, 2>(a, I, J, t, lds);
        return;
    }
    f64_cut<128>(a, nmain, lds);
}
// Every 64-tile cut, stages in rows of ROW bytes (see k_square_f64_lead).  As the refinement
// of a solve, two layers, against cut tiles in the LDS of whole ones: n = 256 5 us less, 513 8, 777 6.
template <int ROW>
__global__ __launch_bounds__(256) void k_square_f64_cut(SquareArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F64Cfg<32, 2, 2, 2, ROW>::LDS];
    f64_cut<ROW>(a, 0, lds);
}

// All of a small problem's 64-tiles as four 32-tiles each, with leading control: at these sizes
// the chain of memory trips at a launch's end (sums stored, counted, read back, state written)
// costs more (n = 256: 12.1 us per layer with the control in the last tile, 10.9 us here).  With
// few workgroups per CU a stage lasts as long as its direct loads are under way (about 1000
// cycles, for 256 of products), so while there are at most two (few_cut_tiles) the rows of a stage
// are 256 bytes in place of 128: n = 256 9.0 us, 513 15.2 (18.6), 777 22.6 (25.7); at
// n = 1024 both take 34 us, and at 1300 the larger stages' LDS leaves fewer workgroups on a CU
// (65 against 55 us).  FP32: n = 256 7.5 (8.1), 513 11.3 (12.5), 777 17.7 (17.7), 1024 24.3 (23.4).
template <int ROW>
__global__ __launch_bounds__(256) void k_square_f64_lead(SquareArgs a, LeadArgs lead) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];   // lead_bytes
    __shared__ __attribute__((aligned(16))) unsigned char lds[F64Cfg<32, 2, 2, 2, ROW>::LDS];
    const int u = xcd_tile_index(blockIdx.x, (a.ntiles + 7) >> 3, a.ntiles);
    if (u < 0) return;
    int I, J;
    tile_of(u >> 2, a.T, F64Main::STRIP, &I, &J);
    const int i = 2 * I + ((u >> 1) & 1), j = 2 * J + (u & 1);
    if (i > j) {   // below the diagonal: its mirror computes it
        if (threadIdx.x < 2) a.parts[2 * u + threadIdx.x] = 0.0;
        return;
    }
    f64_body<32, 2, 2, 2, ROW, true>(a, i, j, u, lds, &lead, dyn);
}

// grouped: block b computes the 64-tile that the tile map names for it (see TileRef)
__global__ __launch_bounds__(256) void k_square_f64_g(const SquareArgs* __restrict__ descs,
                                                      const TileRef* __restrict__ map, int per) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F64Main::LDS];
    const TileRef e = map[(blockIdx.x & 7) * per + (blockIdx.x >> 3)];
    if (e.problem < 0) return;
    const SquareArgs a = descs[e.problem];
    const int t = e.tile;
    int I, J;
    tile_of(t, a.T, F64Main::STRIP, &I, &J);
    f64_body<64, 2, 2, 2>(a, I, J, t, lds);
}

}  // namespace

// Grid of the mixed FP64 and FP32 launches over `edge` rows: a.T 64-tiles per edge; the largest whole
// number of 64-tiles per CU stays whole, the rest is cut.  (The CU count only shapes the
// schedule: every choice gives the same bits.)
constexpr int kMixCus = 256;
void square_mix_grid(int edge, int* T, int* nmain, int* ntiles) {
    *T = (edge + 63) / 64;
    const int nt = ntiles_upper(*T);
    *nmain = nt / kMixCus * kMixCus;
    *ntiles = *nmain + 4 * (nt - *nmain);
}

hipError_t launch_square_f64_mix(const SquareArgs& a, hipStream_t s) {
    int T, nmain, ntiles;
    square_mix_grid(64 * a.T, &T, &nmain, &ntiles);
    if (ntiles != a.ntiles || a.np % 64 || 64 * T > a.np) return hipErrorInvalidValue;
    const int nsub = ntiles - nmain;
    const dim3 grid(nmain + (nsub + 7) / 8 * 8);
    if (nmain > 0) hipLaunchKernelGGL(k_square_f64_mix, grid, dim3(256), 0, s, a, nmain);
    else if (few_cut_tiles(a.T)) hipLaunchKernelGGL(k_square_f64_cut<256>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_square_f64_cut<128>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

bool square_leads(int edge) {
    int T, nmain, ntiles;
    square_mix_grid(edge, &T, &nmain, &ntiles);
    return nmain == 0;
}
bool few_cut_tiles(int T) { return 4 * ntiles_upper(T) <= 2 * kMixCus; }
hipError_t launch_square_f64_lead(const SquareArgs& a, const LeadArgs& lead, hipStream_t s) {
    if (!square_leads(64 * a.T) || a.ntiles != 4 * ntiles_upper(a.T) || !a.parts) return hipErrorInvalidValue;
    const dim3 grid((a.ntiles + 7) / 8 * 8);
    if (few_cut_tiles(a.T)) hipLaunchKernelGGL(k_square_f64_lead<256>, grid, dim3(256), lead_bytes(lead), s, a, lead);
    else hipLaunchKernelGGL(k_square_f64_lead<128>, grid, dim3(256), lead_bytes(lead), s, a, lead);
    return hipGetLastError();
}

hipError_t launch_square_f64_g(const SquareArgs* descs, const TileRef* map, int per, hipStream_t s) {
    hipLaunchKernelGGL(k_square_f64_g, dim3(8 * per), dim3(256), 0, s, descs, map, per);
    return hipGetLastError();
}

// FP64 layer on 128 tiles (n_p a multiple of 128).  variant 0: 4 waves, 2 LDS stages;
// 1: 4 waves, 4 stages (128 KB); 2: 8 waves, 4 stages.
hipError_t launch_square_f64(int variant, const SquareArgs& a, hipStream_t s) {
    if (a.np % 128) return hipErrorInvalidValue;
    const int grid = 8 * a.per;
    if (variant == 0) hipLaunchKernelGGL((k_square_f64<128, 2, 2, 2>), dim3(grid), dim3(256), 0, s, a);
    else if (variant == 1) hipLaunchKernelGGL((k_square_f64<128, 2, 2, 4>), dim3(grid), dim3(256), 0, s, a);
    else if (variant == 2) hipLaunchKernelGGL((k_square_f64<128, 2, 4, 4>), dim3(grid), dim3(512), 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sp2

// FP32 squaring layer Y = alpha X^2 + beta X + gamma I (gfx950), for the FP32 mode, the FP32
// network and single FP32 layers.  Upper-triangle output tiles, mirrored on store.
//
//  * Bound: the matrix pipes (157.3 TFLOP/s).  As for the FP64 layers (k_square_f64.hip),
//    several independent workgroups of 4 waves per CU keep them busy: 64 x 64 tiles, two 16 KB
//    stages of 32 floats per row (one 128-byte line) filled by global_load_lds_dwordx4, the
//    tiles beyond the last whole round of one per CU cut into 32 x 32 ones.  One layer with its
//    control, against the register-staged 128 x 128 (64 x 64 up to n = 512) workgroups and control
//    launch used before: n = 256 15 -> 7.5 us, 777 65 -> 18 us, 1300 113 -> 35 us, 2112 167 ->
//    81 us, 4096 773 -> 510 us (135 TFLOP/s; the clock holds about 2.1 GHz), 5000 1190 -> 950 us.
//  * Each element is the chain of fused multiply-adds over ascending K, whichever instruction
//    computes it, so the tiling changes no bit.  A wave of a 64-tile holds 2 x 2 blocks of
//    v_mfma_f32_16x16x4f32, four chains (one chain of v_mfma_f32_32x32x2f32 took 610 us at
//    n = 4096), a wave of a 32-tile one block.
//  * Lanes read the K they take, 4 t + lane / 16.  The loop over stages is unrolled until buffers
//    and fragment sets are back, so that LDS addresses are constants (550 -> 510 us).
#include "lds_stage.h"
#include "sp2_control.h"
#include "sp2_internal.h"

namespace sp2 {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// BT x BT output tile, four waves with a B x B part each (B = BT / 2: 2 x 2 blocks of 16, or one), ST
// LDS stages of 2 BT rows (panels I and J) of ROW bytes.
template <int BT, int ST, int ROW = 128>
struct F32Cfg {
    static constexpr int B = BT / 2, NT = 256;
    static constexpr int BK = ROW / 4;                   // floats per row per stage
    static constexpr int CH = ROW / 16;                  // 16-byte chunks per row
    static constexpr int RPB = 1024 / ROW;               // rows per 1 KB direct-load block
    static constexpr int ARR = BT * ROW;                 // bytes of one panel stage
    static constexpr int STAGE = 2 * ARR;
    static constexpr int BPR = BT / RPB;                 // 1 KB blocks per panel stage
    static constexpr int LPW = 2 * BPR / 4;              // direct loads per wave per stage
    static constexpr int LDS = ST * STAGE;
    static constexpr int STRIP = 1024 / BT;              // tile_of strip: 1024 columns
    static_assert(B == 32 || B == 16, "one or four 16 x 16 blocks per wave");
    static_assert(ROW == 128 || ROW == 256, "a line of the cache, or two");
    // chunk c of row r is stored at c ^ swz(r)
    static __device__ __forceinline__ int swz(int r) { return (ROW == 128 ? r >> 1 : r) & (CH - 1); }
};

// Output tile (I, J) of edge BT over all of K; t is the tile's slot in a.parts.  LEAD: the
// layer's control at its head (`lead`, lead_bytes of LDS at `dyn`).
template <int BT, int ST, int ROW = 128, bool LEAD = false>
__device__ __forceinline__ void f32_body(const SquareArgs& a, int I, int J, int t, unsigned char* __restrict__ lds,
                                         const LeadArgs* lead = nullptr, unsigned char* __restrict__ dyn = nullptr) {
    typedef F32Cfg<BT, ST, ROW> C;
    constexpr int LPW = C::LPW, VM = LPW * (ST - 1), B = C::B, MB = B / 16, kRow = ROW, kBK = C::BK;
    const int np = a.np;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const float* x = (const float*)a.x0;
    const unsigned char* src_a = (const unsigned char*)(x + (size_t)I * BT * np);
    const unsigned char* src_b = (const unsigned char*)(x + (size_t)J * BT * np);
    const int nsl = ((a.k_all ? np : a.n_real) + kBK - 1) / kBK;
    // direct load l of this wave: lane L fills bytes [16 L, 16 L + 16) of a 1 KB block:
    // panel row q * RPB + L / CH, physical chunk L % CH = logical chunk (L % CH) ^ swz(row)
    unsigned voff[LPW];
#pragma unroll
    for (int l = 0; l < LPW; ++l) {
        const int row = ((wave * LPW + l) % C::BPR) * C::RPB + lane / C::CH;
        voff[l] = (unsigned)row * (unsigned)np * 4u + (unsigned)(((lane & (C::CH - 1)) ^ C::swz(row)) << 4);
    }
    auto load_one = [&](int l, int buf, int ks) {
        const int j = wave * LPW + l;
        const int arr = j / C::BPR, qd = j % C::BPR;
        dma16s(voff[l], (arr ? src_b : src_a) + (size_t)ks * kRow,
               lds_addr(lds + buf * C::STAGE + arr * C::ARR + qd * 1024));
    };
    // A unit is UK indices of K: product s takes K UK g + 4 s + lane / 16.  A wave's next unit is
    // read from LDS behind the products of this one; with one block per wave (32-tiles) it takes
    // eight products to cover those reads.
    constexpr int UK = MB == 1 ? kBK / 2 : 8, UNITS = kBK / UK, SU = UK / 4, NM = SU * MB * MB;
    struct Frag {
        float a[SU][MB], b[SU][MB];
    };
    const int r16 = lane & 15, kq = (lane >> 4) << 2;
    auto frags = [&](int buf, int g, Frag& f) {
        const unsigned char* base = lds + buf * C::STAGE;
#pragma unroll
        for (int s = 0; s < SU; ++s)
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int ra = wm * B + 16 * m + r16, rb = wn * B + 16 * m + r16, c = SU * g + s;
                f.a[s][m] = *(const float*)(base + ra * kRow + ((c ^ C::swz(ra)) << 4) + kq);
                f.b[s][m] = *(const float*)(base + C::ARR + rb * kRow + ((c ^ C::swz(rb)) << 4) + kq);
            }
    };
    f32x4 acc[MB][MB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < MB; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.f;
    // the products of one unit, with (doit) the direct loads of stage ks into buffer buf behind them
    auto mma = [&](const Frag& f, int buf, int ks, bool doit) {
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int s = i / (MB * MB), m = (i / MB) % MB, n = i % MB;
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[s][m], f.b[s][n], acc[m][n], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (doit)
#pragma unroll
                for (int l = i; l < LPW; l += NM) load_one(l, buf, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int pro = nsl < ST ? nsl : ST;
    if (LEAD && wave == 0) lead_load(*lead, lds_addr(dyn));
    for (int q = 0; q < pro; ++q)
#pragma unroll
        for (int l = 0; l < LPW; ++l) load_one(l, q, q);
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
    Frag f[2];
    frags(0, 0, f[0]);
    // Stage st + ST refills the buffer of stage st among the last unit's products, once every wave
    // has read it.
    auto stage = [&](int st, int buf, int first) {   // buf = st % ST
#pragma unroll
        for (int u = 0; u + 1 < UNITS; ++u) {
            frags(buf, u + 1, f[(first + u + 1) & 1]);
            mma(f[(first + u) & 1], 0, 0, false);
        }
        if (st + 1 < nsl) {
            const int last = (st + ST - 1 < nsl - 1) ? st + ST - 1 : nsl - 1;
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<VM>((last - st - 1) * LPW);
            stage_barrier();
            frags((buf + 1) % ST, 0, f[(first + UNITS) & 1]);
            mma(f[(first + UNITS - 1) & 1], buf, st + ST, st + ST < nsl);
        } else {
            mma(f[(first + UNITS - 1) & 1], 0, 0, false);
        }
    };
    constexpr int R = ST % 2 ? 2 * ST : ST;   // stages after which buffers and fragment sets are back
    int st = 0;
    for (; st + R <= nsl; st += R)
#pragma unroll
        for (int k = 0; k < R; ++k) stage(st + k, k % ST, (k * UNITS) & 1);
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (st + k < nsl) stage(st + k, k % ST, (k * UNITS) & 1);

    // ------------------------------------------------------------------- epilogue
    if (!LEAD)
        for (int i = 0; i < 3; ++i) cf.f[i] = a.coef[i];
    const float alpha = cf.f[0], beta = cf.f[1], gamma = cf.f[2];
    float* so = (float*)a.s_out;
    const float* si = (const float*)a.s_in;
    const int ldo = a.ld_out, nv = a.n_valid;
    double tr = 0.0, fr = 0.0;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
#pragma unroll
        for (int n = 0; n < MB; ++n) {
            const int bi = I * BT + wm * B + 16 * m, bj = J * BT + wn * B + 16 * n;
            if (bi > bj) continue;   // below the diagonal
            const int col = bj + r16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = bi + kq + r;
                if (row > col) continue;
                const float xv = acc[m][n][r];
                float y = (beta != 0.f) ? alpha * xv + beta * si[(size_t)row * np + col] : alpha * xv;
                if (row == col && col < a.n_real) y += gamma;
                if (row < nv && col < nv) {
                    so[(size_t)row * ldo + col] = y;
                    if (row != col) so[(size_t)col * ldo + row] = y;
                }
                const double yd = (double)y;
                if (row == col) {
                    tr += yd;
                    fr += yd * yd;
                } else {
                    fr += 2.0 * yd * yd;
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
            for (int w = 0; w < 4; ++w) {
                s0 += red[2 * w];
                s1 += red[2 * w + 1];
            }
            st_agent(a.parts + 2 * t, s0);
            st_agent(a.parts + 2 * t + 1, s1);
        }
        if (!LEAD) tile_done<C::NT>(a, t, (double*)lds, s_done);
    }
}

typedef F32Cfg<64, 2> F32Main;

// Cut tile u of those behind `nmain` whole 64-tiles (blocks from nmain on).
template <int ROW>
__device__ __forceinline__ void f32_cut(const SquareArgs& a, int nmain, unsigned char* lds) {
    const int nsub = a.ntiles - nmain;
    const int u = xcd_tile_index(blockIdx.x - nmain, (nsub + 7) >> 3, nsub);
    if (u < 0) return;
    int I, J;
    tile_of(nmain + (u >> 2), a.T, F32Main::STRIP, &I, &J);
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
    f32_body<32, 2, ROW>(a, i, j, slot, lds);
}

// 64-tiles [0, nmain) whole (nmain a multiple of 8), the others as four 32-tiles each.
__global__ __launch_bounds__(256) void k_square_f32_mix(SquareArgs a, int nmain) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F32Main::LDS];
    int I, J;
    if ((int)blockIdx.x < nmain) {
        const int t = (blockIdx.x & 7) * (nmain >> 3) + (blockIdx.x >> 3);
        tile_of(t, a.T, F32Main::STRIP, &I, &J);
        f32_body<64, 2>(a, I, J, t, lds);
        return;
    }
    f32_cut<128>(a, nmain, lds);
}
// Every 64-tile cut, stages in rows of ROW bytes.
template <int ROW>
__global__ __launch_bounds__(256) void k_square_f32_cut(SquareArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F32Cfg<32, 2, ROW>::LDS];
    f32_cut<ROW>(a, 0, lds);
}

// All of a small problem's 64-tiles as four 32-tiles each, with leading control, in rows of 128
// or 256 bytes (see k_square_f64_lead).
template <int ROW>
__global__ __launch_bounds__(256) void k_square_f32_lead(SquareArgs a, LeadArgs lead) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];   // lead_bytes
    __shared__ __attribute__((aligned(16))) unsigned char lds[F32Cfg<32, 2, ROW>::LDS];
    const int u = xcd_tile_index(blockIdx.x, (a.ntiles + 7) >> 3, a.ntiles);
    if (u < 0) return;
    int I, J;
    tile_of(u >> 2, a.T, F32Main::STRIP, &I, &J);
    const int i = 2 * I + ((u >> 1) & 1), j = 2 * J + (u & 1);
    if (i > j) {   // below the diagonal: its mirror computes it
        if (threadIdx.x < 2) a.parts[2 * u + threadIdx.x] = 0.0;
        return;
    }
    f32_body<32, 2, ROW, true>(a, i, j, u, lds, &lead, dyn);
}

// grouped: block b computes the 64-tile that the tile map names for it (see TileRef)
__global__ __launch_bounds__(256) void k_square_f32_g(const SquareArgs* __restrict__ descs,
                                                      const TileRef* __restrict__ map, int per) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F32Main::LDS];
    const TileRef e = map[(blockIdx.x & 7) * per + (blockIdx.x >> 3)];
    if (e.problem < 0) return;
    const SquareArgs a = descs[e.problem];
    int I, J;
    tile_of(e.tile, a.T, F32Main::STRIP, &I, &J);
    f32_body<64, 2>(a, I, J, e.tile, lds);
}

}  // namespace

hipError_t launch_square_f32_mix(const SquareArgs& a, hipStream_t s) {
    int T, nmain, ntiles;
    square_mix_grid(64 * a.T, &T, &nmain, &ntiles);
    if (ntiles != a.ntiles || a.np % 64 || 64 * T > a.np) return hipErrorInvalidValue;
    const int nsub = ntiles - nmain;
    const dim3 grid(nmain + (nsub + 7) / 8 * 8);
    if (nmain > 0) hipLaunchKernelGGL(k_square_f32_mix, grid, dim3(256), 0, s, a, nmain);
    else if (few_cut_tiles(a.T)) hipLaunchKernelGGL(k_square_f32_cut<256>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_square_f32_cut<128>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_square_f32_lead(const SquareArgs& a, const LeadArgs& lead, hipStream_t s) {
    if (!square_leads(64 * a.T) || a.ntiles != 4 * ntiles_upper(a.T) || !a.parts) return hipErrorInvalidValue;
    const dim3 grid((a.ntiles + 7) / 8 * 8);
    if (few_cut_tiles(a.T)) hipLaunchKernelGGL(k_square_f32_lead<256>, grid, dim3(256), lead_bytes(lead), s, a, lead);
    else hipLaunchKernelGGL(k_square_f32_lead<128>, grid, dim3(256), lead_bytes(lead), s, a, lead);
    return hipGetLastError();
}

hipError_t launch_square_f32_g(const SquareArgs* descs, const TileRef* map, int per, hipStream_t s) {
    hipLaunchKernelGGL(k_square_f32_g, dim3(8 * per), dim3(256), 0, s, descs, map, per);
    return hipGetLastError();
}

}  // namespace sp2

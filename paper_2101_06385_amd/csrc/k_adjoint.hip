// One reverse layer of the differentiable generalized-SP2 network (gfx950).  With G =
// dL/dX_{k+1} (symmetric),
//     M = G X_k + X_k G,  G_k = W_k M + B_k G,
// and the FP64 tile partials of Tr G (= dL/dc_k), <G, X_k>_F (= dL/dB_k) and
// <M, X_k>_F / 2 = <G, X_k^2>_F (= dL/dW_k).
//
//  * FP32 operands on the FP32 matrix instructions: the adjoint can grow by up to a factor 2
//    per layer in the eigenbasis, which half-precision planes could not hold, and FP32 keeps
//    the gradients accurate.
//  * Bound: the matrix pipes (157.3 TFLOP/s).  Output tiles I <= J of the symmetric M (rows of a
//    symmetric matrix are its columns, so all four operands are K-contiguous row panels), cut
//    as in k_square_f32.hip: 64 x 64 tiles, several workgroups per CU, and the tiles beyond the
//    last whole round of one per CU as 32 x 32 ones.  Two MFMA chains per wave (G_I X_J^T and
//    X_I G_J^T).  The four panels (G_I, X_I, X_J, G_J) go into LDS with global_load_lds_dwordx4,
//    32 floats per row and stage, two stages.  One layer with its sums, against persistent
//    workgroups with a split-K tail (64-tiles up to n = 4096, 128-tiles above) and a launch for
//    the sums: n = 512 37 -> 12 us, 1400 74 -> 55 us, 2048 221 -> 161 us, 4096 1.30 -> 1.07 ms
//    (129 TFLOP/s).  Stages of 16 floats (four workgroups of 64-tiles per CU in place of two) took
//    6 % longer at n = 4096; cut tiles in the LDS of whole ones 10 % longer at n = 1000.
//  * One 16-byte read feeds four products of a fragment: a lane's K order is permuted, for A and
//    B alike.  Rows are XOR-swizzled in 16-byte chunks, so that 16 lanes hit distinct banks.
//  * The sums of the layer's partials ride in the next launch (its last workgroup), so a layer is
//    one launch.
#include "lds_stage.h"
#include "sp2_internal.h"

namespace sp2 {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 32;            // floats per row per stage
constexpr int kRow = kBK * 4;      // 128 bytes
constexpr int kRPB = 1024 / kRow;  // rows per 1 KB direct-load block (8)
constexpr int kCh = kRow / 16;     // 16-byte chunks per row

// chunk c of row r is stored at c ^ swz8(r)
__device__ inline int swz8(int r) { return (r >> 1) & 7; }

// BT x BT output tile, four waves with one B x B block each (B = BT / 2), two stages
template <int BT>
struct AdjCfg {
    static constexpr int B = BT / 2, ST = 2;
    static constexpr int ARR = BT * kRow;
    static constexpr int STAGE = 4 * ARR;
    static constexpr int BPR = BT / kRPB;     // 1 KB blocks per panel stage
    static constexpr int LPW = BPR;           // direct loads per wave per stage: wave w loads panel w
    static constexpr int LDS = ST * STAGE;
};

template <int B>
struct Mfma;
template <>
struct Mfma<32> {
    static constexpr int REGS = 16;
    typedef f32x16 Acc;
    static __device__ __forceinline__ Acc mma(float a, float b, const Acc& c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
};
template <>
struct Mfma<16> {
    static constexpr int REGS = 4;
    typedef f32x4 Acc;
    static __device__ __forceinline__ Acc mma(float a, float b, const Acc& c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + r; }
};

// Output tile (I, J) of edge BT; t is its slot in a.parts.
template <int BT>
__device__ __forceinline__ void adjoint_body(const AdjointArgs& a, int I, int J, int t, unsigned char* __restrict__ lds) {
    typedef AdjCfg<BT> C;
    constexpr int B = C::B, ST = C::ST, LPW = C::LPW, VM = LPW * (ST - 1);
    typedef Mfma<B> M;
    constexpr int UK = 4 * (64 / B);        // K per unit: one 16-byte read per lane and fragment
    constexpr int UNITS = kBK / UK;         // units per stage
    const int np = a.np;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int nsl = (a.n + kBK - 1) / kBK;   // G and X are zero beyond n
    // stage panels: 0 = G rows I, 1 = X rows I, 2 = X rows J, 3 = G rows J
    const float* panel = (wave == 0 || wave == 3 ? a.g : a.x) + (size_t)(wave < 2 ? I : J) * BT * np;
    unsigned voff[LPW];
#pragma unroll
    for (int l = 0; l < LPW; ++l) {
        const int row = l * kRPB + lane / kCh;
        voff[l] = (unsigned)row * (unsigned)np * 4u + (unsigned)(((lane & (kCh - 1)) ^ swz8(row)) << 4);
    }
    auto load_one = [&](int l, int buf, int ks) {
        dma16s(voff[l], (const unsigned char*)panel + (size_t)ks * kRow,
               lds_addr(lds + buf * C::STAGE + wave * C::ARR + l * 1024));
    };
    struct Frags {
        f32x4 gi, xi, xj, gj;
    };
    const int ra = wm * B + (lane & (B - 1)), rb = wn * B + (lane & (B - 1)), kc = lane / B;
    auto frags = [&](int buf, int u, Frags& f) {
        const unsigned char* base = lds + buf * C::STAGE;
        const int c = u * (64 / B) + kc;
        const int oa = ra * kRow + ((c ^ swz8(ra)) << 4), ob = rb * kRow + ((c ^ swz8(rb)) << 4);
        f.gi = *(const f32x4*)(base + oa);
        f.xi = *(const f32x4*)(base + C::ARR + oa);
        f.xj = *(const f32x4*)(base + 2 * C::ARR + ob);
        f.gj = *(const f32x4*)(base + 3 * C::ARR + ob);
    };
    typename M::Acc acc0, acc1;
#pragma unroll
    for (int r = 0; r < M::REGS; ++r) acc0[r] = acc1[r] = 0.f;
    // the eight products of one unit, with (doit) the direct loads of stage ks into buffer buf
    // behind them
    auto mma = [&](const Frags& f, int buf, int ks, bool doit) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s & 1) acc1 = M::mma(f.xi[s >> 1], f.gj[s >> 1], acc1);
            else acc0 = M::mma(f.gi[s >> 1], f.xj[s >> 1], acc0);
            __builtin_amdgcn_sched_barrier(0);
            if (doit)
#pragma unroll
                for (int l = s; l < LPW; l += 8) load_one(l, buf, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int pro = nsl < ST ? nsl : ST;
    for (int q = 0; q < pro; ++q)
#pragma unroll
        for (int l = 0; l < LPW; ++l) load_one(l, q, q);
    wait_vm<VM>((pro - 1) * LPW);
    __syncthreads();
    Frags f[2];
    frags(0, 0, f[0]);
    // units alternate between two fragment sets; stage st + ST refills the buffer of stage st
    // among the last unit's products, once every wave has read it
    auto stage = [&](int st, int first) {
        const int buf = st % ST;
#pragma unroll
        for (int u = 0; u + 1 < UNITS; ++u) {
            frags(buf, u + 1, f[(first + u + 1) & 1]);
            mma(f[(first + u) & 1], 0, 0, false);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (st + 1 < nsl) {
            const int last = (st + ST - 1 < nsl - 1) ? st + ST - 1 : nsl - 1;
            wait_vm<VM>((last - st - 1) * LPW);
            stage_barrier();
            frags((st + 1) % ST, 0, f[(first + UNITS) & 1]);
            mma(f[(first + UNITS - 1) & 1], buf, st + ST, st + ST < nsl);
        } else {
            mma(f[(first + UNITS - 1) & 1], 0, 0, false);
        }
    };
    int st = 0;
    for (; st + 1 < nsl; st += 2) {
        stage(st, 0);
        stage(st + 1, UNITS & 1);
    }
    if (st < nsl) stage(st, 0);
#pragma unroll
    for (int r = 0; r < M::REGS; ++r) acc0[r] += acc1[r];

    // G_k = W M + B G over row <= col, mirrored; FP64 partials
    const float wk = a.coef[0], bk = a.coef[1];
    const int col = J * BT + wn * B + (lane & (B - 1));
    const int bi = I * BT + wm * B, bj = J * BT + wn * B;
    double p_tr = 0.0, p_gx = 0.0, p_mx = 0.0;
    if (bi <= bj) {
        const bool diag = bi == bj;
#pragma unroll
        for (int r4 = 0; r4 < M::REGS; r4 += 4) {
            f32x4 gn;
            const int row0 = bi + M::row(r4, lane);   // rows row0 .. row0 + 3
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = row0 + e;
                const size_t off = (size_t)row * np + col;
                const float mv = acc0[r4 + e], gv = a.g[off], xv = a.x[off];
                gn[e] = fmaf(wk, mv, bk * gv);
                if (diag && row > col) continue;
                a.g_out[off] = gn[e];
                if (diag && row != col) a.g_out[(size_t)col * np + row] = gn[e];
                const double wgt = (row == col) ? 1.0 : 2.0;
                if (row == col) p_tr += (double)gv;
                p_gx += wgt * (double)gv * (double)xv;
                p_mx += 0.5 * wgt * (double)mv * (double)xv;
            }
            if (!diag) *(f32x4*)(a.g_out + (size_t)col * np + row0) = gn;
        }
    }
    p_tr = wave_sum(p_tr);
    p_gx = wave_sum(p_gx);
    p_mx = wave_sum(p_mx);
    double* red = (double*)lds;   // the stages' LDS, once every wave has left them
    __syncthreads();
    if (lane == 0) {
        red[3 * wave + 0] = p_tr;
        red[3 * wave + 1] = p_gx;
        red[3 * wave + 2] = p_mx;
    }
    __syncthreads();
    if (tid < 3) a.parts[3 * t + tid] = red[tid] + red[3 + tid] + red[6 + tid] + red[9 + tid];
}

// dc = sum of the Tr G partials, dB of <G, X>, dW of <G, X^2>, in fixed order
__device__ __forceinline__ void reduce3(const double* __restrict__ parts, int nparts, float* dw, float* db, float* dc,
                                        double* sh /* 3 x 256 */) {
    const int t = threadIdx.x;
    double v[3] = {0.0, 0.0, 0.0};
    for (int i = t; i < nparts; i += 256)
        for (int c = 0; c < 3; ++c) v[c] += parts[3 * i + c];
    for (int c = 0; c < 3; ++c) sh[256 * c + t] = v[c];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w)
            for (int c = 0; c < 3; ++c) sh[256 * c + t] += sh[256 * c + t + w];
        __syncthreads();
    }
    if (t == 0) {
        *dc = (float)sh[0];
        *db = (float)sh[256];
        *dw = (float)sh[512];
    }
}

// 64-tiles [0, nmain) whole (CUT: none), the others as four 32-tiles each; the last block sums
// the partials of the layer before (prev, null at the first).
template <bool CUT>
__global__ __launch_bounds__(256) void k_adjoint(AdjointArgs a, int nmain, AdjointSums prev) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[AdjCfg<CUT ? 32 : 64>::LDS];
    constexpr int STRIP = 1024 / 64;
    if (blockIdx.x == gridDim.x - 1) {
        if (prev.parts) reduce3(prev.parts, a.ntiles, prev.dw, prev.db, prev.dc, (double*)lds);
        return;
    }
    int I, J;
    if (!CUT && (int)blockIdx.x < nmain) {
        const int t = (blockIdx.x & 7) * (nmain >> 3) + (blockIdx.x >> 3);
        tile_of(t, a.T, STRIP, &I, &J);
        adjoint_body<CUT ? 32 : 64>(a, I, J, t, lds);
        return;
    }
    const int nsub = a.ntiles - nmain;
    const int u = xcd_tile_index(blockIdx.x - nmain, (nsub + 7) >> 3, nsub);
    if (u < 0) return;
    tile_of(nmain + (u >> 2), a.T, STRIP, &I, &J);
    const int i = 2 * I + ((u >> 1) & 1), j = 2 * J + (u & 1), slot = nmain + u;
    if (i > j) {   // below the diagonal: its mirror computes it
        if (threadIdx.x < 3) a.parts[3 * slot + threadIdx.x] = 0.0;
        return;
    }
    adjoint_body<32>(a, i, j, slot, lds);
}

__global__ __launch_bounds__(256) void k_reduce3(AdjointSums p, int nparts) {
    __shared__ double sh[3 * 256];
    reduce3(p.parts, nparts, p.dw, p.db, p.dc, sh);
}

}  // namespace

hipError_t launch_adjoint(const AdjointArgs& a, const AdjointSums& prev, hipStream_t s) {
    int T, nmain, ntiles;
    square_mix_grid(64 * a.T, &T, &nmain, &ntiles);
    if (ntiles != a.ntiles || a.np % 64 || 64 * T > a.np || a.n > 64 * T) return hipErrorInvalidValue;
    const int nsub = ntiles - nmain;
    const dim3 grid(nmain + (nsub + 7) / 8 * 8 + 1);
    if (nmain == 0) hipLaunchKernelGGL(k_adjoint<true>, grid, dim3(256), 0, s, a, nmain, prev);
    else hipLaunchKernelGGL(k_adjoint<false>, grid, dim3(256), 0, s, a, nmain, prev);
    return hipGetLastError();
}

hipError_t launch_reduce3(const AdjointSums& p, int nparts, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce3, dim3(1), dim3(256), 0, s, p, nparts);
    return hipGetLastError();
}

}  // namespace sp2

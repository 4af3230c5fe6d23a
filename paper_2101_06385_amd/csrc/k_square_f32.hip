// FP32 squaring layer Y = alpha X^2 + beta X + gamma I (gfx950), for the FP32 mode, the FP32
// network and single FP32 layers.  Upper-triangle output tiles, mirrored on store.
//
//  * Bound: the matrix pipes (157.3 TFLOP/s).  As for the FP64 layers (k_square_f64.hip),
//    several independent workgroups of 4 waves per CU keep them busy: 64 x 64 tiles, two 16 KB
//    stages of 32 floats per row (one 128-byte line) filled by global_load_lds_dwordx4, the
//    tiles beyond the last whole round of one per CU cut into 32 x 32 ones.  The launch keeps
//    every CU at four workgroups to the end; the clock (1.8 - 2.1 GHz under this load) and the
//    stages' LDS traffic take the rest.  One layer with its control, against the register-staged
//    128 x 128 (64 x 64 up to n = 512) workgroups and control launch used before: n = 256 15 ->
//    8.1 us, 777 65 -> 18 us, 1300 113 -> 37 us, 2112 167 -> 100 us, 4096 773 -> 610 us
//    (113 TFLOP/s), 5000 1190 -> 1116 us.
//  * Each element is the chain of fused multiply-adds over ascending K, whichever instruction
//    computes it, so the tiling changes no bit: a 64-tile's waves hold one 32 x 32 block each
//    (v_mfma_f32_32x32x2f32), a 32-tile's one 16 x 16 block (v_mfma_f32_16x16x4f32).
//  * Lanes read the K they take, 2 t + lane / 32 or 4 t + lane / 16, two per ds_read2_b32.  (One
//    16-byte read per lane and v_permlane32_swap to sort it took 660 us at n = 4096; four stages
//    for the 32-tiles 56 us at n = 1300, where fewer workgroups then fit a CU.)
#include "sp2_control.h"
#include "sp2_internal.h"

namespace sp2 {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 32;            // floats per row per stage
constexpr int kRow = kBK * 4;      // 128 bytes
constexpr int kRPB = 1024 / kRow;  // rows per 1 KB direct-load block (8)

// BT x BT output tile, four waves with one B x B block each (B = BT / 2), ST LDS stages of
// 2 BT rows (panels I and J).
template <int BT, int ST>
struct F32Cfg {
    static constexpr int B = BT / 2, NT = 256;
    static constexpr int ARR = BT * kRow;                // bytes of one panel stage
    static constexpr int STAGE = 2 * ARR;
    static constexpr int BPR = BT / kRPB;                // 1 KB blocks per panel stage
    static constexpr int LPW = 2 * BPR / 4;              // direct loads per wave per stage
    static constexpr int LDS = ST * STAGE;
    static constexpr int STRIP = 1024 / BT;              // tile_of strip: 1024 columns
    static_assert(B == 32 || B == 16, "one MFMA block per wave");
    static_assert(LPW * (ST - 1) <= 24, "vmcnt range of wait_vm");
};

__device__ inline int swz8(int r) { return (r >> 1) & 7; }

typedef __attribute__((address_space(3))) unsigned char lds_byte;
__device__ __forceinline__ unsigned lds_addr(const unsigned char* p) {
    return (unsigned)(uintptr_t)(const lds_byte*)p;
}
// wave-uniform base in SGPRs and a 32-bit per-lane byte offset
__device__ __forceinline__ void dma16s(unsigned voff, const void* sbase, unsigned lds_base) {
    asm volatile(
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(voff), "s"(sbase), "s"(lds_base)
        : "memory", "m0");
}

#define SP2_VMCNT(n) asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory")
// waits until at most n (rounded down to an available immediate) vector-memory
// instructions of this wave are outstanding
__device__ __forceinline__ void wait_vm(int n) {
    if (n >= 24) SP2_VMCNT(24);
    else if (n >= 16) SP2_VMCNT(16);
    else if (n >= 12) SP2_VMCNT(12);
    else if (n >= 8) SP2_VMCNT(8);
    else if (n >= 6) SP2_VMCNT(6);
    else if (n >= 4) SP2_VMCNT(4);
    else if (n >= 2) SP2_VMCNT(2);
    else SP2_VMCNT(0);
}
#undef SP2_VMCNT

__device__ inline double wsum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// One wave's B x B block.  A unit is 8 K indices; p(s), s < STEPS, is what a lane gives to the
// unit's product s.
template <int B>
struct Block;
template <>
struct Block<32> {
    static constexpr int REGS = 16, STEPS = 4;
    typedef f32x16 Acc;
    struct Frag {
        float v[4];
        __device__ __forceinline__ void load(const unsigned char* base, int row, int g, int lane) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                v[s] = *(const float*)(base + row * kRow + (((2 * g + (s >> 1)) ^ swz8(row)) << 4) + ((s & 1) << 3) +
                                       ((lane >> 5) << 2));
        }
        __device__ __forceinline__ float p(int s) const { return v[s]; }
    };
    static __device__ __forceinline__ Acc mma(float a, float b, const Acc& c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
};
template <>
struct Block<16> {
    static constexpr int REGS = 4, STEPS = 2;
    typedef f32x4 Acc;
    struct Frag {
        float v[2];
        __device__ __forceinline__ void load(const unsigned char* base, int row, int g, int lane) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
                v[s] = *(const float*)(base + row * kRow + (((2 * g + s) ^ swz8(row)) << 4) + ((lane >> 4) << 2));
        }
        __device__ __forceinline__ float p(int s) const { return v[s]; }
    };
    static __device__ __forceinline__ Acc mma(float a, float b, const Acc& c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + r; }
};

// Output tile (I, J) of edge BT over all of K; t is the tile's slot in a.parts.  LEAD: the
// layer's control at its head (`lead`, lead_bytes of LDS at `dyn`).
template <int BT, int ST, bool LEAD = false>
__device__ __forceinline__ void f32_body(const SquareArgs& a, int I, int J, int t, unsigned char* __restrict__ lds,
                                         const LeadArgs* lead = nullptr, unsigned char* __restrict__ dyn = nullptr) {
    typedef F32Cfg<BT, ST> C;
    typedef Block<C::B> M;
    typedef typename M::Frag Frag;
    constexpr int LPW = C::LPW, B = C::B;
    const int np = a.np;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const float* x = (const float*)a.x0;
    const unsigned char* src_a = (const unsigned char*)(x + (size_t)I * BT * np);
    const unsigned char* src_b = (const unsigned char*)(x + (size_t)J * BT * np);
    const int nsl = ((a.k_all ? np : a.n_real) + kBK - 1) / kBK;
    // direct load l of this wave: lane L fills bytes [16 L, 16 L + 16) of a 1 KB block:
    // panel row q * 8 + L / 8, physical chunk L % 8 = logical chunk (L % 8) ^ swz8(row)
    unsigned voff[LPW];
#pragma unroll
    for (int l = 0; l < LPW; ++l) {
        const int row = ((wave * LPW + l) % C::BPR) * kRPB + (lane >> 3);
        voff[l] = (unsigned)row * (unsigned)np * 4u + (unsigned)(((lane & 7) ^ swz8(row)) << 4);
    }
    auto load_one = [&](int l, int buf, int ks) {
        const int j = wave * LPW + l;
        const int arr = j / C::BPR, qd = j % C::BPR;
        dma16s(voff[l], (arr ? src_b : src_a) + (size_t)ks * kRow,
               lds_addr(lds + buf * C::STAGE + arr * C::ARR + qd * 1024));
    };
    auto frags = [&](int buf, int g, Frag& fa, Frag& fb) {
        const unsigned char* base = lds + buf * C::STAGE;
        fa.load(base, wm * B + (lane & (B - 1)), g, lane);
        fb.load(base + C::ARR, wn * B + (lane & (B - 1)), g, lane);
    };
    typename M::Acc acc;
#pragma unroll
    for (int r = 0; r < M::REGS; ++r) acc[r] = 0.f;
    // the products of one unit, with (doit) the direct loads of stage ks into buffer buf behind them
    auto mma = [&](Frag fa, Frag fb, int buf, int ks, bool doit) {
#pragma unroll
        for (int s = 0; s < M::STEPS; ++s) {
            acc = M::mma(fa.p(s), fb.p(s), acc);
            __builtin_amdgcn_sched_barrier(0);
            if (doit)
#pragma unroll
                for (int l = s; l < LPW; l += M::STEPS) load_one(l, buf, ks);
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
        wait_vm(0);
        return;
    }
    wait_vm((pro - 1) * LPW);
    __syncthreads();
    Coefs cf;
    if (LEAD && !lead_finish(*lead, dyn, blockIdx.x == 0 && wave == 0, &cf)) {   // Alg. 1 has stopped
        wait_vm(0);
        return;
    }
    Frag pa, pb, qa, qb;
    frags(0, 0, pa, pb);
    // units alternate between fragment sets P and Q, four per stage.  Stage st + ST refills the
    // buffer of stage st among the last unit's products, once every wave has read it.
    for (int st = 0; st < nsl; ++st) {
        const int buf = st % ST;
        frags(buf, 1, qa, qb);
        mma(pa, pb, 0, 0, false);
        frags(buf, 2, pa, pb);
        mma(qa, qb, 0, 0, false);
        frags(buf, 3, qa, qb);
        mma(pa, pb, 0, 0, false);
        if (st + 1 < nsl) {
            const int last = (st + ST - 1 < nsl - 1) ? st + ST - 1 : nsl - 1;
            __builtin_amdgcn_sched_barrier(0);
            wait_vm((last - st - 1) * LPW);
            __syncthreads();
            frags((st + 1) % ST, 0, pa, pb);
            mma(qa, qb, buf, st + ST, st + ST < nsl);
        } else {
            mma(qa, qb, 0, 0, false);
        }
    }

    // ------------------------------------------------------------------- epilogue
    if (!LEAD)
        for (int i = 0; i < 3; ++i) cf.f[i] = a.coef[i];
    const float alpha = cf.f[0], beta = cf.f[1], gamma = cf.f[2];
    float* so = (float*)a.s_out;
    const float* si = (const float*)a.s_in;
    const int ldo = a.ld_out, nv = a.n_valid;
    const int col = J * BT + wn * B + (lane & (B - 1));
    double tr = 0.0, fr = 0.0;
    if (I * BT + wm * B <= J * BT + wn * B) {   // not wholly below the diagonal
#pragma unroll
        for (int r = 0; r < M::REGS; ++r) {
            const int row = I * BT + wm * B + M::row(r, lane);
            if (row > col) continue;
            const float xv = acc[r];
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
    if (a.parts) {
        // in the stages, which every wave has left: the LDS of a workgroup stays a fifth of a CU's
        double* red = (double*)(lds + C::LDS - 256);
        int* s_done = (int*)(lds + C::LDS - 64);
        tr = wsum(tr);
        fr = wsum(fr);
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

// 64-tiles [0, nmain) whole (nmain a multiple of 8), the others as four 32-tiles each.
typedef F32Cfg<64, 2> F32Main;
typedef F32Cfg<32, 2> F32Sub;
__global__ __launch_bounds__(256) void k_square_f32_mix(SquareArgs a, int nmain) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[F32Main::LDS];
    int I, J;
    if ((int)blockIdx.x < nmain) {
        const int t = (blockIdx.x & 7) * (nmain >> 3) + (blockIdx.x >> 3);
        tile_of(t, a.T, F32Main::STRIP, &I, &J);
        f32_body<64, 2>(a, I, J, t, lds);
        return;
    }
    const int nsub = a.ntiles - nmain;
    const int u = xcd_tile_index(blockIdx.x - nmain, (nsub + 7) >> 3, nsub);
    if (u < 0) return;
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
    f32_body<32, 2>(a, i, j, slot, lds);
}

// All of a small problem's 64-tiles as four 32-tiles each, with leading control (see
// k_square_f64_lead).
__global__ __launch_bounds__(256) void k_square_f32_lead(SquareArgs a, LeadArgs lead) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];   // lead_bytes
    __shared__ __attribute__((aligned(16))) unsigned char lds[F32Sub::LDS];
    const int u = xcd_tile_index(blockIdx.x, (a.ntiles + 7) >> 3, a.ntiles);
    if (u < 0) return;
    int I, J;
    tile_of(u >> 2, a.T, F32Main::STRIP, &I, &J);
    const int i = 2 * I + ((u >> 1) & 1), j = 2 * J + (u & 1);
    if (i > j) {   // below the diagonal: its mirror computes it
        if (threadIdx.x < 2) a.parts[2 * u + threadIdx.x] = 0.0;
        return;
    }
    f32_body<32, 2, true>(a, i, j, u, lds, &lead, dyn);
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
    hipLaunchKernelGGL(k_square_f32_mix, dim3(nmain + (nsub + 7) / 8 * 8), dim3(256), 0, s, a, nmain);
    return hipGetLastError();
}

hipError_t launch_square_f32_lead(const SquareArgs& a, const LeadArgs& lead, hipStream_t s) {
    if (!square_leads(64 * a.T) || a.ntiles != 4 * ntiles_upper(a.T) || !a.parts) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_square_f32_lead, dim3((a.ntiles + 7) / 8 * 8), dim3(256), lead_bytes(lead), s, a, lead);
    return hipGetLastError();
}

hipError_t launch_square_f32_g(const SquareArgs* descs, const TileRef* map, int per, hipStream_t s) {
    hipLaunchKernelGGL(k_square_f32_g, dim3(8 * per), dim3(256), 0, s, descs, map, per);
    return hipGetLastError();
}

}  // namespace sp2

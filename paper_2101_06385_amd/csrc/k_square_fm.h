// Split (dual half-precision) squaring layer of small and medium problems (gfx950), n_p < 3072.
//
// Computes the same layer as k_square_dp (Y = alpha X^2 + beta X + gamma I from the planes
// X0, X1, X0 X0 + X0 X1 + X1 X0 of Eq. Square over the upper triangle), with the same chain of
// products per element, hence the same bits.  Such a layer is bound by latency (dependent
// trips to memory, launches), not by the matrix pipes or the LDS (counters at n = 777: 91 busy CUs,
// matrix pipes busy 0.20 and LDS reads under way 0.18 of their cycles, waves waiting for memory
// counters or barriers 0.49):
//
//  * Fragment-major planes: a plane is stored as 32-row x 16-column blocks of 1 KB in the
//    order in which v_mfma_f32_32x32x16 takes them (lane l = row + 32 (k / 8), 8 halves each),
//    K-consecutive per 32 rows.  A fragment is one 1 KB load, a 1 KB run of LDS without bank
//    conflicts, or one coalesced load into registers.
//  * The state S is kept as 32 x 32 blocks of the upper triangle in accumulator order: 1 KB
//    loads and stores, no mirrored copy (k_select_fm expands it).
//  * Layers of the network (NET) keep S row-major, which their adjoint reads, and take their
//    coefficients from memory: no control and no sums.
//  * Leading control: every workgroup derives its layer's sigma_n from the partial sums of the
//    previous launch behind its first products (the same fixed-order sums in every workgroup);
//    workgroup 0 records it.  No control launch, no arrival counter, no wait for stores at the
//    end of a launch.  The state's hot block and the partial sums are double buffered, since a
//    late workgroup may still read what an early one would overwrite.
//
// Measured, one layer of a solve with its control, against the register-staged or 128-tile
// per-tile kernel with control launches: n = 65 6.9 against 11.2 us, 400 8.8 against 16.1, 777
// 11.8 against 24, 1000 13.4 against 24.8, 1400 18 against 30, 2000 38 against 66, 2100 41
// against 55 us.  A layer of the network, against k_square_dp on 128-tiles: n = 512 8 against 27,
// 1400 16 against 39, 2048 38 against 50, 2900 102 against 122 us.  The clock holds about 1.65 GHz.
// Tried and not kept: one wave per 32 x 32 block (equal up to n = 550, half as fast at 1700), two
// waves of 64 x 32 (10-20 % slower below n = 2000; not timed above, where the one-wave kernel
// serves), the tiles beyond a whole round of one per CU cut into 32 x 32 blocks (40 against 28 us at
// n = 1700), all fragments in registers (their loads return 16 bytes per clock and wave: 512 cycles
// per unit for 384 of products).
#pragma once

#include "lds_stage.h"
#include "sp2_control.h"
#include "sp2_internal.h"

#include <type_traits>

namespace sp2 {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T16>
struct FmOps;
template <>
struct FmOps<_Float16> {
    typedef _Float16 vec8 __attribute__((ext_vector_type(8)));
    typedef _Float16 vec4 __attribute__((ext_vector_type(4)));
    __device__ static inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
template <>
struct FmOps<__bf16> {
    typedef __bf16 vec8 __attribute__((ext_vector_type(8)));
    typedef __bf16 vec4 __attribute__((ext_vector_type(4)));
    __device__ static inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

// 16 bytes per lane from sbase + voff straight to LDS bytes [lds_base + off + 16 lane, + 16)
__device__ __forceinline__ void fm_dma16(unsigned voff, const void* sbase, unsigned lds_base, unsigned off) {
    asm volatile(
        "s_add_u32 m0, %2, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(voff), "s"(sbase), "s"(lds_base), "s"(off)
        : "memory", "m0", "scc");
}

template <int B, int E, typename F>
__device__ __forceinline__ void fm_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        fm_for<B + 1, E>(f);
    }
}

// Epilogue of one 32 x 32 block (bi, bj), bi <= bj, of a wave: Y = alpha X^2 + beta X + gamma I
// from the products in `acc` and the block's S, stored as a block of S, split into the planes
// at (bi, bj) and (bj, bi); adds the block's trace and square sums per lane.  tr: kFmTranspose
// bytes of LDS of this wave.
// NET (layers of the network): S is row-major, both triangles, and there are no sums.
constexpr int kFmTH = 40;                           // transpose pitch in halves (80 bytes: 16-byte aligned rows)
constexpr int kFmTranspose = 2 * 32 * kFmTH * 2;
template <typename T16, bool NET>
__device__ __forceinline__ void fm_store_block(const FmArgs& a, const Coefs& cf, int bi, int bj, const f32x16& acc,
                                               const f32x4 (&s4)[4], size_t ps, T16* __restrict__ tr0, double* tr,
                                               double* fr) {
    typedef typename FmOps<T16>::vec8 vec8;
    typedef typename FmOps<T16>::vec4 vec4;
    constexpr int TH = kFmTH;
    const float alpha = cf.f[0], beta = cf.f[1], gamma = cf.f[2], osc = a.out_scale, isc = a.in_scale;
    T16* tr1 = tr0 + 32 * TH;
    T16* p0 = (T16*)a.p0_out;
    T16* p1 = (T16*)a.p1_out;
    const int lane = threadIdx.x & 63, c = lane & 31, hi = lane >> 5;
    f32x4* so = (f32x4*)(a.s_out + ((size_t)bi * a.sb + bj) * 1024) + lane;
    float* row0 = a.s_out + (size_t)(32 * bi) * a.ld + 32 * bj + c;            // NET: this lane's column
    float* col0 = a.s_out + (size_t)(32 * bj + c) * a.ld + 32 * bi + 4 * hi;   // and its mirror
    auto block = [&](auto diag_) {
        constexpr bool diag = decltype(diag_)::value;
        fm_for<0, 4>([&](auto g) {
            f32x4 y4;
            vec4 h0, h1;
            fm_for<0, 4>([&](auto e) {
                const int r = 8 * g + 4 * hi + e;
                const float x = acc[4 * g + e] * osc;
                float y = (beta != 0.f) ? fmaf(alpha, x, beta * s4[g][(int)e]) : alpha * x;
                if (diag && r == c && 32 * bj + c < a.n_real) y += gamma;
                y4[(int)e] = y;
                const float ys = y * isc;
                const T16 a0 = (T16)ys;
                h0[(int)e] = a0;
                h1[(int)e] = (T16)(ys - (float)a0);
                if (NET) {
                    if (!diag || r <= c) row0[(size_t)r * a.ld] = y;
                    if (diag && r < c) col0[8 * g + e] = y;
                } else if (!diag || r < c) {
                    *fr += 2.0 * (double)y * (double)y;
                } else if (r == c) {
                    *tr += (double)y;
                    *fr += (double)y * (double)y;
                }
            });
            if (!NET) so[64 * g] = y4;
            else if (!diag) *(f32x4*)(col0 + 8 * g) = y4;
            // block (bj, bi) of the planes: rows are this block's columns
            if (!diag) {
                const size_t o = (size_t)bj * ps + (size_t)(2 * bi + (g >> 1)) * 512 + (c + 32 * (g & 1)) * 8 + 4 * hi;
                *(vec4*)(p0 + o) = h0;
                *(vec4*)(p1 + o) = h1;
            }
            // rows of block (bi, bj) through LDS; a diagonal block keeps its upper part and
            // mirrors it
            fm_for<0, 4>([&](auto e) {
                const int r = 8 * g + 4 * hi + e;
                if (!diag || r <= c) {
                    tr0[r * TH + c] = h0[(int)e];
                    tr1[r * TH + c] = h1[(int)e];
                }
                if (diag && r < c) {
                    tr0[c * TH + r] = h0[(int)e];
                    tr1[c * TH + r] = h1[(int)e];
                }
            });
        });
    };
    if (bi == bj) block(std::true_type{});
    else block(std::false_type{});
    // one wave: its LDS operations are in order
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fm_for<0, 2>([&](auto k) {   // unit 2 bj + k: lane = row + 32 (column / 8)
        const size_t o = (size_t)bi * ps + (size_t)(2 * bj + k) * 512 + lane * 8;
        *(vec8*)(p0 + o) = *(const vec8*)(tr0 + c * TH + 16 * k + 8 * hi);
        *(vec8*)(p1 + o) = *(const vec8*)(tr1 + c * TH + 16 * k + 8 * hi);
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// This wave's S of block (bi, bj) for the beta term.
template <bool NET>
__device__ __forceinline__ void fm_load_block(const FmArgs& a, int bi, int bj, f32x4 (&s4)[4]) {
    const int lane = threadIdx.x & 63;
    fm_for<0, 4>([&](auto g) {
        if (NET) s4[g] = *(const f32x4*)(a.s_in + (size_t)(32 * bj + (lane & 31)) * a.ld + 32 * bi + 8 * g + 4 * (lane >> 5));
        else s4[g] = ((const f32x4*)(a.s_in + ((size_t)bi * a.sb + bj) * 1024))[64 * g + lane];
    });
}
// NET: a block of a 64-tile beyond the data holds zeros (the adjoint layers read it)
__device__ __forceinline__ void fm_zero_block(const FmArgs& a, int bi, int bj) {
    const int lane = threadIdx.x & 63, c = lane & 31, hi = lane >> 5;
    for (int r = 0; r < 16; ++r) {
        a.s_out[(size_t)(32 * bi + 2 * r + hi) * a.ld + 32 * bj + c] = 0.f;
        if (bi != bj) a.s_out[(size_t)(32 * bj + 2 * r + hi) * a.ld + 32 * bi + c] = 0.f;
    }
}

// One wave per workgroup, a 64 x 64 tile of Y (2 x 2 blocks): for problems with more 64-tiles
// than the 4-wave workgroups' LDS lets a CU hold.  The last tile runs the next layer's control
// (the sums of so many tiles would take every wave longer than that).  A wave's loads return 16 bytes per clock
// into registers and 32 from LDS (measured: a ring of registers alone runs at 512 cycles per
// unit, whatever its depth, against 384 of the unit's 12 products), so the A fragments come
// straight into registers, DA units ahead, and the B fragments through a ring of R units in
// LDS; reads and loads go between the products.
// Bound: the chain of products of a wave.  n = 2100 (counters): 561 waves, four to a CU, so 140 CUs work;
// their matrix pipes are busy 0.69 and their LDS reads under way 0.14 of the cycles, without bank
// conflicts.
template <typename T16, int R, int DA, int ORD, bool NET = false>
__global__ __launch_bounds__(64) void k_square_fm1(FmArgs a) {
    typedef FmOps<T16> Ops;
    typedef typename Ops::vec8 vec8;
    static_assert((R & (R - 1)) == 0 && R >= 2 && R % 2 == 0 && DA % 2 == 0, "slot index by mask, pairs of units");
    constexpr int SLOT = 4 * 1024;
    static_assert(R * SLOT >= kFmTranspose && R * SLOT >= kControlLds * 8, "transpose and control fit the ring");
    __shared__ __attribute__((aligned(16))) unsigned char ring[R * SLOT];
    __shared__ int s_done;
    const int lane = threadIdx.x;
    const int t = xcd_tile_index(blockIdx.x, a.per, a.ntiles);
    if (t < 0) return;
    int I, J;
    tile_of(t, a.T, 8, &I, &J);
    DevState* st = (DevState*)a.ctl;
    const int KU = a.ku;
    const size_t ps = (size_t)a.pstride * 512;
    const char* abase[4];   // X0 of rows 2 I, 2 I + 1, X1 of the same
    const char* bbase[4];
    fm_for<0, 4>([&](auto k) {
        const T16* pl = (const T16*)(k >> 1 ? a.x1 : a.x0);
        abase[k] = (const char*)(pl + (size_t)(2 * I + (k & 1)) * ps);
        bbase[k] = (const char*)(pl + (size_t)(2 * J + (k & 1)) * ps);
    });
    const unsigned lo = lane * 16, ring0 = lds_addr(ring);
    auto off = [&](int u) { return lo + (unsigned)(u < KU ? u : KU - 1) * 1024u; };   // past the end: the last unit
    vec8 fa[DA][4], fb[2][4];
    auto load_a = [&](auto d, auto k, unsigned o) { fa[d][k] = *(const vec8*)(abase[k] + o); };
    auto load_b = [&](auto k, int u, unsigned o) { fm_dma16(o, bbase[k], ring0 + (u & (R - 1)) * SLOT, k * 1024); };
    auto read_b = [&](auto s, auto k, int u) { fb[s][k] = *(const vec8*)(ring + (u & (R - 1)) * SLOT + k * 1024 + lo); };
    f32x16 acc[2][2];
    fm_for<0, 4>([&](auto i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i >> 1][i & 1][r] = 0.f;
    });
    auto mma_one = [&](auto i, auto d, auto s) {
        constexpr int p = i >> 2, m = (i >> 1) & 1, n = i & 1;
        constexpr int kind = ORD == 0 ? p : (p == 0 ? 1 : p == 1 ? 0 : 2);
        acc[m][n] = Ops::mfma(fa[d][(kind == 2 ? 2 : 0) + m], fb[s][(kind == 1 ? 2 : 0) + n], acc[m][n]);
    };
    // unit u: A in fa[d], B in fb[s]; reads B of u + 1, loads B of u + R and A of u + DA
    auto step = [&](int u, auto d, auto s) {
        // B of unit u + 1 has landed: behind it at most R - 2 units' loads (A and B)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((R - 2) * 8) : "memory");
        const unsigned ob = off(u + R), oa = off(u + DA);
        fm_for<0, 12>([&](auto i) {
            mma_one(i, d, s);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i < 4) read_b(std::integral_constant<int, 1 - s>{}, i, u + 1);
            else if constexpr (i < 8) load_b(std::integral_constant<int, i - 4>{}, u + R, ob);
            // the A registers: X0 is free after the first 8 products, X1 after the last
            else if constexpr (i < 10) load_a(d, std::integral_constant<int, i - 8>{}, oa);
            __builtin_amdgcn_sched_barrier(0);
        });
        load_a(d, std::integral_constant<int, 2>{}, oa);
        load_a(d, std::integral_constant<int, 3>{}, oa);
        __builtin_amdgcn_sched_barrier(0);
    };
    // prologue: units in the order in which the loop issues them
    fm_for<0, (R > DA ? R : DA)>([&](auto w) {
        if constexpr (w < R) fm_for<0, 4>([&](auto k) { load_b(k, w, off(w)); });
        if constexpr (w < DA) fm_for<0, 4>([&](auto k) { load_a(w, k, off(w)); });
    });
    Coefs cf;   // read while the first loads are in flight
    for (int i = 0; i < 3; ++i) cf.f[i] = NET ? a.coef[i] : st->coef[i];
    const bool skip = !NET && st->skip;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (skip) return;   // Alg. 1 has stopped
    fm_for<0, 4>([&](auto k) { read_b(std::integral_constant<int, 0>{}, k, 0); });
    int u = 0;
    auto round = [&] {
        fm_for<0, DA>([&](auto d) { step(u + d, d, std::integral_constant<int, d & 1>{}); });
        u += DA;
    };
    while (u + DA < KU) round();
    fm_for<0, DA>([&](auto d) {   // the last units
        constexpr int s = d & 1;
        if (u + d < KU) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            if (u + d + 1 < KU)
                fm_for<0, 4>([&](auto k) { read_b(std::integral_constant<int, 1 - s>{}, k, u + d + 1); });
            fm_for<0, 12>([&](auto i) { mma_one(i, d, std::integral_constant<int, s>{}); });
        }
    });
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // the ring is free
    f32x4 s4[4][4];
    fm_for<0, 4>([&](auto q) {
        const int bi = 2 * I + (q >> 1), bj = 2 * J + (q & 1);
        fm_load_block<NET>(a, bi, bj, s4[q]);
    });
    double tt = 0.0, ft = 0.0;
    fm_for<0, 4>([&](auto q) {
        const int bi = 2 * I + (q >> 1), bj = 2 * J + (q & 1);
        if (bi > bj) return;
        if (32 * bj >= a.n_real) {
            if (NET) fm_zero_block(a, bi, bj);
            return;
        }
        double tr = 0.0, fr = 0.0;
        fm_store_block<T16, NET>(a, cf, bi, bj, acc[q >> 1][q & 1], s4[q], ps, (T16*)ring, &tr, &fr);
        if (NET) return;
        tt += wave_sum0(tr);
        ft += wave_sum0(fr);
    });
    if (NET) return;
    if (lane == 0) {
        st_agent(a.parts_out + 2 * (size_t)t, tt);
        st_agent(a.parts_out + 2 * (size_t)t + 1, ft);
    }
    tile_done<64>(st, a.parts_out, a.ntiles, t, a.host_flag, (double*)ring, &s_done);
}

// One 64 x 64 tile of Y per workgroup, in 4 waves of one 32 x 32 block each.  R slots of US
// units of 16 K in the LDS ring.  ORD 0: products X0 X0, X0 X1, X1 X0 per unit (the order of
// the 64-tile kernels), 1: X0 X1, X0 X0, X1 X0 (128-tile kernels).
template <typename T16, int R, int US, int ORD, bool NET = false>
__global__ __launch_bounds__(256) void k_square_fm(FmArgs a) {
    typedef FmOps<T16> Ops;
    typedef typename Ops::vec8 vec8;
    static_assert((R & (R - 1)) == 0 && R >= 2, "slot index by mask");
    constexpr int NW = 4;                          // waves
    constexpr int FPU = 8;                         // fragments (1 KB direct loads) per unit
    constexpr int LPW = FPU * US / NW;             // direct loads per wave and slot
    constexpr int SLOT = FPU * US * 1024;
    static_assert((R - 1) * LPW <= 63, "vmcnt");
    static_assert(R * SLOT >= NW * kFmTranspose, "transpose fits the ring");
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];   // lead_bytes
    __shared__ __attribute__((aligned(16))) unsigned char ring[R * SLOT];
    __shared__ double red[4][2];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = xcd_tile_index(blockIdx.x, a.per, a.ntiles);
    if (t < 0) return;
    int I, J;
    tile_of(t, a.T, 8, &I, &J);
    if (64 * J >= a.n_real) return;   // padding
    const int wi = wave >> 1, wj = wave & 1;
    const int ra = 2 * I, rb = 2 * J;   // first staged panels
    const int bi0 = ra + wi, bj0 = rb + wj;

    f32x4 s4[4];
    fm_load_block<NET>(a, bi0, bj0, s4);
    if (!NET && wave == 0) lead_load(a.lead, lds_addr(dyn));

    const int KU = a.ku;
    const size_t ps = (size_t)a.pstride * 512;   // halves per 32-row panel
    // fragments in slot order: X0 rows of A, X1 of A, X0 of B, X1 of B; this wave copies every
    // NW-th of a slot
    const char* base[LPW];
    unsigned slot_off[LPW];
    int unit_of[LPW];
    fm_for<0, LPW>([&](auto l) {
        const int j = l * NW + wave, f = j % FPU;
        const int op = f >= 4, k = f & 3;
        const int row = op ? rb : ra;
        const T16* pl = (const T16*)(k >> 1 ? a.x1 : a.x0);
        base[l] = (const char*)(pl + (size_t)(row + (k & 1)) * ps);
        slot_off[l] = j * 1024;
        unit_of[l] = j / FPU;
    });
    const unsigned lo = lane * 16, ring0 = lds_addr(ring);
    const int KS = (KU + US - 1) / US;   // slots' worth of K
    // direct load l of this wave's share of slot w (units US w ..; past the end: the last unit
    // again) into slot w mod R
    auto issue_one = [&](auto l, int w, unsigned sl) {
        const int u = US * w + unit_of[l];
        fm_dma16(lo + (unsigned)(u < KU ? u : KU - 1) * 1024u, base[l], sl, slot_off[l]);
    };
    auto slot_addr = [&](int w) { return ring0 + (w & (R - 1)) * SLOT; };
    constexpr int FPW = 4;   // fragments of a wave per unit: X0, X1 of A, X0, X1 of B
    struct Frags {
        vec8 f[US * FPW];
    };
    auto read_one = [&](auto i, int w, Frags& f) {
        constexpr int k = i / FPW, j = i % FPW;
        const int at = k * FPU + 2 * j + (j >= 2 ? wj : wi);
        f.f[i] = *(const vec8*)(ring + (w & (R - 1)) * SLOT + at * 1024 + lo);
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    constexpr int MPU = 3;   // products per unit
    auto mma_one = [&](auto i, const Frags& f) {
        constexpr int k = i / MPU, p = i % MPU;
        constexpr int kind = ORD == 0 ? p : (p == 0 ? 1 : p == 1 ? 0 : 2);
        acc = Ops::mfma(f.f[k * FPW + (kind == 2)], f.f[k * FPW + 2 + (kind == 1)], acc);
    };
    auto mma_last = [&](const Frags& f) {   // the last slot: only the units that exist
        fm_for<0, US>([&](auto k) {
            if (US * (KS - 1) + k < KU) fm_for<0, MPU>([&](auto i) { mma_one(std::integral_constant<int, k * MPU + i>{}, f); });
        });
    };
    // One slot: every wave's fragments of it are in registers (lgkmcnt(0) and the barrier), so it
    // takes slot w + R's units; slot w + 1 has landed once at most the R - 2 slots behind it are
    // outstanding in every wave.  Its fragment reads and then the direct loads go between this
    // slot's products (issued in front of them they add their issue time to the products': 600
    // against 384 cycles per unit on a 64 x 64 wave tile); scheduling barriers pin the order.
    auto step = [&](int w, const Frags& cur, Frags& next) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((R - 2) * LPW) : "memory");
        asm volatile("s_barrier" ::: "memory");
        const unsigned sl = slot_addr(w + R);
        constexpr int NM = MPU * US, NR = FPW * US, NS = NR + LPW;
        fm_for<0, NM>([&](auto i) {
            mma_one(i, cur);
            __builtin_amdgcn_sched_barrier(0);
            fm_for<i * NS / NM, (i + 1) * NS / NM>([&](auto k) {
                if constexpr (k < NR) read_one(std::integral_constant<int, k>{}, w + 1, next);
                else issue_one(std::integral_constant<int, k - NR>{}, w + R, sl);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    for (int w = 0; w < R; ++w) {
        const unsigned sl = slot_addr(w);
        fm_for<0, LPW>([&](auto l) { issue_one(l, w, sl); });
    }
    Frags fp, fq;
    // a layer behind the stop (workgroup 0 still hands the state on)
    if (!NET && ((const StateHot*)a.lead.hot_in)->stopped && blockIdx.x != 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 1) * LPW) : "memory");
    asm volatile("s_barrier" ::: "memory");
    fm_for<0, FPW * US>([&](auto i) { read_one(i, 0, fp); });
    int u = 0;
    auto pair = [&] {
        step(u, fp, fq);
        step(u + 1, fq, fp);
        u += 2;
    };
    // the control runs behind the first units' products, with the next loads in flight
    if (u + 2 < KS) pair();
    Coefs cf;
    if (NET) {
        for (int i = 0; i < 3; ++i) cf.f[i] = a.coef[i];
    } else if (!lead_finish(a.lead, dyn, blockIdx.x == 0 && wave == 0, &cf)) {   // Alg. 1 has stopped
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }
    while (u + 2 < KS) pair();
    if (u + 1 < KS) {   // two slots left
        step(u, fp, fq);
        mma_last(fq);
    } else {
        mma_last(fp);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the ring is free
    if (NET) {
        if (bi0 > bj0) return;
        if (32 * bj0 >= a.n_real) return fm_zero_block(a, bi0, bj0);
        double tr = 0.0, fr = 0.0;
        return fm_store_block<T16, true>(a, cf, bi0, bj0, acc, s4, ps, (T16*)(ring + wave * kFmTranspose), &tr, &fr);
    }
    if (threadIdx.x < 8) red[threadIdx.x >> 1][threadIdx.x & 1] = 0.0;   // a block below the diagonal adds nothing
    stage_barrier();
    double tr = 0.0, fr = 0.0;
    if (bi0 <= bj0 && 32 * bj0 < a.n_real) {
        fm_store_block<T16, false>(a, cf, bi0, bj0, acc, s4, ps, (T16*)(ring + wave * kFmTranspose), &tr, &fr);
        const double s0 = wave_sum0(tr), s1 = wave_sum0(fr);
        if (lane == 0) {
            red[wave][0] = s0;
            red[wave][1] = s1;
        }
    }
    stage_barrier();
    if (threadIdx.x < 2)   // the tile's sums, blocks in row-major order
        a.parts_out[2 * (size_t)t + threadIdx.x] =
            ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
}

}  // namespace

// variant: ORD + 2 x (0: 4-wave workgroups, 1: one wave) (see fm_variant in k_square2.hip); a.coef: a
// layer of the network
template <typename T16>
hipError_t launch_fm_t(int variant, const FmArgs& a, hipStream_t s) {
    if (a.coef) {
#define SP2_L(K, NT) hipLaunchKernelGGL((K), dim3(8 * a.per), dim3(NT), 0, s, a)
        switch (variant) {
            case 0: SP2_L((k_square_fm<T16, 4, 2, 0, true>), 256); break;
            case 1: SP2_L((k_square_fm<T16, 4, 2, 1, true>), 256); break;
            case 2: SP2_L((k_square_fm1<T16, 4, 4, 0, true>), 64); break;
            case 3: SP2_L((k_square_fm1<T16, 4, 4, 1, true>), 64); break;
            default: return hipErrorInvalidValue;
        }
#undef SP2_L
        return hipGetLastError();
    }
#define SP2_L(K, NT, LDS) hipLaunchKernelGGL((K), dim3(8 * a.per), dim3(NT), LDS, s, a)
    switch (variant) {
        case 0: SP2_L((k_square_fm<T16, 4, 2, 0>), 256, lead_bytes(a.lead)); break;
        case 1: SP2_L((k_square_fm<T16, 4, 2, 1>), 256, lead_bytes(a.lead)); break;
        case 2: SP2_L((k_square_fm1<T16, 4, 4, 0>), 64, 0); break;
        case 3: SP2_L((k_square_fm1<T16, 4, 4, 1>), 64, 0); break;
        default: return hipErrorInvalidValue;
    }
#undef SP2_L
    return hipGetLastError();
}

}  // namespace sp2

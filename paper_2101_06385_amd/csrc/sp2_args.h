// Arguments of the squaring kernels and of their persistent schedule (the parts of the
// interface the kernel code depends on).
#pragma once

namespace sp2 {

// ---------------------------------------------------------------------------------
// Arguments of the squaring kernels: Y = alpha X^2 + beta X + gamma I, written to
// both triangles (exactly symmetric), optionally split into half-precision planes, with
// FP64 partial sums of Tr Y and ||Y||_F^2 per output tile.
// ---------------------------------------------------------------------------------
struct SquareArgs {
    const void* x0;       // split modes: high plane of X (np x np, row stride plane_ld(np)); plain: X itself
    const void* x1;       // split modes: low plane of X
    const void* s_in;     // X in the state precision (beta term), ld = np
    void* s_out;          // Y in the state precision, ld = ld_out
    void* p0_out;         // split modes: planes of Y (row stride plane_ld(np)), or null
    void* p1_out;
    double* parts;        // 2 doubles per tile, or null
    const float* coef;    // (alpha, beta, gamma)
    const double* coef64; // FP64 layer kernels: (alpha, beta, gamma) in FP64 when non-null
    const int* skip;      // null, or a flag that makes every workgroup return at once
    int np;               // padded edge (multiple of the tile)
    int ld_out;           // leading dimension of s_out
    int n_valid;          // rows/cols >= n_valid of s_out are not written
    int n_real;           // logical edge: the gamma I term stops here so the padding stays zero
    int k_all;            // FP64 / FP32: nonzero = products over all np columns, 0 = X is zero beyond n_real
    int T;                // tiles per edge
    int ntiles;           // T (T + 1) / 2
    int per;              // ceil(ntiles / 8)
    float out_scale;      // split modes: 2^-2s applied to the accumulated products
    float in_scale;       // split modes: 2^s applied before splitting Y
    // control of the next layer by the launch's last finished tile (sp2_control.h)
    int arrivals;         // workgroups that count themselves done (tile_done)
    void* ctl;            // DevState of the call, or null: no control in this launch
    int* host_flag;       // mapped host flag set when Alg. 1 stops, or null
};

// Leading control of a layer: its sigma_n from the partial sums of the launch before.
struct LeadArgs {
    void* st;               // DevState (histories; its hot block is hot[0])
    const void* hot_in;     // hot block that the layer before left
    void* hot_out;          // where this layer's goes (another block)
    const double* parts;    // nparts pairs, `stride` doubles apart
    int* host_flag;         // mapped host flag set when Alg. 1 stops, or null
    int nparts, stride;
    int layer;              // this layer (1 ..)
};

// Arguments of the fragment-major split kernel (k_square_fm.h).
struct FmArgs {
    LeadArgs lead;          // leading control (4-wave workgroups)
    void* ctl;              // DevState: control of the next layer by the last tile (one wave per tile)
    int* host_flag;
    const void* x0;         // planes of X, fragment-major
    const void* x1;
    void* p0_out;           // planes of Y
    void* p1_out;
    const float* s_in;      // X, 32 x 32 blocks of the upper triangle in accumulator order
    float* s_out;           // Y                               (coef: row-major, ld floats per row)
    const float* coef;      // layers without control (network): (alpha, beta, gamma); else null
    int ld;
    double* parts_out;      // a pair per 64-tile; those of padding tiles stay zero
    int pstride;            // 1 KB blocks per 32-row panel of a plane
    int sb;                 // 32-blocks per row of blocks of S
    int ku;                 // units of 16 K that hold data
    int n_real;             // logical edge
    int T, ntiles, per;     // 64-tiles per edge, in all, per XCD
    float out_scale, in_scale;
};
// 1 KB blocks per 32-row panel: one more than the K units, so that panels do not start on
// the same L2 channel
__host__ __device__ inline int fm_pstride(int np) { return np / 16 + 1; }

// Schedule of the persistent split-square kernel: G workgroups run `rounds` whole rounds
// of tiles, then the `tail_tiles` leftover tiles are each cut into `chunks` K-chunks.
// `partial` holds one FP32 tile accumulator per tail chunk, `counter` one arrival count
// per tail tile (zeroed at the start of every call; each executed layer adds `chunks`).
constexpr int kMaxSkGrid = 1024;
// The int array `counter` of the persistent split square: arrivals per split tile at
// [0, kMaxSkGrid), then the ticket counter of the tail-chunk queue at kSkQueueSlot.
constexpr int kSkQueueSlot = kMaxSkGrid;
constexpr int kSkCounterInts = kMaxSkGrid + 64;
// Two-level split tail: group arrival counters at [kSkGroupCounter, kMaxSkGrid) of
// `counter`, group partial tiles from slot kSkGroupSlot of `partial` (chunk partials use
// slots below it: at most one per workgroup).
constexpr int kSkGroupCounter = kMaxSkGrid / 2;
constexpr int kSkGroupSlot = kMaxSkGrid / 2;

// Tile maps of the grouped (many-problem) launches: block b computes tile `tile` of problem
// `problem` in entry (b mod 8) * per + b / 8 (problem -1: no work), so the blocks that the
// hardware sends to one XCD (b mod 8 fixed) walk that XCD's part of the map.
struct TileRef {
    int problem, tile;
};

// Row stride (elements) of the half-precision planes of an np x np matrix.  With a row
// pitch of a power of two kilobytes, the rows of one K-slice of a panel fall on the same
// L2 channel; one extra 128-byte line per row spreads them.  One squaring layer at
// n = 16384 measured 14.5 ms with pitch np and 12.0 ms with this one (no change at 8192).
__host__ __device__ inline int plane_ld(int np) { return np + 64; }
constexpr int kSkVariants = 6;
// Stream-K form (split squaring, stream_k = Q > 0): the ntiles x (KS / Q) units of Q
// K-slices, tile-major, are cut into G contiguous ranges, one per workgroup; a tile that
// several ranges share is finished by the last of its contributors, which sums their FP32
// partials in K order.  Workgroup v keeps its partials in slots 2v (first tile of its
// range) and 2v + 1 (last tile); `counter` then counts arrivals per tile.
struct StreamK {
    int grid = 0, rounds = 0, tail_tiles = 0, chunks = 0;
    float* partial = nullptr;     // FP32 partial tiles
    int* counter = nullptr;       // arrivals per tail tile, counted modulo chunks
    int stream_k = 0;             // slices per stream-K unit; 0: whole rounds + split tail
    int pad = 0;
};
constexpr int kSkMaxContrib = 16;   // most stream-K ranges that may share one tile

}  // namespace sp2

// common.hpp -- shared definitions of the gfx950 CUBE2 force library.
//
// Geometry used by every kernel:
//   * fine mesh: n_f cells per side, positions q in units of 2^-15 fine cells;
//   * IOS cells of 2x2x2 fine cells (n_ios = n_f/2 per side), the unit of the
//     particle order; tiles of 8^3 IOS cells (16^3 fine cells) group them;
//   * key of IOS cell c = tile index * 512 + cell-in-tile index, both x fastest.
// Every particle-side kernel runs one workgroup per tile: the tile's particles
// are the contiguous range cell_start[key0] .. cell_start[key0 + 512].
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/cube2.h"

namespace cube2 {

constexpr int kFracBits = 15;     // in-cell fraction of a fine cell
constexpr int kTileIos = 8;       // IOS cells per tile side
constexpr int kTileFine = 16;     // fine cells per tile side
constexpr int kTileCells = 512;   // IOS cells per tile
constexpr int kBlock = 256;       // threads of the particle-side kernels

struct Level {
    int n = 0;          // cells per side
    int H = 1;          // spacing in fine cells
    int hshift = 0;     // log2(H)
    int pitch = 0;      // complex row pitch of the half spectrum
    double b_a = 0;     // softening of the level (fine cells)
    double b_prev = 0;  // truncation (fine cells); <= 0 means infinity
    size_t tw_off = 0;  // byte offset of the twiddle table in `tables`
    size_t g_off = 0;   // byte offset of the octant Green's table
    size_t gz_off = 0;  // the same values in the z pass's order (FP32, see fft.hip)
    size_t tw64_off = 0, g64_off = 0;  // FP64 copies (CUBE2_FP64_FORM only)
};

}  // namespace cube2

namespace cube2 {
// Pair-law table of the PP kernels (built on the host, see pp.hip).
constexpr int kPairKMax = 128;     // grid intervals of [0, b_f)
constexpr int kPairRow = 12;       // floats per interval: 9 coefficients, y map, pad
// FP32 pair law tables of the PP kernels by s = r^2 (pp.hip): one row of four
// floats per 2^-kSMant of an octave of s.  A row's place is its float exponent
// and top mantissa bits modulo kSOctaves octaves.
constexpr int kSMant = 6;          // forward: 64 rows per octave
constexpr int kSMantAdj = 7;       // adjoint: 128 rows per octave
constexpr int kSOctaves = 32;
constexpr int kSRows = 20 << kSMant;         // rows held (20 octaves)
constexpr int kSRowsAdj = 20 << kSMantAdj;
// Light tiles of the PP kernels (pp.hip): most z-layers of a tile's cells that
// a wave takes at once, and how many particles their box may hold.
constexpr int kPPLightLayers = 2;
constexpr int kPPLightCap = 520, kPPLightCapAdj = 512;
// Words of the PP kernels' lists: a tile in the low bits; above it, in the list of parts,
// the part, the tile's parts less one and whether lanes share a particle; in the order,
// what the list is made from.
constexpr int kTileBits = 18, kPartBits = 5;
constexpr uint32_t kTileMask = (1u << kTileBits) - 1u, kMaxParts = 1u << kPartBits;
constexpr uint32_t kLanesBit = 1u << (kTileBits + 2 * kPartBits);
constexpr int kPPListMax = 8192;             // entries of the list of parts
}  // namespace cube2

struct cube2_ctx {
    cube2_config cfg;
    int pp_K = 0;                      // intervals of the pair-law grid
    // the FP32 pair law's units (pp.hip): position scale and scale of g (powers
    // of two), and whether s is clamped to the table
    float pp_pscale = 1.f, pp_unit = 1.f;
    bool pp_clamp = false;
    uint32_t pp_bmax = 0, pp_bmax_adj = 0;   // float bits of s that the clamped form stops at
    int pp_halo = 1;                   // PP neighbour reach in IOS cells: 1 (b_f <= 2), 2 (b_f <= 4)
    size_t pp_soff = 0, pp_aoff = 0;   // byte offsets of the FP32 tables (forward, adjoint) in `tables`
    std::vector<double> pp_rows64;     // the exact pair law by r, in FP64
    size_t pp64_off = 0;               // FP64 rows (CUBE2_FP64_FORM only)
    bool fp64 = false;                 // CUBE2_FP64_FORM
    bool tsc = false;                  // CUBE2_ASSIGN_TSC: TSC instead of CIC on every PM level
    bool isolated = false;             // CUBE2_ISOLATED: isolated boundaries (appendix A)
    int n_f = 0, n_ios = 0, nt = 0;   // fine cells, IOS cells, tiles per side
    int64_t n_cells = 0;               // IOS cells
    int n_levels = 1;                  // 1 or 2; level 0 = fine, 1 = coarse
    cube2::Level lv[2];
    size_t table_bytes = 0;
    unsigned char *tables = nullptr;   // device; set by cube2_init_tables
    hipStream_t side = nullptr;        // cube2_force's PP stream (default priority), made by cube2_init_tables
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    // the PM adjoint's second stream (default priority) and its fork/join
    // events: the cotangent scatter beside the recomputed forward potentials
    hipStream_t side2 = nullptr;
    hipEvent_t ev_fork2 = nullptr, ev_join2 = nullptr;
};

namespace cube2 {

// Byte layout of the work buffer for n particles.
struct WorkLayout {
    size_t real_f, real_c, bar_f, bar_c, spec, coarse_acc;
    size_t real64_f, real64_c, spec64;  // FP64 form (zero-sized without it)
    size_t keys, vals, keys2, vals2, hist, scan_tmp, offs_tmp, red;
    size_t pp_order, pp_hist, pp_scan, acc_pp;  // cube2_force's concurrent PP: own tile queue, output
    size_t tile_parts, pp_parts;        // the PP's list of parts, and that of the concurrent PP
    size_t tile_order;  // 4 x (tiles) + 64 uint32: PP tile order, its sort buffers, work counter
    size_t vel_tmax;    // velocity codec: one FP32 maximum per tile
    size_t total;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

WorkLayout work_layout(const cube2_ctx *ctx, int64_t n);

// In-cell offsets of the particles to sort, 8 bytes each (in the area of the
// concurrent PP output, which no sort overlaps).
inline ushort4 *sort_offsets(unsigned char *work, const WorkLayout &L) {
    return reinterpret_cast<ushort4 *>(work + L.acc_pp);
}

// bits of the device status word
constexpr uint32_t kStatusOverflow = 1u;    // a deposit or codec accumulator could overflow
constexpr uint32_t kStatusNonFinite = 2u;   // a kick-drift met a non-finite velocity or step

inline uint32_t *status_word(const cube2_ctx *ctx) {
    return reinterpret_cast<uint32_t *>(ctx->tables);
}

// ---- device helpers ------------------------------------------------------

__device__ __forceinline__ uint32_t cell_key(int cx, int cy, int cz, int nt) {
    int tx = cx >> 3, ty = cy >> 3, tz = cz >> 3;
    int ux = cx & 7, uy = cy & 7, uz = cz & 7;
    return (uint32_t)(((tz * nt + ty) * nt + tx) * kTileCells + (uz * 8 + uy) * 8 + ux);
}

// Tile coordinates of workgroup b.  Blocks are dealt to the 8 XCDs round
// robin; this mapping gives each XCD a contiguous slab of tiles so that the
// halos shared between neighbouring tiles stay in one L2.
__device__ __forceinline__ void tile_of_block(int b, int nt, int &tx, int &ty, int &tz) {
    int ntiles = nt * nt * nt;
    int t = b;
    if ((ntiles & 7) == 0) t = (b & 7) * (ntiles >> 3) + (b >> 3);
    tx = t % nt;
    ty = (t / nt) % nt;
    tz = t / (nt * nt);
}

// TSC weights (eq. 5, 16-bit fixed point as the deposit) of the 15-bit
// fraction f of one axis: nearest-node shift hi and the three weights.
template <typename T>
__device__ __forceinline__ int tsc_axis(int f, T (&w)[3]) {
    const int hi = f >= 16384 ? 1 : 0;
    const int m = f - (hi << 15);
    const uint32_t a = (uint32_t)(16384 - m), b = (uint32_t)(16384 + m);
    const uint32_t w0 = (a * a + 16384u) >> 15, w2 = (b * b + 16384u) >> 15;
    const T inv = T(1.0 / 65536.0);
    w[0] = (T)w0 * inv;
    w[2] = (T)w2 * inv;
    w[1] = (T)(65536u - w0 - w2) * inv;
    return hi;
}

// The same weights with their derivatives in the particle coordinate (level
// units): d = m 2^-15 is the offset from the nearest node, and the slopes of
// eq. 5 at the three nodes are -(1/2 - d), -2d and 1/2 + d.
template <typename T>
__device__ __forceinline__ int tsc_axis_grad(int f, T (&w)[3], T (&dw)[3]) {
    const int hi = tsc_axis<T>(f, w);
    const T d = (T)(f - (hi << 15)) * T(1.0 / 32768.0);
    dw[0] = -(T(0.5) - d);
    dw[1] = T(-2) * d;
    dw[2] = T(0.5) + d;
    return hi;
}

__device__ __forceinline__ int wrapn(int i, int n) {  // n is a power of two
    return i & (n - 1);
}

// Largest s in [0, cnt) with pre[s] <= v (pre nondecreasing, pre[0] <= v).
__device__ __forceinline__ int seg_search(const uint32_t *pre, int cnt, uint32_t v) {
    int lo = 0, hi = cnt;  // invariant: pre[lo] <= v, answer in [lo, hi)
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (pre[mid] <= v) lo = mid; else hi = mid;
    }
    return lo;
}

// The same index for a count known at compile time: the last u in [0, CNT)
// with pre[u] <= v, found bit by bit from the highest power of two below
// CNT (pre non-decreasing, so pre[u] <= v holds exactly up to the answer).
// Unrolled and branch-free: no loop control, and the LDS reads of
// independent searches in one thread interleave.  When CNT is not a power
// of two, pre must hold CNT + 1 entries with pre[CNT] > v (the end of the
// last segment): a candidate at or beyond CNT reads pre[CNT] instead, which
// fails the test, so no step needs a branch.
template <int CNT>
__device__ __forceinline__ int seg_search_n(const uint32_t *pre, uint32_t v) {
    static_assert(CNT >= 1, "empty range");
    constexpr int TOP = [] {
        int t = 1;
        while (2 * t < CNT) t *= 2;
        return CNT > 1 ? t : 0;
    }();
    int lo = 0;
#pragma unroll
    for (int step = TOP; step > 0; step >>= 1) {
        const int c = lo + step;
        if (2 * TOP - step < CNT) {   // c < CNT whatever steps were taken (folds once unrolled)
            if (pre[c] <= v) lo = c;
        } else {
            if (pre[c < CNT ? c : CNT] <= v) lo = c;
        }
    }
    return lo;
}

// Index of this thread's wave in its workgroup, known uniform (a scalar).
__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Inclusive sums over the lanes of a wave (every lane active): DPP shifts within the
// rows of 16 lanes, then the rows' sums broadcast to the rows above.  6 additions; by
// shuffles, 6 dependent LDS round trips.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return x;
}

// Block-wide exclusive scan of one uint32 per thread (blockDim == BLOCK).
template <int BLOCK = kBlock>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh /*BLOCK/64+1*/,
                                                         uint32_t &total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint32_t x = wave_inclusive_scan(v);
    if (lane == 63) sh[wid] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) {
        uint32_t s = sh[w];
        if (w < wid) off += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return off + x - v;
}

// A tile of more particles than this, of n in all, is more than one workgroup's in the
// sorts and in the drift: one workgroup is the longer the fewer there are in all.
inline uint32_t heavy_limit(int64_t n) { return n > (1 << 20) ? 8192u : 4096u; }

// Stable sort by cell of one tile's `total` elements, the first of which comes to
// particle `start` (all kBlock threads call it): each wave takes a contiguous part of
// them; the cells' counts per wave give the starts of the cells (written to
// cell_start, or given in `base`) and of each wave's part of them, and a second pass
// ranks equal cells by wave ballots.  cell_of(e) is the cell (0..511) of element e, emit(e,
// i) writes element e to sorted place i (counted from first_place).
template <class CellOf, class Emit>
__device__ __forceinline__ void tile_cell_sort(uint32_t (*hist)[kTileCells] /*[kBlock / 64]*/,
                                               uint32_t *scan_sh /*kBlock / 64 + 1*/, uint32_t total,
                                               uint32_t first_place, uint32_t start,
                                               uint32_t *__restrict__ cell_start,
                                               CellOf cell_of, Emit emit,
                                               const uint32_t *base = nullptr) {
    constexpr int W = kBlock / 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int i = tid; i < W * kTileCells; i += kBlock) hist[i / kTileCells][i % kTileCells] = 0u;
    __syncthreads();
    const uint32_t per = (total + 64 * W - 1) / (64 * W) * 64;
    const uint32_t e0 = min(w * per, total), e1 = min(e0 + per, total);
    // (kAhead words of 64 elements at a time: their loads are issued together)
    constexpr int kAhead = 4;
    for (uint32_t b = e0; b < e1; b += 64 * kAhead) {
        uint32_t c[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) c[k] = cell_of(min(b + 64 * k + lane, e1 - 1));
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (b + 64 * k + lane < e1) atomicAdd(&hist[w][c[k]], 1u);
    }
    __syncthreads();
    // thread i: cells 2i, 2i + 1
    uint32_t tot[2] = {0, 0};
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int v = 0; v < W; ++v) tot[k] += hist[v][2 * tid + k];
    uint32_t all;
    uint32_t at = block_exclusive_scan(tot[0] + tot[1], scan_sh, all);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (base)
            at = base[2 * tid + k];
        else
            cell_start[2 * tid + k] = start + at;
#pragma unroll
        for (int v = 0; v < W; ++v) {
            const uint32_t c = hist[v][2 * tid + k];
            hist[v][2 * tid + k] = at;
            at += c;
        }
    }
    __syncthreads();
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (uint32_t b0 = e0; b0 < e1; b0 += 64 * kAhead) {
        uint32_t cell[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) cell[k] = cell_of(min(b0 + 64 * k + lane, e1 - 1));
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const uint32_t e = b0 + 64 * k + lane, c = cell[k];
            if (b0 + 64 * k >= e1) break;        // wave-uniform
            const bool valid = e < e1;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const bool bit = (c >> i) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t rank = (uint32_t)__popcll(peers & lt);
            const uint32_t first = hist[w][c];
            if (valid && rank == 0) hist[w][c] = first + (uint32_t)__popcll(peers);
            if (valid) emit(e, first_place + first + rank);
            // this wave's counts are written before its next loads (the LDS serves a
            // wave in order; this keeps the compiler from reordering them)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Tile scheduling of the per-tile kernels: persistent workgroups (or, for light
// PP tiles, waves) take the tiles of the heaviest-first order
// (launch_order_tiles) until they are exhausted.

// One claim on a work counter (a single thread calls it): the position in
// `order` of the next tile, or a value >= ntiles when all are taken.
__device__ __forceinline__ int claim_slot(uint32_t *queue, int ntiles) {
    const uint32_t v = atomicAdd(queue, 1u);
    return v < (uint32_t)ntiles ? (int)v : ntiles;
}

// Claims that come often use a counter per XCD (the deposit's here, the light PP tiles' in
// light_claims.hpp): one counter serves only some 70
// million claims a second (14 ns each; the deposit's 262144 tiles of a 1024^3
// mesh took 3.4 ms whatever they held).  Workgroups b = g (mod 8) run on one XCD
// and take every 8th tile of the order, the XCD's slab of the mesh
// (tile_of_block) where the order is that of the blocks.
// When a group's share is taken, its workgroups go on with the next group's.
struct XcdShare {
    int ng, g;                 // groups, this workgroup's
    int done = 0;              // groups found exhausted
    __device__ __forceinline__ XcdShare() : ng(gridDim.x >= 8 ? 8 : 1), g((int)blockIdx.x % ng) {}
    // items of the group out of n
    __device__ __forceinline__ int share(int n) const { return n > g ? (n - g + ng - 1) / ng : 0; }
    // place in the order of the group's i-th item
    __device__ __forceinline__ int place(int i) const { return i * ng + g; }
    // a claim on the group's counter
    __device__ __forceinline__ int claim(uint32_t *queues) const {
        return (int)min(atomicAdd(queues + 32 * g, 1u), 0x3FFFFFFFu);
    }
    // on to the next group; false when all are exhausted
    __device__ __forceinline__ bool next_group() {
        g = g + 1 < ng ? g + 1 : 0;
        return ++done < ng;
    }
};

// Sums over the 64 lanes of a wave (butterfly; every lane must be active).
// The order of the additions is fixed, so float sums are deterministic.
// One DPP lane permutation within rows of 16 lanes, applied to both halves
// of a 64-bit value.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xF, 0xF, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, false);
    return ((unsigned long long)hi << 32) | lo;
}

// Sum of a 64-bit integer over the 64 lanes of a wave (every lane active),
// returned to every lane.  Within each row of 16 lanes, DPP butterflies
// (quad_perm [1,0,3,2] and [2,3,0,1], then the half-row and row mirrors)
// leave the row's sum in all its lanes; the four row sums are then read from
// lanes 0, 16, 32 and 48.  No LDS traffic; the integer sum is exact, so its
// order does not matter.
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
    v += dpp_u64<0xB1>(v);
    v += dpp_u64<0x4E>(v);
    v += dpp_u64<0x141>(v);
    v += dpp_u64<0x140>(v);
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    unsigned long long s = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        s += ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)hi, 16 * r) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)lo, 16 * r);
    return s;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// The particles of a box of cells as one list, cell after cell in box order: position v
// of the list belongs to cell `cell` and is particle `from + v`.  The nonempty cells are
// kept in LDS, and one bit per position tells where a cell begins, kBoxSpan positions
// at a time; a wave then finds its 64 positions' cells by counting bits of one word
// (two lane reads, a bit count and one LDS read, most lanes of the same address),
// where a binary search of the cells' first positions is ten dependent LDS reads.
constexpr int kBoxSpan = 4096;
template <int SEGS, int BLOCK> struct BoxList {
    static constexpr int PER = (SEGS + BLOCK - 1) / BLOCK;   // cells per thread
    struct Shared {
        uint2 seg[SEGS];                     // {from, the caller's word for the cell}
        uint32_t head[kBoxSpan / 32];        // bit: a cell begins here
        uint32_t before;                     // nonempty cells wholly before the span
        uint2 scan[BLOCK / 64];
    };
    uint32_t total, first[PER], rank;        // this thread's cells: first positions, nonempty cells before
    uint32_t pfx;                            // of head word pair `lane` of the span
    unsigned long long word;

    // the list of this thread's cells tid * PER + k (starts src, counts cnt, words tag);
    // the first span is ready after it.  All threads call it; the LDS is free before.
    __device__ __forceinline__ void build(Shared &sh, const uint32_t (&src)[PER], const uint32_t (&cnt)[PER],
                                          const uint32_t (&tag)[PER]) {
        const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
        if (tid < kBoxSpan / 32) sh.head[tid] = 0u;
        uint32_t c = 0, ne = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            c += cnt[k];
            ne += cnt[k] != 0u;
        }
        const uint32_t xc = wave_inclusive_scan(c), xn = wave_inclusive_scan(ne);
        if (lane == 63) sh.scan[w] = make_uint2(xc, xn);
        __syncthreads();
        uint32_t at = xc - c, all = 0;
        rank = xn - ne;
#pragma unroll
        for (int i = 0; i < BLOCK / 64; ++i) {
            const uint2 t = sh.scan[i];
            if (i < w) {
                at += t.x;
                rank += t.y;
            }
            all += t.x;
        }
        total = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
        uint32_t r = rank;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            first[k] = at;
            if (cnt[k]) sh.seg[r++] = make_uint2(src[k] - at, tag[k]);
            at += cnt[k];
        }
        mark(sh, cnt, 0u);
    }
    // the heads of the span of positions [base, base + kBoxSpan); sh.head is clear
    __device__ __forceinline__ void mark(Shared &sh, const uint32_t (&cnt)[PER], uint32_t base) {
        uint32_t r = rank;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t end = first[k] + cnt[k];
            if (cnt[k] && end > base && first[k] < base + kBoxSpan) {
                const uint32_t i = first[k] > base ? first[k] - base : 0u;
                atomicOr(&sh.head[i >> 5], 1u << (i & 31u));
                if (first[k] <= base) sh.before = r;
            }
            r += cnt[k] != 0u;
        }
        __syncthreads();
        const int lane = threadIdx.x & 63;
        word = ((unsigned long long)sh.head[2 * lane + 1] << 32) | sh.head[2 * lane];
        const uint32_t c = (uint32_t)__popcll(word);
        pfx = sh.before + wave_inclusive_scan(c) - c;
    }
    // moves on to the span at `base`; all threads call it
    __device__ __forceinline__ void span(Shared &sh, const uint32_t (&cnt)[PER], uint32_t base) {
        __syncthreads();
        if (threadIdx.x < kBoxSpan / 32) sh.head[threadIdx.x] = 0u;
        __syncthreads();
        mark(sh, cnt, base);
    }
    // {from, word} of the cell of position 64 i + lane of the span (i wave-uniform,
    // 64 i < the span's positions; a lane past the list's end gets its last cell)
    __device__ __forceinline__ uint2 cell(const Shared &sh, int i) const {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, i),
                       hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(word >> 32), i);
        const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)pfx, i) + (lo & 1u) - 1u;
        // heads at or below the lane: those of the word shifted down below it, and bit 0
        const uint32_t l1 = (lo >> 1) | (hi << 31), h1 = hi >> 1;
        return sh.seg[__builtin_amdgcn_mbcnt_hi(h1, __builtin_amdgcn_mbcnt_lo(l1, p))];
    }
};

// Lane of the first set bit of a nonzero wave mask.
__device__ __forceinline__ int first_lane(unsigned long long mask) {
    return __ffsll((long long)mask) - 1;
}

// The kTileCells + 1 particle starts of one tile (cs[key0 .. key0 + 512])
// into LDS, every load of a thread issued before its LDS stores.
template <int BLOCK>
__device__ __forceinline__ void stage_cell_starts(uint32_t *__restrict__ dst,
                                                  const uint32_t *__restrict__ cs, uint32_t key0) {
    constexpr int PER = (kTileCells + 1 + BLOCK - 1) / BLOCK;
    uint32_t v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {  // unconditional loads (clamped index)
        const int i = (int)threadIdx.x + k * BLOCK;
        v[k] = cs[key0 + (i <= kTileCells ? i : kTileCells)];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = (int)threadIdx.x + k * BLOCK;
        if (i <= kTileCells) dst[i] = v[k];
    }
}


// The coarse level at a tile's particles.  Tens of particles share each coarse cell,
// so the finite-difference force (eq. 7) is formed once per node of the tile's
// coarse footprint, (16/H + 1)^3 nodes (TSC: + 3), from the potential in the
// caches, and staged as (E_x, E_y, E_z, extra): a particle then reads 8 (27) nodes
// of four words instead of the 72 (189) potential values of its lines (512^3 particles,
// CIC: interpolation 3.80 -> 3.69 ms, adjoint gather 6.57 -> 6.05; TSC on 512^3 cells:
// 741 -> 694 us and 1964 -> 1680).
template <typename T> struct alignas(4 * sizeof(T)) Vec4 { T x, y, z, w; };
template <int P> constexpr int coarse_field_lo() { return P == 3 ? 1 : 0; }
template <int P, int HS> constexpr int coarse_field_max() {   // nodes per axis; HS = 0: at ratio 2
    return (kTileFine >> (HS > 0 ? HS : 1)) + 1 + 2 * coarse_field_lo<P>();
}
template <int P, int BLOCK, typename T>
__device__ __forceinline__ void stage_coarse_field(Vec4<T> *__restrict__ dst, const T *__restrict__ phi,
                                                   const T *__restrict__ extra, int n, int hshift,
                                                   int ax0, int ay0, int az0) {
    constexpr int LO = coarse_field_lo<P>();
    const int NC = (kTileFine >> hshift) + 1 + 2 * LO, m = n - 1;
    const int x0 = (ax0 >> hshift) - LO, y0 = (ay0 >> hshift) - LO, z0 = (az0 >> hshift) - LO;
    const T c1 = T(2.0 / 3.0), c2 = T(1.0 / 12.0);
    for (int i = threadIdx.x; i < NC * NC * NC; i += BLOCK) {
        const int x = x0 + i % NC, y = y0 + (i / NC) % NC, z = z0 + i / (NC * NC);
        auto at = [&](const T *f, int xx, int yy, int zz) {
            return f[((int64_t)(zz & m) * n + (yy & m)) * n + (xx & m)];
        };
        Vec4<T> e = {T(0), T(0), T(0), T(0)};
        if (phi) {
            e.x = -(c1 * (at(phi, x + 1, y, z) - at(phi, x - 1, y, z)) -
                    c2 * (at(phi, x + 2, y, z) - at(phi, x - 2, y, z)));
            e.y = -(c1 * (at(phi, x, y + 1, z) - at(phi, x, y - 1, z)) -
                    c2 * (at(phi, x, y + 2, z) - at(phi, x, y - 2, z)));
            e.z = -(c1 * (at(phi, x, y, z + 1) - at(phi, x, y, z - 1)) -
                    c2 * (at(phi, x, y, z + 2) - at(phi, x, y, z - 2)));
        }
        if (extra) e.w = at(extra, x, y, z);
        dst[i] = e;
    }
}

// Copy the periodic S^3 block of an n^3 mesh starting at node (x0, y0, z0)
// (wrapped) into LDS, x fastest.  Each wave copies 64/S whole x-rows per pass
// (lane -> (row, x) fixed for the whole copy, so a row is one contiguous
// read), the row's (y, z) is advanced incrementally, and the loads of one
// thread are issued in batches (all in flight before the LDS stores).  A
// block that does not wrap (most of them) is read through one base address
// and a 32-bit offset advanced by constants; a wrapping one through the
// wrapped node indices.
template <int S, int BLOCK, typename T, int MAXB = 20>
__device__ __forceinline__ void stage_block(T *__restrict__ dst, const T *__restrict__ mesh, int n,
                                            int x0, int y0, int z0) {
    static_assert(S <= 64 && BLOCK % 64 == 0, "rows must fit a wave");
    constexpr int RPW = 64 / S;          // rows per wave and pass
    constexpr int RPP = RPW * (BLOCK / 64);
    constexpr int ROWS = S * S;
    constexpr int PASSES = (ROWS + RPP - 1) / RPP;
    constexpr int BATCH = PASSES < MAXB ? PASSES : MAXB;
    constexpr int DY = RPP % S, DZ = RPP / S;
    // every lane loads in every pass, also lanes whose value is not stored
    // (rr == RPW, rows past ROWS): the rows it visits are r0 + j RPP <=
    // PASSES RPP, so their z stays at most LZMAX
    constexpr int LZMAX = (PASSES * RPP) / S;
    const int lane = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6);
    const int rr = lane / S, lx = lane - rr * S;
    const bool act = rr < RPW;
    const int r0 = w * RPW + rr;
    const int m = n - 1;
    const int gx = (x0 + lx) & m;
    int ly = r0 % S, lz = r0 / S;       // (y, z) of this thread's current row
    const bool inside = x0 >= 0 && y0 >= 0 && z0 >= 0 && x0 + S <= n && y0 + S <= n &&
                        z0 + LZMAX < n;   // block-uniform
    const T *__restrict__ base = mesh + ((size_t)(inside ? z0 : 0) * n + (inside ? y0 : 0)) * n +
                                 (inside ? x0 : 0);
    const uint32_t nn = (uint32_t)n * (uint32_t)n;
    uint32_t off = (uint32_t)lz * nn + (uint32_t)ly * (uint32_t)n + (uint32_t)lx;
    const uint32_t dstep = (uint32_t)DY * (uint32_t)n + (uint32_t)DZ * nn;
    const uint32_t dwrap = nn - (uint32_t)S * (uint32_t)n;   // ly passed S: one z up
#pragma unroll
    for (int p0 = 0; p0 < PASSES; p0 += BATCH) {
        T v[BATCH];
        if (inside) {
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                v[k] = base[off];
                ly += DY;
                off += dstep;
                if (ly >= S) {
                    ly -= S;
                    off += dwrap;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                // the wrapped (y, z, x) is a node of the mesh for every lane
                const uint32_t row =
                    (uint32_t)((z0 + lz) & m) * (uint32_t)n + (uint32_t)((y0 + ly) & m);
                v[k] = mesh[row * (uint32_t)n + (uint32_t)gx];
                ly += DY;
                lz += DZ;
                if (ly >= S) {
                    ly -= S;
                    ++lz;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            const int r = r0 + (p0 + k) * RPP;
            if (act && p0 + k < PASSES && r < ROWS) dst[r * S + lx] = v[k];
        }
    }
}

// ---- launch helpers (host) -------------------------------------------------

#define CUBE2_CHECK_HIP(expr)                                  \
    do {                                                       \
        hipError_t e_ = (expr);                                \
        if (e_ != hipSuccess) return CUBE2_EHIP;               \
    } while (0)

#define CUBE2_LAUNCH_CHECK() CUBE2_CHECK_HIP(hipGetLastError())

// Host entry points of the kernel files (return CUBE2_* codes).
int launch_pack(cube2_ctx *ctx, const float *x, int64_t n, uint16_t *pos, uint32_t *cell_start,
                int32_t *perm, unsigned char *work, const WorkLayout &L, hipStream_t s);
// The stable sort by IOS cell of the keys (work) with the offsets of the
// unsorted particles (sort_offsets); with vel != NULL the final gather also forms the kicked
// velocities vel_out[i] = vel[p] + kick acc[p] (FP64, separately rounded) of
// the sorted particles, p = perm[i].  run != NULL (device): nothing is done
// where *run is 0.  counted: the first digit's block counts are in the
// histogram area.
int launch_sort_by_cell(cube2_ctx *ctx, int64_t n, uint16_t *pos, uint32_t *cell_start, int32_t *perm,
                        unsigned char *work, const WorkLayout &L, hipStream_t s,
                        const float *vel = nullptr, const float *acc = nullptr, double kick = 0.0,
                        float *vel_out = nullptr, const uint32_t *run = nullptr,
                        bool counted = false);
// as_f64: rho_f_fx and rho_c_fx receive the FP64 density instead of the integers
int launch_deposit(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                   float *rho_f, uint64_t *rho_f_fx, float *rho_c, uint64_t *rho_c_fx,
                   unsigned char *work, const WorkLayout &L, hipStream_t s, bool as_f64 = false);
int launch_green(cube2_ctx *ctx, hipStream_t s);
int launch_fft_r2c(cube2_ctx *ctx, int level, const float *mesh, float2 *spec, hipStream_t s);
int launch_potential(cube2_ctx *ctx, int level, const float *rho, float *phi, float2 *spec,
                     hipStream_t s);
int launch_potential64(cube2_ctx *ctx, int level, const double *rho, double *phi, double2 *spec,
                       hipStream_t s);
int launch_interp64(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                    const double *phi_f, const double *phi_c, double *acc, int accumulate,
                    hipStream_t s);
int launch_pp64(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n, double *acc,
                int accumulate, hipStream_t s);
// acc (+)= the interpolated force, + extra where that is given (3 n floats; the PP part,
// ready once ev_join has passed)
int launch_interp(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                  const float *phi_f, const float *phi_c, float *acc, int accumulate,
                  const float *extra, hipStream_t s);
// The PP kernels' order of the tiles (launch_order_tiles): heavy ones by estimated work,
// then the light ones, and a list of the heavy ones' parts.
struct PPOrder {
    uint32_t light_cap;    // light: every box of kPPLightLayers cell layers holds at most so many
    uint32_t smallest;     // own particles of the smallest part
    float pairs;           // candidate pairs per product of an x-row's particles and those around it
    float gain;            // pairs per staged particle that a part must have
    float chip, threads;   // workgroups that the chip holds, threads of each
    // set by launch_order_tiles (device): {heavy tiles, those of them in the list, its
    // entries}, and the list
    const uint32_t *counts;
    const uint32_t *parts;
};
int launch_order_tiles(cube2_ctx *ctx, const uint32_t *cs, unsigned char *work,
                       const WorkLayout &L, hipStream_t s, PPOrder *pp = nullptr);
int launch_reset_tile_queue(cube2_ctx *ctx, unsigned char *work, const WorkLayout &L,
                            hipStream_t s);
// Device-wide exclusive scan of m uint32 (in may equal out); tmp: the
// scan_tmp work region.
int launch_exclusive_scan(const uint32_t *in, uint32_t *out, int64_t m, uint32_t *tmp,
                          hipStream_t s);
int launch_interp_levels(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                         const float *phi_f, const float *phi_c, float *acc, int accumulate,
                         int levels, hipStream_t s);
int launch_tile_gather(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                       const int32_t *r0_host, int T, int R, float *x_local, int32_t *idx,
                       int64_t m_max, int64_t *m_out, unsigned char *work, const WorkLayout &L,
                       hipStream_t s);
// side k of the k^3 grid of slots that holds T tiles (a power of two)
int tile_slots(int T);
int launch_tile_scatter_add(int64_t m, const int32_t *perm_local, const float *x_local,
                            const int32_t *idx, int T, int lo, int hi, int n_slot, float scale,
                            const float *acc_local, float *acc, int64_t n, hipStream_t s);

// The tile order and work counter written by launch_order_tiles.
inline const uint32_t *tile_order_ptr(unsigned char *work, const WorkLayout &L) {
    return reinterpret_cast<const uint32_t *>(work + L.tile_order);
}
inline uint32_t *tile_queue_ptr(const cube2_ctx *ctx, unsigned char *work, const WorkLayout &L) {
    return reinterpret_cast<uint32_t *>(work + L.tile_order) + 4 * (size_t)ctx->nt * ctx->nt * ctx->nt;
}

// The XCDs' work counters (XcdShare), 8 of them 128 bytes apart, cleared by
// launch_order_tiles: in the part of the tile order region that the sort no
// longer needs (the keys and values before it).  Meshes of fewer tiles than
// kXcdQueueWords have none: their items are taken at fixed strides.
constexpr int kXcdQueueWords = 8 * 32;
inline uint32_t *xcd_queue_ptr(const cube2_ctx *ctx, unsigned char *work, const WorkLayout &L) {
    return reinterpret_cast<uint32_t *>(work + L.tile_order) + (size_t)ctx->nt * ctx->nt * ctx->nt;
}

// Workgroups of `kernel` (block threads, no dynamic LDS) that fit on the
// device at once, at most `ntiles`: the grid of a persistent launch.
template <typename K>
inline unsigned persistent_grid(K kernel, int block, int ntiles) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess)
        return (unsigned)ntiles;
    const long g = (long)(cus > 0 ? cus : 1) * (per_cu > 0 ? per_cu : 1);
    return (unsigned)(g < ntiles ? g : ntiles);
}
// max |x| over m > 0 floats into *out (device, zero before), as the bits of a
// non-negative float.
int launch_absmax(const float *x, int64_t m, unsigned int *out, hipStream_t s);
int vel_bulk_side(const cube2_ctx *ctx);
int vel_layout_check(const cube2_ctx *ctx, const WorkLayout &L);
int launch_vel_encode(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                      const float *vel, int16_t *vq, float *v_bulk, float *v_scale,
                      unsigned char *work, const WorkLayout &L, hipStream_t s);
int launch_vel_decode(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                      const int16_t *vq, const float *v_bulk, const float *v_scale, float *vel,
                      hipStream_t s);
int launch_pp_concurrent(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                         const float *abar, float *acc_pp, unsigned char *work, const WorkLayout &L,
                         hipStream_t s, hipStream_t order_stream);
// skip (device, one byte per tile, index (tz nt + ty) nt + tx, may be NULL):
// tiles whose own particles the kernel leaves alone
int launch_pp(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n, float *acc,
              int accumulate, unsigned char *work, const WorkLayout &L, hipStream_t s,
              const uint8_t *skip = nullptr);
// Address of the no-allocation entry point's scratch array on the current
// device (taken once per device); out may be NULL.
int noalloc_setup(unsigned char **out);
int build_pair_table(cube2_ctx *ctx);
int launch_pair_tables(cube2_ctx *ctx, hipStream_t s);
int launch_kick_drift(cube2_ctx *ctx, const uint16_t *pos_in, const uint32_t *cs_in,
                      const float *vel_in, const float *acc, int64_t n, double kick,
                      double drift, uint16_t *pos_out, uint32_t *cs_out, float *vel_out,
                      int32_t *perm_out, unsigned char *work, const WorkLayout &L,
                      hipStream_t s);
int launch_reduce(cube2_ctx *ctx, const float *vel, const float *acc, int64_t n, double *out8,
                  unsigned char *work, const WorkLayout &L, hipStream_t s);
int launch_deposit_backward(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                            int level, const float *rho_bar, float *x_bar, int accumulate,
                            hipStream_t s);
int launch_pm_backward(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                       const float *acc_bar, float *x_bar, int accumulate, unsigned char *work,
                       const WorkLayout &L, const float *extra, hipStream_t s);
int launch_pp_backward(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                       const float *acc_bar, float *x_bar, int accumulate, unsigned char *work,
                       const WorkLayout &L, hipStream_t s);
int launch_kick_drift_backward(cube2_ctx *ctx, int64_t n, const int32_t *perm,
                               const float *xbar_out, const float *vbar_out, double kick,
                               double drift, float *xbar_in, float *vbar_in, float *acc_bar,
                               hipStream_t s);

}  // namespace cube2

// kick.hip -- leapfrog kick and drift on integer positions (section 2.2.3:
// kick after each force, drift; section 2.3: positions and velocities at
// interlaced times, positions as in-cell integers), the re-sort that keeps
// the IOS order, and the FP64 diagnostics used for time-step control
// (section 3.2: the step follows the maximum acceleration and velocity).
//
// v' = v + kick * a and dq = rint(drift * v' * 2^15) are evaluated in FP64
// with separately rounded operations (FMA contraction is switched off in
// these kernels), so the integer displacement and the stored velocity are
// deterministic functions of the FP32 inputs.  A particle whose v' or
// displacement is not finite (a non-finite acceleration or velocity, or a
// displacement beyond 2^62 units) is not moved, and the status word records
// it (cube2_status then returns CUBE2_ENONFINITE).
#include <algorithm>

#include "common.hpp"

namespace cube2 {
namespace {

// One particle of IOS cell (cx, cy, cz) kicked and drifted: its new cell,
// offsets and velocity; bad is set if it could not be moved.
__device__ __forceinline__ void drifted(const uint16_t *__restrict__ pos, const float *__restrict__ vel,
                                        const float *__restrict__ acc, int n, uint32_t p, int cx, int cy,
                                        int cz, int n_f, double kick, double drift, int (&c)[3],
                                        uint16_t (&o)[3], float (&v)[3], bool &bad) {
#pragma clang fp contract(off)
    const int64_t mask = ((int64_t)n_f << kFracBits) - 1;   // a power of two less one
    const int uc[3] = {cx, cy, cz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int64_t i = (int64_t)d * n + p;
        const double kv = kick * (double)acc[i];
        const double v1 = (double)vel[i] + kv;
        double dq = rint((drift * v1) * 32768.0);
        if (!(fabs(dq) < 0x1p62)) {   // also NaN: the particle stays where it is
            dq = 0.0;
            bad = true;
        }
        const int64_t q = (((int64_t)uc[d] << 16) + pos[i] + (int64_t)dq) & mask;
        c[d] = (int)(q >> 16);
        o[d] = (uint16_t)(q & 0xFFFF);
        v[d] = (float)v1;
    }
}

// Tiles of more than `limit` particles, with which a step is the radix sort's: the entries
// {tile, slice} of all their slices of kHeavySlice.  One workgroup of the local re-sort
// takes ~15 ns a particle, the radix sort in its place ~15 ns per thousand of all
// (heavy_limit).  us, local and radix: 133 thousand, one tile of 7026 109 and 79; 8.5 million,
// one of 8063 372 and 484 (sorts of the whole key 98, 486).
constexpr uint32_t kHeavySlice = 2048;
struct HeavySlices {
    uint32_t *count;
    uint2 *list;
    uint32_t limit;
};

__global__ __launch_bounds__(kBlock) void kick_drift_kernel(
    const uint16_t *__restrict__ pos, const uint32_t *__restrict__ cs,
    const float *__restrict__ vel, const float *__restrict__ acc, int n, int nt, int n_f,
    double kick, double drift, uint32_t *__restrict__ keys, ushort4 *__restrict__ offs,
    uint32_t *__restrict__ status, HeavySlices heavy, const uint32_t *__restrict__ run) {
    __shared__ uint32_t cst[kTileCells + 1];
    if (run && *run == 0u) return;      // the fallback of the local re-sort, not needed
    const int tid = threadIdx.x;
    bool bad = false;
    const int ntiles = nt * nt * nt, items = ntiles + (run ? (int)*heavy.count : 0);
    for (int b = blockIdx.x; b < items; b += gridDim.x) {
        int tx, ty, tz;
        uint32_t slice = 0;
        if (b < ntiles) {
            tile_of_block(b, nt, tx, ty, tz);
        } else {
            const uint2 h = heavy.list[b - ntiles];
            tx = (int)h.x % nt;
            ty = ((int)h.x / nt) % nt;
            tz = (int)h.x / (nt * nt);
            slice = h.y;
        }
        const uint32_t key0 = (uint32_t)((tz * nt + ty) * nt + tx) * kTileCells;
        stage_cell_starts<kBlock>(cst, cs, key0);
        __syncthreads();
        uint32_t p0 = cst[0], p1 = cst[kTileCells];
        if (run && p1 - p0 > heavy.limit) {
            p0 = b < ntiles ? p1 : p0 + slice * kHeavySlice;
            p1 = min(p1, p0 + kHeavySlice);
        }
        for (uint32_t p = p0 + tid; p < p1; p += kBlock) {
            const int u = seg_search_n<kTileCells>(cst, p);
            int c[3];
            uint16_t o[3];
            float v1[3];
            drifted(pos, vel, acc, n, p, tx * kTileIos + (u & 7), ty * kTileIos + ((u >> 3) & 7),
                    tz * kTileIos + (u >> 6), n_f, kick, drift, c, o, v1, bad);
            offs[p] = make_ushort4(o[0], o[1], o[2], 0);
            keys[p] = cell_key(c[0], c[1], c[2], nt);
        }
        __syncthreads();
    }
    if (bad) atomicOr(status, kStatusNonFinite);
}

// ---------------------------------------------------------------------------
// The local re-sort: a step moves particles by a fraction of a tile, so a
// tile's new particles come from itself and its 26 neighbours, and two passes
// over the particles replace the passes of the radix sort (each a count
// and a scatter) and its final gather:
//   local_split   one workgroup per old tile kicks and drifts its particles
//                 and writes them, in their order, grouped by the tile they go
//                 to (27 groups, within the tile's own particle range); those that
//                 leave the 27 tiles come last, and a list tells their tiles;
//   local_starts  the new tiles' particle counts from the groups and the list, scanned;
//   local_merge   one workgroup per new tile sorts its up to 27 groups, taken
//                 in the order of their old tiles with the listed particles among
//                 them, stably by cell.
// Both orders are that of the input, so the result is the stable sort's.  If more
// particles than the list holds leave the 27 tiles, or more than a few into one tile, or a
// tile holds very many, the radix sort runs instead (its kernels are launched either way and end at once if
// they are not needed: the host does not wait), and the local kernels end as soon as
// they see it.  Both passes are bound by HBM, ~100 bytes per particle together; the
// radix sort moved ~200.  512^3 particles: 8.17 ms by a radix sort of the whole key (all
// particles far: 21.8), 4.1 so, 4.1 with one far particle (9.4 when one sent all to the
// radix sort), 21.7 with all.
// ---------------------------------------------------------------------------

constexpr int kDirs = 27;            // (dz + 1) * 9 + (dy + 1) * 3 + dx + 1
constexpr int kFarDir = kDirs;       // the group of those that leave the 27 tiles
constexpr uint32_t kFarMax = 2048;   // of them in the list
constexpr int kFarTile = 32;         // of them into one tile
constexpr int kSplitItems = 4;       // particles per thread and chunk
constexpr int kSplitChunk = kBlock * kSplitItems;
constexpr int kGroups = kSplitChunk / 64;   // waves' worths per chunk

// new tile minus old on one axis of nt tiles, -1..1 (with two tiles: 0 or 1);
// 2 if they are not neighbours
__device__ __forceinline__ int tile_step(int from, int to, int nt) {
    const int d = (to - from) & (nt - 1);
    return d == 0 ? 0 : (d == 1 ? 1 : (d == nt - 1 ? -1 : 2));
}

// tile t + (dx, dy, dz), periodic
__device__ __forceinline__ int tile_at(int tx, int ty, int tz, int nt) {
    const int m = nt - 1;
    return (((tz & m) * nt) + (ty & m)) * nt + (tx & m);
}

// Moved particles of the old tiles in group order: index, cell in the new tile,
// offsets and kicked velocity, SoA over n.
struct Moved {
    uint32_t *idx;
    uint16_t *cell, *offs;
    float *vel;
};

// Particles that left the 27 tiles around theirs: how many, and the new tile and the slot
// of each of the first kFarMax, in any order.
struct Far {
    uint32_t *count;
    uint2 *list;
};

__global__ void far_clear(uint32_t *count, uint32_t *heavy) {
    *count = 0u;
    *heavy = 0u;
}

// The heavy tiles' slices listed; if there are any the count of far particles is past its
// list, so that the local kernels end at once.  (Heavy tiles found by local_split itself let
// the tiles before them do their work in vain, a quarter of the step.)  A single workgroup
// (alone) also clears the counts; on a 512^3 mesh one took 75 us for the cell
// starts of 32768 tiles, each in a page of its own.
constexpr int kListBlock = 512;
__global__ __launch_bounds__(kListBlock) void list_heavy(const uint32_t *__restrict__ cs, int ntiles,
                                                         uint32_t *__restrict__ far_count,
                                                         HeavySlices heavy, bool alone) {
    __shared__ uint32_t found, base;
    const int t = (int)blockIdx.x * kListBlock + (int)threadIdx.x;
    if (threadIdx.x == 0) found = 0u;
    __syncthreads();
    const uint32_t cnt = t < ntiles ? cs[(size_t)(t + 1) * kTileCells] - cs[(size_t)t * kTileCells] : 0u;
    const uint32_t slices = cnt > heavy.limit ? (cnt + kHeavySlice - 1) / kHeavySlice : 0u;
    const uint32_t at = slices ? atomicAdd(&found, slices) : 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        base = 0u;
        if (alone) {
            *heavy.count = found;
            *far_count = found ? kFarMax + 1u : 0u;
        } else if (found) {
            base = atomicAdd(heavy.count, found);
            atomicMax(far_count, kFarMax + 1u);
        }
    }
    __syncthreads();
    for (uint32_t k = 0; k < slices; ++k) heavy.list[base + at + k] = make_uint2((uint32_t)t, k);
}

// pre[t * 28 + d]: first particle of group d (kFarDir: the far ones) relative to the
// tile's first.
__global__ __launch_bounds__(kBlock) void local_split(
    const uint16_t *__restrict__ pos, const uint32_t *__restrict__ cs,
    const float *__restrict__ vel, const float *__restrict__ acc, int n, int nt, int n_f,
    double kick, double drift, Moved out, uint32_t *__restrict__ pre, Far far,
    uint32_t *__restrict__ status) {
    __shared__ uint32_t cst[kTileCells + 1];
    __shared__ uint32_t cnt[kDirs + 1][kGroups + 1];   // per group of 64 particles, then before it
    __shared__ uint32_t base[kDirs + 1];               // next slot of each direction
    __shared__ uint32_t far_sh;
    int tx, ty, tz;
    tile_of_block(blockIdx.x, nt, tx, ty, tz);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t t = (uint32_t)((tz * nt + ty) * nt + tx);
    stage_cell_starts<kBlock>(cst, cs, t * kTileCells);
    if (tid == 0) far_sh = __hip_atomic_load(far.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid <= kDirs) base[tid] = 0u;
    __syncthreads();
    const uint32_t p0 = cst[0], p1 = cst[kTileCells];
    if (far_sh > kFarMax) return;      // the radix sort does it
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    bool bad = false;
    // a tile of one chunk keeps its particles in registers between the count
    // and the write; a denser one counts all its chunks first
    const bool one = p1 - p0 <= (uint32_t)kSplitChunk;
    for (int pass = one ? 1 : 0; pass < 2; ++pass) {
        for (uint32_t c0 = p0; c0 < p1; c0 += kSplitChunk) {
            int dir[kSplitItems], c[kSplitItems][3];
            uint16_t o[kSplitItems][3];
            float v1[kSplitItems][3];
            uint32_t rank[kSplitItems];
            for (int i = tid; i < (kDirs + 1) * (kGroups + 1); i += kBlock) (&cnt[0][0])[i] = 0u;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kSplitItems; ++k) {
                const uint32_t p = c0 + k * kBlock + tid;
                dir[k] = -1;
                if (p < p1) {
                    const int u = seg_search_n<kTileCells>(cst, p);
                    drifted(pos, vel, acc, n, p, tx * kTileIos + (u & 7),
                            ty * kTileIos + ((u >> 3) & 7), tz * kTileIos + (u >> 6), n_f, kick,
                            drift, c[k], o[k], v1[k], bad);
                    const int dx = tile_step(tx, c[k][0] >> 3, nt), dy = tile_step(ty, c[k][1] >> 3, nt),
                              dz = tile_step(tz, c[k][2] >> 3, nt);
                    dir[k] = dx == 2 || dy == 2 || dz == 2 ? kFarDir : (dz + 1) * 9 + (dy + 1) * 3 + dx + 1;
                }
                // rank among the group's earlier particles of the same direction
                uint64_t peers = __ballot(dir[k] >= 0);
#pragma unroll
                for (int b = 0; b < 5; ++b) {
                    const bool bit = (dir[k] >> b) & 1;
                    const uint64_t m = __ballot(bit);
                    peers &= bit ? m : ~m;
                }
                rank[k] = (uint32_t)__popcll(peers & lt);
                if (dir[k] >= 0 && rank[k] == 0)
                    cnt[dir[k]][k * (kBlock / 64) + w] = (uint32_t)__popcll(peers);
            }
            __syncthreads();
            if (tid <= kDirs) {
                uint32_t sum = 0;
#pragma unroll
                for (int g = 0; g < kGroups; ++g) {
                    const uint32_t v = cnt[tid][g];
                    cnt[tid][g] = sum;
                    sum += v;
                }
                cnt[tid][kGroups] = sum;
                if (pass == 0) base[tid] += sum;
            }
            __syncthreads();
            if (pass == 0) continue;
            if (one && tid < 64) {      // group starts from the chunk's counts
                uint32_t x = lane <= kDirs ? cnt[lane][kGroups] : 0u;
                const uint32_t v = x;
#pragma unroll
                for (int s = 1; s < 32; s <<= 1) {
                    const uint32_t y = __shfl_up(x, s, 64);
                    if (lane >= s) x += y;
                }
                if (lane <= kDirs) {
                    base[lane] = x - v;
                    pre[t * 28 + lane] = x - v;
                }
            }
            // one claim of the list's places per chunk
            if (tid == 0 && cnt[kFarDir][kGroups]) far_sh = atomicAdd(far.count, cnt[kFarDir][kGroups]);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kSplitItems; ++k) {
                if (dir[k] < 0) continue;
                const uint32_t p = c0 + k * kBlock + tid;
                const uint32_t s = p0 + base[dir[k]] + cnt[dir[k]][k * (kBlock / 64) + w] + rank[k];
                out.idx[s] = p;
                out.cell[s] = (uint16_t)(((c[k][2] & 7) * 8 + (c[k][1] & 7)) * 8 + (c[k][0] & 7));
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    out.offs[(int64_t)d * n + s] = o[k][d];
                    out.vel[(int64_t)d * n + s] = v1[k][d];
                }
                if (dir[k] == kFarDir) {
                    const uint32_t i = far_sh + cnt[kFarDir][k * (kBlock / 64) + w] + rank[k];
                    if (i < kFarMax)
                        far.list[i] = make_uint2((uint32_t)tile_at(c[k][0] >> 3, c[k][1] >> 3, c[k][2] >> 3, nt), s);
                }
            }
            __syncthreads();
            if (!one && tid <= kDirs) base[tid] += cnt[tid][kGroups];
            __syncthreads();
        }
        if (pass == 0) {                // counts to starts
            if (tid < 64) {
                uint32_t x = lane <= kDirs ? base[lane] : 0u;
                const uint32_t v = x;
#pragma unroll
                for (int s = 1; s < 32; s <<= 1) {
                    const uint32_t y = __shfl_up(x, s, 64);
                    if (lane >= s) x += y;
                }
                if (lane <= kDirs) {
                    base[lane] = x - v;
                    pre[t * 28 + lane] = x - v;
                }
            }
            __syncthreads();
        }
    }
    if (p0 == p1 && tid <= kDirs) pre[t * 28 + tid] = 0u;
    if (bad) atomicOr(status, kStatusNonFinite);
}

// Particle counts of the new tiles, scanned within blocks of kStartTiles tiles,
// with the blocks' sums and whether a tile of the block gets too many far particles.
constexpr int kStartTiles = 1024;
__global__ __launch_bounds__(kStartTiles) void local_starts(const uint32_t *__restrict__ pre, Far far, int nt,
                                                            uint32_t *__restrict__ starts,
                                                            uint32_t *__restrict__ sums,
                                                            uint32_t *__restrict__ fars) {
    __shared__ uint32_t sh[kStartTiles / 64 + 1];
    __shared__ uint32_t extra[kStartTiles];
    __shared__ uint32_t far_sh;
    const int ntiles = nt * nt * nt, t0 = (int)blockIdx.x * kStartTiles, t = t0 + (int)threadIdx.x;
    const uint32_t nfar = *far.count;
    if (nfar > kFarMax) return;
    if (threadIdx.x == 0) far_sh = 0u;
    extra[threadIdx.x] = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nfar; i += kStartTiles) {
        const uint32_t to = far.list[i].x - (uint32_t)t0;
        if (to < (uint32_t)kStartTiles) atomicAdd(&extra[to], 1u);
    }
    __syncthreads();
    uint32_t sum = 0;
    if (t < ntiles) {
        const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
        for (int d = 0; d < kDirs; ++d) {
            const int dx = d % 3 - 1, dy = (d / 3) % 3 - 1, dz = d / 9 - 1;
            const uint32_t *g = pre + (size_t)tile_at(tx - dx, ty - dy, tz - dz, nt) * 28 + d;
            sum += g[1] - g[0];
        }
        sum += extra[threadIdx.x];
        if (extra[threadIdx.x] > (uint32_t)kFarTile) far_sh = 1u;
    }
    uint32_t total;
    const uint32_t at = block_exclusive_scan<kStartTiles>(sum, sh, total);
    if (t < ntiles) starts[t] = at;
    __syncthreads();
    if (threadIdx.x == 0) {
        sums[blockIdx.x] = total;
        fars[blockIdx.x] = far_sh;
    }
}

// The new tile's groups and far particles in the order of their slots, which is that of
// their old tiles, sorted stably by cell (tile_cell_sort).
__global__ __launch_bounds__(kBlock) void local_merge(
    const uint32_t *__restrict__ cs, int n, int nt, Moved in, const uint32_t *__restrict__ pre,
    const uint32_t *__restrict__ starts, const uint32_t *__restrict__ sums,
    const uint32_t *__restrict__ fars, int nblocks, Far far, uint16_t *__restrict__ pos,
    uint32_t *__restrict__ cell_start, float *__restrict__ vel, int32_t *__restrict__ perm,
    uint32_t *__restrict__ run) {
    constexpr int W = kBlock / 64;
    __shared__ uint32_t hist[W][kTileCells];
    __shared__ uint32_t seg_pre[64], seg_src[64];  // groups in order: first element, first slot
    __shared__ uint32_t scan_sh[W + 1];
    __shared__ uint32_t red_sh[3], far_slot[kFarTile];
    int tx, ty, tz;
    tile_of_block(blockIdx.x, nt, tx, ty, tz);
    const int t = (tz * nt + ty) * nt + tx;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t nfar = *far.count;
    if (nfar > kFarMax) {            // the radix sort does it
        if (t == 0 && tid == 0) *run = 1u;
        return;
    }
    if (tid < 3) red_sh[tid] = 0u;
    __syncthreads();
    for (uint32_t i = tid; i < nfar; i += kBlock)
        if (far.list[i].x == (uint32_t)t) {
            const uint32_t k = atomicAdd(&red_sh[2], 1u);
            if (k < (uint32_t)kFarTile) far_slot[k] = far.list[i].y;
        }
    {   // start of the tile's block of tiles, and the flag (at most 256 blocks)
        const bool in_range = tid < nblocks;
        uint32_t s = in_range && tid < t / kStartTiles ? sums[tid] : 0u;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += (uint32_t)__shfl_xor((int)s, o, 64);
        const bool f = __ballot(in_range && fars[in_range ? tid : 0] != 0u) != 0ull;
        if (lane == 0) {
            atomicAdd(&red_sh[0], s);
            if (f) red_sh[1] = 1u;
        }
    }
    __syncthreads();
    const int nseg = kDirs + (int)min(red_sh[2], (uint32_t)kFarTile);
    if (w == 0) {
        // lane d: the group that came in direction d; then the far particles
        uint32_t cnt = 0, first = 0xFFFFFFFFu;
        if (lane < kDirs) {
            const int dx = lane % 3 - 1, dy = (lane / 3) % 3 - 1, dz = lane / 9 - 1;
            const uint32_t src = (uint32_t)tile_at(tx - dx, ty - dy, tz - dz, nt);
            const uint32_t a = pre[(size_t)src * 28 + lane];
            cnt = pre[(size_t)src * 28 + lane + 1] - a;
            first = cs[(size_t)src * kTileCells] + a;
        } else if (lane < nseg) {
            cnt = 1u;
            first = far_slot[lane - kDirs];
        }
        // (with fewer than three tiles per axis several directions meet the same
        // tile, but only one of them has particles: tile_step)
        uint32_t at = 0, rank = 0;
        for (int j = 0; j < nseg; ++j) {
            const uint32_t fj = (uint32_t)__builtin_amdgcn_readlane((int)first, j),
                           cj = (uint32_t)__builtin_amdgcn_readlane((int)cnt, j);
            if (fj < first || (fj == first && j < lane)) {
                at += cj;
                ++rank;
            }
        }
        if (lane < nseg) {
            seg_pre[rank] = at;
            seg_src[rank] = first;
        } else {
            seg_pre[lane] = 0xFFFFFFFFu;
        }
    }
    __syncthreads();
    if (t == 0 && tid == 0) *run = red_sh[1];
    if (red_sh[1]) return;           // the radix sort does it
    const uint32_t start = starts[t] + red_sh[0];
    // all of the tile's elements: the last group's end
    const uint32_t next = t + 1 < nt * nt * nt && (t + 1) % kStartTiles != 0
                              ? starts[t + 1] : sums[t / kStartTiles];
    const uint32_t total = next - starts[t];
    auto slot_of = [&](uint32_t e) {
        int s = nseg > 32 && seg_pre[32] <= e ? 32 : 0;
#pragma unroll
        for (int step = 16; step > 0; step >>= 1)
            if (seg_pre[s + step] <= e) s += step;
        return seg_src[s] + (e - seg_pre[s]);
    };
    tile_cell_sort(hist, scan_sh, total, start, start, cell_start + (size_t)t * kTileCells,
                   [&](uint32_t e) -> uint32_t { return in.cell[slot_of(e)]; },
                   [&](uint32_t e, uint32_t i) {
                       const uint32_t s = slot_of(e);
                       perm[i] = (int32_t)in.idx[s];
#pragma unroll
                       for (int d = 0; d < 3; ++d) {
                           pos[(int64_t)d * n + i] = in.offs[(int64_t)d * n + s];
                           vel[(int64_t)d * n + i] = in.vel[(int64_t)d * n + s];
                       }
                   });
    if (t == nt * nt * nt - 1 && tid == 0) cell_start[(size_t)(t + 1) * kTileCells] = (uint32_t)n;
}

constexpr int kRedBlocks = 1024;

// Per-block partial sums in FP64 over a fixed grid-stride partition, then a
// fixed-order tree: the result does not depend on scheduling.
__global__ __launch_bounds__(kBlock) void reduce_partial(const float *__restrict__ vel,
                                                         const float *__restrict__ acc, int n,
                                                         double *__restrict__ part) {
    __shared__ double sh[8][kBlock];
    double r[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        double v2 = 0.0, a2 = 0.0;
        for (int d = 0; d < 3; ++d) {
            const double v = vel ? (double)vel[(int64_t)d * n + i] : 0.0;
            const double a = (double)acc[(int64_t)d * n + i];
            r[d] += v;
            r[4 + d] += a;
            v2 += v * v;
            a2 += a * a;
        }
        r[3] += v2;
        r[7] = fmax(r[7], sqrt(a2));
    }
    for (int k = 0; k < 8; ++k) sh[k][threadIdx.x] = r[k];
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st)
            for (int k = 0; k < 8; ++k) {
                const double o = sh[k][threadIdx.x + st];
                sh[k][threadIdx.x] = (k == 7) ? fmax(sh[k][threadIdx.x], o) : sh[k][threadIdx.x] + o;
            }
        __syncthreads();
    }
    if (threadIdx.x < 8) part[(int64_t)blockIdx.x * 8 + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ void reduce_final(const double *__restrict__ part, int nb, double m,
                             double *__restrict__ out) {
    const int k = threadIdx.x;
    if (k >= 8) return;
    double s = 0.0;
    for (int b = 0; b < nb; ++b) {
        const double v = part[(int64_t)b * 8 + k];
        s = (k == 7) ? fmax(s, v) : s + v;
    }
    out[k] = (k == 3) ? 0.5 * m * s : (k == 7 ? s : m * s);
}

__global__ void kd_backward(const int32_t *__restrict__ perm, const float *__restrict__ xbo,
                            const float *__restrict__ vbo, int n, float kick, float drift,
                            float *__restrict__ xbi, float *__restrict__ vbi,
                            float *__restrict__ ab) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int p = perm[i];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int64_t o = (int64_t)d * n;
        const float xb = xbo[o + i];
        const float vb = vbo[o + i] + drift * xb;
        xbi[o + p] = xb;
        vbi[o + p] = vb;
        ab[o + p] = kick * vb;
    }
}

}  // namespace

// The local re-sort has a workgroup per tile in both passes; with only a few particles
// per tile the radix sort costs less.  us, local and radix: 34 per tile 254 and 166 on a
// 512^3 mesh, 43 and 33 on 128^3; 109 per tile 301 and 243, 43 and 34; 181 per tile, local,
// 350 (sorts of the whole key 395); 512 per tile 521 (869).
constexpr int64_t kLocalPerTile = 128;

int launch_kick_drift(cube2_ctx *ctx, const uint16_t *pos_in, const uint32_t *cs_in,
                      const float *vel_in, const float *acc, int64_t n64, double kick,
                      double drift, uint16_t *pos_out, uint32_t *cs_out, float *vel_out,
                      int32_t *perm_out, unsigned char *work, const WorkLayout &L,
                      hipStream_t s) {
    const int n = (int)n64;
    const int nt = ctx->nt;
    const int ntiles = nt * nt * nt;
    uint32_t *run = nullptr;
    HeavySlices heavy{nullptr, nullptr, heavy_limit(n64)};
    // Where neither a heavy tile nor, with at most two tiles per axis, a far particle is
    // possible, the radix sort's kernels are not launched: 16^3 mesh, 512 particles 47 us
    // with them, 22 without; so that also with a few particles per tile the local re-sort
    // is the faster there.  One heavy tile is left to the radix sort from the start.
    const bool heavies = n64 > (int64_t)heavy.limit, sure = nt <= 2 && !heavies;
    if (n > 0 && (sure || (n64 >= kLocalPerTile * (int64_t)ntiles && !(heavies && ntiles == 1)))) {
        // the groups and the tiles' tables take the places of the sort's
        // buffers and of the fine mesh
        Moved m;
        m.idx = reinterpret_cast<uint32_t *>(work + L.keys);
        m.cell = reinterpret_cast<uint16_t *>(work + L.vals);
        m.offs = reinterpret_cast<uint16_t *>(work + L.offs_tmp);
        m.vel = reinterpret_cast<float *>(work + L.acc_pp);
        // (29 words per tile and 516 of the mesh's 4096 per tile, then the list's 4096; one
        // tile, on the smallest mesh, has no far particles and so no list)
        uint32_t *pre = reinterpret_cast<uint32_t *>(work + L.real_f);
        uint32_t *starts = pre + (size_t)28 * ntiles, *sums = starts + ntiles, *fars = sums + 256;
        run = fars + 256;
        Far far;
        far.count = run + 1;
        heavy.count = run + 2;
        far.list = reinterpret_cast<uint2 *>(run + 4);
        heavy.list = reinterpret_cast<uint2 *>(work + L.keys2);   // at most 3 n / 4096 entries
        const int nblocks = (ntiles + kStartTiles - 1) / kStartTiles;
        const int lists = heavies ? (ntiles + kListBlock - 1) / kListBlock : 0;
        if (lists != 1) {
            far_clear<<<1, 1, 0, s>>>(far.count, heavy.count);
            CUBE2_LAUNCH_CHECK();
        }
        if (lists) {
            list_heavy<<<(unsigned)lists, kListBlock, 0, s>>>(cs_in, ntiles, far.count, heavy, lists == 1);
            CUBE2_LAUNCH_CHECK();
        }
        local_split<<<(unsigned)ntiles, kBlock, 0, s>>>(pos_in, cs_in, vel_in, acc, n, nt, ctx->n_f,
                                                        kick, drift, m, pre, far,
                                                        status_word(ctx));
        CUBE2_LAUNCH_CHECK();
        local_starts<<<(unsigned)nblocks, kStartTiles, 0, s>>>(pre, far, nt, starts, sums, fars);
        CUBE2_LAUNCH_CHECK();
        local_merge<<<(unsigned)ntiles, kBlock, 0, s>>>(cs_in, n, nt, m, pre, starts, sums, fars, nblocks,
                                                        far, pos_out, cs_out, vel_out, perm_out, run);
        CUBE2_LAUNCH_CHECK();
        if (sure) return CUBE2_OK;
    }
    if (n > 0) {
        kick_drift_kernel<<<(unsigned)(run ? std::min(ntiles, 2048) : ntiles), kBlock, 0, s>>>(
            pos_in, cs_in, vel_in, acc, n, nt, ctx->n_f, kick, drift,
            reinterpret_cast<uint32_t *>(work + L.keys), sort_offsets(work, L), status_word(ctx),
            heavy, run);
        CUBE2_LAUNCH_CHECK();
    }
    // the re-sort's final gather also forms the kicked velocities
    return launch_sort_by_cell(ctx, n, pos_out, cs_out, perm_out, work, L, s, vel_in, acc,
                               kick, vel_out, run);
}

int launch_reduce(cube2_ctx *ctx, const float *vel, const float *acc, int64_t n64, double *out8,
                  unsigned char *work, const WorkLayout &L, hipStream_t s) {
    const int n = (int)n64;
    double *part = reinterpret_cast<double *>(work + L.red);
    double *dout = part + (size_t)kRedBlocks * 8;
    if (n > 0) {
        reduce_partial<<<kRedBlocks, kBlock, 0, s>>>(vel, acc, n, part);
        CUBE2_LAUNCH_CHECK();
        reduce_final<<<1, 64, 0, s>>>(part, kRedBlocks, ctx->cfg.m_p, dout);
        CUBE2_LAUNCH_CHECK();
        CUBE2_CHECK_HIP(hipMemcpyAsync(out8, dout, 8 * sizeof(double), hipMemcpyDeviceToHost, s));
        CUBE2_CHECK_HIP(hipStreamSynchronize(s));
    } else {
        for (int k = 0; k < 8; ++k) out8[k] = 0.0;
    }
    return CUBE2_OK;
}

int launch_kick_drift_backward(cube2_ctx *ctx, int64_t n, const int32_t *perm,
                               const float *xbar_out, const float *vbar_out, double kick,
                               double drift, float *xbar_in, float *vbar_in, float *acc_bar,
                               hipStream_t s) {
    (void)ctx;
    kd_backward<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(perm, xbar_out, vbar_out, (int)n,
                                                          (float)kick, (float)drift, xbar_in,
                                                          vbar_in, acc_bar);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

}  // namespace cube2

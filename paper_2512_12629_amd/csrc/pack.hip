// pack.hip -- IOS particle order (section 2.3): quantise positions to integer
// in-cell offsets and sort particles stably by IOS cell, so that the particle
// order encodes cell membership and a prefix count per cell (cell_start)
// replaces per-particle cell indices.
//
// The sort is a stable radix sort of the cell key, written for 64-wide
// wavefronts: per 4096-key block a digit histogram, one scan per digit row, then
// a scatter in which each wave ranks its own 1024 keys by wave ballots (a
// 64-lane match on the digit) and counts of its own in LDS; the block's keys are
// staged in LDS in digit order and written out in runs.  It sorts by the tile
// only (two passes of up to 9 bits); one workgroup per tile then sorts the
// tile's particles by cell in LDS, which also gives cell_start, and gathers
// them; a tile of very many is left to several workgroups, by chunks.  One tile alone
// is sorted by the whole key and cell_start read off the sorted keys.  Ties keep their input order, so the
// result equals a stable argsort.  No global atomics.
#include <algorithm>

#include "common.hpp"

namespace cube2 {
namespace {

constexpr int kSortItems = 16;                   // keys per thread per block
constexpr int kSortTile = kBlock * kSortItems;   // 4096 keys per block
constexpr int kScanItems = 4;                    // items per thread in the scan
constexpr int kScanTile = kBlock * kScanItems;   // 1024

__global__ void fill_u32(uint32_t *p, uint32_t v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// q = floor(x * n_f * 2^15) mod (n_f * 2^15); key of the IOS cell; offsets; and
// the block's histogram of the first digit (BITS bits at `shift`) of the sort.
template <int BITS>
__global__ __launch_bounds__(kBlock) void quantize_kernel(const float *__restrict__ x, int n, int n_f,
                                                          int nt, uint32_t *__restrict__ keys,
                                                          ushort4 *__restrict__ offs, int shift,
                                                          int nblk, uint32_t *__restrict__ ghist) {
    __shared__ uint32_t h[1 << BITS];
    for (int i = threadIdx.x; i < (1 << BITS); i += kBlock) h[i] = 0;
    __syncthreads();
    const double span = (double)n_f * 32768.0;
    const int64_t mask = (int64_t)n_f * 32768 - 1;
#pragma unroll 4
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t i = (int64_t)blockIdx.x * kSortTile + r * kBlock + threadIdx.x;
        if (i >= n) break;
        int c[3];
        uint16_t o[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int64_t q = (int64_t)floor((double)x[(int64_t)d * n + i] * span) & mask;
            c[d] = (int)(q >> 16);
            o[d] = (uint16_t)(q & 0xFFFF);
        }
        offs[i] = make_ushort4(o[0], o[1], o[2], 0);   // one line per particle for the final gather
        const uint32_t key = cell_key(c[0], c[1], c[2], nt);
        keys[i] = key;
        atomicAdd(&h[(key >> shift) & ((1u << BITS) - 1u)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < (1 << BITS); i += kBlock) ghist[(int64_t)i * nblk + blockIdx.x] = h[i];
}

// Exclusive scan, phase 1: scan each 1024-element tile, record tile sums.
__global__ void scan_tiles(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                           int64_t m, uint32_t *__restrict__ sums) {
    __shared__ uint32_t sh[kBlock / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems], s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < m) ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t total;
    uint32_t pre = block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < m) out[base + k] = pre;
        pre += v[k];
    }
    if (threadIdx.x == 0 && sums) sums[blockIdx.x] = total;
}

__global__ void scan_add(uint32_t *__restrict__ out, int64_t m, const uint32_t *__restrict__ offs) {
    const int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
    const uint32_t o = offs[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t j = i + (int64_t)k * kBlock;
        if (j < m) out[j] += o;
    }
}

// Device-wide exclusive scan of m entries (in may equal out); tmp holds
// the per-level tile sums.
int exclusive_scan(const uint32_t *in, uint32_t *out, int64_t m, uint32_t *tmp, hipStream_t s) {
    const int64_t tiles = (m + kScanTile - 1) / kScanTile;
    if (tiles <= 1) {
        scan_tiles<<<1, kBlock, 0, s>>>(in, out, m, nullptr);
        CUBE2_LAUNCH_CHECK();
        return CUBE2_OK;
    }
    uint32_t *sums = tmp;
    scan_tiles<<<(unsigned)tiles, kBlock, 0, s>>>(in, out, m, sums);
    CUBE2_LAUNCH_CHECK();
    int r = exclusive_scan(sums, sums, tiles, tmp + align_up((size_t)tiles, 64), s);
    if (r) return r;
    scan_add<<<(unsigned)tiles, kBlock, 0, s>>>(out, m, sums);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

// A fallback's kernels run only if *run is not zero (run == NULL: always);
// their grids are then small, so that a launch that has nothing to do costs
// little, and every kernel strides over its blocks.
__device__ __forceinline__ bool runs(const uint32_t *run) { return !run || *run != 0u; }

template <int BITS>
__global__ __launch_bounds__(kBlock) void radix_count(const uint32_t *__restrict__ keys, int n, int shift,
                                                      int nblk, uint32_t *__restrict__ ghist,
                                                      const uint32_t *__restrict__ go) {
    __shared__ uint32_t h[1 << BITS];
    if (!runs(go)) return;
    for (int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        for (int i = threadIdx.x; i < (1 << BITS); i += kBlock) h[i] = 0;
        __syncthreads();
        const int64_t base = (int64_t)blk * kSortTile;
        for (int r = 0; r < kSortItems; ++r) {
            const int64_t i = base + r * kBlock + threadIdx.x;
            // later digits come in runs (of the earlier pass's order): lanes that
            // share the first lane's digit add once
            const uint32_t dig = i < n ? (keys[i] >> shift) & ((1u << BITS) - 1u) : ~0u;
            const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)dig);
            const uint64_t same = __ballot(dig == first);
            if (dig != first && i < n)
                atomicAdd(&h[dig], 1u);
            else if (dig == first && first != ~0u && (int)(threadIdx.x & 63) == first_lane(same))
                atomicAdd(&h[first], (uint32_t)__popcll(same));
        }
        __syncthreads();
        for (int i = threadIdx.x; i < (1 << BITS); i += kBlock) ghist[(int64_t)i * nblk + blk] = h[i];
        __syncthreads();
    }
}

// Exclusive scan of each digit's row of block counts, one workgroup per digit,
// and the row's total: the scatter adds the totals of the digits before.
constexpr int kRowBlock = 1024;
__global__ __launch_bounds__(kRowBlock) void radix_scan_rows(uint32_t *__restrict__ ghist, int nblk,
                                                             uint32_t *__restrict__ totals,
                                                             const uint32_t *__restrict__ run) {
    __shared__ uint32_t sh[kRowBlock / 64 + 1];
    if (!runs(run)) return;
    uint32_t *row = ghist + (int64_t)blockIdx.x * nblk;
    uint32_t carry = 0;
    for (int i0 = 0; i0 < nblk; i0 += kRowBlock) {
        const int i = i0 + (int)threadIdx.x;
        uint32_t total;
        const uint32_t pre = block_exclusive_scan<kRowBlock>(i < nblk ? row[i] : 0u, sh, total);
        if (i < nblk) row[i] = carry + pre;
        carry += total;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Scatter of one 4096-key block.  The row-scanned digit-major histogram goff
// and the digits' totals give each (digit, block) its global start.  Each wave
// ranks its own 1024 consecutive keys against its counts of the digits so far
// (wave ballots give the rank among equal digits of 64 keys), without a
// barrier; the waves' counts then give every key its place in digit order in
// LDS, from where consecutive threads write consecutive addresses of one digit's
// run.  vin == NULL: the values are the keys' own indices.  (With a barrier
// per 256 keys and the ranks of all four waves taken together the pass ran at
// 2.1 TB/s; 27 million keys 212 us.)
template <int BITS>
__global__ __launch_bounds__(kBlock) void radix_scatter(
    const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint32_t *__restrict__ kout,
    uint32_t *__restrict__ vout, int n, int shift, int nblk, const uint32_t *__restrict__ goff,
    uint32_t *__restrict__ totals, const uint32_t *__restrict__ go) {
    constexpr int BINS = 1 << BITS, W = kBlock / 64, PER = BINS / kBlock;
    __shared__ uint32_t gbase[BINS];       // global start of each digit of this block, less lpre
    __shared__ uint32_t lpre[BINS];        // block-local start of each digit
    __shared__ uint32_t wcnt[W][BINS];     // each wave's counts, then its start within the digit
    __shared__ uint32_t scan_sh[W + 1];
    __shared__ uint32_t sk[kSortTile], sv[kSortTile];
    if (!runs(go)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t dstart[PER], total, sum = 0;  // starts of digits tid PER + i
#pragma unroll
    for (int i = 0; i < PER; ++i) sum += totals[tid * PER + i];
    sum = block_exclusive_scan(sum, scan_sh, total);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        dstart[i] = sum;
        sum += totals[tid * PER + i];
    }
    if (blockIdx.x == 0 && tid == kBlock - 1) totals[BINS] = dstart[PER - 1];
    for (int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        for (int i = tid; i < W * BINS; i += kBlock) wcnt[i / BINS][i % BINS] = 0;
        __syncthreads();
        const int64_t blk0 = (int64_t)blk * kSortTile;
        const int cnt = (int)min((int64_t)kSortTile, (int64_t)n - blk0);
        uint32_t key[kSortItems], place[kSortItems];
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const int li = w * (kSortTile / W) + r * 64 + lane;
            key[r] = li < cnt ? kin[blk0 + li] : 0u;
        }
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const bool valid = w * (kSortTile / W) + r * 64 + lane < cnt;
            const uint32_t dig = (key[r] >> shift) & (BINS - 1);
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                const bool bit = (dig >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t rank = (uint32_t)__popcll(peers & lt);
            const uint32_t before = wcnt[w][dig];
            if (valid && rank == 0) wcnt[w][dig] = before + (uint32_t)__popcll(peers);
            place[r] = before + rank;
            // written before this wave's next loads (the LDS serves a wave in
            // order; this keeps the compiler from reordering them)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        uint32_t mine[PER], at = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            mine[i] = 0;
#pragma unroll
            for (int v = 0; v < W; ++v) {
                const uint32_t c = wcnt[v][tid * PER + i];
                wcnt[v][tid * PER + i] = mine[i];
                mine[i] += c;
            }
            at += mine[i];
        }
        at = block_exclusive_scan(at, scan_sh, total);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            lpre[tid * PER + i] = at;
            gbase[tid * PER + i] = dstart[i] + goff[(int64_t)(tid * PER + i) * nblk + blk] - at;
            at += mine[i];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const int li = w * (kSortTile / W) + r * 64 + lane;
            if (li >= cnt) continue;
            const uint32_t dig = (key[r] >> shift) & (BINS - 1);
            const uint32_t o = lpre[dig] + wcnt[w][dig] + place[r];
            sk[o] = key[r];
            sv[o] = vin ? vin[blk0 + li] : (uint32_t)(blk0 + li);
        }
        __syncthreads();
        for (int j = tid; j < cnt; j += kBlock) {
            const uint32_t k = sk[j];
            const uint32_t o = gbase[(k >> shift) & (BINS - 1)] + (uint32_t)j;
            kout[o] = k;
            vout[o] = sv[j];
        }
        __syncthreads();   // the next block's counts
    }
}

// Particle p to place i of the sorted ones; with vel, the kicked velocity vel[p] + kick
// acc[p] in FP64 with separately rounded operations (the value the kick-drift kernel
// drifted with).
__device__ __forceinline__ void put_particle(const ushort4 *__restrict__ offs, int n,
                                             uint16_t *__restrict__ pos, int32_t *__restrict__ perm,
                                             const float *__restrict__ vel, const float *__restrict__ acc,
                                             double kick, float *__restrict__ vout, uint32_t p,
                                             uint32_t i) {
#pragma clang fp contract(off)
    const ushort4 o = offs[p];
    perm[i] = (int32_t)p;
    pos[i] = o.x;
    pos[(int64_t)n + i] = o.y;
    pos[2 * (int64_t)n + i] = o.z;
    if (vel)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double kv = kick * (double)acc[(int64_t)d * n + p];
            vout[(int64_t)d * n + i] = (float)((double)vel[(int64_t)d * n + p] + kv);
        }
}

// Tiles of more than `limit` particles: the entries {tile, chunk} of all their chunks, a
// tile's in order, and each entry's counts of the cells.  A tile of T has at most 3 T / 4096
// chunks, so that 3 n / 4096 entries and 3 n / 8 counts hold any input.  (A chunk is the
// work of one workgroup, 39 us for 8192, but reads the counts of all chunks of its tile:
// from 65537 on they are larger.)
__device__ __forceinline__ uint32_t heavy_chunk(uint32_t total) { return total <= 65536u ? 2048u : 8192u; }
struct HeavyTiles {
    uint32_t *count;
    uint2 *list;
    uint32_t *hist;
    uint32_t limit;      // heavy_limit, at least 4096
};

// The particles of each tile (keys and vals sorted by tile) sorted by cell, with
// cell_start; offsets gathered, velocities kicked (put_particle).
constexpr int kTileStage = 1536;
__global__ __launch_bounds__(kBlock) void tile_sort_kernel(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals,
    const uint32_t *__restrict__ tstart, const ushort4 *__restrict__ offs, int n, int nt,
    uint16_t *__restrict__ pos, uint32_t *__restrict__ cell_start, int32_t *__restrict__ perm,
    const float *__restrict__ vel, const float *__restrict__ acc, double kick,
    float *__restrict__ vout, HeavyTiles heavy, const uint32_t *__restrict__ go) {
    __shared__ uint32_t hist[kBlock / 64][kTileCells];
    __shared__ uint32_t scan_sh[kBlock / 64 + 1];
    __shared__ uint32_t staged[kTileStage];   // sorted indices: the gather then runs without order
    __shared__ uint32_t at_sh;
    if (!runs(go)) return;
    const int ntiles = nt * nt * nt;
    for (int b = blockIdx.x; b < ntiles; b += gridDim.x) {
        int tx, ty, tz;
        tile_of_block(b, nt, tx, ty, tz);   // neighbouring tiles gather from the same lines
        const int t = (tz * nt + ty) * nt + tx;
        const uint32_t start = tstart[t], total = tstart[t + 1] - start;
        auto cell_of = [&](uint32_t e) -> uint32_t { return keys[start + e] % kTileCells; };
        auto put = [&](uint32_t p, uint32_t i) { put_particle(offs, n, pos, perm, vel, acc, kick, vout, p, i); };
        if (heavy.count && total > heavy.limit) {
            const uint32_t per = heavy_chunk(total), chunks = (total + per - 1) / per;
            if (threadIdx.x == 0) at_sh = atomicAdd(heavy.count, chunks);
            __syncthreads();
            for (uint32_t k = threadIdx.x; k < chunks; k += kBlock) heavy.list[at_sh + k] = make_uint2((uint32_t)t, k);
            if (t == ntiles - 1 && threadIdx.x == 0) cell_start[(size_t)ntiles * kTileCells] = (uint32_t)n;
            __syncthreads();
            continue;
        }
        if (total <= (uint32_t)kTileStage) {
            tile_cell_sort(hist, scan_sh, total, 0u, start, cell_start + (size_t)t * kTileCells, cell_of,
                           [&](uint32_t e, uint32_t i) { staged[i] = vals[start + e]; });
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < total; i += kBlock) put(staged[i], start + i);
        } else {
            tile_cell_sort(hist, scan_sh, total, start, start, cell_start + (size_t)t * kTileCells,
                           cell_of, [&](uint32_t e, uint32_t i) { put(vals[start + e], i); });
        }
        if (t == ntiles - 1 && threadIdx.x == 0) cell_start[(size_t)ntiles * kTileCells] = (uint32_t)n;
        __syncthreads();
    }
}

// The chunks of the heavy tiles: each chunk's counts of the cells; then each chunk to its
// place, which the counts of the tile's chunks before it and of its cells before give.
// (131072 of 2.1 million particles in one tile: one workgroup per tile 890 us, with the
// chunks 165; the radix sort of the whole key 209.  8682 of 133 thousand: 83 in chunks of
// 8192, 55 of 2048, whole key 67.  27 million with 1000 halos, tiles from 4097 on: 813, from
// 8193 on 797.  Where there is none the two launches cost 5 to 10 us.)
__global__ __launch_bounds__(kBlock) void heavy_count_kernel(const uint32_t *__restrict__ keys,
                                                             const uint32_t *__restrict__ tstart,
                                                             HeavyTiles heavy,
                                                             const uint32_t *__restrict__ go) {
    __shared__ uint32_t h[kTileCells];
    if (!runs(go)) return;
    const uint32_t entries = *heavy.count;
    for (uint32_t i = blockIdx.x; i < entries; i += gridDim.x) {
        const uint2 c = heavy.list[i];
        const uint32_t start = tstart[c.x], end = tstart[c.x + 1], per = heavy_chunk(end - start);
        const uint32_t e0 = start + c.y * per, e1 = min(e0 + per, end);
        for (int k = threadIdx.x; k < kTileCells; k += kBlock) h[k] = 0u;
        __syncthreads();
#pragma unroll 8
        for (uint32_t e = e0 + threadIdx.x; e < e1; e += kBlock) atomicAdd(&h[keys[e] % kTileCells], 1u);
        __syncthreads();
        for (int k = threadIdx.x; k < kTileCells; k += kBlock) heavy.hist[(size_t)i * kTileCells + k] = h[k];
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void heavy_sort_kernel(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals,
    const uint32_t *__restrict__ tstart, const ushort4 *__restrict__ offs, int n,
    uint16_t *__restrict__ pos, uint32_t *__restrict__ cell_start, int32_t *__restrict__ perm,
    const float *__restrict__ vel, const float *__restrict__ acc, double kick,
    float *__restrict__ vout, HeavyTiles heavy, const uint32_t *__restrict__ go) {
    __shared__ uint32_t hist[kBlock / 64][kTileCells];
    __shared__ uint32_t scan_sh[kBlock / 64 + 1];
    __shared__ uint32_t base[kTileCells];
    if (!runs(go)) return;
    const int tid = threadIdx.x;
    const uint32_t entries = *heavy.count;
    for (uint32_t i = blockIdx.x; i < entries; i += gridDim.x) {
        const uint2 c = heavy.list[i];
        const uint32_t start = tstart[c.x], total = tstart[c.x + 1] - start;
        const uint32_t per = heavy_chunk(total), chunks = (total + per - 1) / per, e0 = c.y * per,
                       cnt = min(per, total - e0);
        // thread tid: cells 2 tid, 2 tid + 1
        uint2 all = make_uint2(0u, 0u), before = all;
        const uint2 *h = reinterpret_cast<const uint2 *>(heavy.hist + (size_t)(i - c.y) * kTileCells) + tid;
#pragma unroll 8
        for (uint32_t k = 0; k < chunks; ++k) {
            const uint2 v = h[(size_t)k * (kTileCells / 2)];
            all.x += v.x;
            all.y += v.y;
            if (k < c.y) {
                before.x += v.x;
                before.y += v.y;
            }
        }
        uint32_t sum;
        const uint32_t at = block_exclusive_scan(all.x + all.y, scan_sh, sum);
        base[2 * tid] = at + before.x;
        base[2 * tid + 1] = at + all.x + before.y;
        if (c.y == 0) {
            cell_start[(size_t)c.x * kTileCells + 2 * tid] = start + at;
            cell_start[(size_t)c.x * kTileCells + 2 * tid + 1] = start + at + all.x;
        }
        __syncthreads();
        tile_cell_sort(hist, scan_sh, cnt, start, start, nullptr,
                       [&](uint32_t e) -> uint32_t { return keys[start + e0 + e] % kTileCells; },
                       [&](uint32_t e, uint32_t j) {
                           put_particle(offs, n, pos, perm, vel, acc, kick, vout, vals[start + e0 + e], j);
                       },
                       base);
        __syncthreads();
    }
}

// cell_start (shift = 0, n_cells entries and the end), or the tiles' starts
// (shift = 9), from the sorted keys: entry c is the first index whose key >> shift
// is >= c, so index i (0..n) writes the entries (key[i-1], key[i]] (with key[-1]
// = -1 and key[n] = n_cells).  Every entry has exactly one writer.  A run of
// more than 64 entries (a stretch of empty cells) is written by the whole
// wave, so that sparse inputs do not leave one lane writing most of the mesh.  A word
// that the next kernel counts in may be cleared as well.
__global__ void cell_starts_kernel(const uint32_t *__restrict__ keys, int n, int shift, int64_t n_cells,
                                   uint32_t *__restrict__ cell_start, uint32_t *__restrict__ clear,
                                   const uint32_t *__restrict__ run) {
    if (!runs(run)) return;
    if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0u;
    const int lane = threadIdx.x & 63;
    constexpr int PER = 4;                 // consecutive indices per lane
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x * PER; i0 <= n;
         i0 += (int64_t)gridDim.x * blockDim.x * PER) {
        const int64_t i1 = i0 + (int64_t)threadIdx.x * PER;
        uint4 k4 = make_uint4(0, 0, 0, 0);
        if (i1 + 3 < n)
            k4 = *reinterpret_cast<const uint4 *>(keys + i1);
        else if (i1 < n) {
            k4.x = keys[i1];
            k4.y = i1 + 1 < n ? keys[i1 + 1] : 0u;
            k4.z = i1 + 2 < n ? keys[i1 + 2] : 0u;
        }
        const uint32_t k[PER] = {k4.x >> shift, k4.y >> shift, k4.z >> shift, k4.w >> shift};
        uint32_t before = __shfl_up(k[PER - 1], 1, 64);
        if (lane == 0 && i1 > 0 && i1 <= n) before = keys[i1 - 1] >> shift;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int64_t i = i1 + j;
            int64_t lo = 0, hi = -1;
            if (i <= n) {
                lo = i == 0 ? 0 : (int64_t)(j ? k[j - 1] : before) + 1;
                hi = i == n ? n_cells : (int64_t)k[j];
            }
            const bool wide = hi - lo >= 64;
            if (!wide)
                for (int64_t c = lo; c <= hi; ++c) cell_start[c] = (uint32_t)i;
            uint64_t m = __ballot(wide);
            while (m) {
                const int l = __ffsll((long long)m) - 1;
                m &= m - 1;
                const long long a = __shfl((long long)lo, l, 64), b = __shfl((long long)hi, l, 64);
                const uint32_t v = (uint32_t)__shfl((int)i, l, 64);
                for (long long c = a + lane; c <= b; c += 64) cell_start[c] = v;
            }
        }
    }
}

__global__ void gather_offsets(const uint32_t *__restrict__ perm, const ushort4 *__restrict__ offs,
                               int n, uint16_t *__restrict__ pos, int32_t *__restrict__ perm_out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t p = perm[i];
    const ushort4 o = offs[p];
    pos[i] = o.x;
    pos[(int64_t)n + i] = o.y;
    pos[2 * (int64_t)n + i] = o.z;
    if (perm_out) perm_out[i] = (int32_t)p;
}

// gather_offsets and the kick of the velocities in one pass over the
// permutation: vout[i] = vel[p] + kick acc[p] in FP64 with separately rounded
// operations (the value the kick-drift kernel drifted with), p = perm[i].
__global__ void gather_offsets_kick(const uint32_t *__restrict__ perm,
                                    const ushort4 *__restrict__ offs, int n,
                                    uint16_t *__restrict__ pos, int32_t *__restrict__ perm_out,
                                    const float *__restrict__ vel, const float *__restrict__ acc,
                                    double kick, float *__restrict__ vout,
                                    const uint32_t *__restrict__ run) {
#pragma clang fp contract(off)
    if (!runs(run)) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = perm[i];
        const ushort4 q = offs[p];
        pos[i] = q.x;
        pos[(int64_t)n + i] = q.y;
        pos[2 * (int64_t)n + i] = q.z;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int64_t o = (int64_t)d * n;
            const double kv = kick * (double)acc[o + p];
            vout[o + i] = (float)((double)vel[o + p] + kv);
        }
        perm_out[i] = (int32_t)p;
    }
}

// Tiles in dispatch order b (the XCD-slab order of tile_of_block), keyed by
// how many thousand particles they own, largest first.
__global__ void tile_keys_kernel(const uint32_t *__restrict__ cs, int nt, uint32_t *__restrict__ keys,
                                 uint32_t *__restrict__ vals) {
    const int ntiles = nt * nt * nt;
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= ntiles) return;
    int tx, ty, tz;
    tile_of_block(b, nt, tx, ty, tz);
    const uint32_t t = (uint32_t)((tz * nt + ty) * nt + tx);
    const uint32_t cnt = cs[(t + 1) * kTileCells] - cs[t * kTileCells];
    keys[b] = 255u - min(cnt >> 10, 255u);
    vals[b] = t;
}

// ---------------------------------------------------------------------------
// The PP kernels' order.  A heavy tile's work is estimated in candidate pairs: the sum
// over its 64 x-rows of cells of their particles times those of the 9 rows around them
// (10 cells long; `pairs` scales it to the 3 or 5 cells in reach: between the 0.3 of a
// uniform density and the 1 of a halo inside one cell), and what staging its box costs.
// Tiles with the most work come first, and those with more than a share of the whole
// work per workgroup are listed in parts.  A part stages the whole box again, so a tile
// has at most as many as leave each `gain` pairs per staged particle: halos are split, a
// tile of a uniform density is not.  Where halos are so few that the neighbours of one
// particle would take half as long as the work per thread, their tiles are split as finely
// as they can be and lanes share a particle (kLanesBit); so they do in parts of at most
// half a block, and larger parts are whole blocks.
//
// The PP alone, us, with a rule on the number of heavy tiles alone (all in quarters of
// blocks up to 1024, in blocks up to 2048 or, two-cell reach, 4096, else the 128 with the
// most particles in 8 blocks), without any parts, and so.  The rule offered up to 32 parts
// for each heavy tile, at 14 ns a claim.
//   uniform, 0.53 / 0.6 / 1.0 particles per cell side: 128^3 cells 110 68 70, 227 78 73,
//   639 488 373; adjoint 134 82 86, 225 76 79, 785 461 454; two-cell reach 183 135 129,
//   280 182 129, 1420 2179 1336; 256^3 cells 769 205 220, 305 279 297, 2387 2220 2414.
//   halos of 2048: 256^3 cells with 5 170 695 162, 40 272 1184 249, 100 428 1172 404, 400
//   1139 2436 1156; adjoint 237 776 221, 350 1353 330, 606 1161 582, 1672 3283 1805;
//   two-cell reach 313 944 312, 583 1679 545, 839 1343 834, 1705 3941 1680; 512^3 with
//   1000 2884 2743 2829, adjoint 4588 4485 4485; two-cell reach 5481 5311 5192.
// Measured besides: gains of half and twice those of launch_pp_kernel_h (twice: uniform
// 64^3 cells at 0.7, 74 us instead of 50; half: adjoint of 128^3 at 0.56, 111 instead of
// 89); 2 shares (256^3 with 400 halos 1270 us) and 8 (1178).
// ---------------------------------------------------------------------------

constexpr float kStagePairs = 8.0f;    // pairs that staging a particle costs as much as
constexpr float kWorkShares = 4.0f;    // a part is at most the work per workgroup over this
constexpr uint32_t kNearLanes = 9;     // lanes share a particle from 2^9 neighbours on
constexpr uint32_t kWorkFirst = (127u + 12u) << 3;   // work class 0: 2^12 pairs, 8 classes an octave

// work class of a tile (0..254) and its middle
__device__ __forceinline__ uint32_t work_class(float w) {
    const uint32_t c = __float_as_uint(w) >> 20;
    return min(c > kWorkFirst ? c - kWorkFirst : 0u, 254u);
}
__device__ __forceinline__ float work_of_key(uint32_t key) {
    return __uint_as_float((kWorkFirst + 254u - min(key, 254u)) << 20 | 1u << 19);
}

// Keys of the tiles in dispatch order b, one wave per tile: light tiles get the last key,
// the others 254 less their work class; values: the tile, the parts that its particles make,
// the most that pay (each less one) and the log2 of the most neighbours, limited to 15.
// A tile is light if each of its boxes of kPPLightLayers layers of cells and the halo
// holds at most light_cap particles.
__global__ __launch_bounds__(256) void pp_tile_keys_kernel(const uint32_t *__restrict__ cs, int nt,
                                                           PPOrder pp, uint32_t *__restrict__ keys,
                                                           uint32_t *__restrict__ vals) {
    __shared__ uint32_t rows[4][100], own_rows[4][100];   // particles: 10 cells of an x-row, its own 8
    const int ntiles = nt * nt * nt;
    const int w = (int)(threadIdx.x >> 6), b = (int)blockIdx.x * 4 + w;
    const int lane = threadIdx.x & 63;
    if (b >= ntiles) return;
    int tx, ty, tz;
    tile_of_block(b, nt, tx, ty, tz);
    const uint32_t t = (uint32_t)((tz * nt + ty) * nt + tx);
    const int n_ios = nt * kTileIos;
    constexpr int NB = kTileIos / kPPLightLayers;
    uint32_t sum[NB] = {}, all = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {            // the 100 x-rows of the 10^3 box
        const int r = lane + 64 * k;
        if (r >= 100) break;
        const int by = r % 10, bz = r / 10;
        const int cy = wrapn(ty * kTileIos + by - 1, n_ios), cz = wrapn(tz * kTileIos + bz - 1, n_ios);
        const uint32_t a = cell_key(wrapn(tx * kTileIos - 1, n_ios), cy, cz, nt),
                       m = cell_key(tx * kTileIos, cy, cz, nt),
                       e = cell_key(wrapn(tx * kTileIos + 8, n_ios), cy, cz, nt);
        const uint32_t o = cs[m + 8] - cs[m], c = (cs[a + 1] - cs[a]) + o + (cs[e + 1] - cs[e]);
        rows[w][r] = c;
        own_rows[w][r] = o;
        all += c;
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (bz >= i * kPPLightLayers && bz < (i + 1) * kPPLightLayers + 2) sum[i] += c;
    }
    uint32_t most = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sum[i] += (uint32_t)__shfl_xor((int)sum[i], o, 64);
        most = max(most, sum[i]);
    }
    if (most <= pp.light_cap) {
        if (lane == 0) {
            keys[b] = 255u;
            vals[b] = t;
        }
        return;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the rows, before they are read
    __builtin_amdgcn_wave_barrier();
    const int r0 = (1 + (lane >> 3)) * 10 + 1 + (lane & 7);   // this lane's own row
    float near = 0.0f;
#pragma unroll
    for (int i = 0; i < 9; ++i) near += (float)rows[w][r0 + (i / 3 - 1) * 10 + i % 3 - 1];
    const float pairs = wave_sum((float)own_rows[w][r0] * near) * pp.pairs, staged = wave_sum((float)all);
    float nearest = own_rows[w][r0] ? near * pp.pairs : 0.0f;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) nearest = fmaxf(nearest, __shfl_xor(nearest, o, 64));
    if (lane == 0) {
        const uint32_t own = cs[(t + 1) * kTileCells] - cs[t * kTileCells];
        const uint32_t by_own = min((own + pp.smallest - 1) / pp.smallest, kMaxParts),
                       by_gain = (uint32_t)fminf(pairs / (pp.gain * staged), (float)by_own);
        const uint32_t log_near = min(31u - (uint32_t)__clz((int)max((uint32_t)nearest, 1u)), 15u);
        keys[b] = 254u - work_class(pairs + kStagePairs * staged);
        vals[b] = t | (max(by_own, 1u) - 1u) << kTileBits |
                  (max(by_gain, 1u) - 1u) << (kTileBits + kPartBits) | log_near << (kTileBits + 2 * kPartBits);
    }
}

constexpr int kOrderBlock = 1024, kOrderOne = 4 * kOrderBlock;

// The whole work, from each thread's part of it.
__device__ __forceinline__ float whole_work(float work, float *sh /*kOrderBlock / 64*/) {
    work = wave_sum(work);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = work;
    __syncthreads();
    float all = 0.0f;
#pragma unroll
    for (int v = 0; v < kOrderBlock / 64; ++v) all += sh[v];
    return fmaxf(all, 1.0f);
}

// The list of the parts of the first heavy tiles in the order (kOrderOne of them at most,
// and as many as the list holds); key(i) and val(i) are the i-th tile's.
template <class Key, class Val>
__device__ __forceinline__ void list_parts(uint32_t n_heavy, float work, const PPOrder &pp, Key key, Val val,
                                           uint32_t *__restrict__ parts, uint32_t *__restrict__ counts,
                                           uint32_t *scan_sh) {
    constexpr int PER = kOrderOne / kOrderBlock;
    const float rate = kWorkShares * pp.chip / work, per_thread = work / (pp.chip * pp.threads);
    uint32_t v[PER], k[PER], sum = 0, total;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t i = threadIdx.x * PER + j;
        k[j] = v[j] = 0u;
        if (i < n_heavy) {
            const uint32_t x = val(i), by_own = (x >> kTileBits & (kMaxParts - 1u)) + 1u,
                           by_gain = (x >> (kTileBits + kPartBits) & (kMaxParts - 1u)) + 1u,
                           log_near = x >> (kTileBits + 2 * kPartBits);
            const float want = ceilf(fminf(work_of_key(key(i)) * rate, (float)kMaxParts));
            bool lanes = log_near >= kNearLanes && (float)(2u << log_near) >= per_thread;
            k[j] = lanes ? by_own : max(min((uint32_t)want, by_gain), 1u);
            if (!lanes && k[j] > 1u) {       // whole blocks, or parts of at most half a one
                lanes = 2u * k[j] >= by_own;
                if (!lanes) k[j] = min(k[j], (by_own + 3u) / 4u);
            }
            v[j] = (x & kTileMask) | (lanes ? kLanesBit : 0u) | (k[j] - 1u) << (kTileBits + kPartBits);
        }
        sum += k[j];
    }
    uint32_t at = block_exclusive_scan<kOrderBlock>(sum, scan_sh, total);
    uint32_t in = 0, entries = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (k[j] && at + k[j] <= (uint32_t)kPPListMax) {
            for (uint32_t p = 0; p < k[j]; ++p) parts[at + p] = v[j] | p << kTileBits;
            ++in;
            entries += k[j];
        }
        at += k[j];
    }
    uint32_t all_in, all_entries;
    block_exclusive_scan<kOrderBlock>(in, scan_sh, all_in);
    block_exclusive_scan<kOrderBlock>(entries, scan_sh, all_entries);
    if (threadIdx.x == 0) {
        counts[1] = all_in;
        counts[2] = all_entries;
    }
}

// The list for an order made by a radix pass: totals are the tiles of each key, sorted the
// sorted keys.
__global__ __launch_bounds__(kOrderBlock) void pp_parts_kernel(
    const uint32_t *__restrict__ totals, const uint32_t *__restrict__ sorted,
    const uint32_t *__restrict__ order, PPOrder pp, uint32_t *__restrict__ counts,
    uint32_t *__restrict__ parts) {
    __shared__ uint32_t scan_sh[kOrderBlock / 64 + 1];
    __shared__ float sum_sh[kOrderBlock / 64];
    const int tid = threadIdx.x;
    const float work = whole_work(tid < 255 ? (float)totals[tid] * work_of_key((uint32_t)tid) : 0.0f, sum_sh);
    list_parts(counts[0], work, pp, [&](uint32_t i) { return sorted[i]; }, [&](uint32_t i) { return order[i]; },
               parts, counts, scan_sh);
}

// The order of up to kOrderOne tiles by their keys in one workgroup, in place of
// the three launches of a radix pass: each wave ranks its tiles as the radix
// scatter does.  keys == NULL: the key of a tile is its particles in thousands,
// most first (tile_keys_kernel).  Else vals are the tiles' words, counts[0] receives
// where the last key starts, and the list of parts is made.
__global__ __launch_bounds__(kOrderBlock) void order_tiles_kernel(
    const uint32_t *__restrict__ cs, const uint32_t *__restrict__ keys,
    const uint32_t *__restrict__ vals, int nt, uint32_t *__restrict__ order,
    uint32_t *__restrict__ queue, uint32_t *__restrict__ xcd_queue, PPOrder pp,
    uint32_t *__restrict__ counts, uint32_t *__restrict__ parts) {
    constexpr int W = kOrderBlock / 64, PER = kOrderOne / kOrderBlock;
    __shared__ uint32_t wcnt[W][256];
    __shared__ uint32_t scan_sh[W + 1];
    __shared__ float sum_sh[W];
    __shared__ uint32_t sv[kOrderOne];       // the sorted tiles' words
    __shared__ uint8_t sk[kOrderOne];        // and keys
    const int ntiles = nt * nt * nt, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int i = tid; i < W * 256; i += kOrderBlock) wcnt[i / 256][i % 256] = 0;
    const int per = (ntiles + 64 * W - 1) / (64 * W);   // rounds of 64 tiles per wave
    uint32_t key[PER], tile[PER], place[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int b = (w * per + r) * 64 + lane;
        key[r] = 256u;
        tile[r] = 0;
        if (r < per && b < ntiles) {
            if (keys) {
                tile[r] = vals[b];
                key[r] = keys[b];
            } else {
                int tx, ty, tz;
                tile_of_block(b, nt, tx, ty, tz);
                tile[r] = (uint32_t)((tz * nt + ty) * nt + tx);
                key[r] = 255u - min((cs[(tile[r] + 1) * kTileCells] - cs[tile[r] * kTileCells]) >> 10, 255u);
            }
        }
    }
    __syncthreads();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        uint64_t peers = __ballot(key[r] < 256u);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (key[r] >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        const uint32_t before = wcnt[w][key[r] & 255u];
        if (key[r] < 256u && rank == 0) wcnt[w][key[r]] = before + (uint32_t)__popcll(peers);
        place[r] = before + rank;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // as in radix_scatter
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t mine = 0, total;
    if (tid < 256) {
#pragma unroll
        for (int v = 0; v < W; ++v) mine += wcnt[v][tid];
    }
    uint32_t at = block_exclusive_scan<kOrderBlock>(mine, scan_sh, total);
    const uint32_t key_start = at;
    if (tid < 256) {
#pragma unroll
        for (int v = 0; v < W; ++v) {
            const uint32_t c = wcnt[v][tid];
            wcnt[v][tid] = at;
            at += c;
        }
    }
    if (tid == 0) *queue = 0u;
    if (xcd_queue && tid < kXcdQueueWords) xcd_queue[tid] = 0u;
    __shared__ uint32_t heavy_sh;
    if (tid == 255) heavy_sh = key_start;
    __syncthreads();
    const bool list = keys && heavy_sh != 0u;
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (key[r] < 256u) {
            const uint32_t i = wcnt[w][key[r]] + place[r];
            order[i] = tile[r];
            if (list) {
                sv[i] = tile[r];
                sk[i] = (uint8_t)key[r];
            }
        }
    if (keys && tid == 0) counts[0] = heavy_sh;
    if (!list) {
        if (keys && tid == 0) counts[1] = counts[2] = 0u;
        return;
    }
    const float work = whole_work(tid < 255 ? (float)mine * work_of_key((uint32_t)tid) : 0.0f, sum_sh);
    list_parts(heavy_sh, work, pp, [&](uint32_t i) { return (uint32_t)sk[i]; }, [&](uint32_t i) { return sv[i]; },
               parts, counts, scan_sh);
}

}  // namespace

int launch_exclusive_scan(const uint32_t *in, uint32_t *out, int64_t m, uint32_t *tmp,
                          hipStream_t s) {
    return exclusive_scan(in, out, m, tmp, s);
}

namespace {

// workgroups of a kernel that may have nothing to do
unsigned strided(int64_t blocks, const uint32_t *run) {
    return (unsigned)(run ? std::min<int64_t>(blocks, 2048) : blocks);
}

// One stable pass over the BITS-bit digit at `shift` of n keys: counts (unless
// they are there already), rows, scatter.  totals: 2^BITS + 1 words; the last
// receives the start of the last digit.
template <int BITS>
int radix_pass(const uint32_t *kin, const uint32_t *vin, uint32_t *kout, uint32_t *vout, int n,
               int shift, uint32_t *ghist, uint32_t *totals, const uint32_t *run, hipStream_t s,
               bool counted = false) {
    const int nblk = (n + kSortTile - 1) / kSortTile;
    if (!counted) {
        radix_count<BITS><<<strided(nblk, run), kBlock, 0, s>>>(kin, n, shift, nblk, ghist, run);
        CUBE2_LAUNCH_CHECK();
    }
    radix_scan_rows<<<1 << BITS, kRowBlock, 0, s>>>(ghist, nblk, totals, run);
    CUBE2_LAUNCH_CHECK();
    radix_scatter<BITS><<<strided(nblk, run), kBlock, 0, s>>>(kin, vin, kout, vout, n, shift, nblk,
                                                              ghist, totals, run);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

// How the particles are sorted: by tile in `passes` digits of `bits` bits from
// key bit `shift` on and then by cell within the tiles, or (one tile) by the whole
// key, 8 bits a pass.  (By the whole key also where a tile has less than 64 particles, pack
// took, us, on a 64^3 mesh with 729 particles 44 and not 24, 256^3 with 8000 123 and 53, with
// 54872 86 and 59, 512^3 with 64000 131 and 109; with 0.44 million 109 and not 115.)
struct SortPlan {
    bool by_tile;
    int bits, shift, passes;
};
SortPlan sort_plan(const cube2_ctx *ctx, int64_t n) {
    const int64_t ntiles = (int64_t)ctx->nt * ctx->nt * ctx->nt;
    int bits = 0;
    while (((int64_t)kTileCells << bits) < ctx->n_cells) ++bits;
    SortPlan p;
    p.by_tile = bits > 0;
    p.shift = p.by_tile ? 9 : 0;
    const int all = p.by_tile ? bits : bits + 9;
    p.bits = p.by_tile && (all == 9 || all > 16) ? 9 : 8;   // 18 bits in two passes
    p.passes = (all + p.bits - 1) / p.bits;
    return p;
}

}  // namespace

// Work order of the persistent per-tile kernels: the tiles sorted (stably,
// one 8-bit radix pass) by their particle count in units of 1024, descending,
// so that the heaviest tiles start first and the light ones keep the
// XCD-slab order; for the PP kernels by work, with a list of parts (PPOrder).  The
// tile words land in the first ntiles words of the tile_order region; the work
// counter (tile_queue_ptr) is reset to zero.
int launch_order_tiles(cube2_ctx *ctx, const uint32_t *cs, unsigned char *work,
                       const WorkLayout &L, hipStream_t s, PPOrder *pp) {
    const int nt = ctx->nt;
    const int ntiles = nt * nt * nt;
    uint32_t *base = reinterpret_cast<uint32_t *>(work + L.tile_order);
    uint32_t *order = base, *vin = base + ntiles, *kin = base + 2 * ntiles, *kout = base + 3 * ntiles;
    uint32_t *tmp = reinterpret_cast<uint32_t *>(work + L.scan_tmp);
    uint32_t *ghist = reinterpret_cast<uint32_t *>(work + L.hist);
    uint32_t *xcd_queue = ntiles >= kXcdQueueWords ? xcd_queue_ptr(ctx, work, L) : nullptr;
    uint32_t *counts = tmp + 256;   // a radix pass writes where the last key starts there
    uint32_t *parts = reinterpret_cast<uint32_t *>(work + L.tile_parts);
    if (pp) {
        pp->counts = counts;
        pp->parts = parts;
        pp_tile_keys_kernel<<<(ntiles + 3) / 4, 256, 0, s>>>(cs, nt, *pp, kin, vin);
        CUBE2_LAUNCH_CHECK();
    }
    if (ntiles <= kOrderOne) {
        // (vin is read before the counters in its place are cleared)
        order_tiles_kernel<<<1, kOrderBlock, 0, s>>>(cs, pp ? kin : nullptr, vin, nt, order,
                                                     tile_queue_ptr(ctx, work, L), xcd_queue,
                                                     pp ? *pp : PPOrder{}, counts, parts);
        CUBE2_LAUNCH_CHECK();
        return CUBE2_OK;
    }
    if (!pp) {
        tile_keys_kernel<<<(ntiles + 255) / 256, 256, 0, s>>>(cs, nt, kin, vin);
        CUBE2_LAUNCH_CHECK();
    }
    const int r = radix_pass<8>(kin, vin, kout, order, ntiles, 0, ghist, tmp, nullptr, s);
    if (r) return r;
    if (pp) {
        pp_parts_kernel<<<1, kOrderBlock, 0, s>>>(tmp, kout, order, *pp, counts, parts);
        CUBE2_LAUNCH_CHECK();
    }
    if (xcd_queue) {
        fill_u32<<<1, kXcdQueueWords, 0, s>>>(xcd_queue, 0u, kXcdQueueWords);
        CUBE2_LAUNCH_CHECK();
    }
    return launch_reset_tile_queue(ctx, work, L, s);
}

int launch_reset_tile_queue(cube2_ctx *ctx, unsigned char *work, const WorkLayout &L,
                            hipStream_t s) {
    fill_u32<<<1, 64, 0, s>>>(tile_queue_ptr(ctx, work, L), 0u, 1);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

// keys and sort_offsets (work) hold the unsorted particles.
int launch_sort_by_cell(cube2_ctx *ctx, int64_t n64, uint16_t *pos, uint32_t *cell_start,
                        int32_t *perm, unsigned char *work,
                        const WorkLayout &L, hipStream_t s, const float *vel, const float *acc,
                        double kick, float *vel_out, const uint32_t *run, bool counted) {
    const int n = (int)n64;
    uint32_t *tmp = reinterpret_cast<uint32_t *>(work + L.scan_tmp);
    uint32_t *k0 = reinterpret_cast<uint32_t *>(work + L.keys);
    uint32_t *v0 = reinterpret_cast<uint32_t *>(work + L.vals);
    uint32_t *k1 = reinterpret_cast<uint32_t *>(work + L.keys2);
    uint32_t *v1 = reinterpret_cast<uint32_t *>(work + L.vals2);
    uint32_t *ghist = reinterpret_cast<uint32_t *>(work + L.hist);
    const ushort4 *offs = sort_offsets(work, L);
    int r = CUBE2_OK;
    if (n == 0) {
        cell_starts_kernel<<<1, 64, 0, s>>>(k0, 0, 0, ctx->n_cells, cell_start, nullptr, nullptr);
        CUBE2_LAUNCH_CHECK();
        return CUBE2_OK;
    }

    const SortPlan plan = sort_plan(ctx, n);
    const uint32_t *vin = nullptr;      // the first pass takes the keys' indices
    for (int k = 0; k < plan.passes; ++k) {
        const int shift = plan.shift + k * plan.bits;
        const bool have = counted && k == 0;
        r = plan.bits == 9 ? radix_pass<9>(k0, vin, k1, v1, n, shift, ghist, tmp, run, s, have)
                           : radix_pass<8>(k0, vin, k1, v1, n, shift, ghist, tmp, run, s, have);
        if (r) return r;
        uint32_t *t = k0; k0 = k1; k1 = t;
        t = v0; v0 = v1; v1 = t;
        vin = v0;
    }
    if (plan.by_tile) {
        const int ntiles = ctx->nt * ctx->nt * ctx->nt;
        uint32_t *tstart = reinterpret_cast<uint32_t *>(work + L.tile_order);
        // (in the buffers that the sorted keys and values are not in)
        HeavyTiles heavy{nullptr, nullptr, nullptr, heavy_limit(n)};
        if (n > (int)heavy.limit) {
            heavy.count = tmp;
            heavy.list = reinterpret_cast<uint2 *>(v1);
            heavy.hist = k1;
        }
        cell_starts_kernel<<<strided(((int64_t)n + 1 + 1023) / 1024, run), 256, 0, s>>>(k0, n, 9, ntiles, tstart,
                                                                                      heavy.count, run);
        CUBE2_LAUNCH_CHECK();
        tile_sort_kernel<<<strided(ntiles, run), kBlock, 0, s>>>(k0, v0, tstart, offs, n, ctx->nt, pos,
                                                                 cell_start, perm, vel, acc, kick,
                                                                 vel_out, heavy, run);
        CUBE2_LAUNCH_CHECK();
        if (heavy.count) {
            const unsigned blocks = (unsigned)std::min(2048, n / 2048);
            heavy_count_kernel<<<blocks, kBlock, 0, s>>>(k0, tstart, heavy, run);
            CUBE2_LAUNCH_CHECK();
            heavy_sort_kernel<<<blocks, kBlock, 0, s>>>(k0, v0, tstart, offs, n, pos, cell_start, perm, vel,
                                                        acc, kick, vel_out, heavy, run);
            CUBE2_LAUNCH_CHECK();
        }
        return CUBE2_OK;
    }
    // cell_start (n_cells + 1 entries, the last = n) from the sorted keys
    cell_starts_kernel<<<strided(((int64_t)n + 1 + 1023) / 1024, run), 256, 0, s>>>(
        k0, n, 0, ctx->n_cells, cell_start, nullptr, run);
    CUBE2_LAUNCH_CHECK();
    if (vel)
        gather_offsets_kick<<<strided(((int64_t)n + 255) / 256, run), 256, 0, s>>>(
            v0, offs, n, pos, perm, vel, acc, kick, vel_out, run);
    else
        gather_offsets<<<(n + 255) / 256, 256, 0, s>>>(v0, offs, n, pos, perm);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

int launch_pack(cube2_ctx *ctx, const float *x, int64_t n64, uint16_t *pos, uint32_t *cell_start,
                int32_t *perm, unsigned char *work, const WorkLayout &L, hipStream_t s) {
    const int n = (int)n64;
    ushort4 *offs = sort_offsets(work, L);
    if (n > 0) {
        const SortPlan plan = sort_plan(ctx, n);
        const int nblk = (n + kSortTile - 1) / kSortTile;
        auto k = plan.bits == 9 ? quantize_kernel<9> : quantize_kernel<8>;
        k<<<nblk, kBlock, 0, s>>>(x, n, ctx->n_f, ctx->nt, reinterpret_cast<uint32_t *>(work + L.keys),
                                  offs, plan.shift, nblk, reinterpret_cast<uint32_t *>(work + L.hist));
        CUBE2_LAUNCH_CHECK();
    }
    return launch_sort_by_cell(ctx, n, pos, cell_start, perm, work, L, s, nullptr, nullptr, 0.0,
                               nullptr, nullptr, true);
}

}  // namespace cube2

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
// them.  With few particles per tile it sorts by the whole key instead and
// reads cell_start off the sorted keys.  Ties keep their input order, so the
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

// The particles of each tile (keys and vals sorted by tile) sorted by cell, with
// cell_start; offsets gathered and, with vel, the kicked velocities formed as
// vel[p] + kick acc[p] in FP64 with separately rounded operations (the value
// the kick-drift kernel drifted with).
constexpr int kTileStage = 1536;
__global__ __launch_bounds__(kBlock) void tile_sort_kernel(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals,
    const uint32_t *__restrict__ tstart, const ushort4 *__restrict__ offs, int n, int nt,
    uint16_t *__restrict__ pos, uint32_t *__restrict__ cell_start, int32_t *__restrict__ perm,
    const float *__restrict__ vel, const float *__restrict__ acc, double kick,
    float *__restrict__ vout, const uint32_t *__restrict__ go) {
#pragma clang fp contract(off)
    __shared__ uint32_t hist[kBlock / 64][kTileCells];
    __shared__ uint32_t scan_sh[kBlock / 64 + 1];
    __shared__ uint32_t staged[kTileStage];   // sorted indices: the gather then runs without order
    if (!runs(go)) return;
    const int ntiles = nt * nt * nt;
    for (int b = blockIdx.x; b < ntiles; b += gridDim.x) {
        int tx, ty, tz;
        tile_of_block(b, nt, tx, ty, tz);   // neighbouring tiles gather from the same lines
        const int t = (tz * nt + ty) * nt + tx;
        const uint32_t start = tstart[t], total = tstart[t + 1] - start;
        auto cell_of = [&](uint32_t e) -> uint32_t { return keys[start + e] % kTileCells; };
        auto put = [&](uint32_t p, uint32_t i) {
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
        };
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

// cell_start (shift = 0, n_cells entries and the end), or the tiles' starts
// (shift = 9), from the sorted keys: entry c is the first index whose key >> shift
// is >= c, so index i (0..n) writes the entries (key[i-1], key[i]] (with key[-1]
// = -1 and key[n] = n_cells).  Every entry has exactly one writer.  A run of
// more than 64 entries (a stretch of empty cells) is written by the whole
// wave, so that sparse inputs do not leave one lane writing most of the mesh.
__global__ void cell_starts_kernel(const uint32_t *__restrict__ keys, int n, int shift, int64_t n_cells,
                                   uint32_t *__restrict__ cell_start,
                                   const uint32_t *__restrict__ run) {
    if (!runs(run)) return;
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

// The same for the PP kernels, one wave per tile: light tiles get the last
// key, the others 254 less their thousands.  A tile is light if each of its
// boxes of kPPLightLayers layers of cells and the halo holds at most light_cap
// particles.
__global__ void pp_tile_keys_kernel(const uint32_t *__restrict__ cs, int nt, uint32_t light_cap,
                                    uint32_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    const int ntiles = nt * nt * nt;
    const int b = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (b >= ntiles) return;
    int tx, ty, tz;
    tile_of_block(b, nt, tx, ty, tz);
    const uint32_t t = (uint32_t)((tz * nt + ty) * nt + tx);
    const int n_ios = nt * kTileIos;
    constexpr int NB = kTileIos / kPPLightLayers;
    uint32_t sum[NB] = {};
#pragma unroll
    for (int k = 0; k < 2; ++k) {            // the 100 x-rows of the 10^3 box
        const int r = lane + 64 * k;
        if (r >= 100) break;
        const int by = r % 10, bz = r / 10;
        const int cy = wrapn(ty * kTileIos + by - 1, n_ios), cz = wrapn(tz * kTileIos + bz - 1, n_ios);
        const uint32_t a = cell_key(wrapn(tx * kTileIos - 1, n_ios), cy, cz, nt),
                       m = cell_key(tx * kTileIos, cy, cz, nt),
                       e = cell_key(wrapn(tx * kTileIos + 8, n_ios), cy, cz, nt);
        const uint32_t c = (cs[a + 1] - cs[a]) + (cs[m + 8] - cs[m]) + (cs[e + 1] - cs[e]);
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
    if (lane == 0) {
        const uint32_t cnt = cs[(t + 1) * kTileCells] - cs[t * kTileCells];
        keys[b] = most <= light_cap ? 255u : 254u - min(cnt >> 10, 254u);
        vals[b] = t;
    }
}

// The order of up to kOrderOne tiles by their keys in one workgroup, in place of
// the three launches of a radix pass: each wave ranks its tiles as the radix
// scatter does.  keys == NULL: the key of a tile is its particles in thousands,
// most first (tile_keys_kernel).  start255 receives where the last key starts.
constexpr int kOrderBlock = 1024, kOrderOne = 4 * kOrderBlock;
__global__ __launch_bounds__(kOrderBlock) void order_tiles_kernel(
    const uint32_t *__restrict__ cs, const uint32_t *__restrict__ keys, int nt,
    uint32_t *__restrict__ order, uint32_t *__restrict__ start255, uint32_t *__restrict__ queue,
    uint32_t *__restrict__ xcd_queue) {
    constexpr int W = kOrderBlock / 64, PER = kOrderOne / kOrderBlock;
    __shared__ uint32_t wcnt[W][256];
    __shared__ uint32_t scan_sh[W + 1];
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
            int tx, ty, tz;
            tile_of_block(b, nt, tx, ty, tz);
            tile[r] = (uint32_t)((tz * nt + ty) * nt + tx);
            key[r] = keys ? keys[b]
                          : 255u - min((cs[(tile[r] + 1) * kTileCells] - cs[tile[r] * kTileCells]) >> 10, 255u);
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
    if (tid == 255) *start255 = at;
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
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (key[r] < 256u) order[wcnt[w][key[r]] + place[r]] = tile[r];
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
// key bit `shift` on and then by cell within the tiles, or (few particles per
// tile, or one tile) by the whole key, 8 bits a pass.
struct SortPlan {
    bool by_tile;
    int bits, shift, passes;
};
SortPlan sort_plan(const cube2_ctx *ctx, int64_t n) {
    const int64_t ntiles = (int64_t)ctx->nt * ctx->nt * ctx->nt;
    int bits = 0;
    while (((int64_t)kTileCells << bits) < ctx->n_cells) ++bits;
    SortPlan p;
    // a workgroup per tile: 64 particles and more pay for it
    p.by_tile = bits > 0 && n >= 64 * ntiles;
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
// XCD-slab order.  The tile indices land in the first ntiles words of the
// tile_order region; the work counter (tile_queue_ptr) is reset to zero.
int launch_order_tiles(cube2_ctx *ctx, const uint32_t *cs, unsigned char *work,
                       const WorkLayout &L, hipStream_t s, int light_cap,
                       const uint32_t **n_heavy) {
    const int nt = ctx->nt;
    const int ntiles = nt * nt * nt;
    uint32_t *base = reinterpret_cast<uint32_t *>(work + L.tile_order);
    uint32_t *order = base, *vin = base + ntiles, *kin = base + 2 * ntiles, *kout = base + 3 * ntiles;
    uint32_t *tmp = reinterpret_cast<uint32_t *>(work + L.scan_tmp);
    uint32_t *ghist = reinterpret_cast<uint32_t *>(work + L.hist);
    uint32_t *xcd_queue = ntiles >= kXcdQueueWords ? xcd_queue_ptr(ctx, work, L) : nullptr;
    if (n_heavy) *n_heavy = tmp + 256;   // where the last key starts
    if (light_cap > 0) {
        pp_tile_keys_kernel<<<(ntiles + 3) / 4, 256, 0, s>>>(cs, nt, (uint32_t)light_cap, kin, vin);
        CUBE2_LAUNCH_CHECK();
    }
    if (ntiles <= kOrderOne) {
        order_tiles_kernel<<<1, kOrderBlock, 0, s>>>(cs, light_cap > 0 ? kin : nullptr, nt, order, tmp + 256,
                                                     tile_queue_ptr(ctx, work, L), xcd_queue);
        CUBE2_LAUNCH_CHECK();
        return CUBE2_OK;
    }
    if (light_cap <= 0) {
        tile_keys_kernel<<<(ntiles + 255) / 256, 256, 0, s>>>(cs, nt, kin, vin);
        CUBE2_LAUNCH_CHECK();
    }
    const int r = radix_pass<8>(kin, vin, kout, order, ntiles, 0, ghist, tmp, nullptr, s);
    if (r) return r;
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
        cell_starts_kernel<<<1, 64, 0, s>>>(k0, 0, 0, ctx->n_cells, cell_start, nullptr);
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
        cell_starts_kernel<<<strided(((int64_t)n + 1 + 1023) / 1024, run), 256, 0, s>>>(k0, n, 9, ntiles,
                                                                                      tstart, run);
        CUBE2_LAUNCH_CHECK();
        tile_sort_kernel<<<strided(ntiles, run), kBlock, 0, s>>>(k0, v0, tstart, offs, n, ctx->nt, pos,
                                                                 cell_start, perm, vel, acc, kick,
                                                                 vel_out, run);
        CUBE2_LAUNCH_CHECK();
        return CUBE2_OK;
    }
    // cell_start (n_cells + 1 entries, the last = n) from the sorted keys
    cell_starts_kernel<<<strided(((int64_t)n + 1 + 1023) / 1024, run), 256, 0, s>>>(
        k0, n, 0, ctx->n_cells, cell_start, run);
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

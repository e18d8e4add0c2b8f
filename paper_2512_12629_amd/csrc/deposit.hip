// deposit.hip -- CIC mass assignment in exact fixed point (section 2.1.2,
// step 1, with the CIC kernel), both PM levels in one particle sweep.
//
// A particle with 15-bit in-cell fraction f (per axis, on the level's mesh)
// gives node j the weight 2^15 - f and node j+1 the weight f; the product of
// three weights (<= 2^45) is added to a uint64 accumulator.  Integer addition
// is associative, so the result is bit-exact and independent of the order of
// the LDS atomics.  The FP32 density is the accumulator rounded to nearest,
// times 2^-45 (particle masses per level cell).
//
// Fine level: one workgroup owns the 16^3 fine nodes of a tile and gathers
// every particle that touches them: its own 8^3 IOS cells plus the layer of
// IOS cells below it on each axis (a particle in fine cell a-1 feeds node a).
// The contributing cells form a 9^3 box of IOS cells, i.e. 729 contiguous
// particle ranges, gathered as one list (BoxList).
// Each fine node is then written once, as FP32: no global atomics and no
// 64-bit mesh in HBM.
// Coarse level: only the tile's own particles are assigned; the tile's
// coarse footprint (16/H + 1 nodes per axis) is accumulated in LDS and added
// to a uint64 coarse mesh with global atomics, then converted to FP32.
//
// TSC (eq. 5, context flag CUBE2_ASSIGN_TSC): a particle with in-cell
// fraction f has nearest node n0 = j + [f >= 1/2] and offset m = f - [f >=
// 1/2] (units 2^-15, m in [-2^14, 2^14)); nodes n0-1, n0, n0+1 get the
// 16-bit weights W- = round((2^14 - m)^2 / 2^15), W+ = round((2^14 + m)^2 /
// 2^15) and W0 = 2^16 - W- - W+ (eq. 5 to 2^-16, summing exactly to one
// particle).  Products are below 2^47, the density is the accumulator times
// 2^-48.  A fine node then also receives particles of the next IOS cell up,
// so the gathered box is 10^3 IOS cells; the coarse footprint has 16/H + 3
// nodes per axis.
#include "common.hpp"

namespace cube2 {
namespace {

// Gathered box of IOS cells per axis: [c0-1, c0+8) for CIC, [c0-1, c0+9) for TSC.
// CR: the smallest coarse ratio the LDS coarse footprint is sized for (2, or
// 4 for ratios 4 and 8, which keeps the block within 40 KB of LDS: four
// workgroups per CU).
template <int P, int CR = 4> struct DepGeo {
    static constexpr int BOX = kTileIos + (P == 3 ? 2 : 1);
    static constexpr int SEGS = BOX * BOX * BOX;              // 729 or 1000
    static constexpr int CMAX = kTileFine / CR + (P == 3 ? 3 : 1);  // coarse nodes per axis
};

// TSC weights of offset m (units 2^-15, m in [-2^14, 2^14)) in units of 2^-16.
__device__ __forceinline__ void tsc_weights(int m, uint32_t (&w)[3]) {
    const uint32_t a = (uint32_t)(16384 - m), b = (uint32_t)(16384 + m);
    w[0] = (a * a + 16384u) >> 15;
    w[2] = (b * b + 16384u) >> 15;
    w[1] = 65536u - w[0] - w[2];
}

// What the integer meshes receive: the accumulator, or, with a unit, its FP64 density
__device__ __forceinline__ unsigned long long fx_word(unsigned long long v, double unit) {
    return unit != 0.0 ? (unsigned long long)__double_as_longlong((double)v * unit) : v;
}

__global__ void fill_u64(unsigned long long *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// Fine CIC weights of one particle of box segment b (IOS cell coordinates
// relative to the tile, own cells at 0..7) with in-cell offsets o, added to the
// tile's fine nodes that it reaches.
__device__ __forceinline__ void deposit_fine(const int (&b)[3], const uint32_t (&o)[3],
                                             unsigned long long *acc_f) {
    int j[3];
    uint32_t w[3][2];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        j[d] = 2 * b[d] + (int)(o[d] >> 15);  // fine cell rel. to the tile
        const uint32_t f = o[d] & 0x7FFFu;
        w[d][0] = 32768u - f;
        w[d][1] = f;
    }
#pragma unroll
    for (int sz = 0; sz < 2; ++sz)
#pragma unroll
        for (int sy = 0; sy < 2; ++sy) {
            const int nz = j[2] + sz, ny = j[1] + sy;
            if ((unsigned)nz >= (unsigned)kTileFine || (unsigned)ny >= (unsigned)kTileFine)
                continue;
            const uint32_t wyz = w[1][sy] * w[2][sz];  // <= 2^30
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                const int nx = j[0] + sx;
                if ((unsigned)nx >= (unsigned)kTileFine) continue;
                atomicAdd(&acc_f[(nz * kTileFine + ny) * kTileFine + nx],
                          (unsigned long long)wyz * w[0][sx]);
            }
        }
}

// Fine TSC weights of one particle of box segment b, added to the tile's
// fine nodes that it reaches (nodes n0-1 .. n0+1 per axis).
__device__ __forceinline__ void deposit_fine_tsc(const int (&b)[3], const uint32_t (&o)[3],
                                                 unsigned long long *acc_f) {
    int j[3];
    uint32_t w[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int f = (int)(o[d] & 0x7FFFu);
        const int hi = f >= 16384 ? 1 : 0;
        j[d] = 2 * b[d] + (int)(o[d] >> 15) + hi - 1;  // node n0 - 1, rel. to the tile
        tsc_weights(f - (hi << 15), w[d]);
    }
#pragma unroll
    for (int sz = 0; sz < 3; ++sz)
#pragma unroll
        for (int sy = 0; sy < 3; ++sy) {
            const int nz = j[2] + sz, ny = j[1] + sy;
            if ((unsigned)nz >= (unsigned)kTileFine || (unsigned)ny >= (unsigned)kTileFine)
                continue;
            const uint32_t wyz = w[1][sy] * w[2][sz];  // < 2^32
#pragma unroll
            for (int sx = 0; sx < 3; ++sx) {
                const int nx = j[0] + sx;
                if ((unsigned)nx >= (unsigned)kTileFine) continue;
                atomicAdd(&acc_f[(nz * kTileFine + ny) * kTileFine + nx],
                          (unsigned long long)wyz * w[0][sx]);
            }
        }
}

// Coarse TSC weights of the wave's own-tile particles, added to the tile's
// coarse footprint (LDS index = coarse node - tile origin + 1), wave-summed
// when every own lane shares its nearest node.
__device__ __forceinline__ void deposit_coarse_wave_tsc(bool own, const int (&b)[3],
                                                        const uint32_t (&o)[3], int hshift, int NC,
                                                        unsigned long long *acc_c) {
    const unsigned long long om = __ballot(own);
    if (om == 0ull) return;
    int j[3];
    uint32_t w[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const uint32_t q = ((uint32_t)b[d] << 16) + o[d];  // tile-relative
        const uint32_t y = q >> hshift;                           // 2^-15 coarse cells
        const int f = (int)(y & 0x7FFFu);
        const int hi = f >= 16384 ? 1 : 0;
        j[d] = (int)(y >> kFracBits) + hi;                        // n0, LDS index of n0 - 1
        tsc_weights(f - (hi << 15), w[d]);
        if (!own) w[d][0] = w[d][1] = w[d][2] = 0u;
    }
    const int key = own ? (j[2] * NC + j[1]) * NC + j[0] : -1;
    const int lead = first_lane(om);
    const int key0 = __builtin_amdgcn_readlane(key, lead);
    const bool uniform = __ballot(own && key != key0) == 0ull;
#pragma unroll
    for (int sz = 0; sz < 3; ++sz)
#pragma unroll
        for (int sy = 0; sy < 3; ++sy) {
            const uint32_t wyz = w[1][sy] * w[2][sz];
#pragma unroll
            for (int sx = 0; sx < 3; ++sx) {
                const unsigned long long v = (unsigned long long)wyz * w[0][sx];
                const int off = (sz * NC + sy) * NC + sx;
                if (uniform) {
                    const unsigned long long t = wave_sum(v);
                    if ((int)(threadIdx.x & 63) == lead) atomicAdd(&acc_c[key0 + off], t);
                } else if (own) {
                    atomicAdd(&acc_c[key + off], v);
                }
            }
        }
}

// Coarse CIC weights of the wave's own-tile particles (own = true), added to
// the tile's coarse footprint.  Called by all 64 lanes.  An IOS cell lies in
// one coarse cell, so in a dense cell every lane feeds the same 8 nodes:
// then the 8 weights are summed over the wave first (exact integer sums) and
// one lane adds them, instead of 64 lanes contending for each node.
__device__ __forceinline__ void deposit_coarse_wave(bool own, const int (&b)[3],
                                                    const uint32_t (&o)[3], int hshift, int NC,
                                                    unsigned long long *acc_c) {
    const unsigned long long om = __ballot(own);
    if (om == 0ull) return;
    int j[3];
    uint32_t w[3][2];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const uint32_t q = ((uint32_t)b[d] << 16) + o[d];  // tile-relative
        j[d] = (int)(q >> (kFracBits + hshift));
        const uint32_t f = (q >> hshift) & 0x7FFFu;
        w[d][0] = own ? 32768u - f : 0u;
        w[d][1] = own ? f : 0u;
    }
    const int key = own ? (j[2] * NC + j[1]) * NC + j[0] : -1;
    const int lead = first_lane(om);
    const int key0 = __builtin_amdgcn_readlane(key, lead);
    const bool uniform = __ballot(own && key != key0) == 0ull;
#pragma unroll
    for (int sz = 0; sz < 2; ++sz)
#pragma unroll
        for (int sy = 0; sy < 2; ++sy) {
            const uint32_t wyz = w[1][sy] * w[2][sz];
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                const unsigned long long v = (unsigned long long)wyz * w[0][sx];
                const int off = (sz * NC + sy) * NC + sx;
                if (uniform) {
                    const unsigned long long t = wave_sum(v);
                    if ((int)(threadIdx.x & 63) == lead) atomicAdd(&acc_c[key0 + off], t);
                } else if (own) {
                    atomicAdd(&acc_c[key + off], v);
                }
            }
        }
}

template <bool FINE, bool COARSE, int P, int CR>
__global__ __launch_bounds__(kBlock) void deposit_kernel(
    const uint16_t *__restrict__ pos, const uint32_t *__restrict__ cs, int n, int n_f, int nt,
    float *__restrict__ rho_f, unsigned long long *__restrict__ rho_f_fx,
    unsigned long long *__restrict__ coarse_acc, int n_c, int hshift, uint32_t *status,
    const uint32_t *__restrict__ order, uint32_t *__restrict__ queue, double fx_unit) {
    using Geo = DepGeo<P, CR>;
    using List = BoxList<Geo::SEGS, kBlock>;
    constexpr int kBox = Geo::BOX, kSegs = Geo::SEGS;
    constexpr int kSegPerThread = List::PER, kCoarseMax = Geo::CMAX;
    __shared__ typename List::Shared list_sh;
    __shared__ unsigned long long acc_f[FINE ? kTileFine * kTileFine * kTileFine : 1];
    __shared__ unsigned long long acc_c[COARSE ? kCoarseMax * kCoarseMax * kCoarseMax : 1];
    __shared__ int next_sh;

    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int n_ios = nt * kTileIos;
    const int NC = (kTileFine >> hshift) + (P == 3 ? 3 : 1);  // coarse nodes per axis touched
    const int ntiles = nt * nt * nt;

    // Particle ranges (start, count) of this thread's segments of the box of
    // IOS cells [c0-1, c0+kBox-1) around tile t, and each segment's IOS cell relative
    // to the tile (a signed byte per axis; bit 24: one of the tile's own).
    uint32_t cnt[kSegPerThread], src[kSegPerThread], tag[kSegPerThread];
    auto load_segments = [&](int t) {
        const int c0x = (t % nt) * kTileIos, c0y = ((t / nt) % nt) * kTileIos,
                  c0z = (t / (nt * nt)) * kTileIos;
#pragma unroll
        for (int k = 0; k < kSegPerThread; ++k) {
            const int s = tid * kSegPerThread + k;
            cnt[k] = src[k] = tag[k] = 0u;
            if (s < kSegs) {
                const int bx = s % kBox, by = (s / kBox) % kBox, bz = s / (kBox * kBox);
                const bool own = bx > 0 && by > 0 && bz > 0 && bx <= kTileIos && by <= kTileIos &&
                                 bz <= kTileIos;
                tag[k] = (uint32_t)((bx - 1) & 0xFF) | (uint32_t)((by - 1) & 0xFF) << 8 |
                         (uint32_t)((bz - 1) & 0xFF) << 16 | (own ? 1u << 24 : 0u);
                if (FINE || own) {
                    const uint32_t key = cell_key(wrapn(c0x + bx - 1, n_ios), wrapn(c0y + by - 1, n_ios),
                                                  wrapn(c0z + bz - 1, n_ios), nt);
                    src[k] = cs[key];
                    cnt[k] = cs[key + 1];  // end; the count is formed where it is used
                }
            }
        }
    };

    // Persistent workgroups over the heaviest-first tile order, each XCD's share of
    // it (XcdShare).  The loop is software-pipelined: the claim of the next tile
    // is in flight while the current one deposits, and the next tile's segment
    // ranges are loaded while the current one writes its nodes.
    XcdShare xcd;
    const bool fixed = ntiles < kXcdQueueWords;
    // thread 0: the order's place of the next tile, ntiles when all are taken
    int at = blockIdx.x;
    auto claim = [&]() {
        while (xcd.done < xcd.ng) {
            const int i = xcd.claim(queue);
            if (i < xcd.share(ntiles)) return xcd.place(i);
            xcd.next_group();
        }
        return ntiles;
    };
    if (tid == 0) {
        if (!fixed) at = claim();
        next_sh = at < ntiles ? (int)order[at] : -1;
    }
    __syncthreads();
    int t = next_sh;
    if (t >= 0) load_segments(t);
    while (t >= 0) {
        const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
        if (tid == 0) at = fixed ? at + (int)gridDim.x : claim();

        if (FINE)
            for (int i = tid; i < kTileFine * kTileFine * kTileFine; i += kBlock) acc_f[i] = 0ull;
        if (COARSE)
            for (int i = tid; i < NC * NC * NC; i += kBlock) acc_c[i] = 0ull;

#pragma unroll
        for (int k = 0; k < kSegPerThread; ++k) cnt[k] -= src[k];
        List list;
        list.build(list_sh, src, cnt, tag);
        if (tid == 0) {
            // Overflow guard: a fine node sums at most `total` weights of 2^45
            // (CIC) or 2^47 (TSC) each; a coarse node sums the own particles
            // of at most 8 tiles.
            const uint32_t own = cs[(uint32_t)(t + 1) * kTileCells] - cs[(uint32_t)t * kTileCells];
            const uint32_t fine_max = P == 3 ? (1u << 17) : (1u << 19);
            const uint32_t own_max = P == 3 ? (1u << 14) : (1u << 16);
            if ((FINE && list.total >= fine_max) || (COARSE && own >= own_max))
                atomicOr(status, kStatusOverflow);
        }

        // The loop runs wave-uniformly (every lane of a wave takes the same
        // trips) so that the coarse weights can be summed over the wave; each
        // trip takes kBatch particles per lane, whose position loads are all
        // issued before the first deposit.
        constexpr int kBatch = 4, kWaves = kBlock / 64;
        for (uint32_t base = 0; base < list.total; base += kBoxSpan) {
            if (base) list.span(list_sh, cnt, base);
            const uint32_t m = min(list.total - base, (uint32_t)kBoxSpan);
            for (uint32_t i0 = wave; 64 * i0 < m; i0 += kBatch * kWaves) {
                uint2 g[kBatch];
                uint32_t o[kBatch][3];
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    // a word past the end: the first word's cells, not used
                    const uint32_t i = i0 + k * kWaves;
                    g[k] = list.cell(list_sh, 64 * i < m ? (int)i : (int)i0);
                }
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    const uint32_t v = 64 * (i0 + k * kWaves) + lane;
                    o[k][0] = o[k][1] = o[k][2] = 0u;
                    if (v >= m) continue;
                    const uint32_t p = g[k].x + base + v;
#pragma unroll
                    for (int d = 0; d < 3; ++d) o[k][d] = pos[(int64_t)d * n + p];
                }
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    const bool valid = 64 * (i0 + k * kWaves) + lane < m;
                    const int b[3] = {(int)(int8_t)g[k].y, (int)(int8_t)(g[k].y >> 8),
                                      (int)(int8_t)(g[k].y >> 16)};
                    const bool own = valid && (g[k].y >> 24) != 0u;
                    if (P == 3) {
                        if (FINE && valid) deposit_fine_tsc(b, o[k], acc_f);
                        if (COARSE) deposit_coarse_wave_tsc(own, b, o[k], hshift, NC, acc_c);
                    } else {
                        if (FINE && valid) deposit_fine(b, o[k], acc_f);
                        if (COARSE) deposit_coarse_wave(own, b, o[k], hshift, NC, acc_c);
                    }
                }
            }
        }
        // the next tile (the claim made at the top of this one has returned)
        if (tid == 0) next_sh = at < ntiles ? (int)order[at] : -1;
        __syncthreads();
        const int t_next = next_sh;
        if (t_next >= 0) load_segments(t_next);

        if (FINE) {
            const int a0x = tx * kTileFine, a0y = ty * kTileFine, a0z = tz * kTileFine;
            for (int i = tid; i < kTileFine * kTileFine * kTileFine; i += kBlock) {
                const int lx = i % kTileFine, ly = (i / kTileFine) % kTileFine,
                          lz = i / (kTileFine * kTileFine);
                const int64_t g = ((int64_t)(a0z + lz) * n_f + (a0y + ly)) * n_f + (a0x + lx);
                const unsigned long long v = acc_f[i];
                // streaming store: a tile row is half a cache line, and the
                // mesh is read back only by the next kernel
                if (rho_f)
                    __builtin_nontemporal_store((float)v * (P == 3 ? 0x1p-48f : 0x1p-45f), &rho_f[g]);
                if (rho_f_fx) rho_f_fx[g] = fx_word(v, fx_unit);
            }
        }
        if (COARSE) {
            const int lo = P == 3 ? 1 : 0;  // footprint starts one node below (TSC)
            const int A0x = ((tx * kTileFine) >> hshift) - lo, A0y = ((ty * kTileFine) >> hshift) - lo,
                      A0z = ((tz * kTileFine) >> hshift) - lo;
            for (int i = tid; i < NC * NC * NC; i += kBlock) {
                const unsigned long long v = acc_c[i];
                if (!v) continue;
                const int lx = i % NC, ly = (i / NC) % NC, lz = i / (NC * NC);
                const int64_t g = ((int64_t)wrapn(A0z + lz, n_c) * n_c + wrapn(A0y + ly, n_c)) * n_c +
                                  wrapn(A0x + lx, n_c);
                atomicAdd(&coarse_acc[g], v);
            }
        }
        t = t_next;
        __syncthreads();  // this tile is done with the LDS arrays
    }  // tiles
}

__global__ void coarse_finalize(const unsigned long long *__restrict__ accum, int64_t m,
                                float *__restrict__ rho, unsigned long long *__restrict__ fx,
                                float unit, double fx_unit) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    const unsigned long long v = accum[i];
    if (rho) rho[i] = (float)v * unit;
    if (fx) fx[i] = fx_word(v, fx_unit);
}

template <bool FINE, bool COARSE, int P, int CR>
void launch_one_deposit(const uint16_t *pos, const uint32_t *cs, int64_t n, int n_f, int nt,
                        float *rho_f, unsigned long long *ffx, unsigned long long *cacc, int n_c,
                        int hshift, uint32_t *status, const uint32_t *order, uint32_t *queue,
                        int ntiles, double fx_unit, hipStream_t s) {
    auto k = deposit_kernel<FINE, COARSE, P, CR>;
    k<<<persistent_grid(k, kBlock, ntiles), kBlock, 0, s>>>(pos, cs, (int)n, n_f, nt, rho_f, ffx, cacc,
                                                          n_c, hshift, status, order, queue, fx_unit);
}

template <int P>
int launch_deposit_kernels(bool fine, bool coarse, const uint16_t *pos, const uint32_t *cs, int64_t n,
                           int n_f, int nt, float *rho_f, unsigned long long *ffx,
                           unsigned long long *cacc, int n_c, int hshift, uint32_t *status,
                           const uint32_t *order, uint32_t *queue, int ntiles, double fx_unit,
                           hipStream_t s) {
    if (coarse && (kTileFine >> hshift) + (P == 3 ? 3 : 1) > DepGeo<P, 2>::CMAX) return CUBE2_EINVAL;
    const bool r2 = hshift < 2;  // coarse ratio 2: the wider footprint
    if (fine && coarse) {
        if (r2)
            launch_one_deposit<true, true, P, 2>(pos, cs, n, n_f, nt, rho_f, ffx, cacc, n_c, hshift,
                                                 status, order, queue, ntiles, fx_unit, s);
        else
            launch_one_deposit<true, true, P, 4>(pos, cs, n, n_f, nt, rho_f, ffx, cacc, n_c, hshift,
                                                 status, order, queue, ntiles, fx_unit, s);
    } else if (fine) {
        launch_one_deposit<true, false, P, 4>(pos, cs, n, n_f, nt, rho_f, ffx, cacc, n_c, hshift,
                                              status, order, queue, ntiles, fx_unit, s);
    } else {
        if (r2)
            launch_one_deposit<false, true, P, 2>(pos, cs, n, n_f, nt, nullptr, nullptr, cacc, n_c,
                                                  hshift, status, order, queue, ntiles, fx_unit, s);
        else
            launch_one_deposit<false, true, P, 4>(pos, cs, n, n_f, nt, nullptr, nullptr, cacc, n_c,
                                                  hshift, status, order, queue, ntiles, fx_unit, s);
    }
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

}  // namespace

int launch_deposit(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                   float *rho_f, uint64_t *rho_f_fx, float *rho_c, uint64_t *rho_c_fx,
                   unsigned char *work, const WorkLayout &L, hipStream_t s, bool as_f64) {
    const double fx_unit = as_f64 ? (ctx->tsc ? 0x1p-48 : 0x1p-45) : 0.0;
    const int nt = ctx->nt;
    const unsigned blocks = (unsigned)(nt * nt * nt);
    uint32_t *status = status_word(ctx);
    const bool coarse = (rho_c || (as_f64 && rho_c_fx)) && ctx->n_levels > 1;
    const bool fine = rho_f || (as_f64 && rho_f_fx);
    auto *cacc = reinterpret_cast<unsigned long long *>(work + L.coarse_acc);
    const int n_c = coarse ? ctx->lv[1].n : 1;
    const int hshift = coarse ? ctx->lv[1].hshift : 0;
    const int64_t mc = (int64_t)n_c * n_c * n_c;
    if (coarse) {
        fill_u64<<<(unsigned)((mc + 255) / 256), 256, 0, s>>>(cacc, mc);
        CUBE2_LAUNCH_CHECK();
    }
    auto *ffx = reinterpret_cast<unsigned long long *>(rho_f_fx);
    if (!fine && !coarse) return CUBE2_EINVAL;
    // persistent workgroups over the tiles, heaviest first
    int r = launch_order_tiles(ctx, cs, work, L, s);
    if (r) return r;
    const uint32_t *order = tile_order_ptr(work, L);
    uint32_t *queue = xcd_queue_ptr(ctx, work, L);
    const int ntiles = (int)blocks;
    if (ctx->tsc)
        r = launch_deposit_kernels<3>(fine, coarse, pos, cs, n, ctx->n_f, nt, rho_f, ffx, cacc, n_c,
                                      hshift, status, order, queue, ntiles, fx_unit, s);
    else
        r = launch_deposit_kernels<2>(fine, coarse, pos, cs, n, ctx->n_f, nt, rho_f, ffx, cacc, n_c,
                                      hshift, status, order, queue, ntiles, fx_unit, s);
    if (r) return r;
    if (coarse) {
        coarse_finalize<<<(unsigned)((mc + 255) / 256), 256, 0, s>>>(
            cacc, mc, rho_c, reinterpret_cast<unsigned long long *>(rho_c_fx),
            ctx->tsc ? 0x1p-48f : 0x1p-45f, fx_unit);
        CUBE2_LAUNCH_CHECK();
    }
    return CUBE2_OK;
}

}  // namespace cube2

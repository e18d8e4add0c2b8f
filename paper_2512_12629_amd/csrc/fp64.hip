// fp64.hip -- the piece of the FP64 plain form that has no FP32 twin: the PP force
// (eq. 4d) in FP64, one thread per particle looping over its neighbour IOS cells
// (27, or 125 for b_f > 2), with the pair law of eq. (2) evaluated from the exact
// piecewise-polynomial table in FP64.  One workgroup per tile, one wave where
// tiles hold few particles.
// It favours plainness over speed: it is the yardstick the FP32 path is
// compared against at sizes the host oracle cannot reach.
#include "common.hpp"

namespace cube2 {
namespace {

// One workgroup per tile.  The box of (8 + 2H)^3 cells is staged in LDS, kBoxSpan
// particles at a time, as integer positions in units of 2^-15 fine cells (below
// 2^20, exact in FP32); a thread takes one particle and loops over the (2H + 1)^2
// x-rows of cells around its own.  One candidate in six or seven is closer than b_f,
// so the candidates are only tested (in FP32 against b_f^2 and a margin of 1e-5;
// beyond b_f the rows are zero), and those that pass go to a list of the thread's own;
// when a list may not take four more, the lanes that are still in the loop evaluate
// theirs.  The square root, the division and the polynomial, 90 instructions of
// mostly FP64, are left out for the others.
// 2.1 million particles on a 256^3 mesh: 290 us with all of it for every
// candidate, read from HBM cell by cell, 118 us now.
constexpr int kPP64Block = 512, kPP64List = 16;

// Where a tile has only a few particles that work is all latency: the box's list, its
// barriers and two workgroups on a CU for 13 particles of 512 threads.  So where the tiles
// outnumber those workgroups and have at most kPP64Mean particles on average, the tiles
// that have at most kPP64Few and no neighbour with more are one wave's, which reads its
// neighbours from memory; the others, if any, are found and done by the workgroups of a
// second launch.  us so and with the boxes alone, one-cell reach: 13 per tile, 256^3 mesh
// 14 and 35, 512^3 60 and 276; 53 per tile 23 and 38, 103 and 294; 107 per tile (boxes alone) 53.
constexpr int kPP64Few = 128, kPP64Grid = 512;
constexpr int64_t kPP64Mean = 64;

// particles of tile (x, y, z), periodic
__device__ __forceinline__ uint32_t tile_count(const uint32_t *__restrict__ cs, int nt, int x, int y, int z) {
    const int m = nt - 1;
    const uint32_t key = (uint32_t)(((z & m) * nt + (y & m)) * nt + (x & m)) * kTileCells;
    return cs[key + kTileCells] - cs[key];
}

// the pair law's g(r) of r^2 > 0 in fine cells, from its rows
__device__ __forceinline__ double pair64(const double *__restrict__ rows, int K, double kinv, double r2) {
    const double r = sqrt(r2);
    const double t = r * kinv;
    const int idx = min((int)t, K);
    const double *q = rows + (int64_t)idx * kPairRow;
    const double y = q[9] + q[10] * (t - floor(t));
    double U = q[8];
#pragma unroll
    for (int e = 7; e >= 0; --e) U = q[e] + y * U;
    return U / (r2 * r);
}

__global__ __launch_bounds__(64) void pp64_few_kernel(
    const uint16_t *__restrict__ pos, const uint32_t *__restrict__ cs, int n, int nt,
    const double *__restrict__ rows, int K, double kinv, double gm, double *__restrict__ acc,
    int accumulate, int H) {
    __shared__ uint32_t cst[kTileCells + 1];
    int tx, ty, tz;
    tile_of_block(blockIdx.x, nt, tx, ty, tz);
    const int lane = threadIdx.x, n_ios = nt * kTileIos;
    const bool many = lane < 27 && tile_count(cs, nt, tx + lane % 3 - 1, ty + lane / 3 % 3 - 1,
                                              tz + lane / 9 - 1) > kPP64Few;
    if (__any(many)) return;
    stage_cell_starts<64>(cst, cs, (uint32_t)((tz * nt + ty) * nt + tx) * kTileCells);
    __syncthreads();
    for (uint32_t p = cst[0] + lane; p < cst[kTileCells]; p += 64) {
        const int u = seg_search_n<kTileCells>(cst, p);
        const int c[3] = {tx * kTileIos + (u & 7), ty * kTileIos + ((u >> 3) & 7), tz * kTileIos + (u >> 6)};
        int oi[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) oi[d] = pos[(int64_t)d * n + p];
        double a[3] = {0.0, 0.0, 0.0};
        for (int dz = -H; dz <= H; ++dz)
            for (int dy = -H; dy <= H; ++dy)
#pragma unroll 5
                for (int dx = -H; dx <= H; ++dx) {
                    const uint32_t key = cell_key(wrapn(c[0] + dx, n_ios), wrapn(c[1] + dy, n_ios),
                                                  wrapn(c[2] + dz, n_ios), nt);
                    const uint32_t j1 = cs[key + 1];
                    for (uint32_t j = cs[key]; j < j1; ++j) {
                        // in units of 2^-15 fine cells, exact
                        const int D[3] = {dx * 65536 + (int)pos[j] - oi[0],
                                          dy * 65536 + (int)pos[(int64_t)n + j] - oi[1],
                                          dz * 65536 + (int)pos[2 * (int64_t)n + j] - oi[2]};
                        const double X = D[0] * 0x1p-15, Y = D[1] * 0x1p-15, Z = D[2] * 0x1p-15;
                        const double r2 = X * X + Y * Y + Z * Z;
                        if (r2 == 0.0) continue;       // the particle itself (or a coincident one)
                        const double g = pair64(rows, K, kinv, r2);
                        a[0] += g * X;
                        a[1] += g * Y;
                        a[2] += g * Z;
                    }
                }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double *dst = acc + (int64_t)d * n + p;
            *dst = accumulate ? *dst + gm * a[d] : gm * a[d];
        }
    }
}

template <int H>
__device__ __forceinline__ void pp64_tile(
    const uint16_t *__restrict__ pos, const uint32_t *__restrict__ cs, int n, int nt,
    const double *__restrict__ rows, int K, double kinv, float cut, double gm,
    double *__restrict__ acc, int accumulate, int block) {
    constexpr int B = kTileIos + 2 * H, SEGS = B * B * B, W = 2 * H + 1;
    using List = BoxList<SEGS, kPP64Block>;
    __shared__ typename List::Shared lsh;
    __shared__ float xs[3][kBoxSpan];
    __shared__ uint32_t pre[SEGS + 1], cst[kTileCells + 1];
    __shared__ uint16_t held_at[kPP64List][kPP64Block];
    int tx, ty, tz;
    tile_of_block(block, nt, tx, ty, tz);
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), n_ios = nt * kTileIos;
    const uint32_t key0 = (uint32_t)((tz * nt + ty) * nt + tx) * kTileCells;
    const uint32_t p0 = cs[key0], own = cs[key0 + kTileCells] - p0;
    if (own == 0) return;
    stage_cell_starts<kPP64Block>(cst, cs, key0);
    uint32_t src[List::PER], cnt[List::PER], tag[List::PER];
#pragma unroll
    for (int k = 0; k < List::PER; ++k) {
        const int s = tid * List::PER + k;
        src[k] = cnt[k] = tag[k] = 0u;
        if (s < SEGS) {
            const int bx = s % B, by = (s / B) % B, bz = s / (B * B);
            const uint32_t key = cell_key(wrapn(tx * kTileIos + bx - H, n_ios),
                                          wrapn(ty * kTileIos + by - H, n_ios),
                                          wrapn(tz * kTileIos + bz - H, n_ios), nt);
            src[k] = cs[key];
            cnt[k] = cs[key + 1] - src[k];
            tag[k] = (uint32_t)(bx | by << 8 | bz << 16);
        }
    }
    List list;
    list.build(lsh, src, cnt, tag);
#pragma unroll
    for (int k = 0; k < List::PER; ++k)
        if (tid * List::PER + k < SEGS) pre[tid * List::PER + k] = list.first[k];
    if (tid == 0) pre[SEGS] = list.total;
    const bool one = list.total <= (uint32_t)kBoxSpan;
    for (uint32_t l0 = 0; l0 < own; l0 += kPP64Block) {
        const bool active = l0 + tid < own;
        const uint32_t p = p0 + (active ? l0 + tid : own - 1);
        float xi[3];
        int row0 = 0;                    // box cell (-H, -H, -H) of the particle's
        double a[3] = {0.0, 0.0, 0.0};
        for (uint32_t base = 0; base < list.total; base += kBoxSpan) {
            const uint32_t m = min(list.total - base, (uint32_t)kBoxSpan);
            const bool first = l0 == 0 && base == 0;
            if (first || !one) {
                if (!first) list.span(lsh, cnt, base);
                for (uint32_t i = wave; 64 * i < m; i += kPP64Block / 64) {
                    const uint2 g = list.cell(lsh, (int)i);
                    const uint32_t v = 64 * i + lane;
                    if (v >= m) continue;
                    const uint32_t j = g.x + base + v;     // g.x is modulo 2^32
#pragma unroll
                    for (int d = 0; d < 3; ++d)
                        xs[d][v] = (float)(((g.y >> (8 * d)) & 255u) << 16 | pos[(int64_t)d * n + j]);
                }
                __syncthreads();
            }
            if (base == 0) {
                const int u = seg_search_n<kTileCells>(cst, p);
                const int c[3] = {u & 7, (u >> 3) & 7, u >> 6};
                row0 = (c[2] * B + c[1]) * B + c[0];
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    xi[d] = (float)((uint32_t)(c[d] + H) << 16 | pos[(int64_t)d * n + p]);
            }
            if (!active) continue;
            int held = 0;
            auto evaluate = [&]() {
                for (int k = 0; k < held; ++k) {
                    const int v = held_at[k][tid];
                    const double X = (xs[0][v] - xi[0]) * 0x1p-15f, Y = (xs[1][v] - xi[1]) * 0x1p-15f,
                                 Z = (xs[2][v] - xi[2]) * 0x1p-15f;          // exact
                    const double r2 = X * X + Y * Y + Z * Z;
                    const double g = pair64(rows, K, kinv, r2);
                    a[0] += g * X;
                    a[1] += g * Y;
                    a[2] += g * Z;
                }
                held = 0;
            };
            for (int r = 0; r < W * W; ++r) {
                const int s = row0 + ((r / W) * B + r % W) * B;
                const int v1 = (int)(min(max(pre[s + W], base), base + m) - base);
                for (int v = (int)(min(max(pre[s], base), base + m) - base); v < v1; v += 4) {
                    float r2[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int j = min(v + k, v1 - 1);
                        const float X = xs[0][j] - xi[0], Y = xs[1][j] - xi[1], Z = xs[2][j] - xi[2];
                        r2[k] = fmaf(Z, Z, fmaf(Y, Y, X * X));
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        // zero: the particle itself (or a coincident one)
                        if (v + k < v1 && r2[k] > 0.0f && r2[k] < cut) held_at[held++][tid] = (uint16_t)(v + k);
                    }
                    if (__any(held > kPP64List - 4)) evaluate();
                }
            }
            evaluate();
        }
        if (!active) continue;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double *dst = acc + (int64_t)d * n + p;
            *dst = accumulate ? *dst + gm * a[d] : gm * a[d];
        }
    }
}

// FEW: the tiles that pp64_few_kernel leaves.
template <int H, bool FEW>
__global__ __launch_bounds__(kPP64Block) void pp64_kernel(
    const uint16_t *__restrict__ pos, const uint32_t *__restrict__ cs, int n, int nt,
    const double *__restrict__ rows, int K, double kinv, float cut, double gm,
    double *__restrict__ acc, int accumulate) {
    if constexpr (!FEW) {
        pp64_tile<H>(pos, cs, n, nt, rows, K, kinv, cut, gm, acc, accumulate, (int)blockIdx.x);
    } else {
        __shared__ uint64_t left[kPP64Block / 64];
        const int ntiles = nt * nt * nt, grid = (int)gridDim.x;
        for (int b0 = (int)blockIdx.x; b0 < ntiles; b0 += grid * kPP64Block) {
            // thread i looks at the workgroup's i-th tile from here
            const int64_t b = b0 + (int64_t)threadIdx.x * grid;
            bool many = false;
            if (b < ntiles) {
                int x, y, z;
                tile_of_block((int)b, nt, x, y, z);
#pragma unroll
                for (int k = 0; k < 27; ++k)
                    many |= tile_count(cs, nt, x + k % 3 - 1, y + k / 3 % 3 - 1, z + k / 9 - 1) > kPP64Few;
            }
            const uint64_t m = __ballot(many);
            __syncthreads();
            if ((threadIdx.x & 63) == 0) left[wave_id()] = m;
            __syncthreads();
            for (int w = 0; w < kPP64Block / 64; ++w)
                for (uint64_t r = left[w]; r; r &= r - 1) {
                    const int i = 64 * w + __ffsll((long long)r) - 1;
                    pp64_tile<H>(pos, cs, n, nt, rows, K, kinv, cut, gm, acc, accumulate, b0 + i * grid);
                    __syncthreads();
                }
        }
    }
}

}  // namespace

int launch_pp64(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n, double *acc,
                int accumulate, hipStream_t s) {
    const double *rows = reinterpret_cast<const double *>(ctx->tables + ctx->pp64_off);
    const int nt = ctx->nt;
    const double bf = ctx->cfg.b_fine * 32768.0;     // in position units, at most 2^17
    const double kinv = (double)ctx->pp_K / ctx->cfg.b_fine, gm = ctx->cfg.g_newton * ctx->cfg.m_p;
    const int ntiles = nt * nt * nt;
    const bool few = ntiles > kPP64Grid && n <= kPP64Mean * ntiles;
    if (few) {
        pp64_few_kernel<<<(unsigned)ntiles, 64, 0, s>>>(pos, cs, (int)n, nt, rows, ctx->pp_K, kinv, gm, acc,
                                                        accumulate, ctx->pp_halo);
        CUBE2_LAUNCH_CHECK();
    }
    auto *k = few ? (ctx->pp_halo == 1 ? pp64_kernel<1, true> : pp64_kernel<2, true>)
                  : (ctx->pp_halo == 1 ? pp64_kernel<1, false> : pp64_kernel<2, false>);
    k<<<(unsigned)(few ? kPP64Grid : ntiles), kPP64Block, 0, s>>>(
        pos, cs, (int)n, nt, rows, ctx->pp_K, kinv, (float)(bf * bf * (1 + 1e-5)), gm, acc, accumulate);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

}  // namespace cube2

// velocity.hip -- IOS velocities (section 2.3): each velocity component is
// stored as a 16-bit integer relative to a bulk velocity field on a mesh.
// The paper defers the conversion to an earlier paper; the codec here is a
// plain linear one:
//   v_bulk(c) = mean velocity of the particles in bulk cell c (FP32),
//   s         = max_i |v_i - v_bulk(c_i)| / 32767 (one global scale, FP32),
//   q_i       = rint((v_i - v_bulk(c_i)) / s)          (int16),
//   decode    : v_i = v_bulk(c_i) + s q_i              (two FP32 roundings),
// so that |decode - v| <= s/2 plus FP32 rounding.  The bulk mesh is the
// coarse PM mesh (cells of coarse_ratio fine cells), or cells of 4 fine cells
// with one level; a bulk cell lies inside one tile, so every tile computes
// the means of its own cells.  The cell sums are exact 64-bit fixed point (a
// scale S = 2^(41 - e) with max|v| < 2^e), so the means are deterministic.
#include "common.hpp"

namespace cube2 {
namespace {

__global__ void vset2_kernel(unsigned int *p) {
    p[0] = 0u;
    p[1] = 0u;
}

// fixed-point scale S = 2^(41 - e) with max|v| < 2^e (1 when max is 0)
__device__ __forceinline__ float vel_scale(unsigned int amax_bits) {
    const float m = __uint_as_float(amax_bits);
    if (!(m > 0.0f) || !(m < 3.0e38f)) return 1.0f;
    int e;
    (void)frexpf(m, &e);
    return ldexpf(1.0f, min(41 - e, 100));
}

// bulk cell, inside its tile, of the particles of IOS cell u (0..511): bulk
// cells have 2^shift fine cells per axis, at least the 2 of an IOS cell, so
// the particle's offsets do not matter
__host__ __device__ __forceinline__ int bulk_cell(int u, int shift, int ct) {
    const int s = shift - 1;
    return (((u >> 6) >> s) * ct + (((u >> 3) & 7) >> s)) * ct + ((u & 7) >> s);
}

__host__ __device__ __forceinline__ int64_t bulk_index(int tx, int ty, int tz, int lc, int ct, int nb) {
    const int cx = tx * ct + lc % ct, cy = ty * ct + (lc / ct) % ct, cz = tz * ct + lc / (ct * ct);
    return ((int64_t)cz * nb + cy) * nb + cx;
}

// Per tile: fixed-point velocity sums of its bulk cells, the means written to
// v_bulk, and max |v - v_bulk| of its particles written to tmax[tile] (one global
// atomic per wave on a single address would serialise; the tile maxima are
// reduced by a second pass).  The counts are those of the cells' particle
// ranges.  A tile of up to kKeep particles per thread keeps its velocities in
// registers between the sums and the maxima.  Reading the positions for the bulk
// cell and summing runs of equal cells by a segmented scan of LDS permutes, this
// took 242 us for 256^3 particles, and the codes 130.
constexpr int kKeep = 4;
__global__ __launch_bounds__(kBlock) void vel_bulk_kernel(
    const uint32_t *__restrict__ cs, const float *__restrict__ vel, int n, int nt, int shift, int nb,
    const unsigned int *__restrict__ amax, float *__restrict__ v_bulk, float *__restrict__ tmax,
    uint32_t *status) {
    __shared__ float wmax[kBlock / 64];
    __shared__ unsigned long long sum[3][kTileCells];
    __shared__ float vb[3][kTileCells];
    __shared__ uint32_t cst[kTileCells + 1];
    int tx, ty, tz;
    tile_of_block(blockIdx.x, nt, tx, ty, tz);
    const int tid = threadIdx.x;
    const int ct = kTileFine >> shift;       // bulk cells per tile axis
    const int ncell = ct * ct * ct;
    for (int i = tid; i < ncell; i += kBlock) sum[0][i] = sum[1][i] = sum[2][i] = 0ull;
    const uint32_t key0 = (uint32_t)((tz * nt + ty) * nt + tx) * kTileCells;
    stage_cell_starts<kBlock>(cst, cs, key0);
    __syncthreads();
    const float S = vel_scale(amax[0]), invS = 1.0f / S;
    const uint32_t p0 = cst[0], p1 = cst[kTileCells];
    const int lane = tid & 63;
    float v[kKeep][3];
    int lc[kKeep];
    // Particles are sorted by IOS cell: in a dense cell a whole wave feeds one
    // bulk cell and adds its sum once, elsewhere a few lanes share one.
    for (uint32_t c0 = p0; c0 < p1; c0 += kBlock * kKeep) {
#pragma unroll
        for (int k = 0; k < kKeep; ++k) {
            const uint32_t p = c0 + k * kBlock + tid;
            lc[k] = -1;
            if (p < p1) {
#pragma unroll
                for (int d = 0; d < 3; ++d) v[k][d] = vel[(int64_t)d * n + p];
                lc[k] = bulk_cell(seg_search_n<kTileCells>(cst, p), shift, ct);
            }
        }
#pragma unroll
        for (int k = 0; k < kKeep; ++k) {
            const unsigned long long on = __ballot(lc[k] >= 0);
            if (on == 0ull) continue;
            const int lead = first_lane(on);
            const int lc0 = __builtin_amdgcn_readlane(lc[k], lead);
            const bool uniform = __ballot(lc[k] >= 0 && lc[k] != lc0) == 0ull;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const unsigned long long f =
                    lc[k] >= 0 ? (unsigned long long)__float2ll_rn(v[k][d] * S) : 0ull;
                if (uniform) {
                    const unsigned long long t = wave_sum(f);
                    if (lane == lead) atomicAdd(&sum[d][lc0], t);
                } else if (lc[k] >= 0) {
                    atomicAdd(&sum[d][lc[k]], f);
                }
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < ncell; i += kBlock) {
        // the bulk cell's particles: its IOS cells' x-rows
        const int w = 1 << (shift - 1), bx = (i % ct) * w, by = ((i / ct) % ct) * w, bz = i / (ct * ct) * w;
        uint32_t c = 0;
        for (int z = 0; z < w; ++z)
            for (int y = 0; y < w; ++y) {
                const int u = ((bz + z) * 8 + by + y) * 8 + bx;
                c += cst[u + w] - cst[u];
            }
        // 2^22 values below 2^41 each keep the sum within 63 bits
        if (c >= (1u << 22)) atomicOr(status, kStatusOverflow);
        const int64_t g = bulk_index(tx, ty, tz, i, ct, nb);
        const int64_t m3 = (int64_t)nb * nb * nb;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float mean =
                c ? __fdiv_rn(__fmul_rn((float)(long long)sum[d][i], invS), (float)c) : 0.0f;
            vb[d][i] = mean;
            v_bulk[d * m3 + g] = mean;
        }
    }
    __syncthreads();
    float dmax = 0.0f;
    if (p1 - p0 <= (uint32_t)(kBlock * kKeep)) {
#pragma unroll
        for (int k = 0; k < kKeep; ++k) {
            if (p0 + k * kBlock + tid >= p1) continue;
#pragma unroll
            for (int d = 0; d < 3; ++d) dmax = fmaxf(dmax, fabsf(__fsub_rn(v[k][d], vb[d][lc[k]])));
        }
    } else {
        for (uint32_t p = p0 + tid; p < p1; p += kBlock) {
            const int b = bulk_cell(seg_search_n<kTileCells>(cst, p), shift, ct);
#pragma unroll
            for (int d = 0; d < 3; ++d)
                dmax = fmaxf(dmax, fabsf(__fsub_rn(vel[(int64_t)d * n + p], vb[d][b])));
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dmax = fmaxf(dmax, __shfl_xor(dmax, m, 64));
    if ((tid & 63) == 0) wmax[tid >> 6] = dmax;
    __syncthreads();
    if (tid == 0) {
        float b = 0.0f;
        for (int w = 0; w < kBlock / 64; ++w) b = fmaxf(b, wmax[w]);
        tmax[blockIdx.x] = b;
    }
}

// the global scale s = max |v - v_bulk| / 32767 (1 when every deviation is 0)
__device__ __forceinline__ float vel_step(unsigned int dmax_bits) {
    const float m = __uint_as_float(dmax_bits);
    return m > 0.0f ? __fdiv_rn(m, 32767.0f) : 1.0f;
}

// Per tile: q = rint((v - v_bulk) / s) (ENCODE: reads vel_in and amax,
// writes vq_out and v_scale_out) or v = v_bulk + s q (decode: reads vq_in and
// v_scale, writes vel_out).  The tile's bulk velocities are staged, but from few particles
// (kStagedPerTile) read where they are: at ratio 2 they are 6 kB a tile.  Decode, us, staged
// and not: 512^3 mesh, ratio 2, 13 per tile 54 and 24, 109 82 and 40, 512 133 and 146; ratio 4,
// 13 per tile 29 and 24.
constexpr int64_t kStagedPerTile = 128;
template <bool ENCODE, bool STAGED>
__global__ __launch_bounds__(kBlock) void vel_code_kernel(
    const uint32_t *__restrict__ cs, int n, int nt, int shift, int nb,
    const float *__restrict__ v_bulk, const unsigned int *__restrict__ amax,
    const float *__restrict__ vel_in, int16_t *__restrict__ vq_out, float *__restrict__ v_scale_out,
    const float *__restrict__ v_scale, const int16_t *__restrict__ vq_in,
    float *__restrict__ vel_out) {
    __shared__ uint32_t cst[kTileCells + 1];
    __shared__ float vb[3][STAGED ? kTileCells : 1];
    int tx, ty, tz;
    tile_of_block(blockIdx.x, nt, tx, ty, tz);
    const int tid = threadIdx.x;
    const int ct = kTileFine >> shift;
    const uint32_t key0 = (uint32_t)((tz * nt + ty) * nt + tx) * kTileCells;
    const int64_t m3 = (int64_t)nb * nb * nb;
    if constexpr (STAGED)
        for (int i = tid; i < ct * ct * ct; i += kBlock) {
            const int64_t g = bulk_index(tx, ty, tz, i, ct, nb);
#pragma unroll
            for (int d = 0; d < 3; ++d) vb[d][i] = v_bulk[d * m3 + g];
        }
    stage_cell_starts<kBlock>(cst, cs, key0);
    __syncthreads();
    const float s = ENCODE ? vel_step(amax[1]) : v_scale[0];
    if (ENCODE && blockIdx.x == 0 && tid == 0) v_scale_out[0] = s;
    const uint32_t p1 = cst[kTileCells];
    constexpr int kBatch = 2;      // particles per thread whose loads are issued together
    for (uint32_t c0 = cst[0] + tid; c0 < p1; c0 += kBlock * kBatch) {
        float v[kBatch][3];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const uint32_t p = min(c0 + k * kBlock, p1 - 1);
#pragma unroll
            for (int d = 0; d < 3; ++d)
                v[k][d] = ENCODE ? vel_in[(int64_t)d * n + p] : (float)vq_in[(int64_t)d * n + p];
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const uint32_t p = c0 + k * kBlock;
            if (p >= p1) continue;
            const int lc = bulk_cell(seg_search_n<kTileCells>(cst, p), shift, ct);
            const int64_t g = STAGED ? 0 : bulk_index(tx, ty, tz, lc, ct, nb);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const float b = STAGED ? vb[d][lc] : v_bulk[d * m3 + g];
                if (ENCODE) {
                    const float r = rintf(__fdiv_rn(__fsub_rn(v[k][d], b), s));
                    vq_out[(int64_t)d * n + p] = (int16_t)fminf(fmaxf(r, -32767.0f), 32767.0f);
                } else {
                    // two roundings, as documented: no contraction into an FMA
#pragma clang fp contract(off)
                    const float sq = s * v[k][d];
                    vel_out[(int64_t)d * n + p] = b + sq;
                }
            }
        }
    }
}

// bulk cells: the coarse mesh's cells, or 4 fine cells with one level
int bulk_shift(const cube2_ctx *ctx) { return ctx->n_levels > 1 ? ctx->lv[1].hshift : 2; }

}  // namespace

int vel_bulk_side(const cube2_ctx *ctx) { return ctx->n_f >> bulk_shift(ctx); }

// The codec's index arithmetic for this context, run on the host with the
// kernels' own functions: every IOS cell of a tile lands in the bulk cell of each
// of its fine cells, one of the tile's ct^3 <= 512 (the LDS arrays), every bulk
// cell of every tile in
// [0, nb^3) (v_bulk), and the tile maxima fit their work area.
int vel_layout_check(const cube2_ctx *ctx, const WorkLayout &L) {
    const int shift = bulk_shift(ctx), nb = ctx->n_f >> shift, nt = ctx->nt;
    const int ct = kTileFine >> shift;
    if (ct < 1 || ct * ct * ct > kTileCells || (int64_t)nt * ct != nb) return CUBE2_EUNSUPPORTED;
    if (shift < 1) return CUBE2_EUNSUPPORTED;
    for (int u = 0; u < kTileCells; ++u)
        for (int a = 0; a < 8; ++a) {
            const int fx = 2 * (u & 7) + (a & 1), fy = 2 * ((u >> 3) & 7) + ((a >> 1) & 1),
                      fz = 2 * (u >> 6) + (a >> 2);
            const int lc = bulk_cell(u, shift, ct);
            if (lc != ((fz >> shift) * ct + (fy >> shift)) * ct + (fx >> shift) || lc < 0 ||
                lc >= ct * ct * ct)
                return CUBE2_EUNSUPPORTED;
        }
    const int64_t nb3 = (int64_t)nb * nb * nb;
    for (int tz = 0; tz < nt; ++tz)
        for (int ty = 0; ty < nt; ++ty)
            for (int tx = 0; tx < nt; ++tx)
                for (int lc = 0; lc < ct * ct * ct; ++lc) {
                    const int64_t g = bulk_index(tx, ty, tz, lc, ct, nb);
                    if (g < 0 || g >= nb3) return CUBE2_EUNSUPPORTED;
                }
    const size_t ntiles = (size_t)nt * nt * nt;
    if (L.vel_tmax + ntiles * sizeof(float) > L.total) return CUBE2_EWORKSPACE;
    return CUBE2_OK;
}

int launch_vel_encode(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                      const float *vel, int16_t *vq, float *v_bulk, float *v_scale,
                      unsigned char *work, const WorkLayout &L, hipStream_t s) {
    const int nt = ctx->nt;
    const unsigned blocks = (unsigned)(nt * nt * nt);
    const int shift = bulk_shift(ctx), nb = ctx->n_f >> shift;
    unsigned int *amax = reinterpret_cast<unsigned int *>(work + L.red);
    vset2_kernel<<<1, 1, 0, s>>>(amax);
    CUBE2_LAUNCH_CHECK();
    if (n > 0) {
        const int r = launch_absmax(vel, 3 * n, amax, s);
        if (r) return r;
    }
    // per-tile maxima in their own work area (one float per tile)
    float *tmax = reinterpret_cast<float *>(work + L.vel_tmax);
    vel_bulk_kernel<<<blocks, kBlock, 0, s>>>(cs, vel, (int)n, nt, shift, nb, amax, v_bulk, tmax,
                                              status_word(ctx));
    CUBE2_LAUNCH_CHECK();
    const int r = launch_absmax(tmax, (int64_t)blocks, amax + 1, s);
    if (r) return r;
    (void)pos;
    auto *code = n >= kStagedPerTile * (int64_t)blocks ? vel_code_kernel<true, true>
                                                       : vel_code_kernel<true, false>;
    code<<<blocks, kBlock, 0, s>>>(cs, (int)n, nt, shift, nb, v_bulk, amax, vel, vq, v_scale, nullptr,
                                   nullptr, nullptr);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

int launch_vel_decode(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                      const int16_t *vq, const float *v_bulk, const float *v_scale, float *vel,
                      hipStream_t s) {
    if (n == 0) return CUBE2_OK;
    const int nt = ctx->nt;
    const unsigned blocks = (unsigned)(nt * nt * nt);
    const int shift = bulk_shift(ctx), nb = ctx->n_f >> shift;
    (void)pos;
    auto *code = n >= kStagedPerTile * (int64_t)blocks ? vel_code_kernel<false, true>
                                                       : vel_code_kernel<false, false>;
    code<<<blocks, kBlock, 0, s>>>(cs, (int)n, nt, shift, nb, v_bulk, nullptr, nullptr, nullptr, nullptr,
                                   v_scale, vq, vel);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

}  // namespace cube2

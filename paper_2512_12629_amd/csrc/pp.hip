// pp.hip -- the short-range particle-particle force (eq. 4d): for every pair
// closer than the fine softening b_f (the cutoff of the finest PM level),
//   a_i += G m [R(r, b_pp) - R(r, b_f)] (x_j - x_i) / r,
// with R of eq. (2).  An IOS cell is 2 fine cells, so for b_f <= 2 every
// pair lies in the same or in adjacent IOS cells (27 neighbour cells), and
// for 2 < b_f <= 4 within two cells (125); the cell-sorted particle order is
// the linked list of the paper (section 2.3).
//
// The particles of a tile and of its halo of H cells (a (8 + 2H)^3 box of IOS
// cells; a light tile: of one or two of its layers of cells) are staged in LDS
// as FP32 positions relative to the tile origin in fine cells.  Offsets are
// multiples of 2^-15 below 2^5, so these floats and their differences are
// exact: the pair separation is the exact integer one.  A thread takes one
// particle (where tiles with much work are few, four threads share one) and
// loops over its neighbour cells, which in the staged box are (2H + 1)^2
// contiguous ranges (x-rows of 2H + 1 cells); neighbours in a dense cell are
// read by all lanes of a wave at the same LDS address (a broadcast).  Per range
// the pair sum is accumulated in FP32 and then added to the total with Kahan
// compensation.  Whole workgroups take the heavy tiles, or listed parts of them,
// single waves the light ones.  Boxes too large for LDS pass through it in
// parts.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>

#include "common.hpp"
#include "light_claims.hpp"

namespace cube2 {
namespace {

// H: the neighbour reach in IOS cells, 1 for b_f <= 2 fine cells (27
// neighbour cells) and 2 for b_f <= 4 (125).  The staged box has
// 8 + 2H IOS cells per axis.
template <int H> struct PPBox {
    static constexpr int PB = kTileIos + 2 * H;   // 10 or 12 IOS cells per axis
    static constexpr int SEGS = PB * PB * PB;      // 1000 or 1728
    static constexpr int W = 2 * H + 1;            // neighbour cells per axis
};
// Forward: 512 threads, 16 bytes per staged particle: 2 blocks (4 waves per
// SIMD) per CU in 160 KB of LDS, of which the pair-law table takes 20 KB each.
// Adjoint: the cotangent is staged too (24 bytes per particle) and the finer
// table takes 40 KB, so it runs 1024-thread blocks, 1 block (4 waves per SIMD).
template <bool ADJ, int H> struct PPGeo {
    static constexpr int BLOCK = ADJ ? 1024 : 512;
    static constexpr int CAP = ADJ ? (H == 1 ? 4800 : 4656) : (H == 1 ? 3376 : 3152);
    static constexpr int SEG_PER_THREAD = (PPBox<H>::SEGS + BLOCK - 1) / BLOCK;
    static constexpr int ROWS = ADJ ? kSRowsAdj : kSRows;
    // bytes of the workgroup-wide arrays (LDS offsets of the kernel below)
    static constexpr int XA = CAP * 16, PRE = XA + (ADJ ? CAP * 8 : 0),
                         DELTA = PRE + (PPBox<H>::SEGS + 1) * 4,
                         CST = DELTA + PPBox<H>::PB * PPBox<H>::PB * 3 * 4,
                         SCAN = CST + (kTileCells + 1) * 4, TILE = SCAN + (BLOCK / 64 + 1) * 4,
                         BYTES = TILE + 8;
};

// The light tiles' form (one-cell reach): waves work on their own, each with
// its own slice of the LDS.  LAYERS z-layers of a tile's cells per item at
// most, LCAP staged particles (forward: x, y and z in arrays of their own, 12
// bytes per particle).
template <bool ADJ> struct PPLight {
    static constexpr int WAVES = ADJ ? 9 : 8;
    static constexpr int LAYERS = kPPLightLayers;
    static constexpr int SEGS = 100 * (LAYERS + 2);
    static constexpr int LCAP = ADJ ? kPPLightCapAdj : kPPLightCap;
    static constexpr int XA = LCAP * (ADJ ? 16 : 12), DELTA = LCAP * (ADJ ? 24 : 12),
                         OWN = DELTA + 30 * (LAYERS + 2) * 4, PRE = OWN + 8 * LAYERS * 4,
                         BYTES = (int)((PRE + (SEGS + 1) * 2 + 15) / 16 * 16);
};

}  // namespace

// The pair law g(r) = [R(r,b_pp) - R(r,b_f)] / r (eqs. 2 and 4d) as
// g = U(r) / r^3 with U = r^3 g.  On each of the intervals delimited by the
// breakpoints of eq. (2) -- b_pp/2, b_pp (PP softening), b_f/2 (fine
// softening) -- and the cutoff b_f, U is an exact polynomial of degree 8 in r:
//   r^3 b^-3 F_in(r/b)  = sum_k a_k b^(-3-k) r^(k+3),
//   r^3 b^-3 F_out(r/b) = 3/35 - 32/5 (r/b)^2 + sum_k c_k b^(-3-k) r^(k+3),
//   r^3 r^-3 = 1 (Newtonian beyond b_pp),
// with F_in, F_out the two polynomial branches of R(r,b)/r in t = r/b.
// [0, b_f) is cut into K equal intervals with every breakpoint on an
// interval edge, and each interval stores its polynomial re-expanded (FP64,
// on the host) in a local variable y in [0, 1]:  y = fract(r K / b_f) (left
// edge, keeps U ~ r^3 accurate at r -> 0) or y = 1 - fract(.) (right edge)
// on the intervals where 1/r^2 - R(r, b_f) vanishes like (1 - r/b_f)^5 at the
// cutoff, which use the exact factorisation r^3 g = s^5 Q(1 - s),
// s = 1 - r/b_f, Q(t) = 32/35 + 32/7 t + 704/35 t^2 + 64/5 t^3.  The row of
// r >= b_f is zero.  This exact table, in FP64, serves the plain FP64 form.
//
// The FP32 kernels evaluate g as a function of s = r^2 instead, which needs
// neither a square root nor r^-3, through its fifth root: g = (unit/4) L(s)^5.
// Near the cutoff g vanishes like (1 - r/b_f)^5, and sparse particles often
// have all their neighbours there, so a table of g itself would lose its
// relative accuracy; L has a simple zero at the cutoff, which a table follows
// to the last bit, and 0.3 times the curvature of g where g ~ 1/r^3.  L is a
// quadratic per row of 1/64 octave of s (the adjoint, which also needs dL/ds:
// 1/128), in y = 0.4 s - k with k, the row's centre, in the row's fourth
// word: L = c0 + t y, t = c1 + c2 y.  Among the floats next to the centre, k is
// the one whose L is nearest to a float, so that c0 adds no error of its own.
// The fifth power would take the rounding of l = fl(L) five times; one of the five
// factors is therefore L - 3/4 l (root_rest), so that the product l^4 (L - 3/4 l) has it
// once, for two instructions.  With y in 0.4 s the derivative comes free: 2 dg/ds = unit
// L^4 (c1 + 2 c2 y).  unit/4 is a power of two that puts L in [0, 1]; in the row that
// holds the cutoff c0 = 0 and k = 0.4 b_f^2, so that the FMA's clamp to [0, 1] gives
// l = 0, and so exactly g = 0, at and beyond b_f, and the rows beyond are zero.
//
// Against a cubic of g / (1 - s/b_f^2)^4 on rows of 1/16 octave: 19 instructions per
// pair instead of 20, 32 instead of 39 in the adjoint.  Errors (FP32 operations against
// extended precision, that cubic -> l^5 -> now; b_f = 2, b_pp = 0.2): of g r, over
// separations uniform in the sphere of b_f, 1.23e-7 -> 1.46e-7 -> 0.90e-7 rms; relative,
// for r < 0.9 b_f, 3.8e-7 -> 3.7e-7 -> 3.5e-7; times 1 - r/b_f beyond it 6.33e-8 ->
// 6.36e-8 -> 6.36e-8 (the rounding of s); the adjoint's derivative term, of the Jacobian,
// 5.8e-6 -> 1.9e-6 -> 1.9e-6.
//
// s0 = 2^e0 is added to s, with e0 at most -13 and at least 3 octaves below
// (b_pp/2)^2: below that g is nearly constant, so the table has no use for finer octaves and a
// coincident pair has a row (g finite, g D = 0).  Positions are staged in
// units of 2^-j fine cells, which are exact too, with j such that s0 has
// float exponent field 128: a row's place in the table is then its bits modulo
// 32 octaves, with no base to subtract.  Every separation in the staged box is
// below 2 (H + 1) fine cells per axis, so s < 2^6 (H = 1) or 2^7.  If the
// octaves from s0 to there exceed the 20 that the table holds (a small b_f or
// b_pp), s is clamped to the first row beyond the cutoff instead (CLAMP, one
// more instruction per pair): cutoff and s0 are at most 19 octaves apart,
// since b_pp / 2 >= b_f / 128.

namespace {

// The pair-law tables in LDS, declared at namespace scope so that every
// access is a 32-bit LDS address.
// s0 in the scaled units: float exponent field 128
constexpr float kPairS0 = 2.0f;
constexpr float kPairY = 0.4f;     // y in units of s
__shared__ float4 pair_srows[kSRows];
__shared__ float4 pair_arows[kSRowsAdj];

__device__ __forceinline__ void kahan_add(float &s, float &c, float v) {
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

__device__ __forceinline__ float unit_clamp(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 1.0f); }

// Place of the row of s (float bits b) in the table of 2^mant rows per octave.
__host__ __device__ __forceinline__ uint32_t row_place(uint32_t b, int mant) {
    return (b >> (23 - mant)) & (uint32_t)((kSOctaves << mant) - 1);
}

// L - 3/4 l for the rounded l of L = c0 + t y: a quarter of L, less three times l's
// rounding error.  The product of it with l^4, which holds that error four times, is a
// quarter of g / unit with the error once instead of five times.  c0 - 3/4 l is exact.
__host__ __device__ __forceinline__ float root_rest(float t, float y, float c0, float l) {
    return fmaf(t, y, fmaf(-0.75f, l, c0));
}

// g(r) D / unit accumulated into (fx, fy, fz).  s0 is staged as the fourth
// word of the neighbour: with all four words in use the position is one
// 128-bit LDS read, which takes 4.7 cycles of the CU's LDS for a wave that
// reads a few addresses (12 for 64 different ones); a 96-bit read takes 8.5
// (20).
template <bool CLAMP>
__device__ __forceinline__ void pair_accumulate(float dx, float dy, float dz, float s0,
                                                uint32_t bmax, float &fx, float &fy, float &fz) {
    const float s = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, s0)));
    uint32_t b = __float_as_uint(s);
    if (CLAMP) b = min(b, bmax);
    const float4 c = pair_srows[row_place(b, kSMant)];
    const float y = fmaf(s, kPairY, c.w);
    const float t = fmaf(c.z, y, c.y);
    const float l = unit_clamp(fmaf(t, y, c.x));
    const float l2 = l * l;
    const float g = (l2 * l2) * root_rest(t, y, c.x, l);
    fx = fmaf(g, dx, fx);
    fy = fmaf(g, dy, fy);
    fz = fmaf(g, dz, fz);
}

// Adjoint of one pair for the cotangents: out += J(D) u / unit with u = abar_j
// - abar_i and J = d(g D)/dD = g I + 2 g_s D D^T, g_s = dg/ds.  Every term
// enters the accumulators through an FMA.
template <bool CLAMP>
__device__ __forceinline__ void pair_adjoint(float dx, float dy, float dz, float ux, float uy,
                                             float uz, uint32_t bmax, float &ox,
                                             float &oy, float &oz) {
    const float s = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, kPairS0)));
    uint32_t b = __float_as_uint(s);
    if (CLAMP) b = min(b, bmax);
    const float4 c = pair_arows[row_place(b, kSMantAdj)];
    const float y = fmaf(s, kPairY, c.w);
    const float t = fmaf(c.z, y, c.y);
    const float l = unit_clamp(fmaf(t, y, c.x));
    const float ls = fmaf(c.z, y, t);                   // 2.5 dL/ds
    const float l2 = l * l;
    const float l4 = l2 * l2;
    const float g = l4 * root_rest(t, y, c.x, l);
    const float du = fmaf(dz, uz, fmaf(dy, uy, dx * ux)) * (l4 * ls);   // D.u 2 g_s
    ox = fmaf(du, dx, fmaf(g, ux, ox));
    oy = fmaf(du, dy, fmaf(g, uy, oy));
    oz = fmaf(du, dz, fmaf(g, uz, oz));
}

// The pairs of one particle with the staged neighbours v0, v0 + STEP, ... below v1:
// four per iteration, so that the loop control and the LDS latency spread over
// more work.  The loops run on the LDS address against precomputed bounds, never
// below xs (LDS addresses compare unsigned).
template <bool ADJ, bool CLAMP, int STEP>
__device__ __forceinline__ void staged_pairs(const float4 *xs, const float2 *xa, uint32_t v0,
                                             uint32_t v1, float xi, float yi, float zi, float aix,
                                             float aiy, float aiz, uint32_t bmax, float &fx, float &fy,
                                             float &fz) {
    const float4 *q = xs + v0;
    const float2 *qa = xa + v0;
    const float4 *const qe = xs + v1;
    const float4 *const qe4 = xs + (v1 > v0 + 3 * STEP ? v1 - 3 * STEP : v0);
    auto pair = [&](const float4 &x, const float2 &a) {
        if constexpr (ADJ)
            pair_adjoint<CLAMP>(x.x - xi, x.y - yi, x.z - zi, x.w - aix, a.x - aiy, a.y - aiz, bmax, fx,
                                fy, fz);
        else
            pair_accumulate<CLAMP>(x.x - xi, x.y - yi, x.z - zi, x.w, bmax, fx, fy, fz);
    };
    auto cot = [&](int t) { return ADJ ? qa[t] : make_float2(0.f, 0.f); };
    for (; q < qe4; q += 4 * STEP, qa += 4 * STEP) {
        float4 x[4];
        float2 a[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            x[t] = q[t * STEP];
            a[t] = cot(t * STEP);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) pair(x[t], a[t]);
    }
    if constexpr (!ADJ && STEP == 1) {   // up to three more: two, then one
        if ((v1 - v0) & 2u) {
            const float4 x = q[0], y = q[1];
            pair(x, cot(0));
            pair(y, cot(1));
            q += 2;
        }
        if ((v1 - v0) & 1u) pair(q[0], cot(0));
    } else {
        for (; q < qe; q += STEP, qa += STEP) pair(q[0], cot(0));
    }
}

// Sum over the four lanes of a quad, the same in each of them.
__device__ __forceinline__ float quad_sum(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
    return v;
}

// Heavy tiles with much work are taken in parts (the list of PPOrder, pack.hip): each
// part stages the tile's box and takes every nparts-th block of its own particles.  In
// small parts, and where a single particle's neighbours would outlast the other work
// (kLanesBit), four lanes share a particle, each taking every fourth neighbour, and their
// sums are added per range (parts of whole blocks would leave a CU to 8 or 16 waves whose
// pair loops wait on the LDS).  The FP32 rounding of a heavy
// tile's sums therefore depends on the work of the others; it is the same for every call
// on the same particles.
constexpr int kFewLanes = 4;

// Most neighbours whose forces are added in plain FP32 before they enter the compensated
// sum, in the forward with the one-cell reach.  Whole rows of three dense cells lost the
// small terms of a halo's edge beside the large ones of its core (a row of 3000 particles
// in a core and 3000 at the cutoff: rms error 2.5e-7 of the force, so 0.5e-7; single
// particles of overlapping halos 2.5e-5).  1024^3 mesh: 21.7 -> 21.3 ms.  The adjoint, whose
// errors are its table's, would lose 1.7%, and the two-cell reach 10% to spilled registers.
constexpr uint32_t kRange = 512;

// The pair law's units (see above): ps = 2^j and its product with the 2^-15 of
// a position unit, the scale of the sums (unit, and for the forward D's
// 2^-j too) and the float bits that the clamped form stops at.
struct PPLaw {
    float ps, ips, unit;
    uint32_t bmax;
};

// The pairs of one particle with the staged neighbours [v0, v1): two per trip.
template <bool ADJ, bool CLAMP>
__device__ __forceinline__ void light_row(const unsigned char *base, uint32_t v0, uint32_t v1, float xi,
                                          float yi, float zi, float aix, float aiy, float aiz,
                                          uint32_t bmax, float &fx, float &fy, float &fz) {
    using P = PPLight<ADJ>;
    if constexpr (ADJ) {
        const float4 *q = reinterpret_cast<const float4 *>(base);
        const float2 *qa = reinterpret_cast<const float2 *>(base + P::XA);
        for (; v0 + 1 < v1; v0 += 2) {
            const float4 x = q[v0], y = q[v0 + 1];
            const float2 a = qa[v0], b = qa[v0 + 1];
            pair_adjoint<CLAMP>(x.x - xi, x.y - yi, x.z - zi, x.w - aix, a.x - aiy, a.y - aiz, bmax,
                                fx, fy, fz);
            pair_adjoint<CLAMP>(y.x - xi, y.y - yi, y.z - zi, y.w - aix, b.x - aiy, b.y - aiz, bmax,
                                fx, fy, fz);
        }
        if (v0 < v1) {
            const float4 x = q[v0];
            const float2 a = qa[v0];
            pair_adjoint<CLAMP>(x.x - xi, x.y - yi, x.z - zi, x.w - aix, a.x - aiy, a.y - aiz, bmax,
                                fx, fy, fz);
        }
    } else {
        const float *x = reinterpret_cast<const float *>(base), *y = x + P::LCAP, *z = y + P::LCAP;
        for (; v0 + 1 < v1; v0 += 2) {
            const float x0 = x[v0], x1 = x[v0 + 1], y0 = y[v0], y1 = y[v0 + 1], z0 = z[v0], z1 = z[v0 + 1];
            pair_accumulate<CLAMP>(x0 - xi, y0 - yi, z0 - zi, kPairS0, bmax, fx, fy, fz);
            pair_accumulate<CLAMP>(x1 - xi, y1 - yi, z1 - zi, kPairS0, bmax, fx, fy, fz);
        }
        if (v0 < v1) pair_accumulate<CLAMP>(x[v0] - xi, y[v0] - yi, z[v0] - zi, kPairS0, bmax, fx, fy, fz);
    }
}

// The ranges of a particle's neighbour rows, length << 16 | start, longest first
// (merge exchange, Knuth vol. 3, 5.2.2 M: 26 comparators for 9 rows, two instructions
// each).  All lanes of a wave go through their rows together, so that a wave's trips are
// the sum over the rows of the longest of its lanes'.  Rows in the order of the cells give
// nine times the densest row to a wave of sparse cells around a halo, where each
// lane meets the halo in another row; longest first, every lane meets it at once
// (512^3 particles with 8000 halos: 25.1 -> 21.9 ms, adjoint 43.8 -> 35.8; two-cell
// reach, 201^3 with 300: 3.52 -> 2.57 ms).  The light tiles' rows are short and
// alike: there it gained nothing (103 us for 128^3 particles, 106 sorted).
template <int N> struct RowSort {
    struct Pair { int i, j; };
    static constexpr int MAX = N * N;
    struct Net { Pair p[MAX]; int n; };
    static constexpr Net make() {
        Net net{};
        int top = 1;
        while (2 * top < N) top *= 2;
        for (int p = top; p > 0; p /= 2) {
            int q = top, r = 0, d = p;
            for (;;) {
                for (int i = 0; i < N - d; ++i)
                    if ((i & p) == r) net.p[net.n++] = Pair{i, i + d};
                if (q == p) break;
                d = q - p;
                q /= 2;
                r = p;
            }
        }
        return net;
    }
    static constexpr Net net = make();
    template <int... K>
    static __device__ __forceinline__ void run(uint32_t (&a)[N], std::integer_sequence<int, K...>) {
        auto step = [&](int i, int j) {
            const uint32_t x = a[i], y = a[j];
            a[i] = max(x, y);
            a[j] = min(x, y);
        };
        (step(net.p[K].i, net.p[K].j), ...);
    }
    static __device__ __forceinline__ void sort(uint32_t (&a)[N]) {
        run(a, std::make_integer_sequence<int, net.n>{});
    }
    // the next row: the first of a, and the others move up
    static __device__ __forceinline__ uint32_t next(uint32_t (&a)[N]) {
        const uint32_t x = a[0];
#pragma unroll
        for (int k = 0; k + 1 < N; ++k) a[k] = a[k + 1];
        a[N - 1] = 0u;
        return x;
    }
};

// LDS stores of this wave are visible to its own later loads (the LDS serves
// a wave in order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Light tiles (few particles in every box, see pp_tile_keys_kernel), each wave
// by itself: `layers` z-layers of a tile's cells per item, 64 own particles at
// a time, the box of 10 x 10 x (layers + 2) cells staged in the wave's slice
// of the LDS.  A whole workgroup per such tile spent most of its time waiting:
// ~500 particles have ~27 candidates each, and between the tile's claim and
// its first pair lay four dependent memory accesses and seven barriers.  Waves
// with an item each overlap these chains without a barrier, and the adjoint's
// 1024-thread workgroup no longer idles half its threads.  What bounds it now
// is the LDS: the reads of the pair loop, whose lanes are in different cells.
// Measured without halos: 480^3 particles on 1024^3 5.5 -> 4.6 ms (adjoint
// 14.3 -> 7.8), 128^3 on 256^3 148 -> 124 us (266 -> 185).  Positions as
// 16-byte words, with room for 7 waves instead of 8: 4.7 ms and 133 us.
template <bool ADJ, bool CLAMP>
__device__ __forceinline__ void light_tiles(unsigned char *lds, const uint16_t *__restrict__ pos,
                                            const uint32_t *__restrict__ cs, int n, int nt,
                                            const PPLaw &law, float gm, const float *__restrict__ abar,
                                            float *__restrict__ acc, int accumulate,
                                            const uint32_t *__restrict__ order,
                                            uint32_t *__restrict__ queue, int ntiles, int layers,
                                            const uint8_t *__restrict__ skip) {
    using P = PPLight<ADJ>;
    constexpr int PER = (P::SEGS + 63) / 64;       // box cells per lane
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    if (wave >= P::WAVES) return;
    unsigned char *const base = lds + wave * P::BYTES;
    float *const x = reinterpret_cast<float *>(base);
    uint32_t *const delta = reinterpret_cast<uint32_t *>(base + P::DELTA);
    uint32_t *const ownp = reinterpret_cast<uint32_t *>(base + P::OWN);   // first particle of each own row
    uint16_t *const pre = reinterpret_cast<uint16_t *>(base + P::PRE);
    const int n_ios = nt * kTileIos;
    const float ps = law.ps, ips = law.ips;
    const int per_tile = kTileIos / layers;
    const int ncell = 100 * (layers + 2), nown = 8 * layers;
    auto part_of = [](int bx) { return bx < 1 ? 0 : (bx < 1 + kTileIos ? 1 : 2); };
    // Claims per XCD (LightClaims): one claim per item from one counter took 31.6 ms
    // instead of 25.0 for 512^3 particles.  Chunks of 4 items at most, so that the waves of
    // an XCD work on neighbouring tiles, whose boxes share lines of its L2 (the same, 64
    // items 21.8 ms, 16 21.3, 8 21.2, 4 21.0, 1 20.5; adjoint 34.9 and 33.4; but with one
    // item 128^3 particles beside PM take 325 us instead of 318).
    LightClaims claims((int)gridDim.x, (int)blockIdx.x, wave, P::WAVES, ntiles, per_tile,
                       nt * nt * nt >= kXcdQueueWords);
    auto claim = [&](int g) { return lane == 0 ? (int)min(atomicAdd(queue + 32 * g, 1u), 0x3FFFFFFFu) : 0; };
    auto first = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    int place, zp;
    while (claims.take(place, zp, claim, first)) {
        const int t = (int)(order[place] & kTileMask);
        if (skip && skip[t]) continue;
        const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
        const int c0x = tx * kTileIos - 1, c0y = ty * kTileIos - 1,
                  c0z = tz * kTileIos - 1 + zp * layers;
        wave_fence();       // the previous item's loads come first
        // particle ranges of the box cells, PER consecutive ones per lane
        uint32_t src[PER], cnt[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int s = min(lane * PER + k, ncell - 1);
            const int r = s / 10, bx = s - r * 10, bz = r / 10, by = r - bz * 10;
            const uint32_t key = cell_key(wrapn(c0x + bx, n_ios), wrapn(c0y + by, n_ios),
                                          wrapn(c0z + bz, n_ios), nt);
            src[k] = cs[key];
            cnt[k] = cs[key + 1];
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            cnt[k] = lane * PER + k < ncell ? cnt[k] - src[k] : 0u;
            sum += cnt[k];
        }
        uint32_t at = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(at, o, 64);
            if (lane >= o) at += y;
        }
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)at, 63);
        at -= sum;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int s = lane * PER + k;
            if (s < ncell) {
                const int r = s / 10, bx = s - r * 10;
                pre[s] = (uint16_t)at;
                if (bx <= 1 || bx == 9) delta[r * 3 + part_of(bx)] = src[k] - at;
            }
            at += cnt[k];
        }
        for (int s = ncell + lane; s <= P::SEGS; s += 64) pre[s] = (uint16_t)total;
        wave_fence();
        if (lane < nown) {   // own rows: box layers 1..layers, y 1..8, x 1..8
            const int r = (1 + (lane >> 3)) * 10 + 1 + (lane & 7);
            ownp[lane] = pre[r * 10 + 1] + delta[r * 3 + 1];
        }
        // stage, four particles per lane at a time
        constexpr int kStage = 4;
        for (uint32_t v0 = (uint32_t)lane; v0 < total; v0 += 64 * kStage) {
            int u[kStage];
            uint32_t p[kStage], o[kStage][3];
            float ab[kStage][3];
#pragma unroll
            for (int k = 0; k < kStage; ++k) {
                const uint32_t v = min(v0 + 64 * k, total - 1);   // past the end: the last again
                int lo = 0;
#pragma unroll
                for (int step = 256; step > 0; step >>= 1) {
                    const int c = min(lo + step, P::SEGS);
                    if (pre[c] <= v && c < P::SEGS) lo = c;
                }
                u[k] = lo;
                const int r = lo / 10;
                p[k] = v + delta[r * 3 + part_of(lo - r * 10)];
            }
#pragma unroll
            for (int k = 0; k < kStage; ++k) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    o[k][d] = pos[(int64_t)d * n + p[k]];
                    if (ADJ) ab[k][d] = abar[(int64_t)d * n + p[k]];
                }
            }
#pragma unroll
            for (int k = 0; k < kStage; ++k) {
                const uint32_t v = min(v0 + 64 * k, total - 1);
                const int r = u[k] / 10, bx = u[k] - r * 10, bz = r / 10, by = r - bz * 10;
                const float qx = (float)(2 * (bx - 1)) * ps + (float)o[k][0] * ips,
                            qy = (float)(2 * (by - 1)) * ps + (float)o[k][1] * ips,
                            qz = (float)(2 * (bz - 1)) * ps + (float)o[k][2] * ips;
                if constexpr (ADJ) {
                    reinterpret_cast<float4 *>(base)[v] = make_float4(qx, qy, qz, ab[k][0]);
                    reinterpret_cast<float2 *>(base + P::XA)[v] = make_float2(ab[k][1], ab[k][2]);
                } else {
                    x[v] = qx;
                    x[P::LCAP + v] = qy;
                    x[2 * P::LCAP + v] = qz;
                }
            }
        }
        wave_fence();
        const int rl = layers * 10 + 8;      // last own row
        const uint32_t p1 = pre[rl * 10 + 9] + delta[rl * 3 + 1];
        for (uint32_t p = ownp[0] + lane; p < p1; p += 64) {
            int i = 0;
#pragma unroll
            for (int step = P::LAYERS * 4; step > 0; step >>= 1)
                if (i + step < nown && ownp[i + step] <= p) i += step;
            const int r = (1 + (i >> 3)) * 10 + 1 + (i & 7);
            const uint32_t v = p - delta[r * 3 + 1];
            int c = r * 10 + 1;
#pragma unroll
            for (int step = 4; step > 0; step >>= 1)
                if (pre[c + step] <= v) c += step;
            float xi, yi, zi, aix = 0.f, aiy = 0.f, aiz = 0.f;
            if constexpr (ADJ) {
                const float4 q = reinterpret_cast<const float4 *>(base)[v];
                const float2 a = reinterpret_cast<const float2 *>(base + P::XA)[v];
                xi = q.x;
                yi = q.y;
                zi = q.z;
                aix = q.w;
                aiy = a.x;
                aiz = a.y;
            } else {
                xi = x[v];
                yi = x[P::LCAP + v];
                zi = x[2 * P::LCAP + v];
            }
            uint32_t v0[9], v1[9];
#pragma unroll
            for (int row = 0; row < 9; ++row) {
                const int sm = c + (row / 3 - 1) * 100 + (row % 3 - 1) * 10;
                v0[row] = pre[sm - 1];
                v1[row] = pre[sm + 2];
            }
            float sx = 0.f, sy = 0.f, sz = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
#pragma unroll
            for (int row = 0; row < 9; ++row) {
                float fx = 0.f, fy = 0.f, fz = 0.f;
                light_row<ADJ, CLAMP>(base, v0[row], v1[row], xi, yi, zi, aix, aiy, aiz, law.bmax, fx,
                                      fy, fz);
                kahan_add(sx, cx, fx);
                kahan_add(sy, cy, fy);
                kahan_add(sz, cz, fz);
            }
            const float a[3] = {gm * (sx * law.unit), gm * (sy * law.unit), gm * (sz * law.unit)};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                float *dst = acc + (int64_t)d * n + p;
                *dst = accumulate ? *dst + a[d] : a[d];
            }
        }
    }
}

// ADJ = false: acc = G m sum_j g D (forward).  ADJ = true: out = G m sum_j
// J(D) (abar_j - abar_i) for the cotangent abar (the adjoint), which stages
// abar_j beside x_j.
template <bool ADJ, int H, bool CLAMP>
__global__ __launch_bounds__((PPGeo<ADJ, H>::BLOCK), 4) void pp_kernel(const uint16_t *__restrict__ pos,
                                                     const uint32_t *__restrict__ cs, int n,
                                                     int nt, const float4 *__restrict__ table,
                                                     PPLaw law, float gm,
                                                     const float *__restrict__ abar,
                                                     float *__restrict__ acc, int accumulate,
                                                     const uint32_t *__restrict__ order,
                                                     uint32_t *__restrict__ queue, int ntiles,
                                                     const uint32_t *__restrict__ counts,
                                                     const uint32_t *__restrict__ parts,
                                                     uint32_t *__restrict__ light_queue,
                                                     int layers, const uint8_t *__restrict__ skip) {
    using G = PPGeo<ADJ, H>;
    constexpr int CAP = PPGeo<ADJ, H>::CAP;
    constexpr int kPPBlock = PPGeo<ADJ, H>::BLOCK;
    constexpr int kPSegPerThread = PPGeo<ADJ, H>::SEG_PER_THREAD;
    constexpr int kPB = PPBox<H>::PB, kPSegs = PPBox<H>::SEGS, kW = PPBox<H>::W;
    // one arena: the workgroup's arrays, then the waves' slices of the light tiles
    constexpr int kArena = H == 1 && PPLight<ADJ>::WAVES * PPLight<ADJ>::BYTES > G::BYTES
                               ? PPLight<ADJ>::WAVES * PPLight<ADJ>::BYTES : G::BYTES;
    __shared__ __align__(16) unsigned char lds[kArena];
    // staged particles: position and s0, or for the adjoint position and
    // cotangent (x, y, z, ax; ay, az)
    float4 *const xs = reinterpret_cast<float4 *>(lds);
    float2 *const xa = reinterpret_cast<float2 *>(lds + G::XA);
    uint32_t *const seg_pre = reinterpret_cast<uint32_t *>(lds + G::PRE);
    // An x-row of the box crosses three tiles (H, 8 and H cells), and a tile's
    // x-consecutive cells are consecutive in the particle order: particle =
    // staged index + seg_delta of the row's part
    uint32_t *const seg_delta = reinterpret_cast<uint32_t *>(lds + G::DELTA);
    uint32_t *const cst = reinterpret_cast<uint32_t *>(lds + G::CST);   // own cells: tile-relative starts
    uint32_t *const scan_sh = reinterpret_cast<uint32_t *>(lds + G::SCAN);
    int &tile_sh = *reinterpret_cast<int *>(lds + G::TILE);
    uint32_t &maxcnt_sh = *reinterpret_cast<uint32_t *>(lds + G::TILE + 4);

    const int tid = threadIdx.x;
    const int n_ios = nt * kTileIos;
    const float ps = law.ps, ips = law.ips;
    const uint32_t bmax = law.bmax;
    for (int i = tid; i < PPGeo<ADJ, H>::ROWS; i += kPPBlock) (ADJ ? pair_arows : pair_srows)[i] = table[i];
    // part of a box row that holds the box coordinate bx
    auto part_of = [](int bx) { return bx < H ? 0 : (bx < H + kTileIos ? 1 : 2); };

    // Persistent workgroups: each takes the next work item (claim_slot) until all are
    // taken (the exit test is block-uniform).  Thread 0 claims the next item while the
    // current one is processed.  Items are the listed parts of the tiles with the most
    // work, then whole tiles in order.
    // counts[0]: the tiles that are not light; only the one-cell reach takes the light
    // ones by waves
    const int nheavy = H == 1 ? (int)counts[0] : ntiles;
    const int nlisted = (int)counts[1], nlist = (int)counts[2], nitems = nheavy - nlisted + nlist;
    // Without heavy tiles there is nothing to claim: the claim's round trip is 4 us
    // (32^3 particles, 64 tiles: 34.5 -> 30.4 us).
    int next = 0;
    if (tid == 0 && nitems > 0) next = claim_slot(queue, nitems);
    while (nitems > 0) {
        if (tid == 0) {
            tile_sh = next;
            maxcnt_sh = 0u;
        }
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(tile_sh);   // block-uniform
        if (item >= nitems) break;
        if (tid == 0) next = claim_slot(queue, nitems);
        const uint32_t word = item < nlist ? parts[item] : order[item - nlist + nlisted] & kTileMask;
        const int t = (int)(word & kTileMask), part = (int)(word >> kTileBits & (kMaxParts - 1u)),
                  nparts = (int)(word >> (kTileBits + kPartBits) & (kMaxParts - 1u)) + 1;
        if (skip && skip[t]) {   // another level's tile
            __syncthreads();     // every thread has read tile_sh
            continue;
        }
        const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
        const int c0x = tx * kTileIos, c0y = ty * kTileIos, c0z = tz * kTileIos;

        // particle ranges of the (8 + 2H)^3 box of IOS cells [c0-H, c0+8+H)
        uint32_t cnt[kPSegPerThread], src[kPSegPerThread], pre_k[kPSegPerThread];
        uint32_t sum = 0, mx = 0;
#pragma unroll
        for (int k = 0; k < kPSegPerThread; ++k) {
            const int s = tid * kPSegPerThread + k;
            cnt[k] = 0;
            src[k] = 0;
            if (s < kPSegs) {
                const int bx = s % kPB, by = (s / kPB) % kPB, bz = s / (kPB * kPB);
                const uint32_t key = cell_key(wrapn(c0x + bx - H, n_ios), wrapn(c0y + by - H, n_ios),
                                              wrapn(c0z + bz - H, n_ios), nt);
                src[k] = cs[key];
                cnt[k] = cs[key + 1] - src[k];
            }
            sum += cnt[k];
            mx = max(mx, cnt[k]);
        }
        atomicMax(&maxcnt_sh, mx);
        uint32_t total;
        uint32_t pre = block_exclusive_scan<kPPBlock>(sum, scan_sh, total);
#pragma unroll
        for (int k = 0; k < kPSegPerThread; ++k) {
            const int s = tid * kPSegPerThread + k;
            if (s < kPSegs) {
                seg_pre[s] = pre;
                const int bx = s % kPB;
                if (bx == 0 || bx == H || bx == H + kTileIos)
                    seg_delta[(s / kPB) * 3 + part_of(bx)] = src[k] - pre;
            }
            pre_k[k] = pre;
            pre += cnt[k];
        }
        if (tid == 0) seg_pre[kPSegs] = total;
        __syncthreads();
        // own cells (box segments with coordinates H..H+7): their particle
        // starts relative to the tile's first particle, from the box ranges
        // (the own cells' particles are one contiguous range)
        const uint32_t p0 = seg_pre[(H * kPB + H) * kPB + H] + seg_delta[(H * kPB + H) * 3 + 1];
        for (int i = tid; i <= kTileCells; i += kPPBlock) {
            const int u = min(i, kTileCells - 1);          // past the end: the last own cell's end
            const int row = ((u >> 6) + H) * kPB + ((u >> 3) & 7) + H;
            cst[i] = seg_pre[row * kPB + (u & 7) + H + (i - u)] + seg_delta[row * 3 + 1] - p0;
        }
        __syncthreads();
        const uint32_t maxcnt = maxcnt_sh;
        const uint32_t own = cst[kTileCells];
        const int lanes = word & kLanesBit ? kFewLanes : 1;           // per particle
        const int sub = tid & (lanes - 1), kOwn = kPPBlock / lanes;   // own particles per block
        const bool single = total <= (uint32_t)CAP;   // the whole box is staged at once

        // Blocks of own particles, one particle per thread; part p of a split
        // tile takes blocks p, p + nparts, ...  A box that fits is staged for the
        // first of them.  Otherwise each block streams the box layers that its
        // cells reach through LDS, CAP particles at a time, its sums staying in
        // registers.
        bool staged = false;
        for (uint32_t l0 = (uint32_t)(part * kOwn); l0 < own; l0 += (uint32_t)(kOwn * nparts)) {
            const uint32_t lp = l0 + tid / lanes;
            const bool active = lp < own;
            const int u = seg_search_n<kTileCells>(cst, active ? lp : own - 1);
            const uint32_t p = p0 + (active ? lp : own - 1);
            const int bx = (u & 7) + H, by = ((u >> 3) & 7) + H, bz = (u >> 6) + H;
            const int su = (bz * kPB + by) * kPB + bx;
            const uint32_t vown = seg_pre[su] + (active ? lp : own - 1) - cst[u];
            uint32_t V0 = 0, V1 = total;
            float xi = 0.f, yi = 0.f, zi = 0.f;
            float aix = 0.f, aiy = 0.f, aiz = 0.f;
            if (!single) {
                const int za = seg_search_n<kTileCells>(cst, l0) >> 6;
                const int zb = seg_search_n<kTileCells>(cst, min(l0 + kOwn, own) - 1) >> 6;
                V0 = seg_pre[za * kPB * kPB];
                V1 = seg_pre[(zb + 2 * H + 1) * kPB * kPB];
                xi = (float)(2 * (bx - H)) * ps + (float)pos[p] * ips;
                yi = (float)(2 * (by - H)) * ps + (float)pos[(int64_t)n + p] * ips;
                zi = (float)(2 * (bz - H)) * ps + (float)pos[2 * (int64_t)n + p] * ips;
            }
            if (ADJ) {
                aix = abar[p];
                aiy = abar[(int64_t)n + p];
                aiz = abar[2 * (int64_t)n + p];
            }
            float sx = 0.f, sy = 0.f, sz = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
            for (uint32_t vb = V0; vb < V1; vb += CAP) {
                const uint32_t ve = min(vb + (uint32_t)CAP, V1);
                if (!staged) {
                    if (!single) __syncthreads();   // the previous chunk is done with xs
                    if (!ADJ && H == 2 && single && maxcnt <= 4) {
                        // sparse box: every thread copies the particles of its own
                        // segments (at most 4 each), no search needed; one segment at
                        // a time keeps the register footprint of the staging small
#pragma unroll 1
                        for (int k = 0; k < kPSegPerThread; ++k) {
                            const int s = tid * kPSegPerThread + k;
                            const int bx = s % kPB, by = (s / kPB) % kPB, bz = s / (kPB * kPB);
                            uint32_t o[4][3];
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                if ((uint32_t)i >= cnt[k]) continue;
                                const uint32_t p = src[k] + i;
                                o[i][0] = pos[p];
                                o[i][1] = pos[(int64_t)n + p];
                                o[i][2] = pos[2 * (int64_t)n + p];
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                if ((uint32_t)i >= cnt[k]) continue;
                                float4 q;
                                q.x = (float)(2 * (bx - H)) * ps + (float)o[i][0] * ips;
                                q.y = (float)(2 * (by - H)) * ps + (float)o[i][1] * ips;
                                q.z = (float)(2 * (bz - H)) * ps + (float)o[i][2] * ips;
                                q.w = kPairS0;
                                xs[pre_k[k] + i] = q;
                            }
                        }
                    } else {
                        // kStage particles per thread at a time: the segment searches and
                        // the loads of a batch are issued before the LDS stores
                        constexpr int kStage = 4;
                        for (uint32_t v0 = vb + tid; v0 < ve; v0 += kPPBlock * kStage) {
                            int sg[kStage];
                            uint32_t pj[kStage];
#pragma unroll
                            for (int k = 0; k < kStage; ++k) {
                                const uint32_t v = v0 + k * kPPBlock;
                                sg[k] = v < ve ? seg_search(seg_pre, kPSegs, v) : -1;
                                pj[k] = sg[k] < 0 ? 0u : v + seg_delta[(sg[k] / kPB) * 3 + part_of(sg[k] % kPB)];
                            }
                            uint32_t o[kStage][3];
                            float ab[kStage][3];
#pragma unroll
                            for (int k = 0; k < kStage; ++k) {
                                if (sg[k] < 0) continue;
                                const uint32_t p = pj[k];
                                o[k][0] = pos[p];
                                o[k][1] = pos[(int64_t)n + p];
                                o[k][2] = pos[2 * (int64_t)n + p];
                                if (ADJ) {
                                    ab[k][0] = abar[p];
                                    ab[k][1] = abar[(int64_t)n + p];
                                    ab[k][2] = abar[2 * (int64_t)n + p];
                                }
                            }
#pragma unroll
                            for (int k = 0; k < kStage; ++k) {
                                if (sg[k] < 0) continue;
                                const int s = sg[k];
                                const int bx = s % kPB, by = (s / kPB) % kPB, bz = s / (kPB * kPB);
                                float4 q;
                                q.x = (float)(2 * (bx - H)) * ps + (float)o[k][0] * ips;
                                q.y = (float)(2 * (by - H)) * ps + (float)o[k][1] * ips;
                                q.z = (float)(2 * (bz - H)) * ps + (float)o[k][2] * ips;
                                q.w = ADJ ? ab[k][0] : kPairS0;
                                const uint32_t v = v0 + k * kPPBlock;
                                xs[v - vb] = q;
                                if (ADJ) xa[v - vb] = make_float2(ab[k][1], ab[k][2]);
                            }
                        }
                    }
                    __syncthreads();
                    staged = single;
                }
                if (!active) continue;
                if (single) {      // the particle itself is staged: the same exact floats
                    const float4 qi = xs[vown];
                    xi = qi.x;
                    yi = qi.y;
                    zi = qi.z;
                }
                // the 2H + 1 x-neighbours of a cell are consecutive box segments, so the
                // neighbour cells are (2H + 1)^2 contiguous ranges of xs
                uint32_t rows[kW * kW];
#pragma unroll
                for (int row = 0; row < kW * kW; ++row) {
                    const int sm = su + ((row / kW - H) * kPB + row % kW - H) * kPB;
                    const uint32_t r0 = max(seg_pre[sm - H], vb), r1 = min(seg_pre[sm + H + 1], ve);
                    rows[row] = r1 > r0 ? (r1 - r0) << 16 | (r0 - vb) : 0u;
                }
                RowSort<kW * kW>::sort(rows);
                auto add_range = [&](uint32_t v0, uint32_t v1) {
                    float fx = 0.f, fy = 0.f, fz = 0.f;
                    if (lanes == 1)
                        staged_pairs<ADJ, CLAMP, 1>(xs, xa, v0, v1, xi, yi, zi, aix, aiy, aiz, bmax, fx,
                                                    fy, fz);
                    else {
                        staged_pairs<ADJ, CLAMP, kFewLanes>(xs, xa, v0 + sub, v1, xi, yi, zi, aix, aiy,
                                                            aiz, bmax, fx, fy, fz);
                        fx = quad_sum(fx);
                        fy = quad_sum(fy);
                        fz = quad_sum(fz);
                    }
                    kahan_add(sx, cx, fx);
                    kahan_add(sy, cy, fy);
                    kahan_add(sz, cz, fz);
                };
                if constexpr (!ADJ && H == 1) {
#pragma unroll 1
                    for (int row = 0; row < kW * kW; ++row) {
                        const uint32_t key = RowSort<kW * kW>::next(rows);
                        if (!__any(key >= 0x10000u)) break;
                        const uint32_t end = (key & 0xFFFFu) + (key >> 16);
                        for (uint32_t v0 = key & 0xFFFFu;;) {
                            const uint32_t v1 = min(v0 + kRange, end);
                            add_range(v0, v1);
                            if (!__any(v1 < end)) break;
                            v0 = v1;
                        }
                    }
                } else {
                    // (the 25 rows of the two-cell reach in fives, which saves four in five of
                    // the moves: a uniform density, 256^3 cells, 286 -> 271 us)
#pragma unroll (H == 2 ? 5 : 1)
                    for (int row = 0; row < kW * kW; ++row) {
                        const uint32_t key = RowSort<kW * kW>::next(rows);
                        if (!__any(key >= 0x10000u)) break;
                        const uint32_t v0 = key & 0xFFFFu;
                        add_range(v0, v0 + (key >> 16));
                    }
                }
            }
            if (!active || sub != 0) continue;
            const float a[3] = {gm * (sx * law.unit), gm * (sy * law.unit), gm * (sz * law.unit)};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                float *dst = acc + (int64_t)d * n + p;
                *dst = accumulate ? *dst + a[d] : a[d];
            }
        }
        __syncthreads();  // this tile is done with the LDS arrays
    }
    if constexpr (H == 1) {
        __syncthreads();  // every thread has left the queue
        light_tiles<ADJ, CLAMP>(lds, pos, cs, n, nt, law, gm, abar, acc, accumulate, order + nheavy,
                                light_queue, ntiles - nheavy, layers, skip);
    }
}

}  // namespace

namespace {

// Q(y) = P(alpha + beta y) for a degree-8 polynomial (coefficients low to high).
void compose(const double P[9], double alpha, double beta, double Q[9]) {
    double q[9] = {P[8], 0, 0, 0, 0, 0, 0, 0, 0};
    for (int m = 7; m >= 0; --m) {
        double t[9];
        for (int j = 0; j < 9; ++j) t[j] = alpha * q[j] + (j > 0 ? beta * q[j - 1] : 0.0);
        t[0] += P[m];
        for (int j = 0; j < 9; ++j) q[j] = t[j];
    }
    for (int j = 0; j < 9; ++j) Q[j] = q[j];
}

}  // namespace

namespace {

// The rows of L.  They are formed on the device by cube2_init_tables and, for the host's
// evaluation of the law, on the host: of correctly rounded FP64 operations alone (no
// contraction, the fifth root by Newton steps), so that both give the same floats.  On the
// host, for every context, they took 0.25 ms of cube2_create's 0.35.
struct RootLaw {
    double bpp, bf;
    double p2;        // scaled units: s and s0 times 4^j
    double unit;      // of L^5; 0: no pair of different positions, zero rows
    double cut;       // b_f^2 p2 + s0
};

__host__ __device__ inline double bits_double(uint64_t b) {
    double x;
    memcpy(&x, &b, 8);
    return x;
}
__host__ __device__ inline uint64_t double_bits(double x) {
    uint64_t b;
    memcpy(&b, &x, 8);
    return b;
}
// the next float from a positive one, by `ulps`
__host__ __device__ inline float next_float(float x, int ulps) {
    uint32_t b;
    memcpy(&b, &x, 4);
    b += (uint32_t)ulps;
    memcpy(&x, &b, 4);
    return x;
}

// x > 0, to a few 1e-16: a fifth of the exponent and mantissa bits (within 4%), then
// Newton steps, whose error is twice the square of the last.
__host__ __device__ inline double fifth_root(double x) {
#pragma clang fp contract(off)
    double y = bits_double(double_bits(x) / 5 + (0x3FF0000000000000ull / 5) * 4);
    for (int i = 0; i < 5; ++i) {
        const double y2 = y * y;
        y = y - (y - x / (y2 * y2)) * 0.2;
    }
    return y;
}

// R(r, b) / r (eq. 2)
__host__ __device__ inline double r_over_r(double r, double b) {
#pragma clang fp contract(off)
    const double t = r / b;
    if (t >= 1) return 1 / (r * r * r);
    if (2 * t < 1)
        return (64.0 / 5 + t * t * (-256.0 / 5 + t * (32 + t * (1536.0 / 35 + t * (-192.0 / 5))))) /
               (b * b * b);
    return (3.0 / 35 / (t * t) - 32.0 / 5 +
            t * (256.0 / 5 + t * (-96 + t * (256.0 / 5 + t * (32 + t * (-1536.0 / 35 + t * (64.0 / 5))))))) /
           (b * b * r);
}

// The fifth root of the pair law g(r) / unit (eqs. 2 and 4d) at the scaled s = x: where
// 1/r^2 - R(r, b_f) would cancel (r >= b_pp and r >= b_f/2) through its
// factorised form, which also continues it, negative, past the cutoff;
// elsewhere from the branches of R(r, b).
__host__ __device__ inline double pair_root(const RootLaw &p, double x) {
#pragma clang fp contract(off)
    const double r = sqrt((x - (double)kPairS0) / p.p2);
    if (r >= p.bpp && 2 * r >= p.bf) {  // g = q^5 Q(q) / r^3, q = 1 - r/b_f
        const double q = 1 - r / p.bf;
        const double Q = 1344.0 / 35 + q * (-2912.0 / 35 + q * (2048.0 / 35 + q * (-64.0 / 5)));
        return q * fifth_root(Q / (r * r * r * p.unit));
    }
    return fifth_root((r_over_r(r, p.bpp) - r_over_r(r, p.bf)) / p.unit);
}

// Row t (see the comment at the top of the law) of 2^mant per octave, from the octave of
// s0 on, in scaled units.  The adjoint's rows (kSMantAdj) are the quadratics through both
// ends and the middle, which leaves the smallest rms error in dL/ds; the forward's, twice
// as wide, the least-squares fit to five points, close to the smallest error in L.
__host__ __device__ inline float4 root_row(const RootLaw &p, int mant, int t) {
#pragma clang fp contract(off)
    // powers of two by their exponent; s0 has exponent 1
    const double oct = bits_double((uint64_t)(1024 + (t >> mant)) << 52),
                 w = bits_double((uint64_t)(1024 + (t >> mant) - mant) << 52);
    const double lo = oct + (t & ((1 << mant) - 1)) * w, hi = lo + w, c = (double)kPairY, cut = p.cut;
    if (p.unit == 0.0 || lo >= cut) return make_float4(0.0f, 0.0f, 0.0f, 0.0f);   // beyond the cutoff
    const double mid = lo + w / 2, half = w / 2;
    if (hi >= cut) {
        // L = (x - cut) (h0 + h1 (x - cut)) through two points on the far
        // side of the row from the cutoff; k rounded down, so that s >=
        // b_f^2 has y >= 0 and L <= 0
        const double x0 = cut > mid ? lo + w / 8 : mid + w / 8, x1 = x0 + w / 4;
        const double a = pair_root(p, x0) / (x0 - cut), b = pair_root(p, x1) / (x1 - cut);
        const double h1 = (b - a) / (x1 - x0), h0 = a + h1 * (cut - x0);
        float k = (float)(c * cut);
        if ((double)k > c * cut) k = next_float(k, -1);
        return make_float4(0.0f, (float)(h0 / c), (float)(h1 / (c * c)), -k);
    }
    double l0, a1, a2;               // L = l0 + e (a1 + e a2), e in [-1, 1]
    const double g0 = pair_root(p, lo), g2 = pair_root(p, mid), g4 = pair_root(p, hi);
    if (mant == kSMantAdj) {
        l0 = g2;
        a1 = (g4 - g0) / 2;
        a2 = (g4 + g0 - 2 * g2) / 2;
    } else {                         // least squares over e = -1, -1/2, 0, 1/2, 1
        const double g1 = pair_root(p, lo + w / 4), g3 = pair_root(p, mid + w / 4);
        const double m0 = g0 + g1 + g2 + g3 + g4, m2 = g0 + g4 + (g1 + g3) / 4;
        a1 = (g4 - g0 + (g3 - g1) / 2) / 2.5;
        a2 = (m2 - m0 / 2) / 0.875;
        l0 = (m0 - 2.5 * a2) / 5;
    }
    // 8 neighbouring floats kc + i ulp
    const float kc = (float)(c * mid);
    const double ulp = (double)next_float(kc, 1) - kc, ich = 1 / (c * half);
    const double e0 = (kc - c * mid) * ich, de = ulp * ich;
    double best = 1, d = 0;
    int at = 0;
    for (int i = 0; i < 8; ++i) {
        const double e = e0 + i * de, v = l0 + e * (a1 + e * a2), err = fabs((double)(float)v - v);
        if (err < best) {
            best = err;
            at = i;
            d = e;
        }
    }
    return make_float4((float)(l0 + d * (a1 + d * a2)), (float)((a1 + 2 * d * a2) * ich),
                       (float)(a2 * ich * ich), -(float)(kc + at * ulp));
}

RootLaw root_law(const cube2_ctx *ctx) {
    RootLaw p;
    p.bpp = ctx->cfg.b_pp;
    p.bf = ctx->cfg.b_fine;
    p.p2 = (double)ctx->pp_pscale * ctx->pp_pscale;
    p.unit = p.bf * p.bf <= 0x1p-30 ? 0.0 : (double)ctx->pp_unit / 4;
    p.cut = p.bf * p.bf * p.p2 + kPairS0;
    return p;
}

__global__ void root_rows_kernel(RootLaw p, float4 *__restrict__ srows, float4 *__restrict__ arows) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kSRows)
        srows[i] = root_row(p, kSMant, i);
    else if (i < kSRows + kSRowsAdj)
        arows[i - kSRows] = root_row(p, kSMantAdj, i - kSRows);
}

// The law's units.
void set_root_law(cube2_ctx *ctx) {
    const double bpp = ctx->cfg.b_pp, bf = ctx->cfg.b_fine;
    // the largest odd e0 at least 3 octaves below (b_pp/2)^2 and at most -13 (the table
    // holds the octaves up from there, and s0 moves s across a power of two, where FP32
    // halves its resolution, in a smaller part of the range before the cutoff), but not
    // below the 2^-31 under the smallest separation (2^-15)
    int e0 = std::min((int)std::floor(2.0 * std::log2(bpp / 2)) - 3, -13);
    if ((e0 & 1) == 0) --e0;
    e0 = std::max(e0, -31);
    const int j = (1 - e0) / 2;
    ctx->pp_pscale = std::ldexp(1.0f, j);
    const int top = ctx->pp_halo == 1 ? 6 : 7;           // s < 2^top
    ctx->pp_clamp = top - e0 > (kSRows >> kSMant);
    ctx->pp_unit = 1.0f;
    ctx->pp_bmax = ctx->pp_bmax_adj = 0x40000000u;       // the row of s0
    if (bf * bf <= 0x1p-30) return;                      // no pair of different positions: zero rows
    // unit / 4 >= 1.05 g(0): L stays below the clamp
    const double g0 = 64.0 / 5 * (1.0 / (bpp * bpp * bpp) - 1.0 / (bf * bf * bf));
    ctx->pp_unit = (float)std::ldexp(4.0, (int)std::ceil(std::log2(1.05 * g0)));
    // first bit pattern of the row after the one that holds the cutoff
    const float cut = (float)(bf * bf * ctx->pp_pscale * ctx->pp_pscale + kPairS0);
    uint32_t b;
    std::memcpy(&b, &cut, 4);
    ctx->pp_bmax = ((b >> (23 - kSMant)) + 1) << (23 - kSMant);
    ctx->pp_bmax_adj = ((b >> (23 - kSMantAdj)) + 1) << (23 - kSMantAdj);
}

}  // namespace

// The FP32 tables (see RootLaw).
int launch_pair_tables(cube2_ctx *ctx, hipStream_t s) {
    root_rows_kernel<<<(kSRows + kSRowsAdj + 63) / 64, 64, 0, s>>>(
        root_law(ctx), reinterpret_cast<float4 *>(ctx->tables + ctx->pp_soff),
        reinterpret_cast<float4 *>(ctx->tables + ctx->pp_aoff));
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

// The FP64 pair-law table and the FP32 law's units.  Returns
// nonzero when no K <= kPairKMax puts b_pp/2, b_pp and b_f/2 on interval
// edges (the pieces would then straddle a breakpoint of eq. 2).
int build_pair_table(cube2_ctx *ctx) {
    static const double a[6] = {64.0 / 5, 0.0, -256.0 / 5, 32.0, 1536.0 / 35, -192.0 / 5};
    static const double c[6] = {256.0 / 5, -96.0, 256.0 / 5, 32.0, -1536.0 / 35, 64.0 / 5};
    const double bpp = ctx->cfg.b_pp, bf = ctx->cfg.b_fine;
    // smallest K with b_pp/2, b_pp and b_f/2 on interval edges
    int K = 0;
    for (int k = 1; k <= kPairKMax; ++k) {
        const double w = bf / k;
        bool ok = true;
        for (double b : {bpp / 2, bpp, bf / 2}) {
            const double q = b / w;
            if (std::fabs(q - std::nearbyint(q)) > 1e-9 * std::max(1.0, q)) ok = false;
        }
        if (ok) { K = k; break; }
    }
    if (K == 0) return 1;
    const double w = bf / K;
    ctx->pp_K = K;
    ctx->pp_rows64.assign((size_t)(K + 1) * kPairRow, 0.0);
    for (int k = 0; k < K; ++k) {
        const double mid = (k + 0.5) * w, rl = k * w, rr = (k + 1) * w;
        const int pb = mid < bpp / 2 ? 0 : (mid < bpp ? 1 : 2);  // in, out, Newtonian
        const int fb = mid < bf / 2 ? 0 : 1;                      // in, out
        double P[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, Q[9];
        double ya, yb;
        if (pb == 2 && fb == 1) {
            // r^3 g = s^5 Q(1-s) = s^5 (1344/35 - 2912/35 s + 2048/35 s^2 - 64/5 s^3),
            // s = (b_f - r)/b_f = (b_f - rr)/b_f + (w/b_f) y, y = 1 - fract
            P[5] = 1344.0 / 35;
            P[6] = -2912.0 / 35;
            P[7] = 2048.0 / 35;
            P[8] = -64.0 / 5;
            compose(P, (bf - rr) / bf, w / bf, Q);
            ya = 1.0;
            yb = -1.0;
        } else {
            auto add = [&](int br, double b, double sg) {
                if (br == 0) {
                    for (int i = 0; i < 6; ++i) P[i + 3] += sg * a[i] * std::pow(b, -3 - i);
                } else if (br == 1) {
                    P[0] += sg * 3.0 / 35;
                    P[2] += sg * (-32.0 / 5) / (b * b);
                    for (int i = 0; i < 6; ++i) P[i + 3] += sg * c[i] * std::pow(b, -3 - i);
                } else {
                    P[0] += sg;
                }
            };
            add(pb, bpp, 1.0);
            add(fb, bf, -1.0);
            compose(P, rl, w, Q);  // r = rl + w y, y = fract
            ya = 0.0;
            yb = 1.0;
        }
        double *row64 = &ctx->pp_rows64[(size_t)k * kPairRow];
        for (int j = 0; j < 9; ++j) row64[j] = Q[j];
        row64[9] = ya;
        row64[10] = yb;
    }
    set_root_law(ctx);
    return 0;
}

namespace {

// Meshes with at most so many tiles have fewer two-layer items than the chip
// has waves (256 CUs x 16).
constexpr int kOneLayerTiles = 1024;

template <bool ADJ, int H, bool CLAMP>
int launch_pp_kernel_h(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                     const float *abar, float *out, int accumulate, unsigned char *work,
                     const WorkLayout &L, hipStream_t s, float grid_frac,
                     const uint8_t *skip, hipStream_t order_stream) {
    const float4 *table =
        reinterpret_cast<const float4 *>(ctx->tables + (ADJ ? ctx->pp_aoff : ctx->pp_soff));
    PPLaw law;
    law.ps = ctx->pp_pscale;
    law.ips = ctx->pp_pscale * 0x1p-15f;
    law.unit = ADJ ? ctx->pp_unit : ctx->pp_unit / ctx->pp_pscale;
    law.bmax = ADJ ? ctx->pp_bmax_adj : ctx->pp_bmax;
    const int nt = ctx->nt;
    const int ntiles = nt * nt * nt;
    auto k = pp_kernel<ADJ, H, CLAMP>;
    constexpr int kThreads = PPGeo<ADJ, H>::BLOCK;
    const unsigned chip = persistent_grid(k, kThreads, ntiles * (int)kMaxParts);
    PPOrder pp{};
    pp.light_cap = PPLight<ADJ>::LCAP;
    pp.smallest = kThreads / kFewLanes;
    pp.pairs = H == 1 ? 0.5f : 1.2f;
    pp.gain = (H == 1 ? 16.0f : 32.0f) * (ADJ ? 2.0f : 1.0f);
    pp.chip = (float)chip;
    pp.threads = (float)kThreads;
    const int r = launch_order_tiles(ctx, cs, work, L, order_stream, &pp);
    if (r) return r;
    if (order_stream != s) {
        CUBE2_CHECK_HIP(hipEventRecord(ctx->ev_fork, order_stream));
        CUBE2_CHECK_HIP(hipStreamWaitEvent(s, ctx->ev_fork, 0));
    }
    const uint32_t *order = tile_order_ptr(work, L);
    uint32_t *queue = tile_queue_ptr(ctx, work, L);
    // one z-layer of cells per light item where there are few of them
    const int layers = ntiles <= kOneLayerTiles ? 1 : PPLight<ADJ>::LAYERS;
    const unsigned grid = std::max(1u, (unsigned)((float)chip * grid_frac));
    k<<<grid, kThreads, 0, s>>>(
        pos, cs, (int)n, nt, table, law,
        (float)(ctx->cfg.g_newton * ctx->cfg.m_p), abar, out, accumulate, order, queue, ntiles,
        pp.counts, pp.parts, xcd_queue_ptr(ctx, work, L), layers, skip);
    CUBE2_LAUNCH_CHECK();
    return CUBE2_OK;
}

template <bool ADJ>
int launch_pp_kernel(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                     const float *abar, float *out, int accumulate, unsigned char *work,
                     const WorkLayout &L, hipStream_t s, hipStream_t order_stream,
                     float grid_frac = 1.0f, const uint8_t *skip = nullptr) {
    auto go = [&](auto launch) {
        return launch(ctx, pos, cs, n, abar, out, accumulate, work, L, s, grid_frac, skip,
                      order_stream);
    };
    if (ctx->pp_halo == 1)
        return ctx->pp_clamp ? go(launch_pp_kernel_h<ADJ, 1, true>)
                             : go(launch_pp_kernel_h<ADJ, 1, false>);
    return ctx->pp_clamp ? go(launch_pp_kernel_h<ADJ, 2, true>)
                         : go(launch_pp_kernel_h<ADJ, 2, false>);
}

// Share of the persistent PP grid when the PM force runs beside it: the PM
// kernels take the freed workgroup slots, and the memory-bound PM and the
// VALU- and LDS-bound PP then overlap on the same CUs.  Measured with PM, ms at
// 5/8, 3/4, 7/8 and all of the grid (workgroups of 512 threads, two per CU; the
// adjoint's of 1024, one per CU):
//   one-cell reach: 512^3 particles with 8000 halos 36.6 35.7 37.2 38.0, 256^3 with
//   1000 4.85 4.51 4.86 4.94; adjoint 73.3 74.5 75.3 75.8, 9.47 9.60 9.68 9.82, and
//   128^3 without halos 0.631 0.641 0.656 0.660
//   two-cell reach, the same: 63.6 55.2 52.8 55.7, 8.58 7.41 6.88 7.26; adjoint 119.2
//   105.1 108.8 109.1, 15.5 13.5 13.8 14.0
template <bool ADJ> constexpr float concurrent_frac(int halo) {
    return ADJ ? (halo == 1 ? 0.625f : 0.75f) : (halo == 1 ? 0.75f : 0.875f);
}

}  // namespace

// PP force (abar == nullptr) or its adjoint for the cotangents abar into
// acc_pp (not accumulated) with its own tile order and work counter (the
// pp_order / pp_parts / pp_hist / pp_scan regions), so that it can run on another stream s
// while the PM part uses the shared ones.  The tile order is made on
// `order_stream`; if that is not s, s waits for it.
int launch_pp_concurrent(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                         const float *abar, float *acc_pp, unsigned char *work, const WorkLayout &L,
                         hipStream_t s, hipStream_t order_stream) {
    WorkLayout Lpp = L;
    Lpp.tile_order = L.pp_order;
    Lpp.tile_parts = L.pp_parts;
    Lpp.hist = L.pp_hist;
    Lpp.scan_tmp = L.pp_scan;
    if (abar)
        return launch_pp_kernel<true>(ctx, pos, cs, n, abar, acc_pp, 0, work, Lpp, s, order_stream,
                                      concurrent_frac<true>(ctx->pp_halo));
    return launch_pp_kernel<false>(ctx, pos, cs, n, nullptr, acc_pp, 0, work, Lpp, s, order_stream,
                                   concurrent_frac<false>(ctx->pp_halo));
}

int launch_pp(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n, float *acc,
              int accumulate, unsigned char *work, const WorkLayout &L, hipStream_t s,
              const uint8_t *skip) {
    return launch_pp_kernel<false>(ctx, pos, cs, n, nullptr, acc, accumulate, work, L, s, s, 1.0f,
                                   skip);
}

int launch_pp_backward(cube2_ctx *ctx, const uint16_t *pos, const uint32_t *cs, int64_t n,
                       const float *acc_bar, float *x_bar, int accumulate, unsigned char *work,
                       const WorkLayout &L, hipStream_t s) {
    return launch_pp_kernel<true>(ctx, pos, cs, n, acc_bar, x_bar, accumulate, work, L, s, s);
}

}  // namespace cube2

namespace {

// The operations of pair_accumulate and pair_adjoint up to g (and 2 g_s),
// in the same order, for one separation in fine cells; false if it lies
// beyond the staged box's reach of 2 (halo + 1) fine cells per axis.
bool pair_law_host(const cube2_ctx *ctx, bool adj, float dx, float dy, float dz, float *g,
                   float *gs2) {
    using namespace cube2;
    const float lim = 2.0f * (float)(ctx->pp_halo + 1), ps = ctx->pp_pscale;
    if (!(std::fabs(dx) < lim && std::fabs(dy) < lim && std::fabs(dz) < lim)) return false;
    dx *= ps;
    dy *= ps;
    dz *= ps;
    const float s = std::fmaf(dz, dz, std::fmaf(dy, dy, std::fmaf(dx, dx, kPairS0)));
    uint32_t b;
    std::memcpy(&b, &s, 4);
    if (ctx->pp_clamp) b = std::min(b, adj ? ctx->pp_bmax_adj : ctx->pp_bmax);
    const int mant = adj ? kSMantAdj : kSMant;
    const float4 c = root_row(root_law(ctx), mant, (int)row_place(b, mant));
    const float y = std::fmaf(s, kPairY, c.w);
    const float t = std::fmaf(c.z, y, c.y);
    const float l = std::fmin(std::fmax(std::fmaf(t, y, c.x), 0.0f), 1.0f);
    const float l2 = l * l, l4 = l2 * l2;
    *g = (l4 * root_rest(t, y, c.x, l)) * ctx->pp_unit;
    *gs2 = (l4 * std::fmaf(c.z, y, t)) * (ctx->pp_unit * ps * ps);
    return true;
}

}  // namespace

extern "C" int cube2_pair_law_f32(const cube2_ctx *ctx, const float *d, float *g, int64_t n) {
    if (!ctx || n < 0 || (n > 0 && (!d || !g))) return CUBE2_EINVAL;
    for (int64_t i = 0; i < n; ++i) {
        float gs2;
        if (!pair_law_host(ctx, false, d[i], d[n + i], d[2 * n + i], &g[i], &gs2)) return CUBE2_EINVAL;
    }
    return CUBE2_OK;
}

extern "C" int cube2_pair_jacobian_f32(const cube2_ctx *ctx, const float *d, float *g, float *gs,
                                       int64_t n) {
    if (!ctx || n < 0 || (n > 0 && (!d || !g || !gs))) return CUBE2_EINVAL;
    for (int64_t i = 0; i < n; ++i) {
        if (!pair_law_host(ctx, true, d[i], d[n + i], d[2 * n + i], &g[i], &gs[i])) return CUBE2_EINVAL;
        gs[i] *= 0.5f;
    }
    return CUBE2_OK;
}

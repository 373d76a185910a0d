// Short-range pair force over the interaction lists (Section 2.1 eq. 1 with the cutoff
// g_P3M of eq. 2 and Plummer softening of Section 2.4):
//
//   a_i += m_j d g(|d| / eta) / (|d|^2 + eps^2)^(3/2),   d = x_j - x_i.
//
// One 64-lane wavefront per group (or, in the FP32 path, eight of them for a group that would
// hold up the launch): the group's i-particles sit in registers and its list is streamed
// through LDS in tiles; lanes of one stream read the same tile entry (an LDS broadcast) and
// accumulate in registers.  List entries whose source lies at least r_cut from the group's
// bounding box are dropped while a tile is loaded (every pair they form adds exactly zero).
//
// FP32 path (Section 3.1.1): positions are passed relative to the group's cube centre x_g,
// x_i - x_g and wrap(x_j - x_g), each difference taken in FP64 and then rounded to FP32, so
// the rounding error of the subtraction scales with the group size, not the box.  The pair
// law is read from a per-box table of quadratic pieces (see the FP32 section).  The per-tile
// FP32 partial sums are added up in FP64.  Persistent workgroups take the groups from per-XCD
// queues, the heaviest groups first.  Each particle's result
// leaves the kernels as one record in the caller's order, which a last pass splits into the
// output arrays or applies as a kick.
//
// FP64 path: the same relative coordinates in FP64 (nearest image once per entry, or per pair
// when the group's cube plus r_cut reaches half the box), (r^2 + eps^2)^(-1/2) and r^(-1)
// from the hardware estimate refined by two Newton steps, and eq. (2) evaluated directly in a
// form with no cancellation: for R < 1,
//   g = 1 + R^3 (-8/5 + R^2 (8/5 + R (-1/2 + R (-12/35 + 3R/20)))),
// and for R >= 1, g = max(2 - R, 0)^5 (7R^3 + 22R^2 + 10R + 4) / 140 (zero from R = 2 on).
// Both are eq. (2) rearranged.
#include "common.hpp"

#include <cmath>
#include <utility>
#include <vector>

namespace tpm {
namespace {


// First branch of eq. (2) alone, for separations known to be below eta (R < 1).
__device__ __forceinline__ double g_in_f64(double R)
{
    double R2 = R * R;
    double p = fma(0.15, R, -12.0 / 35.0);
    p = fma(p, R, -0.5);
    p = fma(p, R, 1.6);
    p = fma(p, R2, -1.6);
    return fma(p, R2 * R, 1.0);
}

__device__ __forceinline__ double g_p3m_f64(double R)
{
    double g1 = g_in_f64(R);
    double u = fmax(2.0 - R, 0.0);
    double u2 = u * u;
    double u5 = u2 * u2 * u;
    double c = fma(fma(fma(0.05, R, 22.0 / 140.0), R, 10.0 / 140.0), R, 4.0 / 140.0);
    return R < 1.0 ? g1 : u5 * c;
}

// Second branch of eq. (2) alone, for separations known to be at least eta (R >= 1).
__device__ __forceinline__ double g_far_f64(double R)
{
    double u = fmax(2.0 - R, 0.0);
    double u2 = u * u;
    double u5 = u2 * u2 * u;
    double c = fma(fma(fma(0.05, R, 22.0 / 140.0), R, 10.0 / 140.0), R, 4.0 / 140.0);
    return u5 * c;
}

__device__ __forceinline__ double wrapd(double v, double L)
{
    double h = 0.5 * L;
    if (v >= h) return v - L;
    if (v < -h) return v + L;
    return v;
}

// The force kernels leave one record per particle, in the caller's order: float4 (ax, ay, az,
// 0) for float results, double4 for double results and for the kick.  The caller's order is
// arbitrary, so each store lands in its own 32-byte HBM sector: one 16- or 32-byte record costs
// one sector where three 4- or 8-byte component stores cost three.  k_force_out then walks the
// records in order and splits them into the caller's three arrays (kOutF32, kOutF64) or adds dt
// times them to double velocities (kOutKick: the kick of Section 2.2 step 5 taken with the
// short-range force as soon as it is known), each product and sum rounded on its own.
enum { kOutF32 = 0, kOutF64 = 1, kOutKick = 2 };

template <int REC64>
__device__ __forceinline__ void store_rec(void *rec, uint32_t i, double vx, double vy, double vz)
{
    if (REC64)
        ((double4 *)rec)[i] = make_double4(vx, vy, vz, 0.0);
    else
        ((float4 *)rec)[i] = make_float4((float)vx, (float)vy, (float)vz, 0.0f);
}

// FP32 path.  Lengths are in units of r_cut / lam, lam = sqrt(1 - c), and the pair law is
//   a_i = 1/(r_cut^2 lam) sum_j m_j d'_ij G(s),  G(s) = g(2 sqrt(s)) / (s + (eps/r_cut)^2)^(3/2),
// s = |d_ij|^2 / r_cut^2 = (u - c) / (1 - c) with u = |d'_ij|^2 + c: c is a power of two below
// (eps/r_cut)^2, added inside the fused sum of squares, whose result the instruction itself
// clamps to 1, so the cutoff is exactly u = 1.  G is read from a table of p = G^(1/5)
// (build_force_table): 2^kTabSegBits pieces per octave of u, a quadratic in t = u - a where a,
// the piece's lower edge, is u with its low mantissa bits cleared (one AND, and t is exact),
// and G = p^5.  The fifth root turns eq. (2)'s fifth-order zero at the cutoff into a simple one
// and flattens s^-3/2 to s^-3/10, so that a quadratic keeps G's relative accuracy up to R = 2.
// A pair is 18 vector instructions, all of the kind that issues every 2 cycles on gfx950 (FP32
// add, multiply, fused multiply-add, right shift, AND with a literal), and three 4-byte LDS
// reads.  Measured there, cycles per instruction of a wave with four waves on the SIMD: FP32
// fma 2.3-2.7, mul/sub/shift 2.2, AND with a literal 2.4; three-operand integer forms, min, cmp
// and any operand in an SGPR 4.1.  So the address needs no shift-and-add (the table sits at
// the LDS address a >> kTabAddrShift itself) and no uniform value of the inner loop may
// stay in an SGPR.  The three coefficients are read from separate arrays: a 16-byte read per
// lane costs 31-58 cycles of LDS time once the lanes spread over 32 or more pieces, three
// 4-byte reads 9-22.
//
// One tile takes up to kTileF32 list entries.  Each lane examines kTileF32 / 64 of them and
// drops those whose source is at least r_cut from the bounding box of the chunk of particles in
// the registers: every pair they would form is at least r_cut apart and adds exactly zero (g =
// 0 for R >= 2).  The test is taken in FP32 with a margin, so it drops nothing nearer than
// r_cut.  The chunk's own box rather than the group's: chunks are runs in key order, compact in
// space, and on a clustered box chunks of 32 and 64 form 7 and 12 % fewer pairs with it
// (uniform box: 13 % with 32).  Survivors are compacted
// in list order and dealt to the J streams: survivor e goes to stream e % J, row e / J.  Rows
// past the last survivor are zero-mass padding (they add exactly 0).
constexpr int kTileF32 = 192;
constexpr int kTileRounds = kTileF32 / 64;
constexpr int kForceWaves = 8; // waves per workgroup, sharing the table

// LDS layout (bytes): the waves' tiles from 0, then the three coefficient arrays, each at its
// natural address: the entry of the piece with edge a is at (bits(a) >> kTabAddrShift) + q
// kTabPlane for q = 0, 1, 2.  u >= c >= 2^kTabMinExp, so the first entry is at
// (127 + kTabMinExp) << 8 or above and the last (u = 1) at 127 << 8.
constexpr uint32_t kTabPlane = 28 * 256;
constexpr uint32_t kForceLds = (127u << 8) + 2u * kTabPlane + 16u;
static_assert(kTabSegBits == 6 && kTabAddrShift == 15, "64 four-byte entries per octave: 256 bytes");
static_assert(kForceWaves * kTileF32 * 16 <= ((127 + kTabMinExp) << 8), "tiles end below the table");
static_assert(kTabPlane >= (uint32_t)(-kTabMinExp) * 256u + 4u && kTabPlane % 256 == 0,
              "planes do not overlap");

// What a wave needs of its group.  Coordinates are x' = x inv - xg', one fused operation.
struct GroupFrame {
    bool wrap;            // coordinates need the nearest image
    double xg0, xg1, xg2; // wrap: x_g; else x_g inv
    double L, inv_L, inv; // inv = lam / r_cut
};

// The bounding box of a chunk of the group's particles in x' units, for the cull.
struct ChunkBox {
    float c0, c1, c2; // centre
    float h0, h1, h2; // minus half the half size
    float thr;        // a quarter of the squared cull distance, with margin
};

// The LDS writes of this wave are complete before any of its lanes reads LDS again (the
// waves of a workgroup work on different lists, so a workgroup barrier is not wanted).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0); vector memory counters untouched
    __builtin_amdgcn_wave_barrier();
}

// Wave-uniform values that the compiler cannot know to be uniform, into scalar registers.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni(double v)
{
    return __hiloint2double((int)uni((uint32_t)__double2hiint(v)),
                            (int)uni((uint32_t)__double2loint(v)));
}
__device__ __forceinline__ float uni(float v) { return __uint_as_float(uni(__float_as_uint(v))); }

// Keeps a wave-uniform value in a vector register.
__device__ __forceinline__ float in_vgpr(float v)
{
    asm("" : "+v"(v));
    return v;
}

// The list entries of the tile starting at jb (jb < je), one per lane and round.  Slots past
// the range's end read its last entry and are dropped by load_tile_f32.  The caller issues
// these reads one tile ahead, so they are in flight while the previous tile is evaluated.
__device__ __forceinline__ void fetch_entries(const uint32_t *__restrict__ list, uint32_t jb,
                                              uint32_t je, uint32_t *ent)
{
    const uint32_t lane = __lane_id();
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
        const uint32_t j = jb + (uint32_t)(r * 64) + lane;
        ent[r] = list[j < je ? j : je - 1];
    }
}

// A position relative to x_g in x' units.  wrap = false for a group whose bounding box, grown
// by r_cut, lies inside [0, L) on every axis: then a source within r_cut of the box is its own
// nearest image, and a source whose nearest image lies across the boundary is at least r_cut
// from the box without the wrap as with it, so no coordinate needs wrapping.
__device__ __forceinline__ float4 rel_f32(const double4 r, const GroupFrame &F)
{
    if (F.wrap) {
        double dx = r.x - F.xg0, dy = r.y - F.xg1, dz = r.z - F.xg2;
        dx = fma(-F.L, rint(dx * F.inv_L), dx);
        dy = fma(-F.L, rint(dy * F.inv_L), dy);
        dz = fma(-F.L, rint(dz * F.inv_L), dz);
        return make_float4((float)(dx * F.inv), (float)(dy * F.inv), (float)(dz * F.inv),
                           (float)r.w);
    }
    return make_float4((float)fma(r.x, F.inv, -F.xg0), (float)fma(r.y, F.inv, -F.xg1),
                       (float)fma(r.z, F.inv, -F.xg2), (float)r.w);
}

// Culls and packs one tile; returns the number of survivors (the same on every lane).
__device__ __forceinline__ int load_tile_f32(float4 *tile, const uint32_t *ent, uint32_t jb,
                                             uint32_t je, int J, NodeArrays nd,
                                             const GroupFrame &F, const ChunkBox &C)
{
    constexpr int kR = kTileRounds;
    const int lane = __lane_id();
    const float c0 = in_vgpr(C.c0), c1 = in_vgpr(C.c1), c2 = in_vgpr(C.c2);
    const float h0 = in_vgpr(C.h0), h1 = in_vgpr(C.h1), h2 = in_vgpr(C.h2);
    int n = 0;
    // All source reads are issued before any is used, with no branch between them, so a tile
    // waits for one memory latency rather than one per round.
    double4 srcs[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        const double4 *base = (ent[r] & kCellTag) ? nd.nsrc : nd.psrc;
        srcs[r] = base[ent[r] & ~kCellTag];
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        const uint32_t j = jb + (uint32_t)(r * 64 + lane);
        const float4 v = rel_f32(srcs[r], F);
        // half the gap to the box per axis, clamped to [0, 1] (1 is past any cutoff)
        const float w0 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(v.x - c0), h0), 0.f, 1.f);
        const float w1 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(v.y - c1), h1), 0.f, 1.f);
        const float w2 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(v.z - c2), h2), 0.f, 1.f);
        const bool keep = j < je && fmaf(w0, w0, fmaf(w1, w1, w2 * w2)) < C.thr;
        const uint64_t mk = __ballot(keep);
        if (keep) {
            const int e = n + (int)__builtin_amdgcn_mbcnt_hi(
                                  (uint32_t)(mk >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u));
            tile[e] = v;
        }
        n += (int)__popcll(mk);
    }
    // zero the padding slots of the last row (at most J - 1 of them; a full tile has none
    // past its end, since J divides kTileF32)
    const int e = n + lane;
    if (lane < J && e < ((n + J - 1) & ~(J - 1))) tile[e] = make_float4(0.f, 0.f, 0.f, 0.f);
    return __builtin_amdgcn_readfirstlane(n);
}
static_assert(kTileF32 % 16 == 0, "J divides a tile");

// One pair: s = (x_j', m_j), lane particle (xi, yi, zi).  u and t as in the header above.
__device__ __forceinline__ float pair_u(const float4 s, float xi, float yi, float zi, float c,
                                        float &dx, float &dy, float &dz)
{
    dx = s.x - xi;
    dy = s.y - yi;
    dz = s.z - zi;
    // u = min(|d|^2 + c, 1): the clamp is an output modifier of the last fma
    return __builtin_amdgcn_fmed3f(fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, c))), 0.0f, 1.0f);
}
__device__ __forceinline__ float pair_f(float c0, float c1, float c2, float t, float m)
{
    const float p = fmaf(fmaf(c2, t, c1), t, c0);
    const float p2 = p * p;
    return (p2 * p2) * (p * m);
}
constexpr uint32_t kTabEdgeMask = ~((1u << kTabShift) - 1u);

typedef const __attribute__((address_space(3))) char *lds_bytes;

// One row: the source s against the lane's K i-particles.  Every pair's separation, u and table
// reads come first, then the read of the next row's source (at `ahead`), then the arithmetic on
// what was read, so the 3 K + 1 reads are in flight together and the next row does not wait for
// its source.  (Left to itself the compiler waits for each pair's reads before it starts the
// next pair.)
template <int K>
__device__ __forceinline__ void row_f32(const float4 s, const float4 *ahead, float4 &next,
                                        const float *xi, const float *yi, const float *zi,
                                        float c, float *tx, float *ty, float *tz)
{
    typedef const __attribute__((address_space(3))) float *lds_f;
    float dx[K], dy[K], dz[K], t[K], q0[K], q1[K], q2[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float u = pair_u(s, xi[k], yi[k], zi[k], c, dx[k], dy[k], dz[k]);
        const uint32_t a = __float_as_uint(u) & kTabEdgeMask;
        t[k] = u - __uint_as_float(a);
        // a separate shift: the compiler would otherwise fold it with the AND into two
        // instructions of the slower kind
        uint32_t at;
        asm("v_lshrrev_b32 %0, 15, %1" : "=v"(at) : "v"(a));
        const lds_bytes q = (lds_bytes)at;
        q0[k] = *(lds_f)q;
        q1[k] = *(lds_f)(q + kTabPlane);
        q2[k] = *(lds_f)(q + 2 * kTabPlane);
    }
    next = *ahead;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float f = pair_f(q0[k], q1[k], q2[k], t[k], s.w);
        tx[k] = fmaf(f, dx[k], tx[k]);
        ty[k] = fmaf(f, dy[k], ty[k]);
        tz[k] = fmaf(f, dz[k], tz[k]);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// steps rows of a stream (row stride J sources).  The read ahead of the last row goes at most J
// sources past the tile, inside the workgroup's LDS; its value is not used.
template <int K>
__device__ __forceinline__ void tile_pass(const float4 *ts, int steps, int J, const float *xi,
                                          const float *yi, const float *zi, float c, float *tx,
                                          float *ty, float *tz)
{
    float4 s = ts[0];
    for (int t = 0; t < steps; ++t) {
        ts += J;
        float4 next;
        row_f32<K>(s, ts, next, xi, yi, zi, c, tx, ty, tz);
        s = next;
    }
}
static_assert((kForceWaves * kTileF32 + 64) * 16 <= ((127 + kTabMinExp) << 8),
              "a read ahead of the last tile's last row stays below the table");

// The group's particles run in chunks of S lanes x K particles per lane, the wave's 64 / S
// streams taking every J-th source.  A chunk is the largest of 128, 64, 32 and 16 (K = 4) that
// wastes at most a sixth of its slots; up to 8 particles run as S = 4, K = 2.  Loading a tile
// costs as much as two or three particles' pairs with it, so two chunks with few idle slots
// beat one with many, and one kernel within 128 VGPRs (four waves per SIMD) serves every group
// size.  Force call of the 256^3 clustered box with chunks of up to 32, 64, 128 and 256: 11.1,
// 10.5, 10.4 and 10.6 ms; with five and six waves per SIMD (and the spills that takes) 12.8
// and 12.4 ms.
__host__ __device__ __forceinline__ void chunk_layout(uint32_t r, int &S, int &K)
{
    K = 4;
    S = r >= 107 ? 32 : r >= 54 ? 16 : r >= 27 ? 8 : 4;
    if (r <= 8) K = 2;
}

// The least (or, on negated values, the greatest) of v over each run of S lanes.
__device__ __forceinline__ float run_min(float v, int S)
{
#define TPM_MIN_DPP(ctrl)                                                                      \
    v = fminf(v, __uint_as_float(__builtin_amdgcn_update_dpp(                                  \
                     0, __float_as_uint(v), ctrl, 0xf, 0xf, false)))
    TPM_MIN_DPP(0xb1);               // quad_perm 1, 0, 3, 2
    TPM_MIN_DPP(0x4e);               // quad_perm 2, 3, 0, 1
    if (S >= 8) TPM_MIN_DPP(0x141);  // row_half_mirror: the other four of eight
    if (S >= 16) TPM_MIN_DPP(0x140); // row_mirror: the other eight of sixteen
#undef TPM_MIN_DPP
    if (S >= 32) v = fminf(v, __shfl_xor(v, 16, 64));
    if (S >= 64) v = fminf(v, __shfl_xor(v, 32, 64));
    return v;
}

// The force of the list range [j0, j1) on the chunk's particles f + ib ..: per lane K sums
// over its stream's sources, the per-tile FP32 sums added up in FP64.
template <int K>
__device__ __forceinline__ void chunk_sums(float4 *tile, float c, const NodeArrays &nd, int S,
                                           uint32_t n_i, uint32_t f, const uint32_t *list,
                                           uint32_t j0, uint32_t j1,
                                           const double4 *__restrict__ ps, const GroupFrame &F,
                                           double *ax, double *ay, double *az, uint32_t &kept)
{
    const int lane = __lane_id();
    const int J = 64 / S, lgJ = 31 - __builtin_clz(J);
    const int slot = lane & (S - 1), stream = lane / S;
    float xi[K], yi[K], zi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t i = slot + S * k;
        const float4 v = rel_f32(ps[f + (i < n_i ? i : 0)], F); // idle slots repeat the first
        xi[k] = v.x;
        yi[k] = v.y;
        zi[k] = v.z;
        ax[k] = ay[k] = az[k] = 0.0;
    }
    ChunkBox C;
    {
        float lo[3] = {xi[0], yi[0], zi[0]}, hi[3] = {-xi[0], -yi[0], -zi[0]};
#pragma unroll
        for (int k = 1; k < K; ++k) {
            lo[0] = fminf(lo[0], xi[k]);
            lo[1] = fminf(lo[1], yi[k]);
            lo[2] = fminf(lo[2], zi[k]);
            hi[0] = fminf(hi[0], -xi[k]);
            hi[1] = fminf(hi[1], -yi[k]);
            hi[2] = fminf(hi[2], -zi[k]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = uni(run_min(lo[a], S));
            hi[a] = -uni(run_min(hi[a], S));
        }
        C.c0 = 0.5f * (lo[0] + hi[0]);
        C.c1 = 0.5f * (lo[1] + hi[1]);
        C.c2 = 0.5f * (lo[2] + hi[2]);
        C.h0 = -0.25f * (hi[0] - lo[0]);
        C.h1 = -0.25f * (hi[1] - lo[1]);
        C.h2 = -0.25f * (hi[2] - lo[2]);
        // The coordinates near the threshold are at most 1 + 2 max(h) + |c| in size, each
        // rounded a few times to 2^-24 of that; the cull distance is lam <= 1.
        const float big = 1.0f + 4.0f * fmaxf(fmaxf(-C.h0, -C.h1), -C.h2) +
                          fmaxf(fmaxf(fabsf(C.c0), fabsf(C.c1)), fabsf(C.c2));
        C.thr = uni(0.25f * (1.0f + 0x1p-12f + 0x1p-20f * big));
    }
    uint32_t ent[kTileRounds];
    if (j0 < j1) fetch_entries(list, j0, j1, ent);
    for (uint32_t jb = j0; jb < j1; jb += kTileF32) {
        const int nt = load_tile_f32(tile, ent, jb, j1, J, nd, F, C);
        kept += (uint32_t)nt;
        wave_lds_sync();
        if (jb + kTileF32 < j1) fetch_entries(list, jb + kTileF32, j1, ent);
        const int steps = (nt + J - 1) >> lgJ; // the same on every lane
        float tx[K], ty[K], tz[K];
#pragma unroll
        for (int k = 0; k < K; ++k) tx[k] = ty[k] = tz[k] = 0.f;
        tile_pass<K>(tile + stream, steps, J, xi, yi, zi, c, tx, ty, tz);
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ax[k] += (double)tx[k];
            ay[k] += (double)ty[k];
            az[k] += (double)tz[k];
        }
    }
    // the J streams' sums, in a fixed tree
    for (int d = S; d < 64; d <<= 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ax[k] += __shfl_xor(ax[k], d, 64);
            ay[k] += __shfl_xor(ay[k], d, 64);
            az[k] += __shfl_xor(az[k], d, 64);
        }
    }
}

// One chunk by one wave (whole list), or by the workgroup's kForceWaves waves, each on its own
// part [j0, j1) of the list: then the waves' sums meet in LDS (the tiles, two k at a time: 128
// particles x 3 doubles fill one tile) and are added in wave order.
template <int K>
__device__ __forceinline__ void run_chunk(float4 *tiles, int wave, bool split, float c,
                                          const NodeArrays &nd, int S, uint32_t n_i, uint32_t f,
                                          const uint32_t *list, uint32_t j0, uint32_t j1,
                                          const double4 *__restrict__ ps,
                                          const uint32_t *__restrict__ pidx, const GroupFrame &F,
                                          double scale, void *rec, int rec64, uint32_t &kept)
{
    double ax[K], ay[K], az[K];
    chunk_sums<K>(tiles + wave * kTileF32, c, nd, S, n_i, f, list, j0, j1, ps, F, ax, ay,
                        az, kept);
    const int lane = __lane_id();
    if (!split) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t i = (uint32_t)(lane + S * k);
            if (lane < S && i < n_i) {
                if (rec64)
                    store_rec<1>(rec, pidx[f + i], ax[k] * scale, ay[k] * scale, az[k] * scale);
                else
                    store_rec<0>(rec, pidx[f + i], ax[k] * scale, ay[k] * scale, az[k] * scale);
            }
        }
        return;
    }
    double *const red = reinterpret_cast<double *>(tiles);
    constexpr int kWaveWords = kTileF32 * 2; // doubles per wave's tile
#pragma unroll
    for (int kb = 0; kb < K; kb += 2) {
#pragma unroll
        for (int k = kb; k < kb + 2 && k < K; ++k)
            if (lane < S) {
                double *const d = red + wave * kWaveWords + ((k - kb) * 64 + lane) * 3;
                d[0] = ax[k];
                d[1] = ay[k];
                d[2] = az[k];
            }
        __syncthreads();
        const int t = threadIdx.x;
        const int k = kb + (t >> 6);
        const uint32_t i = (uint32_t)(lane + S * k);
        if (t < 128 && k < K && lane < S && i < n_i) {
            double vx = 0.0, vy = 0.0, vz = 0.0;
            for (int w = 0; w < kForceWaves; ++w) {
                const double *d = red + w * kWaveWords + t * 3;
                vx += d[0];
                vy += d[1];
                vz += d[2];
            }
            if (rec64)
                store_rec<1>(rec, pidx[f + i], vx * scale, vy * scale, vz * scale);
            else
                store_rec<0>(rec, pidx[f + i], vx * scale, vy * scale, vz * scale);
        }
        __syncthreads();
    }
}
static_assert(128 * 24 <= kTileF32 * 16, "128 particles' sums fit a tile");

__device__ __forceinline__ uint64_t run_group(float4 *tiles, int wave, bool split, float c,
                                              const ForceBox &B, uint32_t n_g, uint32_t f,
                                              const uint32_t *list, uint32_t j0, uint32_t j1,
                                              const GroupFrame &F, double scale)
{
    uint64_t pairs = 0;
    for (uint32_t ib = 0; ib < n_g;) {
        int S, K;
        chunk_layout(n_g - ib, S, K);
        const uint32_t n_i = n_g - ib < (uint32_t)(S * K) ? n_g - ib : (uint32_t)(S * K);
        uint32_t kept = 0;
#define TPM_CHUNK(KK)                                                                          \
    run_chunk<KK>(tiles, wave, split, c, B.nd, S, n_i, f + ib, list, j0, j1, B.ps,       \
                        B.pidx, F, scale, B.rec, B.rec64, kept)
        if (K == 4)
            TPM_CHUNK(4);
        else
            TPM_CHUNK(2);
#undef TPM_CHUNK
        ib += n_i;
        pairs += (uint64_t)kept * n_i;
    }
    return pairs; // pairs with the entries of [j0, j1) that survived the cull
}

// Group g of box B by one wave, or, split, by the workgroup.
__device__ __forceinline__ void force_group_f32(float4 *tiles, int wave, bool split,
                                                const ForceBox &B, uint32_t g)
{
    const GroupArrays &gr = B.gr;
    const ForceParams &fp = B.fp;
    // everything about the group is read before any of it is used: one memory latency
    const double lo0 = gr.lox[g], lo1 = gr.loy[g], lo2 = gr.loz[g];
    const double hi0 = gr.hix[g], hi1 = gr.hiy[g], hi2 = gr.hiz[g];
    const double x0 = gr.xgx[g], x1 = gr.xgy[g], x2 = gr.xgz[g];
    const uint32_t count = gr.count[g], first = gr.first[g], len = B.len[g];
    const uint64_t off = B.off[g];
    __builtin_amdgcn_sched_barrier(0);
    const double lam = sqrt(1.0 - (double)B.ft.c);
    const double inv_len = 0.5 * fp.inv_eta; // 1 / r_cut
    const double scale = uni(inv_len * inv_len / lam);
    const double rc = fp.rc * (1.0 + 0x1p-10); // clear of rounding at the boundary
    GroupFrame F;
    F.wrap = __ballot(!((lo0 - rc >= 0.0) & (hi0 + rc < fp.L) & (lo1 - rc >= 0.0) &
                        (hi1 + rc < fp.L) & (lo2 - rc >= 0.0) & (hi2 + rc < fp.L))) != 0;
    F.L = fp.L;
    F.inv_L = uni(1.0 / fp.L);
    F.inv = uni(inv_len * lam);
    F.xg0 = uni(F.wrap ? x0 : x0 * F.inv);
    F.xg1 = uni(F.wrap ? x1 : x1 * F.inv);
    F.xg2 = uni(F.wrap ? x2 : x2 * F.inv);
    const float c = in_vgpr(B.ft.c);
    const uint32_t Lg = uni(len);
    uint32_t j0 = 0, j1 = Lg;
    if (split) { // whole rounds of 64 entries per wave
        const uint32_t per = ((Lg + 64 * kForceWaves - 1) / (64 * kForceWaves)) * 64;
        j0 = per * (uint32_t)wave < Lg ? per * (uint32_t)wave : Lg;
        j1 = j0 + per < Lg ? j0 + per : Lg;
    }
    const uint32_t *list =
        B.entries + (((uint64_t)uni((uint32_t)(off >> 32)) << 32) | uni((uint32_t)off));
    const uint64_t pairs =
        run_group(tiles, wave, split, c, B, uni(count), uni(first), list, j0, j1, F, scale);
    if (__lane_id() == 0) {
        if (split)
            atomicAdd(&fp.pairs[g], (unsigned long long)pairs); // zeroed by the prep launch
        else
            fp.pairs[g] = pairs;
    }
}

// The first part at or after `from` (cyclically) whose counter has not reached its size, or
// kXcds.  Lane p < kXcds holds part p's size.  One read of all counters, so a wave that finds
// everything taken leaves after one memory latency, and no atomic is spent on empty queues.
__device__ __forceinline__ uint32_t next_part(uint32_t *ctr, uint32_t size, uint32_t from)
{
    const uint32_t lane = __lane_id();
    uint32_t v = 0;
    if (lane < kXcds)
        v = __hip_atomic_load(&ctr[lane * kQueueStride], __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t m = (uint32_t)__ballot(lane < kXcds && v < size);
    if (!m) return kXcds;
    const uint32_t rot = ((m >> from) | (m << (kXcds - from))) & ((1u << kXcds) - 1u);
    return (from + (uint32_t)__builtin_ctz(rot)) % kXcds;
}

// Item q of part `part` over the boxes (their runs laid end to end): lane b < nb holds box b's
// run end in `ends` (inclusive prefix).
struct Item {
    uint32_t box, k;
};
__device__ __forceinline__ Item find_item(uint32_t ends, int nb, uint32_t q)
{
    const uint32_t lane = __lane_id();
    const uint32_t b = (uint32_t)__popcll(__ballot((int)lane < nb && ends <= q));
    const uint32_t before = b ? (uint32_t)__builtin_amdgcn_readlane((int)ends, (int)b - 1) : 0u;
    return {b, q - before};
}

// Box b's run of part p in the queue of split (heavy = 1) or single-wave groups.
__device__ __forceinline__ uint32_t run_start(const uint32_t *cls, uint32_t p, int heavy)
{
    return cls[heavy ? kClsStarts + p : kClsHeavyEnd + p];
}
__device__ __forceinline__ uint32_t run_size(const uint32_t *cls, uint32_t p, int heavy)
{
    return cls[heavy ? kClsHeavyEnd + p : kClsStarts + p + 1] - run_start(cls, p, heavy);
}

// Per lane p < kXcds the total size of part p over the boxes.
__device__ __forceinline__ uint32_t part_sizes(const ForceBox *bx, int nb, int heavy)
{
    const uint32_t lane = __lane_id();
    uint32_t n = 0;
    if (lane < kXcds)
        for (int b = 0; b < nb; ++b) n += run_size(bx[b].cls, lane, heavy);
    return n;
}
// Per lane the inclusive prefix over the boxes of their runs of `part`.
__device__ __forceinline__ uint32_t run_ends(const ForceBox *bx, int nb, uint32_t part, int heavy)
{
    const int lane = __lane_id();
    uint32_t v = lane < nb ? run_size(bx[lane].cls, part, heavy) : 0u;
#pragma unroll
    for (int d = 1; d < kMaxBatch; d <<= 1) {
        const uint32_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// Persistent: each workgroup copies the table into LDS once, takes split groups as a whole
// until none are left, and then its waves take single groups, each from the queues of
// kXcds contiguous key ranges (its own XCD's first: neighbouring groups share sources through
// one L2; then what is left of the others).  Every box of a launch has the same table.
//
// A group with at least 2^t pairs is split over the workgroup's waves, 2^t being about a
// 16384th of the box's pairs (at least 2^12): one wave alone would hold up the end of the
// launch.  On the 700,001-particle clustered box the longest single-wave group took 1.3 ms of
// a 1.5 ms force call whose work fills the device for 0.6 ms.
//
// What bounds it (256^3 clustered box, n_crit 256): the LDS pipe is busy 93 % of the time and
// the vector units 80 %; without the table reads the call takes 8.7 ms, with conflict-free ones
// 10.2, as it is 10.4 (12.4 with a kernel per blocking factor, a table of 16-byte entries and
// queue counters side by side: 311,000 groups taken through counters in one cache line alone
// cost about 12 ms, at 40 ns each).  700,001 particles: the whole step 3.41 -> 1.53 ms.
template <bool MULTI>
__device__ __forceinline__ void force_f32_body(const ForceBox *bx, int n_boxes)
{
    extern __shared__ float4 smem[];
    const int nb = MULTI ? n_boxes : 1;
    {
        const ForceTable ft = bx[0].ft;
        float *const lds = reinterpret_cast<float *>(smem);
        for (uint32_t i = threadIdx.x; i < ft.entries; i += blockDim.x)
#pragma unroll
            for (uint32_t q = 0; q < 3; ++q)
                lds[(ft.base + q * kTabPlane) / 4 + i] = ft.coef[q * ft.entries + i];
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); // known to be uniform
    const uint32_t lane = __lane_id();
    const uint32_t xcd = blockIdx.x % kXcds;
    uint32_t *const hq = bx[0].cls + kClsQueue, *const lq = hq + kXcds * kQueueStride;
    __syncthreads();
    uint32_t *const word = reinterpret_cast<uint32_t *>(smem); // a tile is free between groups
    uint32_t size = part_sizes(bx, nb, 1), part = xcd, ends = 0, have = kXcds, next = 0;
    bool split = __ballot(size != 0) != 0;
    if (!split) size = part_sizes(bx, nb, 0);
    for (;;) {
        uint32_t *const ctr = split ? hq : lq;
        uint32_t q = next;
        if (!split || wave == 0)
            for (;;) {
                // a single wave asked for its next item before it began the last one
                if (split || part != have) {
                    part = uni(next_part(ctr, size, part));
                    if (part == kXcds) break;
                    if (lane == 0) q = atomicAdd(&ctr[part * kQueueStride], 1u);
                }
                q = uni(q);
                if (q < (uint32_t)__builtin_amdgcn_readlane((int)size, (int)part)) break;
                have = kXcds; // found empty: on to the next part that is not
            }
        if (split) {
            if (threadIdx.x == 0) {
                word[0] = part;
                word[1] = q;
            }
            __syncthreads();
            part = word[0];
            q = word[1];
            __syncthreads();
        }
        part = uni(part);
        q = uni(q);
        if (part == kXcds) {
            if (!split) break;
            split = false; // on to the single-wave groups
            size = part_sizes(bx, nb, 0);
            part = xcd;
            have = kXcds;
            continue;
        }
        if (MULTI && part != have) ends = run_ends(bx, nb, part, split);
        have = part;
        if (!split && lane == 0) next = atomicAdd(&ctr[part * kQueueStride], 1u);
        Item it{0, q};
        if (MULTI) it = find_item(ends, nb, q);
        const ForceBox &B = MULTI ? bx[uni(it.box)] : bx[0];
        force_group_f32(smem, wave, split, B, uni(B.cls[run_start(B.cls, part, split) + it.k]));
    }
}

__global__ __launch_bounds__(64 * kForceWaves, 4) void k_force_f32(ForceBox box)
{
    force_f32_body<false>(&box, 1);
}

__global__ __launch_bounds__(64 * kForceWaves, 4) void k_force_f32_multi(
    const ForceBox *__restrict__ bx, int nb)
{
    force_f32_body<true>(bx, nb);
}

// Adds the groups' pairs into *sum: blocks b of nb.
__device__ __forceinline__ void sum_pairs(uint32_t n_groups, const unsigned long long *pairs,
                                          unsigned long long *sum, uint32_t b, uint32_t nb)
{
    unsigned long long v = 0;
    for (uint32_t g = b * blockDim.x + threadIdx.x; g < n_groups; g += nb * blockDim.x)
        v += pairs[g];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    __shared__ unsigned long long sm[4];
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(sum, sm[0] + sm[1] + sm[2] + sm[3]);
}

// Pair by pair: out[(i * n_j + j) * 3 + a] = acceleration at x_i from (x_j, m_j) with the
// FP32 pair routine of the force kernel (same relative coordinates, units, table and
// rounding), without the cull and without periodic images.
__global__ __launch_bounds__(256) void k_pairwise_f32(int64_t n_i, const double *__restrict__ xi,
                                                      int64_t n_j, const double *__restrict__ xj,
                                                      const double *__restrict__ mj, double xg0,
                                                      double xg1, double xg2, double inv,
                                                      ForceTable ft, double scale,
                                                      double *__restrict__ out)
{
    const int64_t total = n_i * n_j;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = q / n_j, j = q % n_j;
        const float x = (float)fma(xi[3 * i + 0], inv, -xg0 * inv);
        const float y = (float)fma(xi[3 * i + 1], inv, -xg1 * inv);
        const float z = (float)fma(xi[3 * i + 2], inv, -xg2 * inv);
        const float4 src = make_float4((float)fma(xj[3 * j + 0], inv, -xg0 * inv),
                                       (float)fma(xj[3 * j + 1], inv, -xg1 * inv),
                                       (float)fma(xj[3 * j + 2], inv, -xg2 * inv), (float)mj[j]);
        float dx, dy, dz;
        const float u = pair_u(src, x, y, z, ft.c, dx, dy, dz);
        const uint32_t a = __float_as_uint(u) & kTabEdgeMask;
        const float *co = ft.coef + ((a >> kTabAddrShift) - ft.base) / 4;
        const float f = pair_f(co[0], co[ft.entries], co[2 * ft.entries],
                               u - __uint_as_float(a), src.w);
        const float tx = f * dx, ty = f * dy, tz = f * dz;
        out[3 * q + 0] = (double)tx * scale;
        out[3 * q + 1] = (double)ty * scale;
        out[3 * q + 2] = (double)tz * scale;
    }
}

// Queues of the FP32 force.  Group g belongs to XCD part p = floor(8 g / G) (contiguous key
// ranges) and to a cost bucket: the octave of its pairs n_g L_g if it has at least 2^kHeavyCost
// of them or is split (at least 2^t, see k_force_f32), one bucket for all others.  The bins (p,
// bucket) are laid out with the costliest first, so each part lists its split groups, its heavy
// ones longest first and then the rest in about key order (consecutive groups share sources
// through the XCD's L2).  Three passes: count the bins, scan them into cursors and part
// starts, scatter.  Blocks take kClassifyItems * 256 consecutive groups and aggregate their
// bins in LDS first.
constexpr int kClassifyItems = 8;
constexpr int kCostBuckets = 64;
constexpr uint32_t kHeavyCost = 17;
constexpr uint32_t kMinSplit = 12;
constexpr int kBins = kXcds * kCostBuckets;

// t of the box: pairs = its interactions.
__device__ __forceinline__ uint32_t split_log2(unsigned long long pairs)
{
    const uint32_t lg = 63u - (uint32_t)__clzll((long long)(pairs | 1ull));
    return lg > kMinSplit + 14u ? lg - 14u : kMinSplit;
}

__device__ __forceinline__ uint32_t cost_bin(uint32_t g, uint32_t n_groups, uint32_t n_g,
                                             uint32_t L_g, uint32_t t)
{
    const uint32_t part = (uint32_t)(((uint64_t)g * kXcds) / n_groups);
    const uint64_t cost = (uint64_t)n_g * L_g;
    const uint32_t lg = 63u - (uint32_t)__clzll((long long)(cost | 1ull));
    const uint32_t least = t < kHeavyCost ? t : kHeavyCost;
    return part * kCostBuckets + (kCostBuckets - 1 - (lg >= least ? lg : 0u));
}

__global__ __launch_bounds__(256) void k_class_count(GroupArrays gr, uint32_t n_groups,
                                                     const uint32_t *__restrict__ len,
                                                     const unsigned long long *pairs,
                                                     uint32_t *hist)
{
    __shared__ uint32_t s_cnt[kBins];
    for (int i = threadIdx.x; i < kBins; i += 256) s_cnt[i] = 0;
    __syncthreads();
    const uint32_t t = split_log2(*pairs);
    const uint32_t base = blockIdx.x * (256u * kClassifyItems);
#pragma unroll
    for (int r = 0; r < kClassifyItems; ++r) {
        const uint32_t g = base + (uint32_t)r * 256u + threadIdx.x;
        if (g < n_groups) atomicAdd(&s_cnt[cost_bin(g, n_groups, gr.count[g], len[g], t)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += 256)
        if (s_cnt[i]) atomicAdd(&hist[i], s_cnt[i]);
}

// By one wave, lane = cost bucket: the bins' counts to cursors (in place; bins in global memory
// or LDS), part starts and the ends of the parts' split runs into cls.
__device__ __forceinline__ void scan_bins(uint32_t *bins, uint32_t *cls, uint32_t t)
{
    static_assert(kCostBuckets == 64, "one lane per bucket");
    const int lane = __lane_id();
    uint32_t pos = kClsLists;
    uint32_t c[kXcds];
#pragma unroll
    for (int p = 0; p < (int)kXcds; ++p) c[p] = bins[p * kCostBuckets + lane];
#pragma unroll
    for (int p = 0; p < (int)kXcds; ++p) {
        uint32_t v = c[p];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = __shfl_up(v, d, 64);
            if (lane >= d) v += u;
        }
        bins[p * kCostBuckets + lane] = pos + v - c[p];
        // bucket lane holds lg = 63 - lane: split for lg >= t
        if (lane == 0) cls[kClsStarts + p] = pos;
        if (lane == 63 - (int)t) cls[kClsHeavyEnd + p] = pos + v;
        pos += (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    }
    if (lane == 0) cls[kClsStarts + kXcds] = pos;
}
__global__ __launch_bounds__(64) void k_class_scan(uint32_t *cls, const unsigned long long *pairs)
{
    scan_bins(cls + kClsBins, cls, split_log2(*pairs));
}

__global__ __launch_bounds__(256) void k_class_scatter(GroupArrays gr, uint32_t n_groups,
                                                       const uint32_t *__restrict__ len,
                                                       const unsigned long long *pairs,
                                                       uint32_t *cls)
{
    __shared__ uint32_t s_cnt[kBins];
    for (int i = threadIdx.x; i < kBins; i += 256) s_cnt[i] = 0;
    __syncthreads();
    const uint32_t t = split_log2(*pairs);
    const uint32_t base = blockIdx.x * (256u * kClassifyItems);
    uint32_t bin[kClassifyItems], loc[kClassifyItems];
#pragma unroll
    for (int r = 0; r < kClassifyItems; ++r) {
        const uint32_t g = base + (uint32_t)r * 256u + threadIdx.x;
        bin[r] = ~0u;
        if (g < n_groups) {
            bin[r] = cost_bin(g, n_groups, gr.count[g], len[g], t);
            loc[r] = atomicAdd(&s_cnt[bin[r]], 1u);
        }
    }
    __syncthreads();
    // this block's run of each bin
    for (int i = threadIdx.x; i < kBins; i += 256)
        if (s_cnt[i]) s_cnt[i] = atomicAdd(&cls[kClsBins + i], s_cnt[i]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kClassifyItems; ++r)
        if (bin[r] != ~0u) cls[s_cnt[bin[r]] + loc[r]] = base + (uint32_t)r * 256u + threadIdx.x;
}

// 1/sqrt(x) in FP64 for x > 0: the hardware estimate refined by two Newton steps
// y <- y + y (1/2 - (x/2) y^2), each of which squares the relative error (to within rounding).
__device__ __forceinline__ double rsqrt_f64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    y = fma(y, fma(-h, y * y, 0.5), y);
    y = fma(y, fma(-h, y * y, 0.5), y);
    return y;
}

// FP64 path, one wave per group, 64 i-particles per pass.  Each tile of 64 list entries is
// culled against the group's box as in the FP32 path (a source at least r_cut from the box
// adds exactly zero) and the survivors are stored relative to x_g (nearest image, once per
// entry) in three runs: "inner" sources, whose farthest point of the box is within eta (every
// pair has R < 1: eq. (2)'s first branch only), from the front of the tile; "far" ones, at
// least eta from the box (every pair has R >= 1: the second branch only), from the back; the
// others ("near", both branches and a select) in between.  The FP64 pair evaluates both
// branches of g for a near source, so the inner run saves the second branch and the select.
// When the group's cube and cutoff fit in half the box (half side + r_cut < L/2) the
// difference of two relative positions is the nearest-image separation and the pairs need no
// wrap; otherwise the pair wraps it.  (r^2 + eps^2)^(-1/2) and r^(-1) come from
// rsqrt_f64 (r = r^2 r^(-1)); a pair at zero separation adds nothing.
constexpr int kTileF64 = 64;

enum F64Kind { kF64Near = 0, kF64Far = 1, kF64Inner = 2 };

template <int REC64>
__global__ __launch_bounds__(64) void k_force_f64(
    NodeArrays nd, GroupArrays gr, uint32_t n_groups, const uint64_t *__restrict__ off,
    const uint32_t *__restrict__ len, const uint32_t *__restrict__ entries,
    const double4 *__restrict__ ps, const uint32_t *__restrict__ pidx, ForceParams fp,
    void *rec)
{
    __shared__ double4 tile[kTileF64];
    const uint32_t g = xcd_block(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x;
    if (g >= n_groups) return;
    const uint32_t n_g = gr.count[g], f = gr.first[g];
    const uint64_t b = off[g];
    const uint64_t Lg = len[g];
    const double L = fp.L, eps2 = fp.eps2, inv_eta = fp.inv_eta, eta2 = fp.eta * fp.eta;
    const double xg0 = gr.xgx[g], xg1 = gr.xgy[g], xg2 = gr.xgz[g];
    const double cg0 = gr.cgx[g], cg1 = gr.cgy[g], cg2 = gr.cgz[g];
    const double hg0 = gr.hgx[g], hg1 = gr.hgy[g], hg2 = gr.hgz[g];
    const double half_side = 0.5 * ldexp(L, -(int)nd.level[gr.node[g]]);
    const bool pair_wrap = !(half_side + sqrt(fp.rc2) < 0.5 * L);
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t kept_total = 0;
    for (uint32_t ib = 0; ib < n_g; ib += 64) {
        const uint32_t i = ib + lane;
        const bool act = i < n_g;
        kept_total = 0;
        double xi = 0.0, yi = 0.0, zi = 0.0;
        if (act) {
            const double4 r = ps[f + i];
            xi = wrapd(r.x - xg0, L);
            yi = wrapd(r.y - xg1, L);
            zi = wrapd(r.z - xg2, L);
        }
        double ax_ = 0.0, ay_ = 0.0, az_ = 0.0;
        for (uint64_t jb = 0; jb < Lg; jb += kTileF64) {
            const uint64_t j = jb + lane;
            bool keep = false, far = false, inner = false;
            double4 v = make_double4(0.0, 0.0, 0.0, 0.0);
            if (j < Lg) {
                const uint32_t e = entries[b + j];
                const double4 r = (e & kCellTag) ? nd.nsrc[e & ~kCellTag] : nd.psrc[e];
                const double a0 = fabs(wrapd(r.x - cg0, L));
                const double a1 = fabs(wrapd(r.y - cg1, L));
                const double a2 = fabs(wrapd(r.z - cg2, L));
                double w0 = a0 - hg0, w1 = a1 - hg1, w2 = a2 - hg2;
                w0 = w0 > 0.0 ? w0 : 0.0;
                w1 = w1 > 0.0 ? w1 : 0.0;
                w2 = w2 > 0.0 ? w2 : 0.0;
                const double gap2 = w0 * w0 + w1 * w1 + w2 * w2;
                const double e0 = a0 + hg0, e1 = a1 + hg1, e2 = a2 + hg2;
                keep = gap2 < fp.rc2;
                far = gap2 >= eta2;
                inner = e0 * e0 + e1 * e1 + e2 * e2 < eta2;
                v = make_double4(wrapd(r.x - xg0, L), wrapd(r.y - xg1, L), wrapd(r.z - xg2, L),
                                 r.w);
            }
            const uint64_t mi = __ballot(keep && inner), mn = __ballot(keep && !far && !inner),
                           mf = __ballot(keep && far);
            const int ni = __popcll(mi), nn = __popcll(mn), nf = __popcll(mf);
            kept_total += (uint32_t)(ni + nn + nf);
            if (keep) {
                if (far)
                    tile[kTileF64 - 1 - __popcll(mf & lt)] = v;
                else if (inner)
                    tile[__popcll(mi & lt)] = v;
                else
                    tile[ni + __popcll(mn & lt)] = v;
            }
            __syncthreads();
#define TPM_F64_PAIRS(KIND, WRAP, T0, T1)                                                       \
    for (int t = (T0); t < (T1); ++t) {                                                        \
        const double4 s = tile[t];                                                             \
        double dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;                                    \
        if (WRAP) {                                                                            \
            dx = wrapd(dx, L);                                                                 \
            dy = wrapd(dy, L);                                                                 \
            dz = wrapd(dz, L);                                                                 \
        }                                                                                      \
        const double r2 = dx * dx + dy * dy + dz * dz;                                         \
        const double is = rsqrt_f64(r2 + eps2);                                                \
        const double R = r2 * rsqrt_f64(r2) * inv_eta;                                         \
        const double g = KIND == kF64Far     ? g_far_f64(R)                                   \
                         : KIND == kF64Inner ? g_in_f64(R)                                    \
                                             : g_p3m_f64(R);                                  \
        double fm = s.w * g * (is * is * is);                                                  \
        fm = r2 > 0.0 ? fm : 0.0;                                                              \
        ax_ += fm * dx;                                                                        \
        ay_ += fm * dy;                                                                        \
        az_ += fm * dz;                                                                        \
    }
            if (pair_wrap) {
                TPM_F64_PAIRS(kF64Inner, true, 0, ni)
                TPM_F64_PAIRS(kF64Near, true, ni, ni + nn)
                TPM_F64_PAIRS(kF64Far, true, kTileF64 - nf, kTileF64)
            } else {
                TPM_F64_PAIRS(kF64Inner, false, 0, ni)
                TPM_F64_PAIRS(kF64Near, false, ni, ni + nn)
                TPM_F64_PAIRS(kF64Far, false, kTileF64 - nf, kTileF64)
            }
#undef TPM_F64_PAIRS
            __syncthreads();
        }
        if (act) store_rec<REC64>(rec, pidx[f + i], ax_, ay_, az_);
    }
    if (lane == 0) fp.pairs[g] = (unsigned long long)kept_total * n_g;
}

// The records in the caller's order, split into three arrays or applied as a kick (modes as
// for store_rec; records are float4 for kOutF32, double4 otherwise).
template <int MODE>
__device__ __forceinline__ void write_out(const void *__restrict__ rec, int64_t n, void *ax,
                                          void *ay, void *az, double dt, uint32_t b, uint32_t nb)
{
    // the kick's product and sum are rounded separately: no fused multiply-add here (the
    // rest of this file contracts)
#pragma clang fp contract(off)
    for (int64_t j = (int64_t)b * 256 + threadIdx.x; j < n; j += (int64_t)nb * 256) {
        if (MODE == kOutF32) {
            const float4 r = ((const float4 *)rec)[j];
            ((float *)ax)[j] = r.x;
            ((float *)ay)[j] = r.y;
            ((float *)az)[j] = r.z;
        } else {
            const double4 r = ((const double4 *)rec)[j];
            if (MODE == kOutF64) {
                ((double *)ax)[j] = r.x;
                ((double *)ay)[j] = r.y;
                ((double *)az)[j] = r.z;
            } else {
                double *const vx = (double *)ax, *const vy = (double *)ay, *const vz = (double *)az;
                vx[j] = vx[j] + dt * r.x;
                vy[j] = vy[j] + dt * r.y;
                vz[j] = vz[j] + dt * r.z;
            }
        }
    }
}

// The last stat_blocks blocks add up the groups' pairs; the others write the results.
template <int MODE>
__global__ __launch_bounds__(256) void k_force_out(const void *__restrict__ rec, int64_t n,
                                                   void *ax, void *ay, void *az, double dt,
                                                   uint32_t n_groups,
                                                   const unsigned long long *__restrict__ pairs,
                                                   unsigned long long *sum, uint32_t stat_blocks)
{
    const uint32_t nb = gridDim.x - stat_blocks;
    if (blockIdx.x < nb)
        write_out<MODE>(rec, n, ax, ay, az, dt, blockIdx.x, nb);
    else
        sum_pairs(n_groups, pairs, sum, blockIdx.x - nb, stat_blocks);
}

// Box blockIdx.y's float outputs and pairs.
__global__ __launch_bounds__(256) void k_force_out_multi(const ForceBox *__restrict__ bx,
                                                         uint32_t stat_blocks)
{
    const ForceBox &B = bx[blockIdx.y];
    const uint32_t nb = gridDim.x - stat_blocks;
    if (blockIdx.x < nb)
        write_out<kOutF32>(B.rec, B.n, B.out[0], B.out[1], B.out[2], 0.0, blockIdx.x, nb);
    else
        sum_pairs(B.n_groups, B.fp.pairs, B.pair_sum, blockIdx.x - nb, stat_blocks);
}

// Statistics, queue bins, queues and their publication by one workgroup (see the class kernels
// and launch_walk_stats for each part).
__device__ __forceinline__ void walk_results(const WalkBox &B)
{
    constexpr int kThreads = 1024, kWaves = kThreads / 64;
    __shared__ uint32_t bin[kBins];
    __shared__ unsigned long long part[4][kWaves], tot[4];
    const uint32_t tid = threadIdx.x, G = B.n_groups;
    const int lane = tid & 63, wave = tid >> 6;
    unsigned long long v[4] = {0, 0, 0, 0}; // cells, particles, pairs, longest list
    for (uint32_t g = tid; g < G; g += kThreads) {
        const unsigned long long l = B.len[g], c = B.gcells[g];
        v[0] += c;
        v[1] += l - c;
        v[2] += l * B.gr.count[g];
        v[3] = l > v[3] ? l : v[3];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        for (int k = 0; k < 3; ++k) v[k] += __shfl_xor(v[k], d, 64);
        const unsigned long long o = __shfl_xor(v[3], d, 64);
        v[3] = o > v[3] ? o : v[3];
    }
    if (lane == 0)
        for (int k = 0; k < 4; ++k) part[k][wave] = v[k];
    for (uint32_t i = tid; i < kBins; i += kThreads) bin[i] = 0;
    __syncthreads();
    if (tid < 4) {
        unsigned long long t = 0;
        for (int w = 0; w < kWaves; ++w)
            t = tid == 3 ? (part[3][w] > t ? part[3][w] : t) : t + part[tid][w];
        tot[tid] = t;
        B.stats[tid] = t;
    }
    __syncthreads();
    const uint32_t t = split_log2(tot[2]);
    for (uint32_t g = tid; g < G; g += kThreads)
        atomicAdd(&bin[cost_bin(g, G, B.gr.count[g], B.len[g], t)], 1u);
    __syncthreads();
    if (wave == 0) scan_bins(bin, B.cls, t);
    __syncthreads();
    for (uint32_t g = tid; g < G; g += kThreads)
        B.cls[atomicAdd(&bin[cost_bin(g, G, B.gr.count[g], B.len[g], t)], 1u)] = g;
    if (tid == 0 && B.mailbox) {
        uint32_t *m = B.mailbox;
        __hip_atomic_store(&m[1], *(volatile unsigned *)B.overflow, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
        for (int k = 0; k < 4; ++k) {
            __hip_atomic_store(&m[2 + 2 * k], (uint32_t)tot[k], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&m[3 + 2 * k], (uint32_t)(tot[k] >> 32), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
        __hip_atomic_store(&m[0], B.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}
__global__ __launch_bounds__(1024) void k_walk_results(WalkBox box) { walk_results(box); }
__global__ __launch_bounds__(1024) void k_walk_results_multi(const WalkBox *__restrict__ bx)
{
    walk_results(bx[blockIdx.x]);
}

__device__ __forceinline__ void force_prep(const ForceBox &B, uint32_t b, uint32_t nb)
{
    const uint32_t i = b * 256u + threadIdx.x;
    if (i < 2 * kXcds) B.cls[kClsQueue + i * kQueueStride] = 0;
    if (i == 0) *B.pair_sum = 0;
    for (uint32_t k = i; k < B.n_groups; k += nb * 256u) B.fp.pairs[k] = 0;
}
__global__ __launch_bounds__(256) void k_force_prep(ForceBox box)
{
    force_prep(box, blockIdx.x, gridDim.x);
}
__global__ __launch_bounds__(256) void k_force_prep_multi(const ForceBox *__restrict__ bx)
{
    force_prep(bx[blockIdx.y], blockIdx.x, gridDim.x);
}

} // namespace

void launch_classify(GroupArrays gr, uint32_t n_groups, const uint32_t *len,
                     const unsigned long long *pairs, uint32_t *cls, hipStream_t s)
{
    if (!n_groups) return;
    const unsigned b = (n_groups + 256u * kClassifyItems - 1) / (256u * kClassifyItems);
    k_class_count<<<b, 256, 0, s>>>(gr, n_groups, len, pairs, cls + kClsBins);
    k_class_scan<<<1, 64, 0, s>>>(cls, pairs);
    k_class_scatter<<<b, 256, 0, s>>>(gr, n_groups, len, pairs, cls);
}

// Two workgroups of eight waves per CU (four waves per SIMD, 92 of the 160 KB of LDS).
void launch_force_f32(const ForceBox &box, uint32_t n_groups, int n_cu, hipStream_t s)
{
    if (!n_groups) return;
    const uint32_t cap = 2u * (uint32_t)n_cu;
    k_force_f32<<<n_groups < cap ? n_groups : cap, 64 * kForceWaves, kForceLds, s>>>(box);
}

void launch_force_f32_multi(const ForceBox *boxes, int nb, uint32_t n_groups, int n_cu,
                            hipStream_t s)
{
    if (!n_groups) return;
    const uint32_t cap = 2u * (uint32_t)n_cu;
    k_force_f32_multi<<<n_groups < cap ? n_groups : cap, 64 * kForceWaves, kForceLds, s>>>(boxes,
                                                                                          nb);
}

void launch_force_prep(const ForceBox &box, hipStream_t s)
{
    const uint32_t b = (box.n_groups + 255) / 256;
    k_force_prep<<<b < 1024 ? (b ? b : 1) : 1024, 256, 0, s>>>(box);
}

void launch_force_prep_multi(const ForceBox *boxes, int nb, hipStream_t s)
{
    k_force_prep_multi<<<dim3(32, nb), 256, 0, s>>>(boxes);
}

void launch_walk_results_one(const WalkBox &box, hipStream_t s)
{
    k_walk_results<<<1, 1024, 0, s>>>(box);
}

void launch_walk_results_multi(const WalkBox *boxes, int nb, hipStream_t s)
{
    if (nb) k_walk_results_multi<<<nb, 1024, 0, s>>>(boxes);
}

void launch_pairwise_f32(int64_t n_i, const double *xi, int64_t n_j, const double *xj,
                         const double *mj, const double *xg, double eta, ForceTable ft,
                         double *out, hipStream_t s)
{
    const double inv_len = 0.5 / eta; // 1 / r_cut
    const double lam = std::sqrt(1.0 - (double)ft.c);
    const int64_t total = n_i * n_j;
    int64_t b = (total + 255) / 256;
    k_pairwise_f32<<<(unsigned)(b < 65536 ? (b > 0 ? b : 1) : 65536), 256, 0, s>>>(
        n_i, xi, n_j, xj, mj, xg[0], xg[1], xg[2], inv_len * lam, ft, inv_len * inv_len / lam,
        out);
}

void launch_force_f64(NodeArrays nd, GroupArrays gr, uint32_t n_groups, const uint64_t *off,
                      const uint32_t *len, const uint32_t *entries, const double4 *ps, const uint32_t *pidx,
                      ForceParams fp, void *rec, int rec64, hipStream_t s)
{
    if (!n_groups) return;
    if (rec64)
        k_force_f64<1><<<n_groups, 64, 0, s>>>(nd, gr, n_groups, off, len, entries, ps, pidx,
                                              fp, rec);
    else
        k_force_f64<0><<<n_groups, 64, 0, s>>>(nd, gr, n_groups, off, len, entries, ps, pidx,
                                              fp, rec);
}

static uint32_t stat_blocks(uint32_t n_groups)
{
    const uint32_t b = (n_groups + 1023) / 1024;
    return b < 1 ? 1 : b < 64 ? b : 64;
}

void launch_force_out(const void *rec, int mode, int64_t n, void *ax, void *ay, void *az,
                      double dt, uint32_t n_groups, const unsigned long long *pairs,
                      unsigned long long *pair_sum, hipStream_t s)
{
    if (n <= 0) return;
    const int64_t want = (n + 255) / 256;
    const uint32_t sb = stat_blocks(n_groups);
    const unsigned b = (unsigned)(want < 4096 ? want : 4096) + sb;
    if (mode == kOutKick)
        k_force_out<kOutKick><<<b, 256, 0, s>>>(rec, n, ax, ay, az, dt, n_groups, pairs,
                                               pair_sum, sb);
    else if (mode == kOutF64)
        k_force_out<kOutF64><<<b, 256, 0, s>>>(rec, n, ax, ay, az, dt, n_groups, pairs,
                                              pair_sum, sb);
    else
        k_force_out<kOutF32><<<b, 256, 0, s>>>(rec, n, ax, ay, az, dt, n_groups, pairs,
                                              pair_sum, sb);
}

void launch_force_out_multi(const ForceBox *boxes, int nb, int64_t most, hipStream_t s)
{
    const int64_t want = (most + 255) / 256;
    k_force_out_multi<<<dim3((unsigned)(want < 1024 ? want : 1024) + 4, nb), 256, 0, s>>>(boxes,
                                                                                         4);
}

// ------------------------------------------------------------------ the pair-law table
namespace {

// p(s) = G(s)^(1/5) = g(R)^(1/5) (s + e2)^(-3/10), R = 2 sqrt(s) < 2 (lengths in units of
// r_cut), in double precision.  On eq. (2)'s first branch g is evaluated in the form without
// cancellation the FP64 kernel uses; on the second, g = (2 - R)^5 (7R^3 + 22R^2 + 10R + 4) / 140,
// whose fifth root has the simple zero 2 - R = 4 (1 - s) / (2 + R) at the cutoff.
double p_host(double s, double one_minus_s, double e2)
{
    const double R = 2.0 * std::sqrt(s);
    double v;
    if (R < 1.0) {
        const double R2 = R * R;
        v = std::log(1.0 + R2 * R * (-1.6 + R2 * (1.6 + R * (-0.5 + R * (-12.0 / 35.0 + 0.15 * R)))));
        return std::exp(0.2 * v - 0.3 * std::log(s + e2));
    }
    v = std::log((((7.0 * R + 22.0) * R + 10.0) * R + 4.0) / 140.0);
    return 4.0 * one_minus_s / (2.0 + R) * std::exp(0.2 * v - 0.3 * std::log(s + e2));
}

} // namespace

bool build_force_table(double eps_over_rcut, std::vector<float> &coef, ForceTable &ft)
{
    const double e2 = eps_over_rcut * eps_over_rcut;
    if (!(e2 > 0.0) || !std::isfinite(e2)) return false;
    const int le = (int)std::floor(std::log2(e2));
    if (le < -26 || le > 5) return false; // the range of eps that an FP32 box may have
    // c: a power of two at most e2 / 2, so G is smooth over the first pieces, and at most 2^-11,
    // so the first piece (s up to c / 64) is too narrow for eq. (2)'s s^(3/2) term to bend it.
    const int kc = le - 1 < -11 ? le - 1 : -11;
    const uint32_t pieces = (uint32_t)(-kc) << kTabSegBits;
    const double c = std::ldexp(1.0, kc);
    ft.entries = pieces + 1;
    ft.base = (uint32_t)(127 + kc) << 8;
    ft.c = (float)c;
    coef.assign(3 * (size_t)ft.entries, 0.f); // the entry of u = 1 stays zero
    // Each piece: the quadratic in t closest, in the relative least-squares sense at 6
    // Chebyshev nodes, to p, with the constant term rounded to float first and the other two
    // fitted to what is left: the rounding of the constant, which G = p^5 would show fivefold,
    // is then made up for over most of the piece.
    constexpr int kNodes = 6;
    const double pi = 3.14159265358979323846;
    const double seg = 1.0 / (1 << kTabSegBits);
    double x[kNodes];
    for (int i = 0; i < kNodes; ++i) x[i] = 0.5 + 0.5 * std::cos(pi * (i + 0.5) / kNodes);
    for (uint32_t k = 0; k < pieces; ++k) {
        const int e = kc + (int)(k >> kTabSegBits);
        const double lo = std::ldexp(1.0 + (double)(k & ((1u << kTabSegBits) - 1)) * seg, e);
        const double w = std::ldexp(seg, e);
        double y[kNodes], c0 = 0.0;
        double m[3][3] = {}, r[3] = {};
        for (int i = 0; i < kNodes; ++i) {
            const double u = lo + x[i] * w;
            y[i] = p_host((u - c) / (1.0 - c), (1.0 - u) / (1.0 - c), e2);
            const double v[3] = {1.0 / y[i], x[i] / y[i], x[i] * x[i] / y[i]};
            for (int a = 0; a < 3; ++a) {
                r[a] += v[a];
                for (int b = 0; b < 3; ++b) m[a][b] += v[a] * v[b];
            }
        }
        // c0 of the full fit (Cramer's rule), rounded; then the 2 x 2 system of the others
        auto det3 = [](const double A[3][3]) {
            return A[0][0] * (A[1][1] * A[2][2] - A[1][2] * A[2][1]) -
                   A[0][1] * (A[1][0] * A[2][2] - A[1][2] * A[2][0]) +
                   A[0][2] * (A[1][0] * A[2][1] - A[1][1] * A[2][0]);
        };
        double m0[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) m0[a][b] = b == 0 ? r[a] : m[a][b];
        c0 = (double)(float)(det3(m0) / det3(m));
        const double r1 = r[1] - m[1][0] * c0, r2 = r[2] - m[2][0] * c0;
        const double d = m[1][1] * m[2][2] - m[1][2] * m[2][1];
        coef[k] = (float)c0;
        coef[ft.entries + k] = (float)((r1 * m[2][2] - r2 * m[1][2]) / d / w);
        coef[2 * ft.entries + k] = (float)((m[1][1] * r2 - m[2][1] * r1) / d / (w * w));
    }
    return true;
}

} // namespace tpm

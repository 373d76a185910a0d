// Short-range pair force over the interaction lists (Section 2.1 eq. 1 with the cutoff
// g_P3M of eq. 2 and Plummer softening of Section 2.4):
//
//   a_i += m_j d g(|d| / eta) / (|d|^2 + eps^2)^(3/2),   d = x_j - x_i.
//
// One 64-lane wavefront takes a group, or a piece of a long one (some of its particles by a
// segment of its list): the i-particles sit in registers, a chunk of them at a time, and the list
// is streamed through LDS in tiles; lanes of one stream read the same tile entry (an LDS
// broadcast) and accumulate in registers.  List entries whose source lies at least r_cut from the
// chunk's bounding box are dropped while a tile is loaded (every pair they form adds exactly zero).
//
// FP32 path (Section 3.1.1): positions are passed relative to the group's cube centre x_g,
// x_i - x_g and wrap(x_j - x_g), each difference taken in FP64 and then rounded to FP32, so
// the rounding error of the subtraction scales with the group size, not the box.  The pair
// law is read from a per-box table of quadratic pieces (see the FP32 section).  The per-tile
// FP32 partial sums are added up in FP64.  The waves of persistent workgroups take the pieces,
// dealt beforehand, and then the whole groups from per-XCD queues, the heaviest first.  Each
// particle's result leaves the kernels as one record in the caller's order, which a last pass
// splits into the output arrays or applies as a kick.
// The FP64 kernel is in k_force64.hip; what they share (chunks, pieces and queues) in
// force_common.hpp.
#include "force_common.hpp"

#include <cmath>
#include <utility>
#include <vector>

namespace tpm {
namespace {

// FP32 path.  Lengths are in units of r_cut / lam, lam = sqrt(1 - c), and the pair law is
//   a_i = 1/(r_cut^2 lam) sum_j m_j d'_ij G(s),  G(s) = g(2 sqrt(s)) / (s + (eps/r_cut)^2)^(3/2),
// s = |d_ij|^2 / r_cut^2 = (u - c) / (1 - c) with u = |d'_ij|^2 + c: c is a power of two below
// (eps/r_cut)^2, added inside the fused sum of squares, whose result the instruction itself
// clamps to 1, so the cutoff is exactly u = 1.  G is read from a table of G = G_a (1 + r)^5
// (build_force_table): 2^kTabSegBits pieces per octave of u, a the piece's lower edge, which is u
// with its low mantissa bits cleared (one AND), G_a about the value there, and r a quadratic
// without a constant in t = u - a, which is exact.  The fifth root 1 + r turns eq. (2)'s
// fifth-order zero at the cutoff into a simple one and flattens s^-3/2 to s^-3/10, so that a
// quadratic keeps G's relative accuracy up to R = 2; and with |r| at most 0.008 but for the last
// pieces, what is rounded in G is G_a and the sum, each once (p = G^(1/5) itself rounded to FP32
// and raised to the fifth power shows its rounding five times, RMS 1.5e-7 in G for R < 1 where
// this is 0.5e-7).
// A pair is 21 vector instructions, all of the kind that issues every 2 cycles on gfx950 (FP32
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

// Culls and packs one tile; returns the number of survivors (the same on every lane).
__device__ __forceinline__ int load_tile_f32(float4 *tile, const uint32_t *ent, uint32_t jb,
                                             uint32_t je, int J, NodeArrays nd,
                                             const FrameF32 &F, const ChunkBox &C)
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

// One pair (see pair_u): the force from its piece's coefficients.
__device__ __forceinline__ float pair_f(float c0, float c1, float c2, float t, float m)
{
    const float r = fmaf(c2, t, c1) * t;
    // (1 + r)^5 - 1
    const float y = r * fmaf(r, fmaf(r, fmaf(r, r + 5.0f, 10.0f), 10.0f), 5.0f);
    return fmaf(c0, y, c0) * m;
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

// The force of the list range [j0, j1) on the chunk's particles f ..: per lane K sums over its
// stream's sources, the per-tile FP32 sums added up in FP64.
template <int K>
__device__ __forceinline__ uint32_t chunk_sums_f32(float4 *tile, int S, uint32_t n_i, uint32_t f,
                                                   const uint32_t *list, uint32_t j0, uint32_t j1,
                                                   const ForceBox &B, const FrameF32 &F,
                                                   double *ax, double *ay, double *az)
{
    const NodeArrays &nd = B.nd;
    const double4 *__restrict__ const ps = B.ps;
    const float c = in_vgpr(F.c);
    uint32_t kept = 0;
    const int lane = __lane_id();
    const int J = 64 / S, lgJ = 31 - __builtin_clz(J);
    const int slot = lane & (S - 1), stream = lane / S;
    uint32_t ent[kTileRounds];
    if (j0 < j1) fetch_entries<kTileRounds>(list, j0, j1, ent);
    double4 pos[K];
    load_chunk<K>(ps, f, n_i, slot, S, pos);
    float xi[K], yi[K], zi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float4 v = rel_f32(pos[k], F);
        xi[k] = v.x;
        yi[k] = v.y;
        zi[k] = v.z;
        ax[k] = ay[k] = az[k] = 0.0;
    }
    const ChunkBox C = chunk_box<K>(xi, yi, zi, S);
    for (uint32_t jb = j0; jb < j1; jb += kTileF32) {
        const int nt = load_tile_f32(tile, ent, jb, j1, J, nd, F, C);
        kept += (uint32_t)nt;
        wave_lds_sync();
        if (jb + kTileF32 < j1) fetch_entries<kTileRounds>(list, jb + kTileF32, j1, ent);
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
    return kept;
}

// What bounds it (256^3 clustered box, n_crit 256): the LDS pipe is busy 91 % of the time and the
// vector units 90 %.  The kernel takes 10.6 ms, 1.85 pairs per ps.  As the fifth power of p, three
// instructions fewer a pair, it was 10.0 ms (93 and 80 %; 8.7 without the table reads); 12.4 with a
// kernel per blocking factor, a table of 16-byte entries and queue counters side by side (311,000
// groups taken through counters in one cache line alone cost about 12 ms, at 40 ns each).
// 700,001 particles, build, walk and force: 3.44 -> 1.06 ms.
struct PolicyF32 {
    static constexpr int kWaves = kForceWaves, kTilesAt = 0, kTileBytes = kTileF32 * 16;
    static constexpr uint32_t kQueueAt = kClsQueue;
    static constexpr bool kAdd = false;
    using Frame = FrameF32;

    static __device__ __forceinline__ void load_table(char *lds, const ForceBox &B)
    {
        const ForceTable ft = B.ft;
        float *const t = reinterpret_cast<float *>(lds);
        for (uint32_t i = threadIdx.x; i < ft.entries; i += blockDim.x)
#pragma unroll
            for (uint32_t q = 0; q < 3; ++q)
                t[(ft.base + q * kTabPlane) / 4 + i] = ft.coef[q * ft.entries + i];
    }

    template <int K>
    static __device__ __forceinline__ uint32_t chunk_sums(char *tile, int S, uint32_t n_i,
                                                          uint32_t f, const uint32_t *list,
                                                          uint32_t j0, uint32_t j1,
                                                          const ForceBox &B, const Frame &F,
                                                          double *ax, double *ay, double *az)
    {
        return chunk_sums_f32<K>(reinterpret_cast<float4 *>(tile), S, n_i, f, list, j0, j1, B, F,
                                 ax, ay, az);
    }

    static __device__ __forceinline__ void group(char *tile, const ForceBox &B, const Piece &w)
    {
        const GroupRead R(B, w.g);
        finish_group<PolicyF32>(tile, B, w, R, frame_f32(B, R));
    }
};

__global__ __launch_bounds__(64 * kForceWaves, 4) void k_force_f32(ForceBox box)
{
    force_body<PolicyF32, false>(&box, 1);
}

__global__ __launch_bounds__(64 * kForceWaves, 4) void k_force_f32_multi(
    const ForceBox *__restrict__ bx, int nb)
{
    force_body<PolicyF32, true>(bx, nb);
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

// Queues of the force.  Group g belongs to XCD part p, about 8 g / G (contiguous key ranges), and,
// unless it is taken in pieces (more than 2^t pairs, see ForceItem), to a cost bucket: the octave
// of its pairs n_g L_g if it has at least 2^kHeavyCost of them or an eighth of 2^t, one bucket for
// all others.  The bins (p, bucket) are laid out with the costliest first, so each part lists its
// heavy groups longest first and then the rest in about key order (consecutive groups share
// sources through the XCD's L2); the pieces, all of about one cost, have a queue of their own
// before them.  Three passes: count the bins, scan them into cursors and part starts, scatter.
// Blocks take kClassifyItems * 256 consecutive groups and aggregate their bins in LDS first.
//
// Why pieces: a wave alone would hold up the end of the launch, and a device of 4096 waves needs
// several items for each.  Shared by the eight waves of a workgroup instead, which meet in LDS
// twice per chunk, a group's waves get a few dozen list entries each and wait most of the time:
// boxes of 250,007, 500,009 and 700,001 particles ran at 0.92, 0.89 and 1.05 pairs per ps against
// 1.14, 1.18 and 1.47 with pieces (1.9 in the 256^3 box).
constexpr int kClassifyItems = 8;
constexpr int kCostBuckets = 64;
constexpr uint32_t kHeavyCost = 17;
constexpr uint32_t kMinPiece = 13;
constexpr int kBins = kXcds * kCostBuckets;
// Up to this many groups, one per thread, k_walk_results writes the queues itself; for more a
// launch of many workgroups follows, and one that publishes the results (one workgroup took 57 us
// to write the 20,000 pieces of a box of 700,001).
constexpr uint32_t kWriteHere = 1024;

// t of the box: its interactions (pairs) are 6,554 to 13,107 times 2^t.  Pieces of half of 2^t to 2^t
// pairs each are two to four for every wave.  A force call's time over the best of all rows, geometric
// mean over 68 boxes of 100,003 to 2,000,003 particles (four octaves of pairs; clustered and uniform,
// groups of up to 64 and 256, with and without quadrupoles), by the least multiple of 2^t:
//   3,277  4,096  4,681  5,461  6,554  8,192  13,107
//   1.100  1.078  1.063  1.047  1.043  1.057   1.093
__device__ __forceinline__ uint32_t piece_log2(unsigned long long pairs)
{
    const unsigned long long v = (pairs >> 13) + (pairs >> 15);
    const uint32_t lg = 63u - (uint32_t)__clzll((long long)(v | 1ull));
    return lg > kMinPiece ? lg : kMinPiece;
}

// ceil(log2(v)), v >= 1.
__device__ __forceinline__ uint32_t log2_up(uint32_t v) { return v > 1 ? 32u - (uint32_t)__clz((int)(v - 1)) : 0u; }

// s of the segments of a chunk of n_c particles against a list of L entries: the longest of at most
// 2^t pairs, but not so short that there are more than kMaxSegs.  (Powers of two: the queues of a
// box are made by one compute unit or a few, and integer divisions were most of it.)
__device__ __forceinline__ uint32_t seg_log2(uint32_t n_c, uint32_t L, uint32_t t)
{
    const uint32_t by_pairs = log2_up(n_c) + 6u, rounds = (L + kSegMin - 1) / kSegMin;
    const uint32_t few = log2_up((rounds + kMaxSegs - 1) / kMaxSegs);
    const uint32_t s = t > by_pairs ? t - by_pairs : 0u;
    return s > few ? (s < 24u ? s : 24u) : few;
}
__device__ __forceinline__ uint32_t seg_count(uint32_t L, uint32_t s)
{
    const uint32_t rounds = (L + kSegMin - 1) / kSegMin;
    return rounds ? (rounds - 1 >> s) + 1 : 1u;
}

// The pieces of a group: its chunks, all alike but the last, in segments.
struct Pieces {
    uint32_t chunks, s, segs, last_n, last_s, last_segs;
    __device__ __forceinline__ Pieces(uint32_t n_g, uint32_t L, uint32_t t)
        : chunks((n_g + kPieceChunk - 1) / kPieceChunk), s(seg_log2(kPieceChunk, L, t)),
          segs(seg_count(L, s)), last_n(n_g - (chunks - 1) * kPieceChunk),
          last_s(seg_log2(last_n, L, t)), last_segs(seg_count(L, last_s))
    {
    }
    __device__ __forceinline__ uint32_t items() const { return (chunks - 1) * segs + last_segs; }
    __device__ __forceinline__ uint32_t rows() const
    {
        return (segs > 1 ? (chunks - 1) * kPieceChunk * segs : 0u) +
               (last_segs > 1 ? last_n * last_segs : 0u);
    }
    __device__ __forceinline__ void write(uint32_t g, ForceItem *out, uint32_t base) const
    {
        for (uint32_t c = 0; c < chunks; ++c) {
            const bool last = c + 1 == chunks;
            const uint32_t m = last ? last_segs : segs, ss = m << 8 | (last ? last_s : s) << 16;
            for (uint32_t q = 0; q < m; ++q) *out++ = ForceItem{g, c, q | ss, base};
            if (m > 1) base += (last ? last_n : kPieceChunk) * m;
        }
    }
};

// Bucket 0 of a part counts pieces.
__device__ __forceinline__ uint32_t cost_bin(uint32_t g, uint32_t n_groups, uint32_t n_g,
                                             uint32_t L_g, uint32_t t)
{
    // any rounding will do, as long as the parts follow the groups' order
    const uint32_t p = (uint32_t)((float)g * ((float)kXcds / (float)n_groups));
    const uint32_t part = p < kXcds ? p : kXcds - 1;
    const uint64_t cost = (uint64_t)n_g * L_g;
    const uint32_t lg = 63u - (uint32_t)__clzll((long long)(cost | 1ull));
    const uint32_t least = t - 3 < kHeavyCost ? t - 3 : kHeavyCost;
    const uint32_t bucket =
        cost > 1ull << t ? 0u : kCostBuckets - 1 - (lg >= least ? lg : 0u);
    return part * kCostBuckets + bucket;
}
__device__ __forceinline__ bool in_pieces(uint32_t bin) { return bin % kCostBuckets == 0; }

__global__ __launch_bounds__(256) void k_class_count(GroupArrays gr, uint32_t n_groups,
                                                     const uint32_t *__restrict__ len,
                                                     unsigned long long *stats, uint32_t *hist)
{
    __shared__ uint32_t s_cnt[kBins], s_rows;
    for (int i = threadIdx.x; i < kBins; i += 256) s_cnt[i] = 0;
    if (threadIdx.x == 0) s_rows = 0;
    __syncthreads();
    const uint32_t t = piece_log2(stats[2]);
    const uint32_t base = blockIdx.x * (256u * kClassifyItems);
#pragma unroll
    for (int r = 0; r < kClassifyItems; ++r) {
        const uint32_t g = base + (uint32_t)r * 256u + threadIdx.x;
        if (g >= n_groups) continue;
        const uint32_t n_g = gr.count[g], L = len[g], bin = cost_bin(g, n_groups, n_g, L, t);
        if (in_pieces(bin)) {
            const Pieces p(n_g, L, t);
            atomicAdd(&s_cnt[bin], p.items());
            atomicAdd(&s_rows, p.rows());
        } else
            atomicAdd(&s_cnt[bin], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += 256)
        if (s_cnt[i]) atomicAdd(&hist[i], s_cnt[i]);
    if (threadIdx.x == 0 && s_rows) atomicAdd(&stats[4], (unsigned long long)s_rows);
}

// By one wave, lane = cost bucket: the bins' counts to cursors (in place; bins in global memory
// or LDS), the part starts of the whole groups and the number of pieces into cls.  Returns the
// latter.
__device__ __forceinline__ uint32_t scan_bins(uint32_t *bins, uint32_t *cls)
{
    static_assert(kCostBuckets == 64, "one lane per bucket");
    const int lane = __lane_id();
    uint32_t pos = kClsLists, items = 0;
    uint32_t c[kXcds];
#pragma unroll
    for (int p = 0; p < (int)kXcds; ++p) c[p] = bins[p * kCostBuckets + lane];
#pragma unroll
    for (int p = 0; p < (int)kXcds; ++p) {
        const uint32_t mine = lane ? c[p] : 0u;
        uint32_t v = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = __shfl_up(v, d, 64);
            if (lane >= d) v += u;
        }
        bins[p * kCostBuckets + lane] = lane ? pos + v - mine : items;
        if (lane == 0) cls[kClsStarts + p] = pos;
        pos += (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
        items += (uint32_t)__builtin_amdgcn_readfirstlane((int)c[p]);
    }
    if (lane == 0) {
        cls[kClsStarts + kXcds] = pos;
        cls[kClsItems] = items;
    }
    return items;
}
__global__ __launch_bounds__(64) void k_class_scan(uint32_t *cls, unsigned long long *stats)
{
    const uint32_t items = scan_bins(cls + kClsBins, cls);
    if (threadIdx.x == 0) stats[5] = items;
}

// Block b's groups, ITEMS per thread; rows are handed out through stats[6].
template <int ITEMS>
__device__ __forceinline__ void class_scatter(const GroupArrays &gr, uint32_t n_groups,
                                              const uint32_t *__restrict__ len,
                                              unsigned long long *stats, uint32_t *cls,
                                              ForceItem *__restrict__ items, uint32_t b)
{
    __shared__ uint32_t s_cnt[kBins], s_rows, s_base;
    for (int i = threadIdx.x; i < kBins; i += 256) s_cnt[i] = 0;
    if (threadIdx.x == 0) s_rows = s_base = 0;
    __syncthreads();
    const uint32_t t = piece_log2(stats[2]);
    const uint32_t base = b * (256u * ITEMS);
    uint32_t bin[ITEMS], loc[ITEMS], row[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t g = base + (uint32_t)r * 256u + threadIdx.x;
        bin[r] = ~0u;
        row[r] = 0;
        if (g < n_groups) {
            const uint32_t n_g = gr.count[g], L = len[g];
            bin[r] = cost_bin(g, n_groups, n_g, L, t);
            if (in_pieces(bin[r])) {
                const Pieces p(n_g, L, t);
                loc[r] = atomicAdd(&s_cnt[bin[r]], p.items());
                row[r] = atomicAdd(&s_rows, p.rows());
            } else
                loc[r] = atomicAdd(&s_cnt[bin[r]], 1u);
        }
    }
    __syncthreads();
    // this block's run of each bin, and of the rows
    for (int i = threadIdx.x; i < kBins; i += 256)
        if (s_cnt[i]) s_cnt[i] = atomicAdd(&cls[kClsBins + i], s_cnt[i]);
    if (threadIdx.x == 0 && s_rows)
        s_base = (uint32_t)atomicAdd(&stats[6], (unsigned long long)s_rows);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (bin[r] == ~0u) continue;
        const uint32_t g = base + (uint32_t)r * 256u + threadIdx.x;
        if (in_pieces(bin[r]))
            Pieces(gr.count[g], len[g], t).write(g, items + s_cnt[bin[r]] + loc[r], s_base + row[r]);
        else
            cls[s_cnt[bin[r]] + loc[r]] = g;
    }
}
__global__ __launch_bounds__(256) void k_class_scatter(GroupArrays gr, uint32_t n_groups,
                                                       const uint32_t *__restrict__ len,
                                                       unsigned long long *stats, uint32_t *cls,
                                                       ForceItem *__restrict__ items)
{
    class_scatter<kClassifyItems>(gr, n_groups, len, stats, cls, items, blockIdx.x);
}
// After k_walk_results, for boxes whose groups it has only counted.
__global__ __launch_bounds__(256) void k_walk_scatter(WalkBox B)
{
    class_scatter<1>(B.gr, B.n_groups, B.len, B.stats, B.cls, B.items, blockIdx.x);
}
__global__ __launch_bounds__(256) void k_walk_scatter_multi(const WalkBox *__restrict__ bx)
{
    const WalkBox &B = bx[blockIdx.y];
    if (B.n_groups > kWriteHere && blockIdx.x * 256u < B.n_groups)
        class_scatter<1>(B.gr, B.n_groups, B.len, B.stats, B.cls, B.items, blockIdx.x);
}

// Adds up the rows of the chunks whose list was taken in segments, a wave per chunk (that of its
// first segment), in the order of the segments, and stores the particles' records.
__device__ __forceinline__ void force_merge(const ForceBox &B, uint32_t k)
{
    if (k >= B.n_items) return;
    const ForceItem f = B.items[k];
    const uint32_t segs = f.seg_segs >> 8 & 0xffu;
    if ((f.seg_segs & 0xffu) != 0 || segs < 2) return;
    const uint32_t n_g = B.gr.count[f.g], i0 = f.chunk * kPieceChunk;
    const uint32_t n_c = n_g - i0 < kPieceChunk ? n_g - i0 : kPieceChunk;
    const uint32_t first = B.gr.first[f.g] + i0;
    for (uint32_t i = __lane_id(); i < n_c; i += 64) {
        const uint32_t o = B.pidx[first + i];
        const double *r = B.rows + 3 * ((uint64_t)f.base + i);
        double x = 0.0, y = 0.0, z = 0.0;
#pragma unroll 4
        for (uint32_t q = 0; q < segs; ++q) {
            const double *p = r + 3 * (uint64_t)q * n_c;
            x += p[0];
            y += p[1];
            z += p[2];
        }
        if (B.rec64)
            store_rec<1, false>(B.rec, o, x, y, z);
        else
            store_rec<0, false>(B.rec, o, x, y, z);
    }
}
__global__ __launch_bounds__(256) void k_force_merge(ForceBox box)
{
    force_merge(box, blockIdx.x * 4 + (threadIdx.x >> 6));
}
__global__ __launch_bounds__(256) void k_force_merge_multi(const ForceBox *__restrict__ bx)
{
    force_merge(bx[blockIdx.y], blockIdx.x * 4 + (threadIdx.x >> 6));
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

// The overflow word and the six statistics to the box's mailbox, from word 1 on, and then its
// sequence number: the host may go on, on any stream, as soon as it sees that, so whatever else
// the walk leaves has to be complete.
__device__ __forceinline__ void publish_results(const WalkBox &B)
{
    uint32_t *m = B.mailbox;
    __hip_atomic_store(&m[1], *(volatile unsigned *)B.overflow, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
    for (int k = 0; k < 6; ++k) {
        const unsigned long long v = *(volatile unsigned long long *)&B.stats[k];
        __hip_atomic_store(&m[2 + 2 * k], (uint32_t)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&m[3 + 2 * k], (uint32_t)(v >> 32), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __hip_atomic_store(&m[0], B.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Statistics, queue bins, queues (kWriteHere) and their publication by one workgroup (see the
// class kernels and launch_walk_stats for each part).
__device__ __forceinline__ void walk_results(const WalkBox &B)
{
    constexpr int kThreads = 1024, kWaves = kThreads / 64;
    __shared__ uint32_t bin[kBins];
    __shared__ unsigned long long part[4][kWaves], tot[4];
    __shared__ uint32_t s_rows;
    const uint32_t tid = threadIdx.x, G = B.n_groups;
    const int lane = tid & 63, wave = tid >> 6;
    unsigned long long v[4] = {0, 0, 0, 0}; // cells, particles, pairs, longest list
    // all of a thread's groups at once, kept for the two passes below: one memory latency
    constexpr int kPer = (int)(kOneBlockGroups / kThreads);
    // neighbouring lanes take groups an eighth of the box apart, of different parts: atomics of
    // a wave on one bin in LDS are served one by one
    const uint32_t eighth = (G + 7) / 8, g0 = (tid & 7) * eighth, g_end = min(G, g0 + eighth);
    auto group = [&](int r) { return g0 + (tid >> 3) + (uint32_t)r * (kThreads / 8); };
    uint32_t n_g[kPer], len[kPer], cells[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const uint32_t g = group(r), at = g < g_end ? g : 0u;
        n_g[r] = B.gr.count[at];
        len[r] = B.len[at];
        cells[r] = B.gcells[at];
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        if (group(r) >= g_end) continue;
        v[0] += cells[r];
        v[1] += len[r] - cells[r];
        v[2] += (unsigned long long)len[r] * n_g[r];
        v[3] = len[r] > v[3] ? len[r] : v[3];
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
    if (tid == 0) s_rows = 0;
    __syncthreads();
    if (tid < 4) {
        unsigned long long t = 0;
        for (int w = 0; w < kWaves; ++w)
            t = tid == 3 ? (part[3][w] > t ? part[3][w] : t) : t + part[tid][w];
        tot[tid] = t;
        B.stats[tid] = t;
    }
    __syncthreads();
    const uint32_t t = piece_log2(tot[2]);
    uint32_t rows = 0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const uint32_t g = group(r);
        if (g >= g_end) continue;
        const uint32_t k = cost_bin(g, G, n_g[r], len[r], t);
        if (in_pieces(k)) {
            const Pieces p(n_g[r], len[r], t);
            atomicAdd(&bin[k], p.items());
            rows += p.rows();
        } else
            atomicAdd(&bin[k], 1u);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) rows += __shfl_xor(rows, d, 64);
    if (lane == 0 && rows) atomicAdd(&s_rows, rows);
    __syncthreads();
    if (wave == 0) {
        const uint32_t items = scan_bins(bin, B.cls);
        if (lane == 0) {
            B.stats[4] = s_rows;
            B.stats[5] = items;
            s_rows = 0;
        }
    }
    __syncthreads();
    if (G <= kWriteHere) {
        const uint32_t g = group(0); // kWriteHere groups: one each
        if (g < g_end) {
            const uint32_t k = cost_bin(g, G, n_g[0], len[0], t);
            if (in_pieces(k)) {
                const Pieces p(n_g[0], len[0], t);
                const uint32_t at = atomicAdd(&bin[k], p.items());
                p.write(g, B.items + at, atomicAdd(&s_rows, p.rows()));
            } else
                B.cls[atomicAdd(&bin[k], 1u)] = g;
        }
    } else { // the cursors for the launch that follows
        for (uint32_t i = tid; i < kBins; i += kThreads) B.cls[kClsBins + i] = bin[i];
    }
    if (G <= kWriteHere && B.mailbox) { // every thread's writes before the publication
        __threadfence();
        __syncthreads();
        if (tid == 0) publish_results(B);
    }
}
__global__ __launch_bounds__(1024) void k_walk_results(WalkBox box) { walk_results(box); }
__global__ __launch_bounds__(1024) void k_walk_results_multi(const WalkBox *__restrict__ bx)
{
    walk_results(bx[blockIdx.x]);
}

// For boxes whose queues k_walk_scatter has written.
__global__ void k_walk_publish(WalkBox box)
{
    if (threadIdx.x == 0) publish_results(box);
}
__global__ void k_walk_publish_multi(const WalkBox *__restrict__ bx)
{
    const WalkBox &B = bx[blockIdx.x];
    if (threadIdx.x == 0 && B.n_groups > kWriteHere && B.mailbox) publish_results(B);
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
                     unsigned long long *stats, uint32_t *cls, ForceItem *items, hipStream_t s)
{
    if (!n_groups) return;
    const unsigned b = (n_groups + 256u * kClassifyItems - 1) / (256u * kClassifyItems);
    k_class_count<<<b, 256, 0, s>>>(gr, n_groups, len, stats, cls + kClsBins);
    k_class_scan<<<1, 64, 0, s>>>(cls, stats);
    k_class_scatter<<<b, 256, 0, s>>>(gr, n_groups, len, stats, cls, items);
}

void launch_force_merge(const ForceBox &box, hipStream_t s)
{
    if (box.n_items) k_force_merge<<<(box.n_items + 3) / 4, 256, 0, s>>>(box);
}

void launch_force_merge_multi(const ForceBox *boxes, int nb, uint32_t most_items, hipStream_t s)
{
    if (most_items) k_force_merge_multi<<<dim3((most_items + 3) / 4, nb), 256, 0, s>>>(boxes);
}

// Two workgroups of eight waves per CU (four waves per SIMD, 92 of the 160 KB of LDS).
static unsigned force_blocks(uint32_t n_work, uint32_t cap) { return n_work < cap ? n_work : cap; }

void launch_force_f32(const ForceBox &box, int n_cu, hipStream_t s)
{
    if (!box.n_groups) return;
    k_force_f32<<<force_blocks(box.n_groups + box.n_items, 2u * (uint32_t)n_cu), 64 * kForceWaves,
                  kForceLds, s>>>(box);
}

void launch_force_f32_multi(const ForceBox *boxes, int nb, uint32_t n_work, int n_cu,
                            hipStream_t s)
{
    if (!n_work) return;
    k_force_f32_multi<<<force_blocks(n_work, 2u * (uint32_t)n_cu), 64 * kForceWaves, kForceLds,
                        s>>>(boxes, nb);
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
    if (box.n_groups <= kWriteHere) {
        k_walk_results<<<1, 1024, 0, s>>>(box);
        return;
    }
    WalkBox quiet = box;
    quiet.mailbox = nullptr;
    k_walk_results<<<1, 1024, 0, s>>>(quiet);
    k_walk_scatter<<<(box.n_groups + 255) / 256, 256, 0, s>>>(box);
    if (box.mailbox) k_walk_publish<<<1, 64, 0, s>>>(box);
}

void launch_walk_results_multi(const WalkBox *boxes, int nb, uint32_t most, hipStream_t s)
{
    if (!nb) return;
    k_walk_results_multi<<<nb, 1024, 0, s>>>(boxes);
    if (most > kWriteHere) {
        k_walk_scatter_multi<<<dim3((most + 255) / 256, nb), 256, 0, s>>>(boxes);
        k_walk_publish_multi<<<nb, 64, 0, s>>>(boxes);
    }
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
    // Chebyshev nodes, to p = G^(1/5) gives G_a, rounded to float; then 1 + r, a quadratic with
    // the constant 1, is fitted to (G / G_a)^(1/5) in the same sense, which makes up for that
    // rounding over most of the piece.
    constexpr int kNodes = 6;
    const double pi = 3.14159265358979323846;
    const double seg = 1.0 / (1 << kTabSegBits);
    double x[kNodes];
    for (int i = 0; i < kNodes; ++i) x[i] = 0.5 + 0.5 * std::cos(pi * (i + 0.5) / kNodes);
    for (uint32_t k = 0; k < pieces; ++k) {
        const int e = kc + (int)(k >> kTabSegBits);
        const double lo = std::ldexp(1.0 + (double)(k & ((1u << kTabSegBits) - 1)) * seg, e);
        const double w = std::ldexp(seg, e);
        double y[kNodes];
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
        // the constant of the full fit (Cramer's rule); then the 2 x 2 system of the others
        auto det3 = [](const double A[3][3]) {
            return A[0][0] * (A[1][1] * A[2][2] - A[1][2] * A[2][1]) -
                   A[0][1] * (A[1][0] * A[2][2] - A[1][2] * A[2][0]) +
                   A[0][2] * (A[1][0] * A[2][1] - A[1][1] * A[2][0]);
        };
        double m0[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) m0[a][b] = b == 0 ? r[a] : m[a][b];
        coef[k] = (float)std::pow(det3(m0) / det3(m), 5.0);
        const double c0 = std::pow((double)coef[k], 0.2);
        const double r1 = r[1] - m[1][0] * c0, r2 = r[2] - m[2][0] * c0;
        const double d = (m[1][1] * m[2][2] - m[1][2] * m[2][1]) * c0;
        coef[ft.entries + k] = (float)((r1 * m[2][2] - r2 * m[1][2]) / d / w);
        coef[2 * ft.entries + k] = (float)((m[1][1] * r2 - m[2][1] * r1) / d / (w * w));
    }
    return true;
}

} // namespace tpm

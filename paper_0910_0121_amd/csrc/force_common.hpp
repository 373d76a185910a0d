// Parts shared by the FP32 and FP64 force kernels: the persistent workgroups and their queues,
// the split of a group into chunks of particles, its pieces, and the output of their sums.
// A kernel is a policy P: kWaves (waves per workgroup), kTilesAt and kTileBytes (the waves' LDS
// tiles), kQueueAt (its queue counters), kAdd (sums are added to the records and no pairs are
// counted), Frame (a group's origin and units, with `scale`, the factor of the sums), load_table,
// group (reads a group, makes its frame and calls finish_group) and chunk_sums<K> (a wave's sums
// for a chunk over a range of the group's list, each lane's own stream's; returns the entries that
// survived the cull).
#pragma once

#include "common.hpp"

namespace tpm {
namespace {

// The force kernels leave one record per particle, in the caller's order: float4 (ax, ay, az,
// 0) for float results, double4 for double results and for the kick.  The caller's order is
// arbitrary, so each store lands in its own 32-byte HBM sector: one 16- or 32-byte record costs
// one sector where three 4- or 8-byte component stores cost three.  k_force_out then walks the
// records in order and splits them into the caller's three arrays (kOutF32, kOutF64) or adds dt
// times them to double velocities (kOutKick: the kick of Section 2.2 step 5 taken with the
// short-range force as soon as it is known), each product and sum rounded on its own.
enum { kOutF32 = 0, kOutF64 = 1, kOutKick = 2 };

template <int REC64, bool ADD>
__device__ __forceinline__ void store_rec(void *rec, uint32_t i, double vx, double vy, double vz)
{
    if (ADD) { // each record belongs to one particle of one chunk
        if (REC64) {
            double4 *const r = (double4 *)rec + i;
            const double4 o = *r;
            *r = make_double4(o.x + vx, o.y + vy, o.z + vz, 0.0);
        } else {
            float4 *const r = (float4 *)rec + i;
            const float4 o = *r;
            *r = make_float4(o.x + (float)vx, o.y + (float)vy, o.z + (float)vz, 0.0f);
        }
        return;
    }
    if (REC64)
        ((double4 *)rec)[i] = make_double4(vx, vy, vz, 0.0);
    else
        ((float4 *)rec)[i] = make_float4((float)vx, (float)vy, (float)vz, 0.0f);
}

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

// The lane, as a value that the compiler does not take for the same from one use to the next: what
// is worked out from it (queue and list addresses) is not kept in vector registers across the
// pair loops, whose 128 are all in use.
__device__ __forceinline__ uint32_t lane_now()
{
    uint32_t l = __lane_id();
    asm volatile("" : "+v"(l));
    return l;
}

// The chunk's particles, K per lane (slot, slot + S, ..; idle slots repeat the first), all on their
// way before any is used.
template <int K>
__device__ __forceinline__ void load_chunk(const double4 *__restrict__ ps, uint32_t f,
                                           uint32_t n_i, int slot, int S, double4 *r)
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t i = (uint32_t)(slot + S * k);
        r[k] = ps[f + (i < n_i ? i : 0)];
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Keeps a wave-uniform value in a vector register.
__device__ __forceinline__ float in_vgpr(float v)
{
    asm("" : "+v"(v));
    return v;
}

// The list entries of the tile starting at jb (jb < je), one per lane and round.  Slots past
// the range's end read its last entry and are dropped when the tile is packed.  The caller issues
// these reads one tile ahead, so they are in flight while the previous tile is evaluated.
template <int ROUNDS>
__device__ __forceinline__ void fetch_entries(const uint32_t *__restrict__ list, uint32_t jb,
                                              uint32_t je, uint32_t *ent)
{
    const uint32_t lane = lane_now();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t j = jb + (uint32_t)(r * 64) + lane;
        ent[r] = list[j < je ? j : je - 1];
    }
}

// The bounding box of a chunk of the group's particles in x' units, for the cull.
struct ChunkBox {
    float c0, c1, c2; // centre
    float h0, h1, h2; // minus half the half size
    float thr;        // a quarter of the squared cull distance, with margin
};

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

// The box of the chunk's particles, K per lane and repeated over the J streams.
template <int K>
__device__ __forceinline__ ChunkBox chunk_box(const float *xi, const float *yi, const float *zi,
                                              int S)
{
    ChunkBox C;
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
    // The coordinates near the threshold are at most 1 + 2 max(h) + |c| in size, each rounded a
    // few times to 2^-24 of that; the cull distance is at most 1.
    const float big = 1.0f + 4.0f * fmaxf(fmaxf(-C.h0, -C.h1), -C.h2) +
                      fmaxf(fmaxf(fabsf(C.c0), fabsf(C.c1)), fabsf(C.c2));
    C.thr = uni(0.25f * (1.0f + 0x1p-12f + 0x1p-20f * big));
    return C;
}

// The J streams' sums on every lane, in a fixed tree.
template <int K>
__device__ __forceinline__ void add_streams(double *ax, double *ay, double *az, int S)
{
    for (int d = S; d < 64; d <<= 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ax[k] += __shfl_xor(ax[k], d, 64);
            ay[k] += __shfl_xor(ay[k], d, 64);
            az[k] += __shfl_xor(az[k], d, 64);
        }
    }
}

// One chunk by one wave: its sums to the particles' records, or, for a segment of the list, to the
// segment's rows (of three doubles, `rows`), which launch_force_merge adds up.
template <class P, int K>
__device__ __forceinline__ uint32_t run_chunk(char *tile, double *rows, int S, uint32_t n_i,
                                              uint32_t f, const uint32_t *list, uint32_t j0,
                                              uint32_t j1, const ForceBox &B,
                                              const typename P::Frame &F)
{
    double ax[K], ay[K], az[K];
    const uint32_t kept =
        P::template chunk_sums<K>(tile, S, n_i, f, list, j0, j1, B, F, ax, ay, az);
    const double scale = F.scale;
    const uint32_t *__restrict__ const pidx = B.pidx;
    void *const rec = B.rec;
    const int rec64 = B.rec64;
    const int lane = (int)lane_now();
    // the places in the caller's order are on their way while the streams are added up
    uint32_t o[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t i = (uint32_t)(lane + S * k);
        o[k] = pidx[f + (i < n_i ? i : 0)];
    }
    __builtin_amdgcn_sched_barrier(0);
    add_streams<K>(ax, ay, az, S);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t i = (uint32_t)(lane + S * k);
        if (lane < S && i < n_i) {
            const double x = ax[k] * scale, y = ay[k] * scale, z = az[k] * scale;
            if (rows) {
                double *const r = rows + 3 * i;
                r[0] = P::kAdd ? r[0] + x : x;
                r[1] = P::kAdd ? r[1] + y : y;
                r[2] = P::kAdd ? r[2] + z : z;
            } else if (rec64)
                store_rec<1, P::kAdd>(rec, o[k], x, y, z);
            else
                store_rec<0, P::kAdd>(rec, o[k], x, y, z);
        }
    }
    return kept;
}

// Particles [i0, i1) of a group over the list range [j0, j1); returns the pairs with the entries
// that survived the cull.
template <class P>
__device__ __forceinline__ uint64_t run_group(char *tile, double *rows, const ForceBox &B,
                                              uint32_t i0, uint32_t i1, uint32_t f,
                                              const uint32_t *list, uint32_t j0, uint32_t j1,
                                              const typename P::Frame &F)
{
    uint64_t pairs = 0;
    for (uint32_t ib = i0; ib < i1;) {
        int S, K;
        chunk_layout(i1 - ib, S, K);
        const uint32_t n_i = i1 - ib < (uint32_t)(S * K) ? i1 - ib : (uint32_t)(S * K);
        uint32_t kept;
        if (K == 4)
            kept = run_chunk<P, 4>(tile, rows, S, n_i, f + ib, list, j0, j1, B, F);
        else
            kept = run_chunk<P, 2>(tile, rows, S, n_i, f + ib, list, j0, j1, B, F);
        ib += n_i;
        if (rows) rows += 3 * n_i;
        pairs += (uint64_t)kept * n_i;
    }
    return pairs;
}

// What the kernels read about a group, all of it before any is used: one memory latency.
struct GroupRead {
    double lo[3], hi[3], xg[3];
    uint32_t count, first, len;
    uint64_t off;
    __device__ __forceinline__ GroupRead(const ForceBox &B, uint32_t g)
    {
        const GroupArrays &gr = B.gr;
        lo[0] = gr.lox[g]; lo[1] = gr.loy[g]; lo[2] = gr.loz[g];
        hi[0] = gr.hix[g]; hi[1] = gr.hiy[g]; hi[2] = gr.hiz[g];
        xg[0] = gr.xgx[g]; xg[1] = gr.xgy[g]; xg[2] = gr.xgz[g];
        count = gr.count[g];
        first = gr.first[g];
        len = B.len[g];
        off = B.off[g];
        __builtin_amdgcn_sched_barrier(0);
    }
    // Whether the bounding box, grown by r_cut (and clear of rounding), leaves [0, L) anywhere:
    // otherwise a source within r_cut of the box is its own nearest image, and a source whose
    // nearest image lies across the boundary is at least r_cut from the box without the wrap as
    // with it, so no coordinate needs wrapping.
    __device__ __forceinline__ bool wraps(const ForceBox &B) const
    {
        const ForceParams &fp = B.fp;
        const double rc = B.units.rc_wrap;
        return __ballot(!((lo[0] - rc >= 0.0) & (hi[0] + rc < fp.L) & (lo[1] - rc >= 0.0) &
                          (hi[1] + rc < fp.L) & (lo[2] - rc >= 0.0) & (hi[2] + rc < fp.L))) != 0;
    }
};

// What a wave of the FP32 kernels needs of its group.  Coordinates are x' = x inv - xg', one fused operation.
struct FrameF32 {
    bool wrap;            // coordinates need the nearest image
    double xg0, xg1, xg2; // wrap: x_g; else x_g inv
    double L, inv_L, inv; // inv = lam / r_cut
    double scale;
    float c;
};

// A position relative to x_g in x' units (wrap: see GroupRead::wraps).
__device__ __forceinline__ float4 rel_f32(const double4 r, const FrameF32 &F)
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

__device__ __forceinline__ FrameF32 frame_f32(const ForceBox &B, const GroupRead &R)
{
    const ForceUnits &U = B.units;
    FrameF32 F;
    F.scale = U.scale;
    F.wrap = R.wraps(B);
    F.L = B.fp.L;
    F.inv_L = U.inv_L;
    F.inv = U.inv;
    F.xg0 = uni(F.wrap ? R.xg[0] : R.xg[0] * F.inv);
    F.xg1 = uni(F.wrap ? R.xg[1] : R.xg[1] * F.inv);
    F.xg2 = uni(F.wrap ? R.xg[2] : R.xg[2] * F.inv);
    F.c = B.ft.c;
    return F;
}

// One pair in x' units: a source s against a particle, and u = min(|d'|^2 + c, 1).
__device__ __forceinline__ float pair_u(const float4 s, float xi, float yi, float zi, float c,
                                        float &dx, float &dy, float &dz)
{
    dx = s.x - xi;
    dy = s.y - yi;
    dz = s.z - zi;
    // u = min(|d|^2 + c, 1): the clamp is an output modifier of the last fma
    return __builtin_amdgcn_fmed3f(fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, c))), 0.0f, 1.0f);
}
// The piece of a group that a wave takes: all of it, or a part of its particles and of its list.
struct Piece {
    uint32_t g;
    bool whole;
    uint32_t chunk, seg, segs, log2_per, base; // see ForceItem
};

// The piece once its group's frame is known.
template <class P>
__device__ __forceinline__ void finish_group(char *tile, const ForceBox &B, const Piece &w,
                                             const GroupRead &R, const typename P::Frame &F)
{
    const uint32_t Lg = uni(R.len), n_g = uni(R.count);
    uint32_t i0 = 0, i1 = n_g, j0 = 0, j1 = Lg;
    double *rows = nullptr;
    if (!w.whole) {
        i0 = w.chunk * kPieceChunk;
        i1 = n_g - i0 < kPieceChunk ? n_g : i0 + kPieceChunk;
        const uint32_t per = kSegMin << w.log2_per;
        j0 = w.seg * per;
        j1 = j0 + per < Lg ? j0 + per : Lg;
        if (w.segs > 1) rows = B.rows + 3 * ((uint64_t)w.base + (uint64_t)w.seg * (i1 - i0));
    }
    const uint32_t *list =
        B.entries + (((uint64_t)uni((uint32_t)(R.off >> 32)) << 32) | uni((uint32_t)R.off));
    // (uniform already, which the compiler loses sight of: the pair loops' counters would be vectors)
    const uint64_t pairs = run_group<P>(tile, rows, B, uni(i0), uni(i1), uni(R.first), list, uni(j0),
                                        uni(j1), F);
    if (!P::kAdd && __lane_id() == 0) {
        if (w.whole)
            B.fp.pairs[w.g] = pairs;
        else
            atomicAdd(&B.fp.pairs[w.g], (unsigned long long)pairs); // zeroed by the prep launch
    }
}

// The first part at or after `from` (cyclically) whose counter has not reached its size, or
// kXcds.  Lane p < kXcds holds part p's size, less what is dealt.  One read of all counters, so a wave that finds
// everything taken leaves after one memory latency, and no atomic is spent on empty queues.
__device__ __forceinline__ uint32_t next_part(uint32_t *ctr, uint32_t size, uint32_t from)
{
    const uint32_t lane = lane_now();
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

// Box b's run of part p in the queue of whole groups.
__device__ __forceinline__ uint32_t run_size(const uint32_t *cls, uint32_t p)
{
    return cls[kClsStarts + p + 1] - cls[kClsStarts + p];
}

// Per lane p < kXcds the total size of part p over the boxes.
__device__ __forceinline__ uint32_t part_sizes(const ForceBox *bx, int nb)
{
    const uint32_t lane = lane_now();
    uint32_t n = 0;
    if (lane < kXcds)
        for (int b = 0; b < nb; ++b) n += run_size(bx[b].cls, lane);
    return n;
}
// Per lane the inclusive prefix over the boxes (lane b < nb: v).
__device__ __forceinline__ uint32_t box_ends(uint32_t v)
{
    const int lane = __lane_id();
#pragma unroll
    for (int d = 1; d < kMaxBatch; d <<= 1) {
        const uint32_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// Waves of the launch on XCD p.
template <class P>
__device__ __forceinline__ uint32_t dealt_waves(uint32_t p)
{
    return (gridDim.x - p + kXcds - 1) / kXcds * P::kWaves;
}

// Persistent: each workgroup copies the table into LDS once; then its waves, each for itself, take
// the pieces of groups that are too long for one wave and after them whole groups.
// The pieces, all of much the same cost, are dealt: an eighth of the list, which is in key order,
// to each XCD's waves in turn.  (From a counter per XCD they would come one per 45 ns: 6000 of
// them, for a box of 250,007 particles, took 0.75 ms where their pairs take 0.16.)
// The whole groups lie in kXcds contiguous key ranges (neighbouring groups share sources through
// one L2).  The first of each are dealt to the waves of its XCD, one each; the others come
// from a queue per range, the own XCD's first and then what is left of the others, and a wave asks
// for its next one before it begins one.  So a small box needs no counter (all 4096 waves asking at
// once took 40 us).  Every box of a launch has the same table.
template <class P, bool MULTI>
__device__ __forceinline__ void force_body(const ForceBox *bx, int n_boxes)
{
    extern __shared__ float4 smem[];
    const int nb = MULTI ? n_boxes : 1;
    char *const lds = reinterpret_cast<char *>(smem);
    P::load_table(lds, bx[0]);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); // known to be uniform
    const uint32_t lane = __lane_id(), xcd = blockIdx.x % kXcds;
    __syncthreads();
    char *const tile = lds + P::kTilesAt + wave * P::kTileBytes;
    // the pieces: places at, at + step, .. below hi
    uint32_t ends = 0, total = bx[0].cls[kClsItems];
    if (MULTI) {
        ends = box_ends((int)lane < nb ? bx[lane].cls[kClsItems] : 0u);
        total = (uint32_t)__builtin_amdgcn_readlane((int)ends, nb - 1);
    }
    total = uni(total);
    const bool by_xcd = gridDim.x >= kXcds; // else some XCD has no workgroup
    const uint32_t hi = by_xcd ? (uint32_t)((uint64_t)total * (xcd + 1) / kXcds) : total;
    const uint32_t blocks = by_xcd ? (gridDim.x - xcd + kXcds - 1) / kXcds : gridDim.x;
    const uint32_t place = (uint32_t)wave * blocks + (by_xcd ? blockIdx.x / kXcds : blockIdx.x);
    uint32_t at = place + (by_xcd ? (uint32_t)((uint64_t)total * xcd / kXcds) : 0u);
    bool pieces = true;
    uint32_t *const ctr = bx[0].cls + P::kQueueAt;
    uint32_t size = 0, part = xcd, have = kXcds, next = 0;
    for (;;) { // one place where a group is taken, whichever way it was found
        Piece w{0, false, 0, 0, 1, 0, 0};
        Item it{0, at};
        bool dealt = false;
        if (pieces && at >= hi) {
            pieces = false;
            size = part_sizes(bx, nb);
            dealt = by_xcd && place < (uint32_t)__builtin_amdgcn_readlane((int)size, (int)xcd);
            // what is left of part p once its XCD's waves have one each
            const uint32_t p = lane_now(), w_p = by_xcd ? dealt_waves<P>(p) : 0u;
            size = p < kXcds && size > w_p ? size - w_p : 0u;
            it.k = place;
        }
        if (!pieces && !dealt) {
            uint32_t q = next;
            for (;;) {
                if (part != have) {
                    part = __ballot(size != 0) ? uni(next_part(ctr, size, part)) : kXcds;
                    if (part == kXcds) break;
                    if (lane == 0) q = atomicAdd(&ctr[part * kQueueStride], 1u);
                }
                q = uni(q);
                if (q < (uint32_t)__builtin_amdgcn_readlane((int)size, (int)part)) break;
                have = kXcds; // found empty: on to the next part that is not
            }
            if (part == kXcds) break;
            if (MULTI && part != have)
                ends = box_ends((int)lane < nb ? run_size(bx[lane].cls, part) : 0u);
            have = part;
            if (lane == 0) next = atomicAdd(&ctr[part * kQueueStride], 1u);
            it.k = uni(q + (by_xcd ? dealt_waves<P>(part) : 0u));
        } else if (MULTI && dealt)
            ends = box_ends((int)lane < nb ? run_size(bx[lane].cls, xcd) : 0u);
        if (MULTI) it = find_item(ends, nb, it.k);
        const ForceBox &B = MULTI ? bx[uni(it.box)] : bx[0];
        if (pieces) {
            const ForceItem f = B.items[it.k];
            const uint32_t ss = uni(f.seg_segs);
            w = Piece{uni(f.g), false, uni(f.chunk), ss & 0xffu, ss >> 8 & 0xffu, ss >> 16,
                      uni(f.base)};
            at += blocks * P::kWaves;
        } else {
            w.g = uni(B.cls[B.cls[kClsStarts + (dealt ? xcd : part)] + it.k]);
            w.whole = true;
        }
        P::group(tile, B, w);
    }
}

} // namespace
} // namespace tpm

// Quadrupole term of the cell entries (Section 4.1: the second-order moment of a cell, whose
// expansion must carry the spatial derivatives of the cutoff function).
//
// For a cell of mass M, centre of mass X and second moment Q = sum m s s^double about X, the
// particles' pair law F(d) = d h(r), h = g(r/eta) (r^2 + eps^2)^(-3/2), summed over the cell is,
// to second order in the offsets s,
//     M F(d) + (Q d) u + (1/2) tr(Q) d u + (1/2) (d.Q.d) d w,   u = h'/r,  w = (h'/r)'/r,
// with d = X - x_i.  The force kernels add the first term for every cell entry; this file
// adds the rest, after them, for boxes that ask for it:
//  * k_second_moments: Q per node in FP64, level by level from the leaves up (a leaf from its
//    particles, an internal node from its children by the parallel-axis theorem);
//  * k_quad_f32 for FP32 boxes, in the FP32 force kernel's units, chunks and queues: u and w from
//    a table, the list's cell entries gathered 64 at a time;
//  * k_quad_f64: one wave per group; its list's cell entries that can reach the group (gap to
//    the group's box < r_cut) are gathered into LDS 64 at a time, and the lanes add their terms to
//    the group's particles' acceleration records (small groups spread each particle's cells over
//    several lanes).
#include "force_common.hpp"

#include <cmath>
#include <vector>

namespace tpm {
namespace {

constexpr int kQuadTile64 = 64;

__device__ __forceinline__ double wrapq(double v, double L)
{
    const double h = 0.5 * L;
    if (v >= h) return v - L;
    if (v < -h) return v + L;
    return v;
}

__device__ __forceinline__ void node_second_moments(const NodeArrays &nd,
                                                    const double4 *__restrict__ ps, uint32_t u,
                                                    double *Q)
{
    const double4 cu = nd.nsrc[u]; // centre of mass, mass
    const double X = cu.x, Y = cu.y, Z = cu.z;
    double q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const uint32_t nch = nd.nchild[u];
    // as for the moments, everything is read before any of it is added (in order, zeros for what
    // there is not)
    if (nch == 0) {
        const uint32_t f = nd.first[u], n = nd.count[u];
        for (uint32_t k = 0; k < n; k += 4) {
            double4 r[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                r[j] = ps[f + (k + j < n ? k + j : k)];
                if (k + j >= n) r[j].w = 0.0;
            }
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const double dx = r[j].x - X, dy = r[j].y - Y, dz = r[j].z - Z, m = r[j].w;
                q[0] += m * dx * dx;
                q[1] += m * dy * dy;
                q[2] += m * dz * dz;
                q[3] += m * dx * dy;
                q[4] += m * dx * dz;
                q[5] += m * dy * dz;
            }
        }
    } else {
        const uint32_t cf = nd.child_first[u];
#pragma unroll
        for (uint32_t h = 0; h < 8; h += 4) {
            double4 cc[4];
            double qc[4][6];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const bool there = h + j < nch;
                const uint32_t c = cf + (there ? h + j : 0);
                cc[j] = nd.nsrc[c];
#pragma unroll
                for (int a = 0; a < 6; ++a) qc[j][a] = Q[6 * (size_t)c + a];
                if (!there) {
                    cc[j].w = 0.0;
#pragma unroll
                    for (int a = 0; a < 6; ++a) qc[j][a] = 0.0;
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const double dx = cc[j].x - X, dy = cc[j].y - Y, dz = cc[j].z - Z, m = cc[j].w;
                q[0] += qc[j][0] + m * dx * dx;
                q[1] += qc[j][1] + m * dy * dy;
                q[2] += qc[j][2] + m * dz * dz;
                q[3] += qc[j][3] + m * dx * dy;
                q[4] += qc[j][4] + m * dx * dz;
                q[5] += qc[j][5] + m * dy * dz;
            }
        }
    }
    for (int a = 0; a < 6; ++a) Q[6 * (size_t)u + a] = q[a];
}

__global__ __launch_bounds__(256) void k_second_moments(NodeArrays nd,
                                                        const double4 *__restrict__ ps,
                                                        uint32_t lo, uint32_t hi, double *Q)
{
    for (uint32_t u = lo + blockIdx.x * blockDim.x + threadIdx.x; u < hi;
         u += gridDim.x * blockDim.x)
        node_second_moments(nd, ps, u, Q);
}

// Consecutive levels of few nodes (l1 down to l0) by one workgroup, a barrier between levels.
__global__ __launch_bounds__(1024) void k_second_moments_levels(NodeArrays nd,
                                                                const double4 *__restrict__ ps,
                                                                TreeOffsets to, int l1, int l0,
                                                                double *Q)
{
    for (int l = l1; l >= l0; --l) {
        for (uint32_t u = to.off[l] + threadIdx.x; u < to.off[l + 1]; u += 1024u)
            node_second_moments(nd, ps, u, Q);
        __syncthreads();
    }
}

// FP32 boxes.  In the FP32 force kernel's units (x' = x lam / r_cut, u = |d'|^2 + c clamped to 1,
// G the pair law as a function of u) and with Q' = Q (lam / r_cut)^2 the terms are
//     (Q'd') U + (1/2) tr(Q') d' U + (d'.Q'd') d' V,   U = 2 dG/du,  V = dU/du,
// times the force's own scale.  V is piecewise quadratic and U its integral, from one set of four
// coefficients (build_quad_table).  A pair is 36 FP32 instructions and four 4-byte LDS reads (about
// 90 cycles of issue and 20 of LDS time); with both laws evaluated it was about 110 instructions.
//
// Each wave first collects its range's cell entries in an LDS queue, 128 list entries at a
// time, and gathers centre and moments for 64 cells at once: on the lists of a clustered box most
// entries are particles, and a tile per 64 list entries would be mostly empty.  Measured on
// 1,000,003 particles (theta 0.7, groups of up to 256): 0.54 ms, of which instruction issue is
// 0.3 and the rest waits for cells (80 bytes each, gathered); with a workgroup of one wave per
// group and the laws evaluated, 1.54 ms.
constexpr int kQuadWaves = 16; // per workgroup: one workgroup, four waves per SIMD
constexpr int kQuadFetch = 2;  // list entries fetched per lane and round
struct QuadCell {
    float4 a, b, c; // x', y', z', tr / 2; Q'xx, Q'yy, Q'zz, Q'xy; Q'xz, Q'yz, -, -
};

// LDS: the waves' tiles, then the four coefficient arrays at their natural addresses (bits of the
// piece's edge >> kQuadAddrShift, as in the force kernel), then the waves' queues.
constexpr uint32_t kQuadPlane = 28 * 512;
constexpr uint32_t kQuadQueues = (127u << 9) + 3u * kQuadPlane + 16u;
constexpr uint32_t kQuadQueueLen = 64 + 64 * kQuadFetch;
constexpr uint32_t kQuadLds = kQuadQueues + kQuadWaves * kQuadQueueLen * 4;
constexpr int kQuadTile = 64;
static_assert(kQuadSegBits == 7 && kQuadAddrShift == 14, "128 entries per octave: 512 bytes");
static_assert(kQuadWaves * kQuadTile * sizeof(QuadCell) <= ((127 + kTabMinExp) << 9),
              "tiles end below the table");
static_assert(kQuadPlane >= (uint32_t)(-kTabMinExp) * 512u + 4u, "planes do not overlap");
constexpr uint32_t kQuadEdgeMask = ~((1u << kQuadShift) - 1u);

typedef const __attribute__((address_space(3))) char *lds_bytes;
typedef const __attribute__((address_space(3))) float *lds_f;

// One row: a cell against two of the lane's particles.
__device__ __forceinline__ void quad_pairs(const QuadCell &s, const float *xi, const float *yi,
                                           const float *zi, float c, float *tx, float *ty,
                                           float *tz)
{
    constexpr int NP = 2;
    float dx[NP], dy[NP], dz[NP], t[NP], q0[NP], q1[NP], q2[NP], q3[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const float u = pair_u(s.a, xi[k], yi[k], zi[k], c, dx[k], dy[k], dz[k]);
        const uint32_t a = __float_as_uint(u) & kQuadEdgeMask;
        t[k] = u - __uint_as_float(a);
        uint32_t at;
        asm("v_lshrrev_b32 %0, 14, %1" : "=v"(at) : "v"(a));
        const lds_bytes q = (lds_bytes)at;
        q0[k] = *(lds_f)q;
        q1[k] = *(lds_f)(q + kQuadPlane);
        q2[k] = *(lds_f)(q + 2 * kQuadPlane);
        q3[k] = *(lds_f)(q + 3 * kQuadPlane);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        // V = q1 + t (q2 + t q3),  U = q0 + t (q1 + (t/2) (q2 + (2t/3) q3))
        const float V = fmaf(fmaf(q3[k], t[k], q2[k]), t[k], q1[k]);
        const float h = fmaf(q3[k], t[k] * (2.0f / 3.0f), q2[k]);
        const float U = fmaf(fmaf(h, 0.5f * t[k], q1[k]), t[k], q0[k]);
        const float qx = fmaf(s.b.x, dx[k], fmaf(s.b.w, dy[k], s.c.x * dz[k]));
        const float qy = fmaf(s.b.w, dx[k], fmaf(s.b.y, dy[k], s.c.y * dz[k]));
        const float qz = fmaf(s.c.x, dx[k], fmaf(s.c.y, dy[k], s.b.z * dz[k]));
        const float dq = fmaf(dx[k], qx, fmaf(dy[k], qy, dz[k] * qz));
        const float sc = fmaf(dq, V, s.a.w * U);
        tx[k] = fmaf(qx, U, fmaf(sc, dx[k], tx[k]));
        ty[k] = fmaf(qy, U, fmaf(sc, dy[k], ty[k]));
        tz[k] = fmaf(qz, U, fmaf(sc, dz[k], tz[k]));
    }
    __builtin_amdgcn_sched_barrier(0);
}

struct PolicyQuad {
    static constexpr int kWaves = kQuadWaves, kTilesAt = 0,
                         kTileBytes = kQuadTile * (int)sizeof(QuadCell);
    static constexpr uint32_t kQueueAt = kClsQuadQueue;
    static constexpr bool kAdd = true;
    using Frame = FrameF32;

    static __device__ __forceinline__ void load_table(char *lds, const ForceBox &B)
    {
        const QuadTable qt = B.qt;
        float *const t = reinterpret_cast<float *>(lds);
        for (uint32_t i = threadIdx.x; i < qt.entries; i += blockDim.x)
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                t[(qt.base + q * kQuadPlane) / 4 + i] = qt.coef[q * qt.entries + i];
    }

    template <int K>
    static __device__ __forceinline__ uint32_t chunk_sums(char *tile_bytes, int S, uint32_t n_i,
                                                          uint32_t f, const uint32_t *list,
                                                          uint32_t j0, uint32_t j1,
                                                          const ForceBox &B, const Frame &F,
                                                          double *ax, double *ay, double *az)
    {
        extern __shared__ float4 smem[];
        QuadCell *const tile = reinterpret_cast<QuadCell *>(tile_bytes);
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        uint32_t *const queue =
            reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(smem) + kQuadQueues) +
            (uint32_t)wave * kQuadQueueLen;
        const double4 *__restrict__ const ps = B.ps;
        const double4 *__restrict__ const nsrc = B.nd.nsrc;
        const double *__restrict__ const moments = B.moments;
        const double to_q = ldexp(F.inv * F.inv, -B.qt.scale_exp);
        const float c = in_vgpr(F.c);
        const int lane = __lane_id();
        const int J = 64 / S, lgJ = 31 - __builtin_clz(J);
        const int slot = lane & (S - 1), stream = lane / S;
        constexpr uint32_t kRound = 64 * kQuadFetch;
        uint32_t ent[kQuadFetch];
        uint32_t jb = j0, nq = 0;
        if (j0 < j1) fetch_entries<kQuadFetch>(list, j0, j1, ent);
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
        for (;;) {
            while (nq < 64 && jb < j1) {
#pragma unroll
                for (int r = 0; r < kQuadFetch; ++r) {
                    const bool cell = jb + (uint32_t)(r * 64 + lane) < j1 && (ent[r] & kCellTag);
                    const uint64_t m = __ballot(cell);
                    if (cell)
                        queue[nq + __builtin_amdgcn_mbcnt_hi(
                                       (uint32_t)(m >> 32),
                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                            ent[r] & ~kCellTag;
                    nq += (uint32_t)__popcll(m);
                }
                jb += kRound;
                if (jb < j1) fetch_entries<kQuadFetch>(list, jb, j1, ent);
            }
            nq = uni(nq);
            if (!nq) break;
            // the last 64 (or fewer) of the queue
            const uint32_t take = nq < 64 ? nq : 64;
            wave_lds_sync();
            const bool mine = (uint32_t)lane < take;
            const uint32_t cell = queue[nq - take + (mine ? (uint32_t)lane : 0u)];
            nq -= take;
            const float4 v = rel_f32(nsrc[cell], F);
            const double *q = moments + 6 * (size_t)cell;
            const double q0 = q[0] * to_q, q1 = q[1] * to_q, q2 = q[2] * to_q, q3 = q[3] * to_q,
                         q4 = q[4] * to_q, q5 = q[5] * to_q;
            const float w0 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(v.x - C.c0), C.h0), 0.f, 1.f);
            const float w1 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(v.y - C.c1), C.h1), 0.f, 1.f);
            const float w2 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(v.z - C.c2), C.h2), 0.f, 1.f);
            const bool keep = mine && fmaf(w0, w0, fmaf(w1, w1, w2 * w2)) < C.thr;
            const uint64_t mk = __ballot(keep);
            const int nt = (int)__popcll(mk);
            if (keep) {
                QuadCell o;
                o.a = make_float4(v.x, v.y, v.z, (float)(0.5 * (q0 + q1 + q2)));
                o.b = make_float4((float)q0, (float)q1, (float)q2, (float)q3);
                o.c = make_float4((float)q4, (float)q5, 0.f, 0.f);
                tile[__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u))] = o;
            }
            // the last row's padding adds zero
            const int e = nt + lane;
            if (lane < J && e < ((nt + J - 1) & ~(J - 1)))
                tile[e].a = tile[e].b = tile[e].c = make_float4(0.f, 0.f, 0.f, 0.f);
            wave_lds_sync();
            const int steps = (nt + J - 1) >> lgJ; // the same on every lane
            float tx[K], ty[K], tz[K];
#pragma unroll
            for (int k = 0; k < K; ++k) tx[k] = ty[k] = tz[k] = 0.f;
            const QuadCell *ts = tile + stream;
            for (int t = 0; t < steps; ++t) {
                const QuadCell s = *ts;
                ts += J;
#pragma unroll
                for (int k = 0; k < K; k += 2)
                    quad_pairs(s, xi + k, yi + k, zi + k, c, tx + k, ty + k, tz + k);
            }
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < K; ++k) {
                ax[k] += (double)tx[k];
                ay[k] += (double)ty[k];
                az[k] += (double)tz[k];
            }
        }
        return 0;
    }

    static __device__ __forceinline__ void group(char *tile, const ForceBox &B, const Piece &w)
    {
        const GroupRead R(B, w.g);
        finish_group<PolicyQuad>(tile, B, w, R, frame_f32(B, R));
    }
};
static_assert(kQuadTile % 16 == 0, "J divides a tile");

__global__ __launch_bounds__(64 * kQuadWaves, 4) void k_quad_f32(ForceBox box)
{
    force_body<PolicyQuad, false>(&box, 1);
}

// FP64 boxes.
// g(R) of eq. (2) and its first two derivatives, each times 140: the expanded first branch,
// and the second branch as (2 - R)^5 P(R), P = 7R^3 + 22R^2 + 10R + 4, differentiated as a
// product so that nothing cancels near R = 2.
__device__ __forceinline__ void g_derivs140(double R, double &g, double &g1, double &g2)
{
    if (R < 1.0) {
        const double R2 = R * R;
        g = 140.0 - R2 * R * (224.0 + R2 * (-224.0 + R * (70.0 + R * (48.0 - 21.0 * R))));
        g1 = -R2 * (672.0 + R2 * (-1120.0 + R * (420.0 + R * (336.0 - 168.0 * R))));
        g2 = -R * (1344.0 + R2 * (-4480.0 + R * (2100.0 + R * (2016.0 - 1176.0 * R))));
    } else if (R < 2.0) {
        const double v = 2.0 - R, v2 = v * v, v3 = v2 * v;
        const double P = 4.0 + R * (10.0 + R * (22.0 + 7.0 * R));
        const double P1 = 10.0 + R * (44.0 + 21.0 * R);
        const double P2 = 44.0 + 42.0 * R;
        g = v3 * v2 * P;
        g1 = v3 * v * (v * P1 - 5.0 * P);
        g2 = v3 * (20.0 * P - 10.0 * v * P1 + v2 * P2);
    } else {
        g = g1 = g2 = 0.0;
    }
}

// The second branch alone, for pairs known to have R >= 1 (clamped to zero from R = 2 on).
__device__ __forceinline__ void g_derivs140_far(double R, double &g, double &g1, double &g2)
{
    const double v = R < 2.0 ? 2.0 - R : 0.0, v2 = v * v, v3 = v2 * v;
    const double P = 4.0 + R * (10.0 + R * (22.0 + 7.0 * R));
    const double P1 = 10.0 + R * (44.0 + 21.0 * R);
    const double P2 = 44.0 + 42.0 * R;
    g = v3 * v2 * P;
    g1 = v3 * v * (v * P1 - 5.0 * P);
    g2 = v3 * (20.0 * P - 10.0 * v * P1 + v2 * P2);
}

__device__ __forceinline__ double rsqrt_f64q(double x) { return 1.0 / sqrt(x); }

// A cell as the kernel uses it: centre of mass relative to the group's cube centre, half the
// trace of the moments, and the six moments.
struct alignas(32) QuadCell64 {
    double x, y, z, htr, q0, q1, q2, q3, q4, q5, pad0, pad1;
};

// One wave per group.  The lanes are S = 64 / J particle slots times J cell phases, J the
// largest power of two with n_g J <= 64 kQuadK: lane (slot, phase) takes up to kQuadK particles
// (slot, slot + S, ...) and every J-th cell of each tile, so a cell read from LDS serves
// several particles and small groups still fill the wave.  The J partial sums of a particle
// are added with lane shuffles at the end.
constexpr int kQuadK = 4;

template <int REC64>
__global__ __launch_bounds__(64) void k_quad_f64(NodeArrays nd, GroupArrays gr, uint32_t n_groups,
                                             const uint64_t *__restrict__ off,
                                             const uint32_t *__restrict__ len,
                                             const uint32_t *__restrict__ entries,
                                             const double4 *__restrict__ ps,
                                             const uint32_t *__restrict__ pidx,
                                             const double *__restrict__ Q, ForceParams fp,
                                             void *rec)
{
    __shared__ QuadCell64 tile[kQuadTile64];
    const uint32_t g = xcd_block(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x;
    if (g >= n_groups) return;
    const uint32_t n_g = gr.count[g], f = gr.first[g];
    const uint64_t b = off[g], Lg = len[g];
    const double L = fp.L;
    const double xg0 = gr.xgx[g], xg1 = gr.xgy[g], xg2 = gr.xgz[g];
    const double cg0 = gr.cgx[g], cg1 = gr.cgy[g], cg2 = gr.cgz[g];
    const double hg0 = gr.hgx[g], hg1 = gr.hgy[g], hg2 = gr.hgz[g];
    const double half_side = 0.5 * ldexp(L, -(int)nd.level[gr.node[g]]);
    // one image per entry (relative to the cube centre) serves every particle of the group
    // unless half the group cube plus r_cut reaches L/2; then each pair takes its own (only
    // the FP64 path: the FP32 force call refuses such boxes)
    const bool pair_wrap = !(half_side + sqrt(fp.rc2) < 0.5 * L);
    const double inv_eta = fp.inv_eta, eps2 = fp.eps2;
    const double inv_eta2 = inv_eta * inv_eta;
    int lj = 0; // log2 J
    while (lj < 6 && (uint64_t)n_g << (lj + 1) <= 64u * kQuadK) ++lj;
    const int J = 1 << lj, S = 64 >> lj;
    const int slot = lane & (S - 1), ph = lane >> (6 - lj);
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    for (uint32_t ib = 0; ib < n_g; ib += (uint32_t)S * kQuadK) {
        double xi[kQuadK], yi[kQuadK], zi[kQuadK], ax_[kQuadK], ay_[kQuadK], az_[kQuadK];
#pragma unroll
        for (int k = 0; k < kQuadK; ++k) {
            const uint32_t i = ib + slot + k * S;
            xi[k] = yi[k] = zi[k] = 0.0;
            ax_[k] = ay_[k] = az_[k] = 0.0;
            if (i < n_g) {
                const double4 r = ps[f + i];
                xi[k] = wrapq(r.x - xg0, L);
                yi[k] = wrapq(r.y - xg1, L);
                zi[k] = wrapq(r.z - xg2, L);
            }
        }
        // particles this wave holds in the block: how many of the kQuadK slots are used
        const uint32_t rest = n_g - ib;
        const int kk = rest >= (uint32_t)S * kQuadK ? kQuadK : (int)((rest + S - 1) / S);
        for (uint64_t jb = 0; jb < Lg; jb += 64) {
            const uint64_t j = jb + lane;
            bool keep = false, far = false;
            QuadCell64 v{};
            if (j < Lg) {
                const uint32_t e = entries[b + j];
                if (e & kCellTag) {
                    const uint32_t c = e & ~kCellTag;
                    const double4 r = nd.nsrc[c];
                    double w0 = fabs(wrapq(r.x - cg0, L)) - hg0;
                    double w1 = fabs(wrapq(r.y - cg1, L)) - hg1;
                    double w2 = fabs(wrapq(r.z - cg2, L)) - hg2;
                    w0 = w0 > 0.0 ? w0 : 0.0;
                    w1 = w1 > 0.0 ? w1 : 0.0;
                    w2 = w2 > 0.0 ? w2 : 0.0;
                    const double gap2 = w0 * w0 + w1 * w1 + w2 * w2;
                    keep = gap2 < fp.rc2;
                    far = gap2 >= fp.eta * fp.eta; // every pair has R >= 1
                    const double *q = Q + 6 * (size_t)c;
                    // the moments carry the 1/140 of g and its derivatives below
                    const double k = 1.0 / 140.0;
                    v = QuadCell64{wrapq(r.x - xg0, L),
                                    wrapq(r.y - xg1, L),
                                    wrapq(r.z - xg2, L),
                                    0.5 * (q[0] + q[1] + q[2]) * k,
                                    q[0] * k,
                                    q[1] * k,
                                    q[2] * k,
                                    q[3] * k,
                                    q[4] * k,
                                    q[5] * k,
                                    0.0,
                                    0.0};
                }
            }
            // near cells from the front of the tile, far ones from the back
            const uint64_t mn = __ballot(keep && !far), mf = __ballot(keep && far);
            if (keep) {
                if (far)
                    tile[kQuadTile64 - 1 - __popcll(mf & lt)] = v;
                else
                    tile[__popcll(mn & lt)] = v;
            }
            const int nn = __popcll(mn), nf = __popcll(mf);
            __syncthreads();
            auto pair = [&](const QuadCell64 &s, bool far_cell, int k) {
                double dx = s.x - xi[k], dy = s.y - yi[k], dz = s.z - zi[k];
                if (pair_wrap) {
                    dx = wrapq(dx, L);
                    dy = wrapq(dy, L);
                    dz = wrapq(dz, L);
                }
                // pairs at or beyond r_cut get g = g' = g'' = 0 from the polynomials (R >= 2)
                const double r2 = dx * dx + dy * dy + dz * dz;
                const double ir = r2 > 0.0 ? rsqrt_f64q(r2) : 0.0, r = r2 * ir, R = r * inv_eta;
                double gv, g1, g2;
                if (far_cell)
                    g_derivs140_far(R, gv, g1, g2);
                else
                    g_derivs140(R, gv, g1, g2);
                const double is = rsqrt_f64q(r2 + eps2), is2 = is * is;
                const double q3 = is2 * is, p5 = q3 * is2, s7 = p5 * is2;
                const double ir2 = ir * ir;
                // 140 u = 140 h'/r and 140 w = 140 (h'/r)'/r (the moments carry 1/140)
                const double A = g1 * inv_eta * ir;
                const bool live = r2 > 0.0; // a cell never sits on a particle; kept safe
                const double ur = live ? A * q3 - 3.0 * gv * p5 : 0.0;
                const double wr =
                    live ? (g2 * inv_eta2 - A) * ir2 * q3 - 6.0 * A * p5 + 15.0 * gv * s7 : 0.0;
                const double qx = s.q0 * dx + s.q3 * dy + s.q4 * dz;
                const double qy = s.q3 * dx + s.q1 * dy + s.q5 * dz;
                const double qz = s.q4 * dx + s.q5 * dy + s.q2 * dz;
                const double sc = s.htr * ur + 0.5 * (dx * qx + dy * qy + dz * qz) * wr;
                ax_[k] += qx * ur + sc * dx;
                ay_[k] += qy * ur + sc * dy;
                az_[k] += qz * ur + sc * dz;
            };
            for (int t = ph; t < nn; t += J) {
                const QuadCell64 s = tile[t];
#pragma unroll
                for (int k = 0; k < kQuadK; ++k)
                    if (k < kk) pair(s, false, k);
            }
            for (int t = kQuadTile64 - nf + ph; t < kQuadTile64; t += J) {
                const QuadCell64 s = tile[t];
#pragma unroll
                for (int k = 0; k < kQuadK; ++k)
                    if (k < kk) pair(s, true, k);
            }
            __syncthreads();
        }
        // add the J phases of each particle (lanes slot, slot + S, slot + 2S, ...)
#pragma unroll
        for (int k = 0; k < kQuadK; ++k) {
            for (int d = S; d < 64; d <<= 1) {
                ax_[k] += __shfl_xor(ax_[k], d, 64);
                ay_[k] += __shfl_xor(ay_[k], d, 64);
                az_[k] += __shfl_xor(az_[k], d, 64);
            }
            const uint32_t i = ib + slot + k * S;
            if (i < n_g && ph == 0) {
                const uint32_t o = pidx[f + i];
                if (REC64) {
                    double4 *const r = (double4 *)rec + o;
                    r->x += ax_[k];
                    r->y += ay_[k];
                    r->z += az_[k];
                } else {
                    float4 *const r = (float4 *)rec + o;
                    r->x += float(ax_[k]);
                    r->y += float(ay_[k]);
                    r->z += float(az_[k]);
                }
            }
        }
    }
}

} // namespace

void launch_second_moments(NodeArrays nd, const double4 *ps, const TreeOffsets &to, int max_level,
                           double *Q, hipStream_t s)
{
    for (int l = max_level; l >= 0;) {
        const uint32_t lo = to.off[l], hi = to.off[l + 1];
        int l0 = l;
        while (l0 >= 0 && to.off[l0 + 1] - to.off[l0] <= kFewNodes) --l0;
        if (l - l0 >= 2) {
            k_second_moments_levels<<<1, 1024, 0, s>>>(nd, ps, to, l, l0 + 1, Q);
            l = l0;
            continue;
        }
        const uint32_t b = (hi - lo + 255) / 256;
        if (b) k_second_moments<<<b < 65535 ? b : 65535, 256, 0, s>>>(nd, ps, lo, hi, Q);
        --l;
    }
}

void build_quad_table(double eps_over_rcut, double c, std::vector<float> &coef, QuadTable &qt)
{
    const double e2 = eps_over_rcut * eps_over_rcut, lam2 = 1.0 - c;
    const int kc = (int)std::lround(std::log2(c));
    const uint32_t pieces = (uint32_t)(-kc) << kQuadSegBits;
    qt.entries = pieces + 1;
    qt.base = (uint32_t)(127 + kc) << (23 - kQuadAddrShift);
    // V's quadratic term is about 60 e2^-5.5: in float's range for every eps with the factor
    qt.scale_exp = e2 < std::ldexp(1.0, -20) ? -32 : 0;
    const double sigma = std::ldexp(1.0, qt.scale_exp);
    // U and V at the s of u
    auto laws = [&](double u, double &U, double &V) {
        const double s = (u - c) / lam2, R = 2.0 * std::sqrt(s), R2 = R * R;
        double g, a, b; // g, g' / R and g'' of eq. (2)
        if (R < 1.0) {
            g = 1.0 + R2 * R * (-1.6 + R2 * (1.6 + R * (-0.5 + R * (-12.0 / 35 + 0.15 * R))));
            a = R * (-4.8 + R2 * (8.0 + R * (-3.0 + R * (-2.4 + 1.2 * R))));
            b = R * (-9.6 + R2 * (32.0 + R * (-15.0 + R * (-14.4 + 8.4 * R))));
        } else {
            const double v = 4.0 * ((1.0 - u) / lam2) / (2.0 + R), v3 = v * v * v; // 2 - R
            const double P = 4.0 + R * (10.0 + R * (22.0 + 7.0 * R));
            const double P1 = 10.0 + R * (44.0 + 21.0 * R), P2 = 44.0 + 42.0 * R;
            g = v3 * v * v * P / 140.0;
            a = v3 * v * (v * P1 - 5.0 * P) / 140.0 / R;
            b = v3 * (20.0 * P - 10.0 * v * P1 + v * v * P2) / 140.0;
        }
        // dg/ds = 2 a, d2g/ds2 = 4 (b - a) / R^2 = (b - a) / s
        const double x = s + e2, f = 1.0 / (x * std::sqrt(x)), f1 = -1.5 * f / x,
                     f2 = -2.5 * f1 / x;
        const double G1 = 2.0 * a * f + g * f1;
        const double G2 = (b - a) / s * f + 4.0 * a * f1 + g * f2;
        U = sigma * 2.0 * G1 / lam2;
        V = sigma * 2.0 * G2 / (lam2 * lam2);
    };
    coef.assign(4 * (size_t)qt.entries, 0.f); // the entry of u = 1 stays zero
    const double third = 0.86602540378443864676; // cos(pi / 6)
    for (uint32_t k = 0; k < pieces; ++k) {
        const int e = kc + (int)(k >> kQuadSegBits);
        const double w = std::ldexp(1.0 / (1 << kQuadSegBits), e);
        const double lo = std::ldexp(1.0, e) + (k & ((1u << kQuadSegBits) - 1u)) * w;
        // V through its values at the three Chebyshev nodes m +- h third, m; U through its value at m
        const double h = 0.5 * w, d = h * third;
        double Um, Vm, U0, Vl, Vr;
        laws(lo + h - d, U0, Vl);
        laws(lo + h + d, U0, Vr);
        laws(lo + h, Um, Vm);
        const double b1 = (Vr - Vl) / (2.0 * d), b2 = (Vr + Vl - 2.0 * Vm) / (2.0 * d * d);
        const double v0 = Vm - h * (b1 - h * b2), v1 = b1 - 2.0 * h * b2; // in t = (u - m) + h
        coef[0 * qt.entries + k] =
            (float)(Um - h * (v0 + h * (0.5 * v1 + h * b2 / 3.0)));
        coef[1 * qt.entries + k] = (float)v0;
        coef[2 * qt.entries + k] = (float)v1;
        coef[3 * qt.entries + k] = (float)b2;
    }
}

void launch_quad(const ForceBox &box, int fp64, int n_cu, hipStream_t s)
{
    const uint32_t n_groups = box.n_groups;
    if (!n_groups) return;
    if (!fp64) {
        const uint32_t cap = (uint32_t)n_cu, work = n_groups + box.n_items;
        k_quad_f32<<<work < cap ? work : cap, 64 * kQuadWaves, kQuadLds, s>>>(box);
    } else if (box.rec64)
        k_quad_f64<1><<<n_groups, 64, 0, s>>>(box.nd, box.gr, n_groups, box.off, box.len,
                                              box.entries, box.ps, box.pidx, box.moments, box.fp,
                                              box.rec);
    else
        k_quad_f64<0><<<n_groups, 64, 0, s>>>(box.nd, box.gr, n_groups, box.off, box.len,
                                              box.entries, box.ps, box.pidx, box.moments, box.fp,
                                              box.rec);
}

} // namespace tpm

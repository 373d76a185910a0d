// Short-range pair force in FP64 over the interaction lists (Section 2.1 eq. 1, eq. 2; Plummer
// softening of Section 2.4), in the work split of the FP32 kernel (force_common.hpp): positions
// relative to x_g are FP64 differences (nearest image once per entry, or per pair when the
// group's cube plus r_cut reaches half the box), and the pair law is
//   * read from a table (force_table64.cpp) where the softening allows one and the box is large
//     enough to be worth making it: G(s) = G_a (1 + r)^5 with r a polynomial of degree 6 in
//     t = u - a, u = 2^18 (c + (1 - c) s) clamped to 2^18, a the piece's lower edge, which is u with
//     its low mantissa bits cleared, so t is exact; or
//   * evaluated pair by pair otherwise: (r^2 + eps^2)^(-1/2) and r^(-1) from the hardware
//     estimate refined by two Newton steps, and eq. (2) in a form with no cancellation: for R < 1,
//     g = 1 + R^3 (-8/5 + R^2 (8/5 + R (-1/2 + R (-12/35 + 3R/20)))), and for R >= 1,
//     g = max(2 - R, 0)^5 (7R^3 + 22R^2 + 10R + 4) / 140.
//
// A pair from the table is 26 FP64 and 9 other vector instructions (about 140 cycles of issue at
// 4.4 per FP64 instruction) and 48 bytes from LDS; evaluated, it is about 50 FP64 instructions, two
// of them 17-cycle estimates.  |r| is at most 0.008 but for the last pieces before the cutoff, so
// its coefficients need not be as exact as G_a: the two highest, whose share of G is at most 6e-10,
// are floats and are summed in FP32 (an error of 3e-17).  A pair's error, of 300,000 each at eps /
// r_cut from 2^-11 to 3 and without that of u: RMS 0.8e-16 for R < 1.9, largest 3.7e-16; as p^5
// with three coefficients in FP32 it was 2.4 to 4.6e-16 and 2.3e-15 below R = 1, and pair by pair
// it is 1.6 to 2.7e-16 and 1.3e-15.  The coefficients are read power by power (4- and 8-byte reads:
// a 16-byte read costs two to three times as much per byte once the lanes spread over pieces).
// Measured on the 128^3 clustered box (2.1 million particles, kernel trace): 3.2 ms, LDS and vector
// units both busy three quarters of it or more; as p^5 it was 3.0, pair by pair, with one group a
// wave, 8.2.
#include "force_common.hpp"

namespace tpm {
namespace {

constexpr int kTile64 = 128;
constexpr int kRounds64 = kTile64 / 64;
constexpr uint32_t kPlaneHi = (kTab64Entries * 8u + 15u) / 16u * 16u;
constexpr uint32_t kPlaneLo = (kTab64Entries * 4u + 15u) / 16u * 16u;
constexpr uint32_t kLoAt = kTab64F64 * kPlaneHi;
constexpr uint32_t kTable64 = kLoAt + (kTab64Deg + 1 - kTab64F64) * kPlaneLo;
static_assert(kTab64Deg == 6 && kTab64F64 == 5, "the Horner steps below");
static_assert(kTable64 <= 81920, "LDS: the table below half of a compute unit's 160 KB");

constexpr double kTop64 = 1 << kTab64Exp; // u at s = 1

struct Frame64 {
    bool wrap;      // coordinates need the nearest image
    bool pair_wrap; // and pairs too
    double xg0, xg1, xg2, L;
    double k2, c;         // table: u = r^2 k2 + c
    double eps2, inv_eta; // pair by pair
    float inv, len;       // 1 / r_cut and L / r_cut, for the cull
    double scale;
};

__device__ __forceinline__ double wrapd(double v, double L)
{
    double h = 0.5 * L;
    if (v >= h) return v - L;
    if (v < -h) return v + L;
    return v;
}

__device__ __forceinline__ double4 rel_f64(const double4 r, const Frame64 &F)
{
    const double x = r.x - F.xg0, y = r.y - F.xg1, z = r.z - F.xg2;
    if (F.wrap) return make_double4(wrapd(x, F.L), wrapd(y, F.L), wrapd(z, F.L), r.w);
    return make_double4(x, y, z, r.w);
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

__device__ __forceinline__ double g_p3m_f64(double R)
{
    const double R2 = R * R;
    double p = fma(0.15, R, -12.0 / 35.0);
    p = fma(p, R, -0.5);
    p = fma(p, R, 1.6);
    p = fma(p, R2, -1.6);
    const double g1 = fma(p, R2 * R, 1.0);
    const double u = fmax(2.0 - R, 0.0);
    const double u2 = u * u;
    const double c = fma(fma(fma(0.05, R, 22.0 / 140.0), R, 10.0 / 140.0), R, 4.0 / 140.0);
    return R < 1.0 ? g1 : u2 * u2 * u * c;
}

// Culls and packs one tile (as load_tile_f32; the cull in FP32 units of r_cut with its margin).
// With pair_wrap the distance along an axis is the nearest image's.
__device__ __forceinline__ int load_tile_f64(double4 *tile, const uint32_t *ent, uint32_t jb,
                                             uint32_t je, int J, const NodeArrays &nd,
                                             const Frame64 &F, const ChunkBox &C)
{
    const int lane = __lane_id();
    int n = 0;
    double4 srcs[kRounds64];
#pragma unroll
    for (int r = 0; r < kRounds64; ++r) {
        const double4 *base = (ent[r] & kCellTag) ? nd.nsrc : nd.psrc;
        srcs[r] = base[ent[r] & ~kCellTag];
    }
#pragma unroll
    for (int r = 0; r < kRounds64; ++r) {
        const uint32_t j = jb + (uint32_t)(r * 64 + lane);
        const double4 v = rel_f64(srcs[r], F);
        float d0 = (float)v.x * F.inv - C.c0, d1 = (float)v.y * F.inv - C.c1,
              d2 = (float)v.z * F.inv - C.c2;
        if (F.pair_wrap) {
            d0 -= F.len * rintf(d0 / F.len);
            d1 -= F.len * rintf(d1 / F.len);
            d2 -= F.len * rintf(d2 / F.len);
        }
        const float w0 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(d0), C.h0), 0.f, 1.f);
        const float w1 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(d1), C.h1), 0.f, 1.f);
        const float w2 = __builtin_amdgcn_fmed3f(fmaf(0.5f, fabsf(d2), C.h2), 0.f, 1.f);
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
    const int e = n + lane;
    if (lane < J && e < ((n + J - 1) & ~(J - 1))) tile[e] = make_double4(0.0, 0.0, 0.0, 0.0);
    return __builtin_amdgcn_readfirstlane(n);
}
static_assert(kTile64 % 16 == 0, "J divides a tile");

typedef const __attribute__((address_space(3))) char *lds_bytes;
typedef const __attribute__((address_space(3))) double *lds_d;
typedef const __attribute__((address_space(3))) float *lds_f;

// NP of the lane's particles against one source.  Table: all reads of the NP pairs first, then
// the arithmetic on them.
template <bool TABLE, bool PW, int NP>
__device__ __forceinline__ void pairs_f64(const double4 s, const double *xi, const double *yi,
                                          const double *zi, const Frame64 &F, uint32_t base,
                                          double *ax, double *ay, double *az)
{
    double dx[NP], dy[NP], dz[NP], r2[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        dx[k] = s.x - xi[k];
        dy[k] = s.y - yi[k];
        dz[k] = s.z - zi[k];
        if (PW) {
            dx[k] = wrapd(dx[k], F.L);
            dy[k] = wrapd(dy[k], F.L);
            dz[k] = wrapd(dz[k], F.L);
        }
        r2[k] = fma(dx[k], dx[k], fma(dy[k], dy[k], dz[k] * dz[k]));
    }
    if (TABLE) {
        double t[NP], q0[NP], q1[NP], q2[NP], q3[NP], q4[NP];
        float q5[NP], q6[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double u = fmin(fma(r2[k], F.k2, F.c), kTop64);
            const uint32_t a = (uint32_t)__double2hiint(u) & 0xffffc000u;
            t[k] = u - __hiloint2double((int)a, 0);
            const uint32_t b = a - base;
            const lds_bytes h = (lds_bytes)(b >> 11), l = (lds_bytes)(b >> 12);
            q0[k] = *(lds_d)h;
            q1[k] = *(lds_d)(h + kPlaneHi);
            q2[k] = *(lds_d)(h + 2 * kPlaneHi);
            q3[k] = *(lds_d)(h + 3 * kPlaneHi);
            q4[k] = *(lds_d)(h + 4 * kPlaneHi);
            q5[k] = *(lds_f)(l + kLoAt);
            q6[k] = *(lds_f)(l + kLoAt + kPlaneLo);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double z = (double)fmaf(q6[k], (float)t[k], q5[k]);
            const double r =
                fma(fma(fma(fma(z, t[k], q4[k]), t[k], q3[k]), t[k], q2[k]), t[k], q1[k]) * t[k];
            // (1 + r)^5 - 1
            const double y = r * fma(r, fma(r, fma(r, r + 5.0, 10.0), 10.0), 5.0);
            const double f = fma(q0[k], y, q0[k]) * s.w;
            ax[k] = fma(f, dx[k], ax[k]);
            ay[k] = fma(f, dy[k], ay[k]);
            az[k] = fma(f, dz[k], az[k]);
        }
        __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double is = rsqrt_f64(r2[k] + F.eps2);
            const double R = r2[k] * rsqrt_f64(r2[k]) * F.inv_eta;
            double f = s.w * g_p3m_f64(R) * (is * is * is);
            f = r2[k] > 0.0 ? f : 0.0; // a pair at zero separation adds nothing
            ax[k] = fma(f, dx[k], ax[k]);
            ay[k] = fma(f, dy[k], ay[k]);
            az[k] = fma(f, dz[k], az[k]);
        }
    }
}

// steps rows of a stream (row stride J sources) against the lane's K particles, two at a time.
template <bool TABLE, bool PW, int K>
__device__ __forceinline__ void tile_pass_f64(const double4 *ts, int steps, int J,
                                              const double *xi, const double *yi,
                                              const double *zi, const Frame64 &F, uint32_t base,
                                              double *ax, double *ay, double *az)
{
    for (int t = 0; t < steps; ++t) {
        const double4 s = *ts;
        ts += J;
#pragma unroll
        for (int k = 0; k < K; k += 2)
            pairs_f64<TABLE, PW, 2>(s, xi + k, yi + k, zi + k, F, base, ax + k, ay + k, az + k);
    }
}

// Waves per workgroup: 16 around one copy of the table (68 KB, and 64 KB of tiles), four per
// SIMD; without the table the tiles alone are in LDS.
template <bool TABLE>
struct Policy64 {
    static constexpr int kWaves = 16, kTilesAt = TABLE ? (int)kTable64 : 0,
                         kTileBytes = kTile64 * 32;
    static constexpr uint32_t kQueueAt = kClsQueue;
    static constexpr bool kAdd = false;
    static constexpr uint32_t kLds = kTilesAt + kWaves * kTileBytes;
    using Frame = Frame64;

    static __device__ __forceinline__ void load_table(char *lds, const ForceBox &B)
    {
        if (!TABLE) return;
        for (uint32_t i = threadIdx.x; i < kTab64Entries; i += blockDim.x) {
#pragma unroll
            for (uint32_t q = 0; q < kTab64F64; ++q)
                reinterpret_cast<double *>(lds + q * kPlaneHi)[i] =
                    B.tab64_hi[q * kTab64Entries + i];
#pragma unroll
            for (uint32_t q = 0; q < kTab64Deg + 1 - kTab64F64; ++q)
                reinterpret_cast<float *>(lds + kLoAt + q * kPlaneLo)[i] =
                    B.tab64_lo[q * kTab64Entries + i];
        }
    }

    template <int K>
    static __device__ __forceinline__ uint32_t chunk_sums(char *tile_bytes, int S, uint32_t n_i,
                                                          uint32_t f, const uint32_t *list,
                                                          uint32_t j0, uint32_t j1,
                                                          const ForceBox &B, const Frame &F,
                                                          double *ax, double *ay, double *az)
    {
        double4 *const tile = reinterpret_cast<double4 *>(tile_bytes);
        const double4 *__restrict__ const ps = B.ps;
        const int lane = __lane_id();
        const int J = 64 / S, lgJ = 31 - __builtin_clz(J);
        const int slot = lane & (S - 1), stream = lane / S;
        uint32_t kept = 0;
        uint32_t ent[kRounds64];
        if (j0 < j1) fetch_entries<kRounds64>(list, j0, j1, ent);
        double4 pos[K];
        load_chunk<K>(ps, f, n_i, slot, S, pos);
        double xi[K], yi[K], zi[K];
        ChunkBox C;
        {
            float fx[K], fy[K], fz[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double4 v = rel_f64(pos[k], F);
                xi[k] = v.x;
                yi[k] = v.y;
                zi[k] = v.z;
                fx[k] = (float)v.x * F.inv;
                fy[k] = (float)v.y * F.inv;
                fz[k] = (float)v.z * F.inv;
                ax[k] = ay[k] = az[k] = 0.0;
            }
            C = chunk_box<K>(fx, fy, fz, S);
        }
        // the table's first edge, kept in a vector register
        uint32_t base = (uint32_t)(1023 - kTab64Oct + kTab64Exp) << 20;
        asm("" : "+v"(base));
        for (uint32_t jb = j0; jb < j1; jb += kTile64) {
            const int nt = load_tile_f64(tile, ent, jb, j1, J, B.nd, F, C);
            kept += (uint32_t)nt;
            wave_lds_sync();
            if (jb + kTile64 < j1) fetch_entries<kRounds64>(list, jb + kTile64, j1, ent);
            const int steps = (nt + J - 1) >> lgJ; // the same on every lane
            if (F.pair_wrap)
                tile_pass_f64<TABLE, true, K>(tile + stream, steps, J, xi, yi, zi, F, base, ax,
                                              ay, az);
            else
                tile_pass_f64<TABLE, false, K>(tile + stream, steps, J, xi, yi, zi, F, base, ax,
                                               ay, az);
            wave_lds_sync();
        }
        return kept;
    }

    static __device__ __forceinline__ void group(char *tile, const ForceBox &B, const Piece &w)
    {
        const GroupRead R(B, w.g);
        const uint32_t node = B.gr.node[w.g];
        const ForceParams &fp = B.fp;
        const ForceUnits &U = B.units;
        Frame F;
        F.wrap = R.wraps(B);
        const double half_side = 0.5 * ldexp(fp.L, -(int)uni((uint32_t)B.nd.level[node]));
        F.pair_wrap = __ballot(!(half_side + fp.rc < 0.5 * fp.L)) != 0;
        F.L = fp.L;
        F.xg0 = uni(R.xg[0]);
        F.xg1 = uni(R.xg[1]);
        F.xg2 = uni(R.xg[2]);
        F.k2 = U.k2;
        F.c = kTop64 / (1u << kTab64Oct);
        F.eps2 = fp.eps2;
        F.inv_eta = fp.inv_eta;
        F.inv = U.inv_f;
        F.len = U.len_f;
        F.scale = U.scale;
        finish_group<Policy64>(tile, B, w, R, F);
    }
};

template <bool TABLE>
__global__ __launch_bounds__(64 * Policy64<TABLE>::kWaves, 4) void k_force_f64(ForceBox box)
{
    force_body<Policy64<TABLE>, false>(&box, 1);
}

} // namespace

void launch_force_f64(const ForceBox &box, int n_cu, hipStream_t s)
{
    if (!box.n_groups) return;
    const uint32_t cap = (uint32_t)n_cu, work = box.n_groups + box.n_items;
    const uint32_t blocks = work < cap ? work : cap;
    constexpr int threads = 64 * Policy64<true>::kWaves;
    if (box.tab64_hi)
        k_force_f64<true><<<blocks, threads, Policy64<true>::kLds, s>>>(box);
    else
        k_force_f64<false><<<blocks, threads, Policy64<false>::kLds, s>>>(box);
}

} // namespace tpm

// Particle-mesh (PM) long-range force on an N^3 periodic mesh (Section 2.2 step 1): TSC
// mass assignment, the potential by FFT with the Green's function of the long-range part of
// the split (the complement of eq. 2), a fourth-order difference for the mesh force and TSC
// interpolation back to the particles.
//
// Mesh layout: point (x, y, z) at (x N + y) N + z, z contiguous; N a power of two.
//  * assignment by owner cells: the mesh is cut into cells of 8^3 points (tree cells, so a
//    cell's particles are contiguous in key order); a workgroup sums a chunk of one cell's
//    particles into the cell's 11^3 box in LDS and stores the box to its own slot, then one
//    workgroup per cell adds, for each of its points, the slot words that cover it.  Masses
//    are 64-bit fixed point and every sum is a fixed set of integer adds, so the mesh is the
//    same on every run; there are no global atomics;
//  * FFT: five passes over bundles of lines (4096 values at most) of the half spectrum kx <= N/2
//    of the real mesh: x forward (reading the fixed-point masses, two real lines as one complex
//    line), y forward, z forward + Green's function + z inverse in one kernel, y inverse,
//    x inverse (writing the real potential).  Bundles along x and y are neighbouring lines in z,
//    so a load of one element row is contiguous; bundles along z are contiguous rows;
//  * mesh force and interpolation: over the assignment's chunks, the potential around the cell
//    is read into LDS, the fourth-order central differences on the cell's 11^3 box formed there,
//    and each particle's 27 points read from those; the 16-byte result goes to the particle's
//    slot in the caller's order through the sort permutation (a scattered write); k_pm_split
//    then writes the three output arrays contiguously.
#include "common.hpp"

namespace tpm {
namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b)
{
    return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 csub(double2 a, double2 b)
{
    return make_double2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ double2 wide(float2 a) { return make_double2(a.x, a.y); }
__device__ __forceinline__ float2 narrow(double2 a) { return make_float2((float)a.x, (float)a.y); }

// Nearest mesh point of coordinate x for inv_h = N / L.  The product is rounded on its own
// (no contraction into the add), so every kernel finds the same point for the same x.
__device__ __forceinline__ int nearest(double x, double inv_h)
{
#pragma clang fp contract(off)
    return (int)floor(x * inv_h + 0.5);
}

// TSC cloud along one axis: the nearest mesh point (returned) and the weights of the points
// before it, at it and after it.
__device__ __forceinline__ int tsc(double x, double inv_h, double w[3])
{
#pragma clang fp contract(off)
    const double u = x * inv_h;
    const double f = floor(u + 0.5);
    const double d = u - f;
    w[0] = 0.5 * (0.5 - d) * (0.5 - d);
    w[1] = 0.75 - d * d;
    w[2] = 0.5 * (0.5 + d) * (0.5 + d);
    return (int)f;
}

// Fixed-point scale for the mesh masses: a power of two S with n m_max S < 2^62, so no sum
// of contributions can overflow 64 bits.
__device__ __forceinline__ double pm_scale(unsigned long long mmax_bits, int64_t n)
{
    const double t = (double)n * __longlong_as_double((long long)mmax_bits);
    return ldexp(1.0, 61 - ilogb(t));
}

// Mass assignment, owner by owner.  The mesh is cut into cells of kCellPts^3 points, which
// are the tree cells of level l_c = log2(N / kCellPts): a particle's cell c (per axis) is its
// key's prefix, and its nearest mesh point i0 = floor(x N / L + 1/2) lies in [8c, 8c + 8] (the
// key's product x 2^21 / L and x N / L differ from the exact values by a relative 2^-52 at
// most, far below the half point of margin; at x -> L the key is clamped and i0 = N, still in
// range).  So the particles of a cell, contiguous in key order, touch only the kBox^3 points
// [8c - 1, 8c + 9] of the cell's box.  One workgroup sums a chunk of a cell's particles into
// its box in LDS and writes the box to the chunk's own slot with plain stores; then each mesh
// point sums the slot words that cover it (one or two cells per axis, every chunk of each) and
// writes its mesh word.  No global atomics, and every sum is a fixed set of integer adds, so
// the mesh is the same on every run.  A thread sums the 27 contributions of a run of its
// particles with the same nearest point in registers (fixed point, rounded once per run and
// point).
constexpr int kCellPts = 8;
constexpr int kBox = kCellPts + 3;             // 11 points per axis
constexpr int kBoxWords = kBox * kBox * kBox;  // 1331
constexpr int kAssignThreads = 256;

// Particles per workgroup at most.  250,007 clustered particles on a 64^3 mesh are 570 workgroups
// of up to 4096, whose fullest decide: assignment and interpolation take 28 us each, 17 with
// workgroups of up to 1024; 16.8 million have enough with 4096, and halves of that only add slots
// to the gather (0.16 to 0.18 ms).  Calls with 1024 and with 4096, clustered: 500,000 particles on
// 128^3 149 and 162 us, 2 million 204 and 203, 4.1 million 323 and 326; on 256^3 4.3 million 823 and
// 822, 6 million 903 and 892, 12 million 1134 and 1077.  Uniform, 4.1 million on 128^3: 297 and 285.
static uint32_t cell_chunk(int64_t n) { return n < (1 << 22) ? 1024u : 4096u; }

__device__ __forceinline__ uint32_t spread3_10(uint32_t v) // 10 bits -> every third bit
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}
__device__ __forceinline__ uint32_t compact3_10(uint32_t v)
{
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030c30c3u;
    v = (v | (v >> 4)) & 0x0300f00fu;
    v = (v | (v >> 8)) & 0x030000ffu;
    v = (v | (v >> 16)) & 0x3ffu;
    return v;
}
// The Morton index of cell (cx, cy, cz), in the keys' bit order (x above y above z).
__device__ __forceinline__ uint32_t cell_index(uint32_t cx, uint32_t cy, uint32_t cz)
{
    return (spread3_10(cx) << 2) | (spread3_10(cy) << 1) | spread3_10(cz);
}

// cell_start[m] = the first particle (key order) of Morton cell m, m = 0 .. ncells; the
// cell of a key is key >> sh.
__global__ __launch_bounds__(256) void k_pm_cells(const uint64_t *__restrict__ key, int64_t n,
                                                  int sh, uint32_t ncells,
                                                  uint32_t *__restrict__ cell_start)
{
    const uint32_t m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m > ncells) return;
    int64_t lo = 0, hi = n; // first i with key[i] >> sh >= m
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((key[mid] >> sh) < (uint64_t)m)
            lo = mid + 1;
        else
            hi = mid;
    }
    cell_start[m] = (uint32_t)lo;
}

// items[m] = chunks of cell m (exclusive prefix taken afterwards).
__global__ __launch_bounds__(256) void k_pm_cell_items(const uint32_t *__restrict__ cell_start,
                                                       uint32_t ncells, uint32_t chunk,
                                                       uint32_t *__restrict__ items)
{
    const uint32_t m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= ncells) return;
    const uint32_t c = cell_start[m + 1] - cell_start[m];
    items[m] = (c + chunk - 1) / chunk;
}

// The cell whose chunks include chunk `item`: the last m with item_start[m] <= item.  Every lane
// of the wave probes one place of the range, so 32768 cells take three memory latencies and not
// fifteen.
__device__ __forceinline__ uint32_t item_cell(const uint32_t *__restrict__ item_start,
                                              uint32_t ncells, uint32_t item)
{
    const uint32_t lane = __lane_id();
    uint32_t lo = 0, len = ncells;
    while (len > 1) {
        const uint32_t step = (len + 63) / 64, at = lane * step;
        const bool before = at < len && item_start[lo + at] <= item;
        const uint32_t k = (uint32_t)__popcll(__ballot(before)) - 1u; // lane 0 always is
        lo += k * step;
        len = min(step, len - k * step);
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// One workgroup per chunk (grid: an upper bound on the chunks; the rest leave).
__global__ __launch_bounds__(kAssignThreads) void k_pm_assign(
    const double4 *__restrict__ ps, int64_t n, int N, double inv_h,
    const unsigned long long *__restrict__ mx, const uint32_t *__restrict__ cell_start,
    const uint32_t *__restrict__ item_start, uint32_t ncells, uint32_t chunk,
    unsigned long long *__restrict__ slots)
{
    __shared__ unsigned long long box[kBoxWords];
    const uint32_t item = blockIdx.x;
    if (item >= item_start[ncells]) return; // the same for the whole workgroup
    const uint32_t m = item_cell(item_start, ncells, item);
    const uint32_t first = cell_start[m] + (item - item_start[m]) * chunk;
    const uint32_t end = min(cell_start[m + 1], first + chunk);
    const int ox = 8 * (int)compact3_10(m >> 2) - 1, oy = 8 * (int)compact3_10(m >> 1) - 1,
              oz = 8 * (int)compact3_10(m) - 1;
    for (int t = threadIdx.x; t < kBoxWords; t += kAssignThreads) box[t] = 0ull;
    __syncthreads();
    const double S = pm_scale(*mx, n);
    const uint32_t per = (end - first + kAssignThreads - 1) / kAssignThreads;
    const uint32_t i0 = first + threadIdx.x * per, i1 = min(end, i0 + per);
    double acc[27];
#pragma unroll
    for (int j = 0; j < 27; ++j) acc[j] = 0.0;
    int cx = 0, cy = 0, cz = 0;
    bool open = false;
    auto add_run = [&]() {
        const int bx = cx - 1 - ox, by = cy - 1 - oy, bz = cz - 1 - oz; // in [0, 8]
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const unsigned long long v = __double2ull_rn(acc[(a * 3 + b) * 3 + c]);
                    if (v) atomicAdd(&box[((bx + a) * kBox + (by + b)) * kBox + (bz + c)], v);
                }
    };
    for (uint32_t i = i0; i < i1; ++i) {
        const double4 p = ps[i];
        double wx[3], wy[3], wz[3];
        const int ix = tsc(p.x, inv_h, wx), iy = tsc(p.y, inv_h, wy), iz = tsc(p.z, inv_h, wz);
        if (open && (ix != cx || iy != cy || iz != cz)) {
            add_run();
#pragma unroll
            for (int j = 0; j < 27; ++j) acc[j] = 0.0;
        }
        cx = ix;
        cy = iy;
        cz = iz;
        open = true;
        const double ms = p.w * S;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const double wab = ms * wx[a] * wy[b];
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[(a * 3 + b) * 3 + c] += wab * wz[c];
            }
    }
    if (open) add_run();
    __syncthreads();
    unsigned long long *dst = slots + (size_t)item * kBoxWords;
    for (int t = threadIdx.x; t < kBoxWords; t += kAssignThreads) dst[t] = box[t];
}

// One workgroup per cell, one thread per mesh point of the cell: the sum of the slot words of
// every chunk of every cell whose box covers the point (its own cell, and the neighbour on
// the low side for the cell's first two planes, on the high side for its last plane, per
// axis): at most two cells per axis, whose first chunks are read together.  The 27 neighbours'
// chunk ranges are read into LDS once.  256^3 mesh, 16.8 million clustered particles: 0.29 ms
// with a loop over the 27 cells and one read in flight a thread, 0.16 as it is.
__global__ __launch_bounds__(kCellPts * kCellPts * kCellPts) void k_pm_gather(
    int N, const uint32_t *__restrict__ item_start, const unsigned long long *__restrict__ slots,
    unsigned long long *__restrict__ mass)
{
    __shared__ uint32_t rng[27][2];
    const int ncell = N / kCellPts, cm = ncell - 1;
    // each XCD takes a contiguous slab of cells, whose neighbours' slots its L2 then shares
    const int cell = (int)xcd_block(blockIdx.x, gridDim.x);
    const int cx = cell / (ncell * ncell), cy = (cell / ncell) % ncell, cz = cell % ncell;
    const int t = threadIdx.x;
    if (t < 27) {
        const int dx = t / 9 - 1, dy = (t / 3) % 3 - 1, dz = t % 3 - 1;
        const uint32_t m = cell_index((uint32_t)((cx + dx) & cm), (uint32_t)((cy + dy) & cm),
                                      (uint32_t)((cz + dz) & cm));
        rng[t][0] = item_start[m];
        rng[t][1] = item_start[m + 1];
    }
    __syncthreads();
    const int x0 = t >> 6, y0 = (t >> 3) & 7, z0 = t & 7; // point within the cell
    auto other = [](int p) { return p < 2 ? -1 : p == kCellPts - 1 ? 1 : 0; };
    const int ox = other(x0), oy = other(y0), oz = other(z0); // 0: only its own cell covers it
    unsigned long long v[8];
    uint32_t next[8], end[8], word[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) { // own or other cell per axis
        const int dx = j & 4 ? ox : 0, dy = j & 2 ? oy : 0, dz = j & 1 ? oz : 0;
        const bool cover = (!(j & 4) || ox) && (!(j & 2) || oy) && (!(j & 1) || oz);
        const int k = ((dx + 1) * 3 + (dy + 1)) * 3 + (dz + 1);
        next[j] = rng[k][0];
        end[j] = cover ? rng[k][1] : 0u;
        word[j] = (uint32_t)(((x0 - 8 * dx + 1) * kBox + (y0 - 8 * dy + 1)) * kBox +
                             (z0 - 8 * dz + 1));
        const bool some = next[j] < end[j];
        v[j] = slots[some ? (size_t)next[j] * kBoxWords + word[j] : 0];
        if (!some) v[j] = 0ull;
    }
    unsigned long long sum = 0ull;
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += v[j];
#pragma unroll
    for (int j = 0; j < 8; ++j) // cells of more than one chunk
#pragma unroll 4
        for (uint32_t it = next[j] + 1; it < end[j]; ++it)
            sum += slots[(size_t)it * kBoxWords + word[j]];
    mass[((size_t)(8 * cx + x0) * N + (size_t)(8 * cy + y0)) * N + (size_t)(8 * cz + z0)] = sum;
}

// ---------------------------------------------------------------- FFT on bundles of lines
//
// A line of N = 2^LOGN points is transformed by N / 16 threads with 16 points each in registers, in
// one to three steps of radix 16, 8 or 4 (Stockham's ordering: natural in, natural out); between
// steps the points change places through LDS once.  Step s with radix R after steps of product
// NS: butterfly j takes points j + r N / R, times exp(-2 pi i r (j mod NS) / (NS R)), to points
// (j / NS) NS R + (j mod NS) + r NS.
// The points are double in registers, and float wherever they are stored (in LDS between the steps,
// in memory between the passes): with float butterflies the half spectrum's rounding, which no
// longer averages over k and -k, made the force of a uniform box on a fine mesh 8 % less exact
// than the full complex transform had it; as it is, that is twice as exact (300,007 particles,
// 256^3 mesh: 3.3e-7 RMS against 6.8e-7, and 6.4e-7 for the full one).
// N = 256, five passes from the masses to the potential: 0.152 ms for 0.75 GB read and written,
// 0.140 with float butterflies; with radix-2 stages through LDS on the full complex mesh 0.59.

template <int LOGN>
struct Radix; // the steps' radices, 0 where there is none
template <> struct Radix<4> { static constexpr int a = 16, b = 0, c = 0; };
template <> struct Radix<5> { static constexpr int a = 8, b = 4, c = 0; };
template <> struct Radix<6> { static constexpr int a = 8, b = 8, c = 0; };
template <> struct Radix<7> { static constexpr int a = 16, b = 8, c = 0; };
template <> struct Radix<8> { static constexpr int a = 16, b = 16, c = 0; };
template <> struct Radix<9> { static constexpr int a = 8, b = 8, c = 8; };
template <> struct Radix<10> { static constexpr int a = 16, b = 8, c = 8; };

// Lines per workgroup; threads per line; LDS points, with a row left free after every 16 (points
// 16 apart would fall on the same banks).
template <int LOGN>
struct Lines {
    static constexpr int N = 1 << LOGN, B = N >= 256 ? 4096 / N : 16, T = N / 16;
    static constexpr int P = B < N / 2 ? B : N / 2; // pairs of real lines per workgroup
    static constexpr int kRows = N + N / 16;
};

// Times exp(-+ i pi / 2).
template <bool INV>
__device__ __forceinline__ double2 quarter(double2 v)
{
    return INV ? make_double2(-v.y, v.x) : make_double2(v.y, -v.x);
}

template <bool INV>
__device__ __forceinline__ void dft4(double2 &a, double2 &b, double2 &c, double2 &d)
{
    const double2 s = cadd(a, c), m = csub(a, c), t = cadd(b, d), u = quarter<INV>(csub(b, d));
    a = cadd(s, t);
    b = cadd(m, u);
    c = csub(s, t);
    d = csub(m, u);
}

// Discrete Fourier transform of R points in registers, natural order in and out.
template <int R, bool INV>
__device__ __forceinline__ void dft(double2 *v)
{
    constexpr double kH = 0.70710678118654752440; // cos(pi / 4)
    constexpr double sg = INV ? 1.0 : -1.0;
    if (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else if (R == 8) {
        double2 e[4], o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            e[i] = cadd(v[i], v[i + 4]);
            o[i] = csub(v[i], v[i + 4]);
        }
        o[1] = cmul(o[1], make_double2(kH, sg * kH));
        o[2] = quarter<INV>(o[2]);
        o[3] = cmul(o[3], make_double2(-kH, sg * kH));
        dft4<INV>(e[0], e[1], e[2], e[3]);
        dft4<INV>(o[0], o[1], o[2], o[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = e[i];
            v[2 * i + 1] = o[i];
        }
    } else {
        constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173; // pi / 8
        const double2 w[10] = {{1.0, 0.0},   {c1, sg * s1},  {kH, sg * kH}, {s1, sg * c1},
                              {0.0, sg},    {-s1, sg * c1}, {-kH, sg * kH}, {-c1, sg * s1},
                              {-1.0, 0.0},  {-c1, -sg * s1}};
        double2 y[4][4]; // y[i][k]: over points i, i + 4, i + 8, i + 12
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int k = 0; k < 4; ++k) y[i][k] = v[i + 4 * k];
            dft4<INV>(y[i][0], y[i][1], y[i][2], y[i][3]);
#pragma unroll
            for (int k = 1; k < 4; ++k)
                if (i) y[i][k] = i * k == 4 ? quarter<INV>(y[i][k]) : cmul(y[i][k], w[i * k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            dft4<INV>(y[0][k], y[1][k], y[2][k], y[3][k]);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[k + 4 * i] = y[i][k];
        }
    }
}

// Calls f(e, v) for the thread's points as a step of radix R reads them (and the last one leaves
// them), or as a step of radix R after NS leaves them.
template <int LOGN, int R, class F>
__device__ __forceinline__ void for_inputs(double2 *v, int jt, F f)
{
#pragma unroll
    for (int q = 0; q < 16 / R; ++q)
#pragma unroll
        for (int r = 0; r < R; ++r)
            f(jt + q * Lines<LOGN>::T + r * (Lines<LOGN>::N / R), v[q * R + r]);
}
template <int LOGN, int R, int NS, class F>
__device__ __forceinline__ void for_outputs(double2 *v, int jt, F f)
{
#pragma unroll
    for (int q = 0; q < 16 / R; ++q) {
        const int j = jt + q * Lines<LOGN>::T;
#pragma unroll
        for (int r = 0; r < R; ++r) f((j / NS) * (NS * R) + j % NS + r * NS, v[q * R + r]);
    }
}

template <int LOGN, int R, int NS, bool INV>
__device__ __forceinline__ void step(double2 *v, int jt, const double2 *tw)
{
    constexpr int N = 1 << LOGN;
#pragma unroll
    for (int q = 0; q < 16 / R; ++q) {
        const int k = (jt + q * Lines<LOGN>::T) % NS;
        if (NS > 1) {
#pragma unroll
            for (int r = 1; r < R; ++r) {
                double2 w = tw[r * k * (N / (NS * R))];
                if (INV) w.y = -w.y;
                v[q * R + r] = cmul(v[q * R + r], w);
            }
        }
        dft<R, INV>(v + q * R);
    }
}

// The points through LDS (at(e): where point e of the thread's line lies), from the order in which
// the step of radix R after NS leaves them to that in which one of radix R2 reads them.
template <int LOGN, int R, int NS, int R2, class AT>
__device__ __forceinline__ void exchange(double2 *v, int jt, float2 *buf, AT at)
{
    for_outputs<LOGN, R, NS>(v, jt, [&](int e, double2 &x) { buf[at(e)] = narrow(x); });
    __syncthreads();
    for_inputs<LOGN, R2>(v, jt, [&](int e, double2 &x) { x = wide(buf[at(e)]); });
    __syncthreads();
}

// The whole line: v as a step of radix A (C from the back with REV) reads it; left as the last
// step leaves it.  REV takes the radices in reverse, so it can follow a plain one in registers.
template <int LOGN, bool INV, bool REV, class AT>
__device__ __forceinline__ void fft_line(double2 *v, int jt, float2 *buf, const double2 *tw,
                                         AT at)
{
    using X = Radix<LOGN>;
    constexpr int n = X::c ? 3 : X::b ? 2 : 1;
    constexpr int r0 = !REV ? X::a : n == 3 ? X::c : n == 2 ? X::b : X::a;
    constexpr int r1 = n < 2 ? 4 : n == 2 ? (REV ? X::a : X::b) : X::b; // 4: not used
    constexpr int r2 = n < 3 ? 4 : REV ? X::a : X::c;
    step<LOGN, r0, 1, INV>(v, jt, tw);
    if (n >= 2) {
        exchange<LOGN, r0, 1, r1>(v, jt, buf, at);
        step<LOGN, r1, r0, INV>(v, jt, tw);
    }
    if (n >= 3) {
        exchange<LOGN, r1, r0, r2>(v, jt, buf, at);
        step<LOGN, r2, r0 * r1, INV>(v, jt, tw);
    }
}
template <int LOGN>
struct Ends { // radices of the first and the last step
    using X = Radix<LOGN>;
    static constexpr int first = X::a, last = X::c ? X::c : X::b ? X::b : X::a;
};

// exp(-2 pi i k / N), k < N, from the table's first half.
template <int LOGN>
__device__ __forceinline__ void load_twiddles(double2 *tw_s, const double2 *tw)
{
    constexpr int N = 1 << LOGN;
    for (int k = threadIdx.x; k < N; k += blockDim.x) {
        const double2 w = tw[k & (N / 2 - 1)];
        tw_s[k] = k < N / 2 ? w : make_double2(-w.x, -w.y);
    }
}

// Forward along x, masses (fixed point, scaled by 1/S) to the half spectrum kx <= N / 2.  The real
// lines of z and z + 1 are transformed as one complex line C; theirs are (C(k) + C(N-k)*) / 2 and
// (C(k) - C(N-k)*) / 2i.
template <int LOGN>
__global__ __launch_bounds__(Lines<LOGN>::P *Lines<LOGN>::T) void k_fft_x_forward(
    const unsigned long long *__restrict__ mass, const unsigned long long *__restrict__ mx,
    int64_t n_part, float2 *__restrict__ grid, const double2 *__restrict__ tw)
{
    using D = Lines<LOGN>;
    constexpr int N = D::N, P = D::P;
    __shared__ float2 buf[D::kRows * P];
    __shared__ double2 tw_s[N];
    load_twiddles<LOGN>(tw_s, tw);
    const int l = threadIdx.x % P, jt = threadIdx.x / P;
    const int y = blockIdx.x / (N / (2 * P)), z0 = (blockIdx.x % (N / (2 * P))) * 2 * P;
    const double inv_s = 1.0 / pm_scale(*mx, n_part);
    auto at = [&](int e) { return (e + (e >> 4)) * P + l; };
    double2 v[16];
    for_inputs<LOGN, Ends<LOGN>::first>(v, jt, [&](int e, double2 &x) {
        const ulonglong2 m2 =
            *reinterpret_cast<const ulonglong2 *>(mass + ((size_t)e * N + y) * N + z0 + 2 * l);
        x = make_double2((double)m2.x * inv_s, (double)m2.y * inv_s);
    });
    __syncthreads();
    fft_line<LOGN, false, false>(v, jt, buf, tw_s, at);
    for_inputs<LOGN, Ends<LOGN>::last>(v, jt, [&](int e, double2 &x) { buf[at(e)] = narrow(x); });
    __syncthreads();
    for (int k = jt; k <= N / 2; k += D::T) {
        const float2 c = buf[at(k)], d = buf[at((N - k) & (N - 1))];
        *reinterpret_cast<float4 *>(grid + ((size_t)k * N + y) * N + z0 + 2 * l) =
            make_float4(0.5f * (c.x + d.x), 0.5f * (c.y - d.y), 0.5f * (c.y + d.y),
                        0.5f * (d.x - c.x));
    }
}

// Inverse along x, from the half spectrum to the real potential, two lines at a time again.
template <int LOGN>
__global__ __launch_bounds__(Lines<LOGN>::P *Lines<LOGN>::T) void k_fft_x_inverse(
    const float2 *__restrict__ grid, float *__restrict__ phi, const double2 *__restrict__ tw)
{
    using D = Lines<LOGN>;
    constexpr int N = D::N, P = D::P;
    __shared__ float2 buf[D::kRows * P];
    __shared__ double2 tw_s[N];
    load_twiddles<LOGN>(tw_s, tw);
    const int l = threadIdx.x % P, jt = threadIdx.x / P;
    const int y = blockIdx.x / (N / (2 * P)), z0 = (blockIdx.x % (N / (2 * P))) * 2 * P;
    auto at = [&](int e) { return (e + (e >> 4)) * P + l; };
    for (int k = jt; k <= N / 2; k += D::T) {
        const float4 g =
            *reinterpret_cast<const float4 *>(grid + ((size_t)k * N + y) * N + z0 + 2 * l);
        if (k == 0 || k == N / 2) { // real, but for rounding
            buf[at(k)] = make_float2(g.x, g.z);
        } else {
            buf[at(k)] = make_float2(g.x - g.w, g.y + g.z);
            buf[at(N - k)] = make_float2(g.x + g.w, g.z - g.y);
        }
    }
    __syncthreads();
    double2 v[16];
    for_inputs<LOGN, Ends<LOGN>::first>(v, jt, [&](int e, double2 &x) { x = wide(buf[at(e)]); });
    __syncthreads();
    fft_line<LOGN, true, false>(v, jt, buf, tw_s, at);
    for_inputs<LOGN, Ends<LOGN>::last>(v, jt, [&](int e, double2 &x) {
        *reinterpret_cast<float2 *>(phi + ((size_t)e * N + y) * N + z0 + 2 * l) = narrow(x);
    });
}

// Along y in the plane of one kx, B neighbouring lines in z.
template <int LOGN, bool INV>
__global__ __launch_bounds__(Lines<LOGN>::B *Lines<LOGN>::T) void k_fft_y(
    float2 *__restrict__ grid, const double2 *__restrict__ tw)
{
    using D = Lines<LOGN>;
    constexpr int N = D::N, B = D::B;
    __shared__ float2 buf[D::kRows * B];
    __shared__ double2 tw_s[N];
    load_twiddles<LOGN>(tw_s, tw);
    const int l = threadIdx.x % B, jt = threadIdx.x / B;
    float2 *const line =
        grid + (size_t)(blockIdx.x / (N / B)) * N * N + (blockIdx.x % (N / B)) * B + l;
    auto at = [&](int e) { return (e + (e >> 4)) * B + l; };
    double2 v[16];
    for_inputs<LOGN, Ends<LOGN>::first>(v, jt,
                                        [&](int e, double2 &x) { x = wide(line[(size_t)e * N]); });
    __syncthreads();
    fft_line<LOGN, INV, false>(v, jt, buf, tw_s, at);
    for_inputs<LOGN, Ends<LOGN>::last>(v, jt,
                                       [&](int e, double2 &x) { line[(size_t)e * N] = narrow(x); });
}

// z forward, times the Green's function, z inverse, for B rows (kx, ky = q0 + l).  The forward
// transform leaves the points in registers where the inverse with its radices reversed reads
// them.  green is the octant table, index (fx H + fy) H + fz with f = min(k, N - k), H = N/2 + 1.
template <int LOGN>
__global__ __launch_bounds__(Lines<LOGN>::B *Lines<LOGN>::T) void k_fft_z_green(
    float2 *__restrict__ grid, const double2 *__restrict__ tw, const float *__restrict__ green)
{
    using D = Lines<LOGN>;
    constexpr int N = D::N, B = D::B, H = N / 2 + 1;
    __shared__ float2 buf[D::kRows * B];
    __shared__ double2 tw_s[N];
    load_twiddles<LOGN>(tw_s, tw);
    const int l = threadIdx.x / D::T, jt = threadIdx.x % D::T;
    const int kx = blockIdx.x / (N / B), ky = (blockIdx.x % (N / B)) * B + l;
    float2 *const line = grid + ((size_t)kx * N + ky) * N;
    const float *const g = green + ((size_t)kx * H + (ky <= N / 2 ? ky : N - ky)) * H;
    auto at = [&](int e) { return l * D::kRows + e + (e >> 4); };
    double2 v[16];
    for_inputs<LOGN, Ends<LOGN>::first>(v, jt, [&](int e, double2 &x) { x = wide(line[e]); });
    __syncthreads();
    fft_line<LOGN, false, false>(v, jt, buf, tw_s, at);
    for_inputs<LOGN, Ends<LOGN>::last>(v, jt, [&](int e, double2 &x) {
        const double gk = g[e <= N / 2 ? e : N - e];
        x.x *= gk;
        x.y *= gk;
    });
    fft_line<LOGN, true, true>(v, jt, buf, tw_s, at);
    for_inputs<LOGN, Ends<LOGN>::first>(v, jt, [&](int e, double2 &x) { line[e] = narrow(x); });
}

// Fourier transform of the S2 cloud of radius eta at x = k eta (Hockney & Eastwood's shape):
// 12 (2 - 2 cos x - x sin x) / x^4, by its Taylor series where the closed form cancels.
__device__ __forceinline__ double s2_hat(double x)
{
    if (x < 0.2) {
        const double x2 = x * x;
        return 1.0 - x2 / 15.0 + x2 * x2 / 560.0 - x2 * x2 * x2 / 37800.0;
    }
    double sn, cs;
    sincos(x, &sn, &cs);
    const double x2 = x * x;
    return 12.0 * (2.0 - 2.0 * cs - x * sn) / (x2 * x2);
}

// Green's function octant table and twiddles.  G(k) = -4 pi S^(k eta)^2 / (k^2 W(k)^2 L^3):
// the long-range potential of a unit mass (the force between two S2 clouds of radius eta,
// whose complement is eq. 2) over the TSC window W = prod sinc^3(k_a h / 2) divided out for
// both the assignment and the interpolation, and 1/L^3 of the inverse transform; G(0) = 0.
// tw[k] = exp(-2 pi i k / N), k < N/2.
__global__ __launch_bounds__(256) void k_pm_green(int N, double L, double eta,
                                                  float *__restrict__ green,
                                                  double2 *__restrict__ tw)
{
    const int H = N / 2 + 1;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (t < (size_t)N / 2) {
        double sn, cs;
        sincospi(2.0 * (double)t / N, &sn, &cs);
        tw[t] = make_double2(cs, -sn);
    }
    if (t >= (size_t)H * H * H) return;
    const int fz = (int)(t % H), fy = (int)((t / H) % H), fx = (int)(t / ((size_t)H * H));
    const double kf = 2.0 * M_PI / L, h = L / N;
    const int f[3] = {fx, fy, fz};
    double k2 = 0.0, W = 1.0;
    for (int a = 0; a < 3; ++a) {
        const double k = kf * f[a];
        k2 += k * k;
        const double x = 0.5 * k * h;
        const double sc = f[a] ? sin(x) / x : 1.0;
        W *= sc * sc * sc;
    }
    if (k2 == 0.0) {
        green[t] = 0.0f;
        return;
    }
    const double S = s2_hat(sqrt(k2) * eta);
    green[t] = (float)(-4.0 * M_PI * S * S / (k2 * W * W * L * L * L));
}

// Mesh force and its TSC interpolation to each particle, written to stage[idx[i]] =
// (ax, ay, az, 0), i.e. already in the caller's order (k_pm_split then writes the three arrays
// contiguously).  One workgroup per chunk of a cell's particles (the chunks of the
// assignment).  The potential of the cell's kBox^3 points, [8c - 1, 8c + 9] per axis, and of two
// more on each side along one axis is read into LDS; from it the force there,
//     F_a = -[(2/3)(phi(i+1) - phi(i-1)) - (1/12)(phi(i+2) - phi(i-2))] / h,
// and each particle's 27 points come from that.  The weights and the order of the sums are those
// of a plain per-particle gather.
// 256^3 mesh, 16.8 million clustered particles: 0.55 ms, of which the boxes take 0.2 and the
// particles 0.35, half of that for scattering their 16-byte records (with the records in key
// order 0.39 in all; stored around the caches 0.92); with the force mesh written out and read
// back, 0.77.  The three components are arrays of their own: a 16-byte read per lane takes
// two to three times the LDS time of three 4-byte ones once the lanes spread over points.
constexpr int kPhi = kBox + 4; // points per axis of the potential
__global__ __launch_bounds__(kAssignThreads) void k_pm_interp(
    const double4 *__restrict__ ps, int N, double inv_h, const float *__restrict__ phi,
    const uint32_t *__restrict__ idx, float4 *__restrict__ stage,
    const uint32_t *__restrict__ cell_start, const uint32_t *__restrict__ item_start,
    uint32_t ncells, uint32_t chunk)
{
    // the force takes the potential's place: 16 KB, so eight workgroups fit a compute unit
    __shared__ float lds[3 * kBoxWords];
    static_assert(3 * kBoxWords >= kPhi * kPhi * kPhi, "the potential fits");
    float *const pot = lds, *const fx = lds, *const fy = lds + kBoxWords, *const fz = fy + kBoxWords;
    // an XCD takes runs of 32 chunks (cells in Morton order): the chunks of one cell and its
    // neighbours then read their boxes through one L2.  With one run per XCD over the whole grid,
    // whose end has no chunks, the XCDs' shares differ: 578 us at 256^3 against 549 (557 in plain
    // order, 562 with one run each over the chunks alone, 558 with runs of 8).
    const uint32_t item = xcd_run<32>(blockIdx.x, gridDim.x);
    if (item >= item_start[ncells]) return; // the same for the whole workgroup
    const uint32_t m = item_cell(item_start, ncells, item);
    const uint32_t first = cell_start[m] + (item - item_start[m]) * chunk;
    const uint32_t end = min(cell_start[m + 1], first + chunk);
    const int ox = 8 * (int)compact3_10(m >> 2) - 1, oy = 8 * (int)compact3_10(m >> 1) - 1,
              oz = 8 * (int)compact3_10(m) - 1;
    const int mask = N - 1;
    {
        // sixteen lanes to a row of fifteen points, sixteen rows (one and a fifteenth of a plane)
        // at a time
        static_assert(kPhi == 15 && kAssignThreads == 256, "a lane more than a row has points");
        const int bz = threadIdx.x & 15, z = (oz - 2 + bz) & mask;
        const int rim_z = bz < 2 || bz >= kBox + 2;
        int bx = 0, by = threadIdx.x >> 4;
        if (by == kPhi) {
            by = 0;
            bx = 1;
        }
        for (; bx < kPhi;) {
            const int rim = (bx < 2 || bx >= kBox + 2) + (by < 2 || by >= kBox + 2) + rim_z;
            if (rim <= 1 && bz < kPhi)
                pot[(bx * kPhi + by) * kPhi + bz] =
                    phi[((uint32_t)((ox - 2 + bx) & mask) * (uint32_t)N +
                         (uint32_t)((oy - 2 + by) & mask)) * (uint32_t)N + (uint32_t)z];
            ++bx;
            if (++by == kPhi) {
                by = 0;
                ++bx;
            }
        }
    }
    // the first particle is under way while the force is formed
    uint32_t i = first + threadIdx.x;
    double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
    uint32_t o = 0;
    if (i < end) {
        p = ps[i];
        o = idx[i];
    }
    __syncthreads();
    const float fh = (float)inv_h;
    constexpr int kPer = (kBoxWords + kAssignThreads - 1) / kAssignThreads;
    float f[kPer][3];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int t = threadIdx.x + k * kAssignThreads;
        if (t < kBoxWords) {
            const int bx = t / (kBox * kBox), by = (t / kBox) % kBox, bz = t % kBox;
            const float *q = pot + ((bx + 2) * kPhi + (by + 2)) * kPhi + (bz + 2);
            const float c1 = 2.0f / 3.0f, c2 = 1.0f / 12.0f;
            auto d = [&](int st) {
                return -(c1 * (q[st] - q[-st]) - c2 * (q[2 * st] - q[-2 * st])) * fh;
            };
            f[k][0] = d(kPhi * kPhi);
            f[k][1] = d(kPhi);
            f[k][2] = d(1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int t = threadIdx.x + k * kAssignThreads;
        if (t < kBoxWords) {
            fx[t] = f[k][0];
            fy[t] = f[k][1];
            fz[t] = f[k][2];
        }
    }
    __syncthreads();
    while (i < end) {
        double wx[3], wy[3], wz[3];
        const int ix = tsc(p.x, inv_h, wx), iy = tsc(p.y, inv_h, wy), iz = tsc(p.z, inv_h, wz);
        const uint32_t out = o;
        i += kAssignThreads;
        if (i < end) { // the next one
            p = ps[i];
            o = idx[i];
        }
        const int at = ((ix - 1 - ox) * kBox + (iy - 1 - oy)) * kBox + (iz - 1 - oz);
        float sx = 0.0f, sy = 0.0f, sz = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const double wab = wx[a] * wy[b];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float w = (float)(wab * wz[c]);
                    const int k = at + (a * kBox + b) * kBox + c;
                    sx += w * fx[k];
                    sy += w * fy[k];
                    sz += w * fz[k];
                }
            }
        }
        stage[out] = make_float4(sx, sy, sz, 0.0f);
    }
}

// The caller's order o: ax[o], ay[o], az[o] = stage[o] (written, or added to with ACC).
template <typename T, int ACC>
__global__ __launch_bounds__(256) void k_pm_split(const float4 *__restrict__ stage, int64_t n,
                                               T *__restrict__ ax, T *__restrict__ ay,
                                               T *__restrict__ az)
{
    const int64_t o = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (o >= n) return;
    const float4 v = stage[o];
    if (ACC) {
        ax[o] += (T)v.x;
        ay[o] += (T)v.y;
        az[o] += (T)v.z;
    } else {
        ax[o] = (T)v.x;
        ay[o] = (T)v.y;
        az[o] = (T)v.z;
    }
}

} // namespace

void launch_pm_green(int N, double L, double eta, float *green, double2 *tw, hipStream_t s)
{
    const size_t H = N / 2 + 1;
    const size_t work = H * H * H > (size_t)N / 2 ? H * H * H : (size_t)N / 2;
    k_pm_green<<<(unsigned)((work + 255) / 256), 256, 0, s>>>(N, L, eta, green, tw);
}

size_t pm_assign_cells(int N) { const size_t c = (size_t)N / kCellPts; return c * c * c; }
size_t pm_assign_items_max(int N, int64_t n)
{
    return pm_assign_cells(N) + (size_t)((n + cell_chunk(n) - 1) / cell_chunk(n));
}
size_t pm_assign_slot_words() { return kBoxWords; }

void launch_pm_assign(const double4 *ps, const uint64_t *key, int64_t n, int N, double L,
                      const unsigned long long *mx, uint32_t *cell_start, uint32_t *item_start,
                      uint32_t *scan_tmp, unsigned long long *slots, unsigned long long *mass,
                      hipStream_t s)
{
    const uint32_t ncells = (uint32_t)pm_assign_cells(N);
    const int lc = __builtin_ctz((unsigned)(N / kCellPts)); // tree level of the cells
    const int sh = 3 * (21 - lc);
    k_pm_cells<<<(ncells + 1 + 255) / 256, 256, 0, s>>>(key, n, sh, ncells, cell_start);
    k_pm_cell_items<<<(ncells + 255) / 256, 256, 0, s>>>(cell_start, ncells, cell_chunk(n),
                                                         item_start);
    scan_u32(item_start, ncells, item_start + ncells, scan_tmp, s); // exclusive; the total last
    const size_t items = pm_assign_items_max(N, n);
    if (n)
        k_pm_assign<<<(unsigned)items, kAssignThreads, 0, s>>>(ps, n, N, N / L, mx, cell_start,
                                                               item_start, ncells, cell_chunk(n), slots);
    k_pm_gather<<<ncells, kCellPts * kCellPts * kCellPts, 0, s>>>(N, item_start, slots, mass);
}

size_t pm_grid_points(int N) { return (size_t)(N / 2 + 1) * N * N; }

template <int LOGN>
static void pm_potential(const unsigned long long *mass, const unsigned long long *mx, int64_t n,
                         float2 *grid, float *phi, const float *green, const double2 *tw,
                         hipStream_t s)
{
    using D = Lines<LOGN>;
    constexpr unsigned pairs = D::N * (D::N / (2 * D::P)), lines = (D::N / 2 + 1) * (D::N / D::B);
    k_fft_x_forward<LOGN><<<pairs, D::P * D::T, 0, s>>>(mass, mx, n, grid, tw);
    k_fft_y<LOGN, false><<<lines, D::B * D::T, 0, s>>>(grid, tw);
    k_fft_z_green<LOGN><<<lines, D::B * D::T, 0, s>>>(grid, tw, green);
    k_fft_y<LOGN, true><<<lines, D::B * D::T, 0, s>>>(grid, tw);
    k_fft_x_inverse<LOGN><<<pairs, D::P * D::T, 0, s>>>(grid, phi, tw);
}

void launch_pm_potential(const unsigned long long *mass, const unsigned long long *mx,
                         int64_t n, int N, float2 *grid, float *phi, const float *green,
                         const double2 *tw, hipStream_t s)
{
    switch (N) {
    case 16: return pm_potential<4>(mass, mx, n, grid, phi, green, tw, s);
    case 32: return pm_potential<5>(mass, mx, n, grid, phi, green, tw, s);
    case 64: return pm_potential<6>(mass, mx, n, grid, phi, green, tw, s);
    case 128: return pm_potential<7>(mass, mx, n, grid, phi, green, tw, s);
    case 256: return pm_potential<8>(mass, mx, n, grid, phi, green, tw, s);
    case 512: return pm_potential<9>(mass, mx, n, grid, phi, green, tw, s);
    default: return pm_potential<10>(mass, mx, n, grid, phi, green, tw, s);
    }
}

void launch_pm_interp(const double4 *ps, int64_t n, int N, double L, const float *phi,
                      const uint32_t *idx, float4 *stage, const uint32_t *cell_start,
                      const uint32_t *item_start, hipStream_t s)
{
    if (!n) return;
    const uint32_t ncells = (uint32_t)pm_assign_cells(N);
    k_pm_interp<<<(unsigned)pm_assign_items_max(N, n), kAssignThreads, 0, s>>>(
        ps, N, N / L, phi, idx, stage, cell_start, item_start, ncells, cell_chunk(n));
}

void launch_pm_split(const float4 *stage, int64_t n, void *ax, void *ay, void *az,
                     int out_fp64, int accumulate, hipStream_t s)
{
    if (!n) return;
    const unsigned b = (unsigned)((n + 255) / 256);
    if (out_fp64) {
        if (accumulate)
            k_pm_split<double, 1><<<b, 256, 0, s>>>(stage, n, (double *)ax, (double *)ay,
                                                (double *)az);
        else
            k_pm_split<double, 0><<<b, 256, 0, s>>>(stage, n, (double *)ax, (double *)ay,
                                                (double *)az);
    } else {
        if (accumulate)
            k_pm_split<float, 1><<<b, 256, 0, s>>>(stage, n, (float *)ax, (float *)ay, (float *)az);
        else
            k_pm_split<float, 0><<<b, 256, 0, s>>>(stage, n, (float *)ax, (float *)ay, (float *)az);
    }
}

} // namespace tpm

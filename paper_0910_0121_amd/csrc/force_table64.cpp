// The FP64 force kernel's table of the pair law, built on the host.
//
// G(s) = g(2 sqrt(s)) / (s + e2)^(3/2), s = (r / r_cut)^2, is given in pieces over u = c + (1 - c) s,
// 64 per octave, in t = u - a with a the piece's lower edge, as G = G_a (1 + r(t))^5: G_a its value
// at the edge and r a polynomial of degree 6 without a constant, so that only one rounding, G_a's,
// and not five times that of a fifth root, is left in G.  u and t are scaled by 2^18, so that the
// floats among the coefficients stay in range for the narrowest pieces and the widest.
//
// 1 + r = g^(1/5) / g_a^(1/5) times ((s + e2) / (s_a + e2))^(-3/10), both as power series in
// tau = t / w, w the piece's width.  The first does not depend on e2: R = 2 sqrt(s), eq. (2) as a
// polynomial of R, split into even and odd powers (R^2 = 4 s is linear in tau), and the fifth root
// from its differential equation, in extended precision, once per process (about 1 ms).  The second
// is a binomial series in tau (w / (1 - c)) / (s_a + e2), at most tau / 64.  Their product, of degree
// 9, is brought to degree 6 by subtracting Chebyshev polynomials, which leaves less than 1e-17; r
// being small, doubles are enough for it, and a table takes 0.1 ms (all of it in extended precision,
// for every e2, took 1.4 to 1.7).  c = 2^-24: g carries (8/5) R^3 = 12.8 s^(3/2), which no polynomial
// follows at s = 0, and a first piece of width 2^-30 keeps what is missed there below 1e-16.
// The two highest coefficients are rounded to float, from the top down, each time putting the
// rounding error times the best lower-degree approximation of that power back into the lower
// coefficients: what remains is below 1e-19.
#include "common.hpp"

#include <cmath>

namespace tpm {
namespace {

typedef long double real;
constexpr int kDeg = 9, kKeep = kTab64Deg;
constexpr uint32_t kPieces = (uint32_t)kTab64Oct * 64u;

struct Series {
    real a[kDeg + 1];
};

Series mul(const Series &f, const Series &g)
{
    Series r{};
    for (int i = 0; i <= kDeg; ++i)
        for (int j = 0; i + j <= kDeg; ++j) r.a[i + j] += f.a[i] * g.a[j];
    return r;
}

// c[0] + c[1] S + ... + c[n] S^n for the linear S = s0 + s1 x.
Series poly(real s0, real s1, const real *c, int n)
{
    Series r{};
    r.a[0] = c[n];
    for (int k = n - 1; k >= 0; --k) {
        for (int i = kDeg; i > 0; --i) r.a[i] = r.a[i] * s0 + r.a[i - 1] * s1;
        r.a[0] = r.a[0] * s0 + c[k];
    }
    return r;
}

// y = (g / g(0))^(1/5), from 5 y' g = y g'.
Series fifth_root(const Series &g)
{
    Series y{};
    y.a[0] = 1;
    for (int n = 1; n <= kDeg; ++n) {
        real v = 0;
        for (int k = 1; k <= n; ++k) v += 0.2L * k * g.a[k] * y.a[n - k];
        for (int k = 1; k < n; ++k) v -= g.a[k] * (n - k) * y.a[n - k];
        y.a[n] = v / (n * g.a[0]);
    }
    return y;
}

// f / g
Series quotient(const Series &f, const Series &g)
{
    Series r{};
    for (int n = 0; n <= kDeg; ++n) {
        real v = f.a[n];
        for (int k = 1; k <= n; ++k) v -= g.a[k] * r.a[n - k];
        r.a[n] = v / g.a[0];
    }
    return r;
}

// Eq. (2) for R < 1.
real g_near(real s)
{
    const real R = 2 * std::sqrt(s), R2 = R * R;
    return 1 + R2 * R * (-1.6L + R2 * (1.6L + R * (-0.5L + R * (-12.0L / 35 + 0.15L * R))));
}

// What of the table does not depend on e2: per piece s and g at the lower edge, and g^(1/5) over
// its value there in powers of tau.
struct Cutoff {
    real s[kPieces], g[kPieces];
    double root[kPieces][kDeg + 1];
    double cheb[kDeg + 1][kDeg + 1]; // shifted Chebyshev polynomials T_n(2 tau - 1) in powers of tau
    Cutoff();
};

Cutoff::Cutoff()
{
    // T_n(2 tau - 1): T_(n+1) = (4 tau - 2) T_n - T_(n-1)
    for (int n = 0; n <= kDeg; ++n)
        for (int i = 0; i <= kDeg; ++i)
            cheb[n][i] = n == 0   ? (i == 0)
                         : n == 1 ? (i == 0 ? -1 : i == 1 ? 2 : 0)
                                  : (i ? 4 * cheb[n - 1][i - 1] : 0) - 2 * cheb[n - 1][i] -
                                        cheb[n - 2][i];
    const real c = std::ldexp(1.0L, -kTab64Oct), pi = 3.14159265358979323846264338327950288L;
    // eq. (2) for R < 1, and its cubic factor for R >= 1, in even and odd powers of R over S = R^2
    const real near_even[5] = {1, 0, 0, -0.5L, 0.15L}, near_odd[4] = {0, -1.6L, 1.6L, -12.0L / 35};
    const real far_even[2] = {4.0L / 140, 22.0L / 140}, far_odd[2] = {10.0L / 140, 7.0L / 140};
    for (uint32_t k = 0; k < kPieces; ++k) {
        const int e = (int)(k >> 6) - kTab64Oct;
        const real edge = std::ldexp(1 + (real)(k & 63u) / 64, e), w = std::ldexp(1.0L / 64, e);
        const real h = w / (1 - c);
        s[k] = (edge - c) / (1 - c);
        for (int i = 0; i <= kDeg; ++i) root[k][i] = 0.0;
        if (k < 4) {
            // the piece is not narrow next to s: interpolation at the Chebyshev nodes of degree 6,
            // with its own value at the edge
            constexpr int N = kKeep + 1;
            g[k] = g_near(s[k]);
            real y[N];
            for (int i = 0; i < N; ++i) {
                const real tau = (1 + std::cos(pi * (i + 0.5L) / N)) / 2;
                y[i] = std::pow(g_near(s[k] + h * tau) / g[k], 0.2L);
            }
            real q[N] = {};
            for (int n = 0; n < N; ++n) {
                real v = 0;
                for (int i = 0; i < N; ++i) v += y[i] * std::cos(pi * n * (i + 0.5L) / N);
                v *= (n ? 2.0L : 1.0L) / N;
                for (int i = 0; i <= n; ++i) q[i] += v * cheb[n][i];
            }
            for (int i = 0; i < N; ++i) root[k][i] = (double)(q[i] / q[0]);
            g[k] *= q[0] * q[0] * q[0] * q[0] * q[0];
            continue;
        }
        Series R{};
        R.a[0] = 2 * std::sqrt(s[k]);
        for (int n = 1; n <= kDeg; ++n) { // R^2 = 4 s
            real v = n == 1 ? 4 * h : 0;
            for (int i = 1; i < n; ++i) v -= R.a[i] * R.a[n - i];
            R.a[n] = v / (2 * R.a[0]);
        }
        const bool near = s[k] + h / 2 < 0.25L;
        Series f = mul(R, near ? poly(4 * s[k], 4 * h, near_odd, 3)
                               : poly(4 * s[k], 4 * h, far_odd, 1));
        const Series even =
            near ? poly(4 * s[k], 4 * h, near_even, 4) : poly(4 * s[k], 4 * h, far_even, 1);
        for (int i = 0; i <= kDeg; ++i) f.a[i] += even.a[i];
        g[k] = f.a[0];
        Series p = fifth_root(f);
        if (!near) { // g = (2 - R)^5 times the cubic, and 2 - R = 4 (1 - s) / (2 + R)
            Series d = R, one{};
            d.a[0] += 2;
            one.a[0] = 4 * (1 - edge) / (1 - c);
            one.a[1] = -4 * h;
            const Series v = quotient(one, d);
            const real v2 = v.a[0] * v.a[0];
            g[k] *= v2 * v2 * v.a[0];
            p = mul(p, v);
        }
        for (int i = 0; i <= kDeg; ++i) root[k][i] = (double)(p.a[i] / p.a[0]);
    }
}

} // namespace

bool build_force_table64(double eps_over_rcut, std::vector<double> &hi, std::vector<float> &lo)
{
    const real e2 = (real)eps_over_rcut * eps_over_rcut;
    if (!(e2 >= std::ldexp(1.0L, 1 - kTab64Oct)) || !std::isfinite(eps_over_rcut) || e2 > 64)
        return false;
    static const Cutoff C; // made by the first caller; the others wait for it
    hi.assign((size_t)kTab64F64 * kTab64Entries, 0.0); // the entry of u = 1 stays zero
    lo.assign((size_t)(kKeep + 1 - kTab64F64) * kTab64Entries, 0.f);
    double binom[kDeg + 1] = {1.0}; // of -3/10
    for (int n = 1; n <= kDeg; ++n) binom[n] = binom[n - 1] * (-0.3 - (n - 1)) / n;
    const real inv = 1 / (1 - std::ldexp(1.0L, -kTab64Oct));
    for (uint32_t k = 0; k < kPieces; ++k) {
        const int e = (int)(k >> 6) - kTab64Oct;
        const real x = C.s[k] + e2;
        hi[k] = (double)(C.g[k] / (x * std::sqrt(x)));
        const double rho = (double)(std::ldexp(inv, e - 6) / x);
        double b[kDeg + 1], q[kDeg + 1] = {};
        double pw = 1.0;
        for (int n = 0; n <= kDeg; ++n, pw *= rho) b[n] = binom[n] * pw;
        const double *const y = C.root[k];
        for (int i = 0; i <= kDeg; ++i)
            for (int j = 0; i + j <= kDeg; ++j) q[i + j] += y[i] * b[j];
        for (int n = kDeg; n > kKeep; --n) {
            const double v = q[n] / C.cheb[n][n];
            for (int i = 1; i < n; ++i) q[i] -= v * C.cheb[n][i];
        }
        // in t: tau = t / w, w a power of two
        const double iw = std::ldexp(1.0, 6 - e - kTab64Exp);
        double scale[kKeep + 1] = {1.0};
        for (int n = 1; n <= kKeep; ++n) scale[n] = scale[n - 1] * iw;
        for (int n = kKeep; n >= kTab64F64; --n) {
            const float v = (float)(q[n] * scale[n]);
            lo[(size_t)(n - kTab64F64) * kTab64Entries + k] = v;
            const double off = (q[n] - (double)v / scale[n]) / C.cheb[n][n]; // what is left over
            for (int i = 1; i < n; ++i) q[i] -= off * C.cheb[n][i];
        }
        for (int n = 1; n < kTab64F64; ++n) hi[(size_t)n * kTab64Entries + k] = q[n] * scale[n];
    }
    return true;
}

} // namespace tpm

// The FP64 force kernel's table of the pair law, built on the host in extended precision.
//
// G(s) = g(2 sqrt(s)) / (s + e2)^(3/2), s = (r / r_cut)^2, is given in pieces over u = c + (1 - c) s,
// 64 per octave, in t = u - a with a the piece's lower edge, as G = G_a (1 + r(t))^5: G_a its value
// at the edge and r a polynomial of degree 6 without a constant, so that only one rounding, G_a's,
// and not five times that of a fifth root, is left in G.  u and t are scaled by 2^18, so that the
// floats among the coefficients stay in range for the narrowest pieces and the widest.  Per piece
// p = G^(1/5) is expanded about the middle as a power series (s = s_m + h x, x in [-1, 1]): R = 2
// sqrt(s), eq. (2) as a polynomial of R, split into even and odd powers (R^2 = 4 s is linear in x),
// and the fractional powers from their differential equation; the series of degree 9 is brought to
// degree 6 by subtracting Chebyshev polynomials, which leaves a relative error below 1e-17 in p.
// c = 2^-24: g carries (8/5) R^3 = 12.8 s^(3/2), which no polynomial follows at s = 0, and a first
// piece of width 2^-30 keeps what is missed there below 1e-16.
// The two highest coefficients are rounded to float, from the top down, each time putting the
// rounding error times the best lower-degree approximation of that power back into the lower
// coefficients: what remains is below 1e-19 of p.
#include "common.hpp"

#include <cmath>

namespace tpm {
namespace {

typedef long double real;
constexpr int kDeg = 9, kKeep = kTab64Deg;

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

// y = g^(1/5) (f0 + f1 x)^(-3/10), from y' A = y B with A = g (f0 + f1 x) and
// B = g' (f0 + f1 x) / 5 - 3 g f1 / 10.
Series root(const Series &g, real f0, real f1)
{
    real A[kDeg + 1], B[kDeg + 1];
    for (int i = 0; i <= kDeg; ++i) {
        A[i] = g.a[i] * f0 + (i ? g.a[i - 1] * f1 : 0);
        B[i] = 0.2L * ((i < kDeg ? (i + 1) * g.a[i + 1] * f0 : 0) + i * g.a[i] * f1) -
               0.3L * g.a[i] * f1;
    }
    Series y{};
    y.a[0] = std::exp(0.2L * std::log(g.a[0]) - 0.3L * std::log(f0));
    for (int n = 1; n <= kDeg; ++n) {
        real v = 0;
        for (int k = 1; k <= n; ++k) v += B[k - 1] * y.a[n - k];
        for (int k = 1; k < n; ++k) v -= A[k] * (n - k) * y.a[n - k];
        y.a[n] = v / (n * A[0]);
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

// Chebyshev T_n in powers of x.
void chebyshev(int n, real *t)
{
    real a[kDeg + 1] = {1}, b[kDeg + 1] = {0, 1};
    for (int i = 0; i <= kDeg; ++i) t[i] = n == 0 ? a[i] : b[i];
    for (int m = 2; m <= n; ++m) {
        for (int i = 0; i <= kDeg; ++i) t[i] = (i ? 2 * b[i - 1] : 0) - a[i];
        for (int i = 0; i <= kDeg; ++i) {
            a[i] = b[i];
            b[i] = t[i];
        }
    }
}

// p at one s, for the first pieces (their width is not small next to s).
real p_at(real s, real e2)
{
    const real R = 2 * std::sqrt(s), R2 = R * R;
    const real g = 1 + R2 * R * (-1.6L + R2 * (1.6L + R * (-0.5L + R * (-12.0L / 35 + 0.15L * R))));
    return std::pow(g, 0.2L) * std::pow(s + e2, -0.3L);
}

} // namespace

bool build_force_table64(double eps_over_rcut, std::vector<double> &hi, std::vector<float> &lo)
{
    const real e2 = (real)eps_over_rcut * eps_over_rcut;
    if (!(e2 >= std::ldexp(1.0L, 1 - kTab64Oct)) || !std::isfinite(eps_over_rcut) || e2 > 64)
        return false;
    constexpr uint32_t pieces = (uint32_t)kTab64Oct * 64u;
    hi.assign((size_t)kTab64F64 * kTab64Entries, 0.0); // the entry of u = 1 stays zero
    lo.assign((size_t)(kKeep + 1 - kTab64F64) * kTab64Entries, 0.f);
    const real c = std::ldexp(1.0L, -kTab64Oct);
    real T[kDeg + 1][kDeg + 1];
    for (int n = 0; n <= kDeg; ++n) chebyshev(n, T[n]);
    // shifted Chebyshev polynomials T_n(2 tau - 1) in powers of tau, for the rounding
    real Ts[kKeep + 1][kKeep + 1] = {};
    for (int n = 0; n <= kKeep; ++n) {
        real v[kKeep + 1] = {}; // Horner in (2 tau - 1)
        for (int k = n; k >= 0; --k) {
            real w[kKeep + 1] = {};
            for (int i = 0; i <= kKeep; ++i) {
                w[i] -= v[i];
                if (i < kKeep) w[i + 1] += 2 * v[i];
            }
            w[0] += T[n][k];
            for (int i = 0; i <= kKeep; ++i) v[i] = w[i];
        }
        for (int i = 0; i <= kKeep; ++i) Ts[n][i] = v[i];
    }
    // eq. (2) for R < 1, and its cubic factor for R >= 1, in even and odd powers of R over S = R^2
    const real near_even[5] = {1, 0, 0, -0.5L, 0.15L}, near_odd[4] = {0, -1.6L, 1.6L, -12.0L / 35};
    const real far_even[2] = {4.0L / 140, 22.0L / 140}, far_odd[2] = {10.0L / 140, 7.0L / 140};
    for (uint32_t k = 0; k < pieces; ++k) {
        const int e = (int)(k >> 6) - kTab64Oct;
        const real edge = std::ldexp(1 + (real)(k & 63u) / 64, e), w = std::ldexp(1.0L / 64, e);
        const real s_m = (edge + w / 2 - c) / (1 - c), h = w / 2 / (1 - c);
        real q[kDeg + 1] = {}; // p in powers of x
        if (k < 4) {
            // interpolation at the Chebyshev nodes of degree 6, by their discrete sums
            constexpr int N = kKeep + 1;
            real y[N], x[N];
            const real pi = 3.14159265358979323846264338327950288L;
            for (int i = 0; i < N; ++i) {
                x[i] = std::cos(pi * (i + 0.5L) / N);
                const real s = s_m + h * x[i];
                y[i] = p_at(s > 0 ? s : 0, e2);
            }
            for (int n = 0; n < N; ++n) {
                real v = 0;
                for (int i = 0; i < N; ++i) v += y[i] * std::cos(pi * n * (i + 0.5L) / N);
                v *= (n ? 2.0L : 1.0L) / N;
                for (int i = 0; i <= n; ++i) q[i] += v * T[n][i];
            }
        } else {
            Series R{};
            R.a[0] = 2 * std::sqrt(s_m);
            for (int n = 1; n <= kDeg; ++n) { // R^2 = 4 s
                real v = n == 1 ? 4 * h : 0;
                for (int i = 1; i < n; ++i) v -= R.a[i] * R.a[n - i];
                R.a[n] = v / (2 * R.a[0]);
            }
            const bool near = R.a[0] < 1;
            Series g = mul(R, near ? poly(4 * s_m, 4 * h, near_odd, 3)
                                   : poly(4 * s_m, 4 * h, far_odd, 1));
            const Series even = near ? poly(4 * s_m, 4 * h, near_even, 4)
                                     : poly(4 * s_m, 4 * h, far_even, 1);
            for (int i = 0; i <= kDeg; ++i) g.a[i] += even.a[i];
            Series p = root(g, s_m + e2, h);
            if (!near) { // g = (2 - R)^5 times the cubic, and 2 - R = 4 (1 - s) / (2 + R)
                Series d = R, one{};
                d.a[0] += 2;
                one.a[0] = 4 * (1 - edge - w / 2) / (1 - c);
                one.a[1] = -4 * h;
                p = mul(p, quotient(one, d));
            }
            for (int i = 0; i <= kDeg; ++i) q[i] = p.a[i];
            for (int n = kDeg; n > kKeep; --n) {
                const real v = q[n] / T[n][n];
                for (int i = 0; i <= n; ++i) q[i] -= v * T[n][i];
            }
        }
        // in tau = t / w: x = 2 tau - 1
        real b[kKeep + 1] = {};
        for (int n = kKeep; n >= 0; --n) {
            real v[kKeep + 1] = {};
            for (int i = 0; i <= kKeep; ++i) {
                v[i] -= b[i];
                if (i < kKeep) v[i + 1] += 2 * b[i];
            }
            v[0] += q[n];
            for (int i = 0; i <= kKeep; ++i) b[i] = v[i];
        }
        real iw[kKeep + 1];
        iw[0] = 1;
        for (int i = 1; i <= kKeep; ++i) iw[i] = iw[i - 1] / std::ldexp(w, kTab64Exp);
        for (int n = kKeep; n >= kTab64F64; --n) {
            const float v = (float)(b[n] / b[0] * iw[n]);
            lo[(size_t)(n - kTab64F64) * kTab64Entries + k] = v;
            const real off = b[n] - (real)v * b[0] / iw[n]; // this much of tau^n is left over
            for (int i = 0; i < n; ++i) b[i] -= off * Ts[n][i] / Ts[n][n];
        }
        // p / b[0] = 1 + r
        const real p2 = b[0] * b[0];
        hi[k] = (double)(p2 * p2 * b[0]);
        for (int n = 1; n < kTab64F64; ++n)
            hi[(size_t)n * kTab64Entries + k] = (double)(b[n] / b[0] * iw[n]);
    }
    return true;
}

} // namespace tpm

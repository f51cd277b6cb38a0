// Host generation of the Rys quadrature tables (layout in hfx_internal.h).
//
// The n-point Rys quadrature (Dupuis, Rys and King, J. Chem. Phys. 65, 111
// (1976)) is the Gauss quadrature of the weight e^{-T t^2} on 0 <= t <= 1 in
// the variable x = t^2: sum_r w_r P(x_r) = int_0^1 P(t^2) e^{-T t^2} dt for
// every polynomial P of degree below 2n, so that sum_r w_r x_r^m = F_m(T).
// For each T the recurrence coefficients of the orthogonal polynomials come
// from the Stieltjes procedure on a 48-point Gauss-Legendre discretisation of
// the weight (exact to rounding for T <= RYS_NT), the roots from bisection
// and secant steps between the roots of the next lower polynomial, and the weights from the
// Christoffel sums, all in long double.  Roots and weights are then
// interpolated in T by one polynomial of degree RYS_NC - 1 per unit interval
// (Chebyshev nodes), stored as powers.  Above RYS_NT the upper limit of the integral may be
// moved to infinity (the tail is below 1.4e-17 of F_8 there): x_r = h_r / T
// and w_r = v_r / sqrt(T) with the half-range Gauss-Hermite nodes h_r = s_r^2
// and weights v_r, which the same procedure gives from the discretised weight
// e^{-s^2} on [0, 12].
#include <algorithm>
#include <cmath>
#include <vector>

#include "hfx_internal.h"

namespace {

typedef long double ld;

void gauss_legendre(int n, std::vector<ld>& x, std::vector<ld>& w) {   // on [0, 1]
    x.resize(n);
    w.resize(n);
    for (int i = 0; i < n; ++i) {
        ld z = cosl((ld)M_PIl * (i + 0.75L) / (n + 0.5L)), dp = 0;
        for (int it = 0; it < 100; ++it) {
            ld p0 = 1, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const ld p2 = ((2 * k - 1) * z * p1 - (k - 1) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (z * p1 - p0) / (z * z - 1);
            const ld dz = p1 / dp;
            z -= dz;
            if (fabsl(dz) < 1e-19L) break;
        }
        x[i] = 0.5L * (1 - z);
        w[i] = 1 / ((1 - z * z) * dp * dp);
    }
}

// Gauss quadrature with n points of the discrete measure (x_i, m_i), x_i in [0, top].
void gauss_of_measure(const std::vector<ld>& x, const std::vector<ld>& m, ld top, int n, ld* root, ld* weight) {
    const size_t N = x.size();
    std::vector<ld> p0(N, 0.0L), p1(N, 1.0L), al(n), be(n);
    ld last = 0;
    for (int k = 0; k < n; ++k) {
        ld s = 0, sx = 0;
        for (size_t i = 0; i < N; ++i) {
            const ld t = m[i] * p1[i] * p1[i];
            s += t;
            sx += t * x[i];
        }
        al[k] = sx / s;
        be[k] = k ? s / last : s;   // be[0]: the total mass
        last = s;
        for (size_t i = 0; i < N; ++i) {
            const ld p2 = (x[i] - al[k]) * p1[i] - (k ? be[k] : 0.0L) * p0[i];
            p0[i] = p1[i];
            p1[i] = p2;
        }
    }
    auto poly = [&](int deg, ld z) {   // monic orthogonal polynomial
        ld a = 0, b = 1;
        for (int k = 0; k < deg; ++k) {
            const ld c = (z - al[k]) * b - (k ? be[k] : 0.0L) * a;
            a = b;
            b = c;
        }
        return b;
    };
    std::vector<ld> r;   // roots of the polynomial of degree deg, ascending
    for (int deg = 1; deg <= n; ++deg) {
        std::vector<ld> nr(deg);
        for (int i = 0; i < deg; ++i) {
            ld lo = i ? r[i - 1] : 0.0L, hi = i + 1 < deg ? r[i] : top;
            const bool up = poly(deg, hi) > 0;
            for (int it = 0; it < 12; ++it) {
                const ld mid = 0.5L * (lo + hi);
                if ((poly(deg, mid) > 0) == up) hi = mid; else lo = mid;
            }
            // secant steps inside the bracket to rounding
            ld u = lo, v = hi, fu = poly(deg, u), fv = poly(deg, v);
            for (int it = 0; it < 12 && fv != fu && u != v; ++it) {
                const ld t = std::min(hi, std::max(lo, v - fv * (v - u) / (fv - fu)));
                u = v;
                fu = fv;
                v = t;
                fv = poly(deg, v);
            }
            nr[i] = v;
        }
        r.swap(nr);
    }
    for (int i = 0; i < n; ++i) {
        ld a = 0, b = 1, norm = be[0], s = 1 / norm;   // sum of the squared orthonormal polynomials
        for (int k = 0; k + 1 < n; ++k) {
            const ld c = (r[i] - al[k]) * b - (k ? be[k] : 0.0L) * a;
            a = b;
            b = c;
            norm *= be[k + 1];
            s += b * b / norm;
        }
        root[i] = r[i];
        weight[i] = 1 / s;
    }
}

}  // namespace

void hfx_rys_table(double* tab) {
    std::vector<ld> gx, gw;
    gauss_legendre(48, gx, gw);
    const size_t N = gx.size();
    std::vector<ld> x(N), m(N);
    for (int n = RYS_NMIN; n <= RYS_NMAX; ++n) {
        double* blk = tab + rys_block(n);
        for (int k = 0; k < RYS_NT; ++k) {
            ld f[2 * RYS_NMAX][RYS_NC];   // values at the interval's Chebyshev nodes: roots, then weights
            for (int j = 0; j < RYS_NC; ++j) {
                const ld T = k + 0.5L + 0.5L * cosl((ld)M_PIl * (j + 0.5L) / RYS_NC);
                for (size_t i = 0; i < N; ++i) {
                    x[i] = gx[i] * gx[i];
                    m[i] = gw[i] * expl(-T * x[i]);
                }
                ld r[RYS_NMAX], w[RYS_NMAX];
                gauss_of_measure(x, m, 1.0L, n, r, w);
                for (int i = 0; i < n; ++i) {
                    f[2 * i][j] = r[i];
                    f[2 * i + 1][j] = w[i];
                }
            }
            for (int q = 0; q < 2 * n; ++q) {
                // Chebyshev coefficients, then powers of z = 2 (T - k) - 1
                ld c[RYS_NC], mono[RYS_NC] = {0}, t0[RYS_NC] = {0}, t1[RYS_NC] = {0};
                for (int i = 0; i < RYS_NC; ++i) {
                    ld s = 0;
                    for (int j = 0; j < RYS_NC; ++j) s += f[q][j] * cosl((ld)M_PIl * i * (j + 0.5L) / RYS_NC);
                    c[i] = s * (i ? 2.0L : 1.0L) / RYS_NC;
                }
                t0[0] = 1;
                t1[1] = 1;
                for (int i = 0; i < RYS_NC; ++i) {   // t0 = T_i, t1 = T_{i+1}
                    for (int d = 0; d <= i; ++d) mono[d] += c[i] * t0[d];
                    ld t2[RYS_NC] = {0};
                    for (int d = 0; d + 1 < RYS_NC; ++d) t2[d + 1] = 2 * t1[d];
                    for (int d = 0; d < RYS_NC; ++d) t2[d] -= t0[d];
                    for (int d = 0; d < RYS_NC; ++d) {
                        t0[d] = t1[d];
                        t1[d] = t2[d];
                    }
                }
                double* o = blk + ((size_t)k * n + q / 2) * RYS_ROW + (q % 2) * RYS_NC;
                for (int d = 0; d < RYS_NC; ++d) o[d] = (double)mono[d];
            }
        }
        // the asymptotic nodes: h_r and v_r
        const ld smax = 12;
        for (size_t i = 0; i < N; ++i) {
            const ld s = smax * gx[i];
            x[i] = s * s;
            m[i] = smax * gw[i] * expl(-x[i]);
        }
        ld r[RYS_NMAX], w[RYS_NMAX];
        gauss_of_measure(x, m, smax * smax, n, r, w);
        double* o = blk + (size_t)RYS_NT * n * RYS_ROW;
        for (int i = 0; i < n; ++i) {
            o[2 * i] = (double)r[i];
            o[2 * i + 1] = (double)w[i];
        }
    }
}

// Host-side set-up arithmetic of the FDLB solver: Gauss-Hermite quadrature, the
// orthonormal Hermite table used by the equilibrium contraction, and the mapping of
// (denseness, Knudsen number) to the model's covolume and reference viscosity.
// Everything here runs once per context, in FP64, on the CPU.
#include "host_math.h"

#include "node_tables.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace elb {

namespace {

// sqrt(l), l <= 257 (the largest order asked for is 256)
struct Roots {
    double v[258];
    Roots() { for (int l = 0; l < 258; ++l) v[l] = std::sqrt((double)l); }
};
const Roots kRoot;

}  // namespace

// Orthonormal probabilists' Hermite values h_l(x) = He_l(x)/sqrt(l!) for l = 0..lmax <= 256,
// from He_{l+1} = x He_l - l He_{l-1} divided through by sqrt((l+1)!).
void hermite_orthonormal(int lmax, double x, double *h)
{
    h[0] = 1.0;
    if (lmax >= 1) h[1] = x;
    for (int l = 1; l < lmax; ++l) h[l + 1] = (x * h[l] - kRoot.v[l] * h[l - 1]) / kRoot.v[l + 1];
}

// Nodes: for the compiled node counts from the table; otherwise the eigenvalues of the
// symmetric Jacobi matrix of the probabilists' Hermite recurrence (zero diagonal, off-diagonal
// sqrt(k)), bracketed by the sign counts of its LDL^T pivots to 1e-7 of the range and refined
// by Newton's method on h_Q (h_Q' = sqrt(Q) h_{Q-1}), which squares the error each time: O(Q^2)
// in all, where rotations of the full matrix cost O(Q^3) per sweep (Q = 96: 98 ms, 1.2 ms
// this way, 20 ns from the table).
int gauss_hermite_nodes(int Q, double *p)
{
    if (Q < 1 || Q > 256) return 1;
    for (const NodeTable &t : kNodeTables)
        if (t.q == Q) {
            for (int k = 0; k < Q / 2; ++k) {
                p[Q / 2 + k] = t.positive[k];
                p[Q / 2 - 1 - k] = -t.positive[k];
            }
            return 0;
        }
    // number of eigenvalues below v
    auto below = [&](double v) {
        double d = -v;
        int n = d < 0;
        for (int k = 1; k < Q; ++k) {
            d = -v - (double)k / (d == 0.0 ? 1e-300 : d);
            n += d < 0;
        }
        return n;
    };
    const double top = 2.0 * kRoot.v[Q];  // the spectrum lies inside (-top, top)
    std::vector<double> h(Q + 2);
    double left = -top;
    for (int k = 0; k < Q / 2; ++k) {
        double lo = left, hi = 0.0;
        while (hi - lo > 1e-7 * top) {
            const double m = 0.5 * (lo + hi);
            if (below(m) > k) hi = m;
            else lo = m;
        }
        double x = 0.5 * (lo + hi);
        for (int it = 0; it < 6; ++it) {
            hermite_orthonormal(Q, x, h.data());
            const double d = kRoot.v[Q] * h[Q - 1];
            if (d == 0.0) break;
            x -= h[Q] / d;
        }
        left = x;
        p[k] = x;
        p[Q - 1 - k] = -x;
    }
    if (Q % 2) p[Q / 2] = 0.0;
    return 0;
}

// Weights: Christoffel numbers w_k = 1 / sum_{l<Q} h_l(p_k)^2, which sum to 1 for the
// normalised weight function exp(-p^2/2)/sqrt(2 pi) of Sec. II.D.
int gauss_hermite(int Q, double *p, double *w)
{
    if (gauss_hermite_nodes(Q, p)) return 1;
    std::vector<double> h(Q + 2);
    for (int k = 0; k < Q; ++k) {
        hermite_orthonormal(Q - 1, p[k], h.data());
        double s = 0.0;
        for (int l = 0; l < Q; ++l) s += h[l] * h[l];
        w[k] = 1.0 / s;
    }
    return 0;
}

// Carnahan-Starling contact value (Sec. II.A, eq. chi).
double chi_set(double eta) { return 0.5 * (2.0 - eta) / ((1.0 - eta) * (1.0 - eta) * (1.0 - eta)); }

// Reduced density eta with E_l = (3/sqrt 2) b n chi = 6 sqrt(2) eta chi(eta) (Sec. II.B),
// by safeguarded Newton iteration on [0, 1/2).
double eta_of_denseness(double El)
{
    if (El <= 0.0) return 0.0;
    const double c = 6.0 * std::sqrt(2.0);
    double lo = 0.0, hi = 0.5, eta = std::min(El / c, 0.25);
    for (int it = 0; it < 200; ++it) {
        double chi = chi_set(eta);
        double f = c * eta * chi - El;
        if (f > 0) hi = eta; else lo = eta;
        double dchi = chi * (3.0 / (1.0 - eta) - 1.0 / (2.0 - eta));
        double fp = c * (chi + eta * dchi);
        double nxt = eta - f / fp;
        if (!(nxt > lo && nxt < hi)) nxt = 0.5 * (lo + hi);
        if (std::fabs(nxt - eta) <= 1e-17 * std::max(1.0, eta)) { eta = nxt; break; }
        eta = nxt;
    }
    return eta;
}

// Covolume b = 4 eta0 / n_ref, and the dilute hard-sphere viscosity at T = 1,
// mu_ref = (5/16) sqrt(2 pi) n_ref l_dilute, where l_dilute = chi0 * Kn * kn_length is the
// Boltzmann mean free path (the Enskog one, l = 1/(sqrt 2 pi sigma^2 n chi), divided by
// chi; Sec. II.B).  With mu_ref, tau = mu / P_i (Sec. II.B) becomes
//   tau = mu_ref (1 + 0.8 y + (4/25)(1 + 12/pi) y^2) / (n chi sqrt T),  y = b n chi.
void map_units(double El, double kn, double kn_length, double n_ref, double *b, double *mu_ref,
               double *eta0, double *chi0)
{
    double e = eta_of_denseness(El);
    double ch = chi_set(e);
    *eta0 = e;
    *chi0 = ch;
    *b = 4.0 * e / n_ref;
    *mu_ref = 5.0 / 16.0 * std::sqrt(2.0 * M_PI) * n_ref * ch * kn * kn_length;
}

// Weights of the Fischer-Methfessel ball average (Sec. II.A, eq. chi_ret) on the grid:
//   nbar_i = 3/(4 S^3) int_{-S}^{S} n(x_i + t dx) (S^2 - t^2) dt = sum_{|j|<=J} w_j n_{i+j},
// S = sigma/dx, the slice area pi (sigma^2 - s^2) of the ball being the weight in 1-D.  On
// each interval [m, m+1] (in cells) n is the cubic through the points m-1 .. m+2; w_j
// collects the exact integrals of its Lagrange basis times the weight over the part of the
// interval inside [-S, S].  Returns J (w has 2J + 1 entries, w[J] belongs to the cell).
int fm_weights(double S, std::vector<double> &w)
{
    if (!(S > 0.0)) {
        w.assign(1, 1.0);
        return 0;
    }
    const int M = (int)std::ceil(S), J = M + 1;
    w.assign(2 * J + 1, 0.0);
    for (int m = -M; m < M; ++m) {
        const double lo = std::max((double)m, -S) - m, hi = std::min((double)(m + 1), S) - m;
        if (!(hi > lo)) continue;
        // weight in x = t - m: (S^2 - m^2) - 2 m x - x^2
        const double wq[3] = {S * S - (double)m * m, -2.0 * m, -1.0};
        for (int a = 0; a < 4; ++a) {
            // Lagrange basis of node a - 1 over the nodes -1, 0, 1, 2, as coefficients in x
            double l[4] = {1.0, 0.0, 0.0, 0.0};
            double den = 1.0;
            for (int c = 0; c < 4; ++c) {
                if (c == a) continue;
                const double xc = c - 1;
                for (int d = 3; d >= 1; --d) l[d] = l[d - 1] - xc * l[d];
                l[0] = -xc * l[0];
                den *= (double)(a - c);
            }
            double integral = 0.0;
            for (int d = 0; d < 4; ++d)
                for (int e = 0; e < 3; ++e) {
                    const int k = d + e + 1;
                    integral += l[d] * wq[e] * (std::pow(hi, k) - std::pow(lo, k)) / k;
                }
            w[J + m - 1 + a] += 0.75 / (S * S * S) * integral / den;
        }
    }
    return J;
}

}  // namespace elb

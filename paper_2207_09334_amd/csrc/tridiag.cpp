// Eigenvalues of the symmetric tridiagonal matrices that the Lanczos iterations of
// cronos_natural_frequencies build: Sturm-sequence bisection for the smallest ones and
// inverse iteration for the last component of their eigenvectors (the Lanczos residual).
#include <cmath>

#include "common.h"

namespace cronos {

namespace {

constexpr int kShifts = 16;   // shifts that one pass over T serves

// Numbers of eigenvalues of T below each x[0..kShifts) (T: diagonal a[0..k), off-diagonal
// b[0..k-1), b2 = b^2).  The ratios of the LDL^T factorisation of T - x I count the negative
// pivots; a zero pivot is replaced by a tiny one, which moves x by far less than the bisection
// tolerance.  One shift alone is a serial chain of divisions (a division latency per row); the
// shifts' chains are independent, so together they run at the divider's throughput.
void sturm_counts(const double* a, const double* b2, int64_t k, const double* x, double tiny, int64_t* count) {
    double q[kShifts], c[kShifts], xs[kShifts];
    for (int l = 0; l < kShifts; ++l) {
        xs[l] = x[l];
        q[l] = a[0] - xs[l];
        c[l] = 0.0;
    }
    for (int64_t i = 0;; ++i) {
        for (int l = 0; l < kShifts; ++l) {
            q[l] = std::fabs(q[l]) < tiny ? -tiny : q[l];
            c[l] += q[l] < 0.0 ? 1.0 : 0.0;
        }
        if (i + 1 == k) break;
        const double ai = a[i + 1], bi = b2[i];
        for (int l = 0; l < kShifts; ++l) q[l] = (ai - xs[l]) - bi / q[l];
    }
    for (int l = 0; l < kShifts; ++l) count[l] = (int64_t)c[l];
}

}  // namespace

// Gershgorin interval [lo, hi] holding every eigenvalue of T.
void gershgorin(const double* a, const double* b, int64_t k, double* lo, double* hi) {
    double l = a[0], h = a[0];
    for (int64_t i = 0; i < k; ++i) {
        const double r = (i > 0 ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < k ? std::fabs(b[i]) : 0.0);
        l = std::min(l, a[i] - r);
        h = std::max(h, a[i] + r);
    }
    *lo = l;
    *hi = h;
}

// (l + h) / 2, also where the sum is beyond the largest double.
static double middle(double l, double h) {
    const double s = l + h;
    return std::isinf(s) ? 0.5 * l + 0.5 * h : 0.5 * s;
}

// The `count` smallest eigenvalues of T, ascending, by section of [lo, hi] down to one ulp: up to
// kShifts of them at a time, each pass over T placing kShifts / m points inside each of m intervals.
void tridiag_smallest(const double* a, const double* b2, int64_t k, int64_t count, double lo, double hi, double tiny,
                      double* theta) {
    for (int64_t j0 = 0; j0 < count; j0 += kShifts) {
        const int m = (int)std::min<int64_t>(kShifts, count - j0), per = kShifts / m;
        double l[kShifts], h[kShifts], x[kShifts];
        int64_t below[kShifts];
        for (int j = 0; j < kShifts; ++j) {
            l[j] = lo;
            h[j] = hi;
            x[j] = hi;
        }
        for (int it = 0; it < 200; ++it) {
            bool open = false;
            for (int j = 0; j < m; ++j) {
                const double mid = middle(l[j], h[j]);
                open = open || (mid > l[j] && mid < h[j]);   // else the interval is at one ulp
                const double width = h[j] - l[j];   // infinite beyond the largest double: halved until it is not
                for (int p = 0; p < per; ++p)
                    x[j * per + p] = std::isinf(width) ? mid : l[j] + width * ((double)(p + 1) / (per + 1));
            }
            if (!open) break;
            sturm_counts(a, b2, k, x, tiny, below);
            for (int j = 0; j < m; ++j) {
                const double l0 = l[j], h0 = h[j];
                for (int p = 0; p < per; ++p) {
                    const double xp = x[j * per + p];
                    if (xp <= l0 || xp >= h0) continue;
                    if (below[j * per + p] > j0 + j) h[j] = std::min(h[j], xp);
                    else l[j] = std::max(l[j], xp);
                }
            }
        }
        for (int j = 0; j < m; ++j) theta[j0 + j] = middle(l[j], h[j]);
    }
}

// |last component| of the unit eigenvector of T for the eigenvalue approximation theta: two
// steps of inverse iteration, (T - theta I) z = z_prev solved by Gaussian elimination with
// partial pivoting (the band then has two super-diagonals).
double eigvec_last_component(const double* a, const double* b, int64_t k, double theta, double tiny) {
    if (k == 1) return 1.0;
    std::vector<double> dd(k), dl(k - 1), du(k - 1), du2(k > 2 ? k - 2 : 1, 0.0), z(k, 1.0 / std::sqrt((double)k));
    std::vector<char> swapped(k - 1, 0);
    for (int64_t i = 0; i < k; ++i) dd[i] = a[i] - theta;
    for (int64_t i = 0; i + 1 < k; ++i) dl[i] = du[i] = b[i];
    for (int64_t i = 0; i + 1 < k; ++i) {
        if (std::fabs(dd[i]) >= std::fabs(dl[i])) {
            if (std::fabs(dd[i]) < tiny) dd[i] = tiny;
            const double m = dl[i] / dd[i];
            dl[i] = m;
            dd[i + 1] -= m * du[i];
            if (i + 2 < k) du2[i] = 0.0;
        } else {
            const double m = dd[i] / dl[i];
            dd[i] = dl[i];
            dl[i] = m;
            const double t = du[i];
            du[i] = dd[i + 1];
            dd[i + 1] = t - m * dd[i + 1];
            if (i + 2 < k) {
                du2[i] = du[i + 1];
                du[i + 1] = -m * du[i + 1];
            }
            swapped[i] = 1;
        }
    }
    if (std::fabs(dd[k - 1]) < tiny) dd[k - 1] = tiny;
    for (int rep = 0; rep < 2; ++rep) {
        // forward: apply the row swaps and multipliers (L^-1 P)
        for (int64_t i = 0; i + 1 < k; ++i) {
            if (swapped[i]) std::swap(z[i], z[i + 1]);
            z[i + 1] -= dl[i] * z[i];
        }
        // back substitution with U (diagonal dd, super-diagonals du, du2)
        z[k - 1] /= dd[k - 1];
        z[k - 2] = (z[k - 2] - du[k - 2] * z[k - 1]) / dd[k - 2];
        for (int64_t i = k - 3; i >= 0; --i) z[i] = (z[i] - du[i] * z[i + 1] - du2[i] * z[i + 2]) / dd[i];
        double nrm = 0.0, big = 0.0;
        for (int64_t i = 0; i < k; ++i) big = std::max(big, std::fabs(z[i]));
        if (!(big > 0.0) || !std::isfinite(big)) return 1.0;
        for (int64_t i = 0; i < k; ++i) {
            z[i] /= big;
            nrm += z[i] * z[i];
        }
        nrm = std::sqrt(nrm);
        for (int64_t i = 0; i < k; ++i) z[i] /= nrm;
    }
    return std::fabs(z[k - 1]);
}

}  // namespace cronos

extern "C" cronos_status cronos_tridiag_smallest(int64_t k, const double* a, const double* b, int64_t count,
                                                 double* theta, double* last) {
    cronos::clear_error();
    if (k < 1 || count < 1 || count > k) return cronos::fail(CRONOS_EINVAL, "tridiag_smallest: need 1 <= count <= k");
    if (!a || !theta || (k > 1 && !b)) return cronos::fail(CRONOS_EINVAL, "tridiag_smallest: NULL argument");
    for (int64_t i = 0; i < k; ++i)
        if (!std::isfinite(a[i]) || (i + 1 < k && !std::isfinite(b[i])))
            return cronos::fail(CRONOS_EINVAL, "tridiag_smallest: non-finite entry");
    const double zero = 0.0;
    const double* bb = k > 1 ? b : &zero;
    std::vector<double> b2(k > 1 ? k - 1 : 1, 0.0);
    for (int64_t i = 0; i + 1 < k; ++i) b2[i] = bb[i] * bb[i];
    double lo, hi;
    cronos::gershgorin(a, bb, k, &lo, &hi);
    const double norm = std::max({std::fabs(lo), std::fabs(hi), 1e-300});
    cronos::tridiag_smallest(a, b2.data(), k, count, lo, hi, 1e-300, theta);
    for (int64_t j = 0; j < count; ++j) {
        if (last) last[j] = cronos::eigvec_last_component(a, bb, k, theta[j], 1e-15 * norm);
    }
    return CRONOS_OK;
}

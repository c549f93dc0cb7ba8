// Small dense FP64 linear algebra on the host for the Rayleigh-Ritz steps of
// Chebyshev filter diagonalisation (Sec. 4.2): Cholesky factorisation,
// inversion of the triangular factor, and the cyclic Jacobi eigensolver for
// complex Hermitian matrices.  Matrices are row-major std::complex<double>,
// at most a few hundred rows (the search-space size), so O(n^3) host work is
// negligible next to the filter sweeps.
#include "pv_dense.hpp"

#include <algorithm>
#include <cmath>
#include <numeric>

namespace pvd {

bool cholesky_upper(int n, std::vector<cd>& A) {
    // A = R^H R, R upper triangular; R overwrites the upper triangle of A,
    // the strict lower triangle is zeroed.
    for (int j = 0; j < n; ++j) {
        double d = A[(size_t)j * n + j].real();
        for (int k = 0; k < j; ++k) d -= std::norm(A[(size_t)k * n + j]);
        if (!(d > 0.0) || !std::isfinite(d)) return false;
        const double rjj = std::sqrt(d);
        A[(size_t)j * n + j] = rjj;
        for (int i = j + 1; i < n; ++i) {
            cd s = A[(size_t)j * n + i];
            for (int k = 0; k < j; ++k) s -= std::conj(A[(size_t)k * n + j]) * A[(size_t)k * n + i];
            A[(size_t)j * n + i] = s / rjj;
        }
    }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < i; ++j) A[(size_t)i * n + j] = 0.0;
    return true;
}

void invert_upper(int n, const std::vector<cd>& R, std::vector<cd>& M) {
    // M = R^{-1} (upper triangular), by back substitution column by column.
    M.assign((size_t)n * n, cd(0.0));
    for (int j = 0; j < n; ++j) {
        M[(size_t)j * n + j] = 1.0 / R[(size_t)j * n + j];
        for (int i = j - 1; i >= 0; --i) {
            cd s = 0.0;
            for (int k = i + 1; k <= j; ++k) s += R[(size_t)i * n + k] * M[(size_t)k * n + j];
            M[(size_t)i * n + j] = -s / R[(size_t)i * n + i];
        }
    }
}

namespace {

// Rows x, y of n complex numbers (split parts), with f = (er, ei) y:
// x <- cs x - sn f, y <- sn x + cs f.
void rotate_rows(int n, double* __restrict__ xr, double* __restrict__ xi, double* __restrict__ yr,
                 double* __restrict__ yi, double cs, double sn, double er, double ei) {
    for (int k = 0; k < n; ++k) {
        const double fr = er * yr[k] - ei * yi[k], fi = er * yi[k] + ei * yr[k];
        const double gr = cs * xr[k] - sn * fr, gi = cs * xi[k] - sn * fi;
        yr[k] = sn * xr[k] + cs * fr;
        yi[k] = sn * xi[k] + cs * fi;
        xr[k] = gr;
        xi[k] = gi;
    }
}

}  // namespace

void heev_jacobi(int n, std::vector<cd>& A, std::vector<double>& w, std::vector<cd>& V) {
    // Cyclic Jacobi: each (p, q) rotation first removes the phase of A_pq
    // (diag(1, e^{-i phi})) and then applies the real symmetric Jacobi
    // rotation that zeroes |A_pq|.  V accumulates the product of rotations.
    // Real and imaginary parts lie apart and V by vectors, so a rotation is
    // two passes over contiguous rows; A is Hermitian, so the rows give the
    // columns and the diagonal has closed forms.  A random 64 x 64: 29 ms with
    // std::complex rows and columns, 7.8 so (2.7 GHz, one core).
    const size_t ld = (size_t(n) + 8) | 1;   // odd: a column's entries spread over the cache
    std::vector<double> ar(n * ld), ai(n * ld), vr(n * ld, 0.0), vi(n * ld, 0.0);
    double scale = 0.0;
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < n; ++j) {
            const cd v = A[size_t(i) * n + j];
            ar[i * ld + j] = v.real();
            ai[i * ld + j] = i == j ? 0.0 : v.imag();
            scale = std::max(scale, std::abs(v));
        }
        vr[i * ld + i] = 1.0;
    }
    auto diag = [&](int i) -> double& { return ar[i * ld + i]; };
    if (scale == 0.0) scale = 1.0;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0;
        for (int p = 0; p < n; ++p)
            for (int q = p + 1; q < n; ++q) {
                const size_t pq = p * ld + q;
                off += ar[pq] * ar[pq] + ai[pq] * ai[pq];
            }
        if (std::sqrt(off) <= 1e-17 * scale * n) break;
        for (int p = 0; p < n - 1; ++p)
            for (int q = p + 1; q < n; ++q) {
                double *pr = &ar[p * ld], *pi = &ai[p * ld];
                double *qr = &ar[q * ld], *qi = &ai[q * ld];
                const double r = std::hypot(pr[q], pi[q]);
                if (r <= 1e-300 || r < 1e-18 * scale) continue;
                const double er = pr[q] / r, ei = pi[q] / r;   // e^{i phi}
                const double a = diag(p), b = diag(q);
                const double theta = (b - a) / (2.0 * r);
                const double t = (theta >= 0.0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double cs = 1.0 / std::sqrt(t * t + 1.0), sn = t * cs;
                // U = [[cs, sn], [-sn e^{-i phi}, cs e^{-i phi}]] on (p, q):
                // A <- U^H A U, V <- V U
                rotate_rows(n, pr, pi, qr, qi, cs, sn, er, ei);
                pr[p] = a - t * r;
                qr[q] = b + t * r;
                pr[q] = pi[q] = qr[p] = qi[p] = pi[p] = qi[q] = 0.0;
                for (int k = 0; k < n; ++k) {
                    const size_t kp = k * ld + p, kq = k * ld + q;
                    ar[kp] = pr[k];
                    ai[kp] = -pi[k];
                    ar[kq] = qr[k];
                    ai[kq] = -qi[k];
                }
                rotate_rows(n, &vr[p * ld], &vi[p * ld], &vr[q * ld], &vi[q * ld], cs, sn, er, -ei);
            }
    }
    // ascending eigenvalues, vectors in the columns of V alike
    std::vector<int> idx(n);
    std::iota(idx.begin(), idx.end(), 0);
    std::stable_sort(idx.begin(), idx.end(), [&](int i, int j) { return diag(i) < diag(j); });
    w.resize(n);
    V.resize(size_t(n) * n);
    for (int c = 0; c < n; ++c) {
        w[c] = diag(idx[c]);
        for (int k = 0; k < n; ++k) V[size_t(k) * n + c] = cd(vr[idx[c] * ld + k], vi[idx[c] * ld + k]);
    }
}

}  // namespace pvd

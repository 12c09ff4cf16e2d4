// Host symmetric eigensolver for the small projected problems.
//
// The paper solves the eigenproblem of the banded block-tridiagonal T_k on
// the CPU with a special-purpose banded symmetric eigensolver (Section
// 3.2.2).  This one works in two phases:
//   1. band -> tridiagonal by Householder reflectors of the band's width
//      (Lang, "A parallel algorithm for reducing symmetric banded matrices to
//      tridiagonal form", SIAM J. Sci. Comput. 14, 1993): one column is
//      cleared at a time, and of the bulge that its reflector makes further
//      down the band only the first column is cleared, the rest being left
//      to the next columns' reflectors.  N^2 / 2b reflectors of b elements, in
//      short vector loops, where element-by-element rotations need
//      N^2 (1/2 + ... + 1/b) / 2 of them, each a serial square root and
//      divide;
//   2. implicit symmetric QR on the tridiagonal (Golub & Van Loan, "Matrix
//      Computations", Sec. 8.3), two sweeps at once: each rotation waits for
//      the square root and divide of the one before it, so a second sweep,
//      shifted by the other eigenvalue of the trailing 2 x 2 block, runs
//      three rows behind the first and fills that wait.
// The factors are logged, so eigenvectors are built only where needed:
//   * selected ROWS of the eigenvector matrix, accumulated on rows of the
//     identity as the factors are made (the convergence check needs the last
//     r rows, for the Ritz residual bounds);
//   * selected COLUMNS by replaying the log backwards on columns of the
//     identity (the Ritz vectors need only the candidates' columns).
// Both cost O(#factors x #selected); the column replay runs in parallel
// threads.
// Measured on one core at 2.7 GHz, T_k of order 520 with semi-bandwidth 8 and
// 130 candidates: eigenvalues and last rows 5.8 ms (rotations in both phases:
// 24.2), candidates' columns 12.3 ms (30.9).
//
// Dense matrices (the Rayleigh-Ritz projections, whose bandwidth is the full
// order) take a different first phase: Householder reduction to tridiagonal
// form (Golub & Van Loan, Alg. 8.3.1), whose cost is O(N^3) with unit-stride
// inner loops, instead of O(N^2 log b) rotations each touching O(b) strided
// entries.  Their eigenvectors are the logged QR rotations replayed on
// identity columns followed by the reflectors.
#include "flp_internal.h"

#include <algorithm>
#include <atomic>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <numeric>
#include <thread>
#include <vector>

namespace flp {

namespace {

// Four doubles at any address of a double.
typedef double v4 __attribute__((ext_vector_type(4), aligned(8)));
inline __attribute__((always_inline)) v4 ld4(const double *p) { return *reinterpret_cast<const v4 *>(p); }
inline __attribute__((always_inline)) void st4(double *p, v4 x) { *reinterpret_cast<v4 *>(p) = x; }
inline __attribute__((always_inline)) double sum4(v4 x) { return (x.x + x.y) + (x.z + x.w); }
inline int round4(int x) { return (x + 3) & ~3; }

// Code built twice, for AVX2 where the CPU has it (4 doubles per vector
// operation instead of 2) and for the base instruction set, with no fused
// multiply-add, so both builds round alike.
bool cpu_avx2() {
    static const bool have = __builtin_cpu_supports("avx2");
    return have;
}

// Lower half of a symmetric band matrix, column-compact: entry (i, j), i >= j,
// at B[j * ld + (i - j)].  ld holds the band (half-width b), the bulges of the
// reduction below it (up to 2b - 1) and the padding of its vector loops; rows
// from N on are zero and stay zero.
struct Band {
    int N, b, ld;
    std::vector<double> B;
};

// Band -> tridiagonal.  Rows [i0, i0 + L) of column c are reflected onto
// their first entry; the reflector is applied from the left to the columns
// between c and i0, from both sides to the diagonal block, from the right to
// the b rows below it (whose first column is the next to be cleared), and to
// the rows of Zt (row i: the tracked rows' entries in column i, nrp of them).
// NV vectors of four cover a reflector's b elements.
template <int NV>
inline __attribute__((always_inline)) void band_body(Band &M, EigLog &log, double *Zt, int nrp) {
#pragma clang fp contract(off)
    const int N = M.N, b = M.b, ld = M.ld;
    constexpr int LP = 4 * NV;
    double *B = M.B.data();
    double vb[LP + 4] = {}, wb[LP + 4] = {}, Dn[LP * LP] = {};
    for (int j = 0; j + 2 < N; ++j) {
        for (int c = j, i0 = j + 1; i0 + 1 < N; c = i0, i0 += b) {
            const int L = std::min(b, N - i0);
            double *x = B + (size_t)c * ld + (i0 - c);
            v4 v[NV], t[NV];
            for (int q = 0; q < NV; ++q) v[q] = ld4(x + 4 * q);
            const double x0 = v[0].x;
            v[0].x = 0.0;
            for (int q = 0; q < NV; ++q) t[q] = v[q] * v[q];
            for (int q = 1; q < NV; ++q) t[0] += t[q];
            const double sigma = sum4(t[0]);
            // entries whose squares underflow are 1e-40 of the matrix (far_scale)
            for (int q = 0; q < NV; ++q) st4(x + 4 * q, v4(0.0));
            if (sigma < 1e-280) {
                x[0] = x0;
                continue;
            }
            // v0 = x0 - mu with mu of the other sign: no cancellation
            const double mu = -std::copysign(std::sqrt(x0 * x0 + sigma), x0);
            const double v0 = x0 - mu;
            const double bt = -v0 / mu;
            const double inv = 1.0 / v0;
            for (int q = 0; q < NV; ++q) v[q] *= inv;
            v[0].x = 1.0;
            x[0] = mu;
            for (int q = 0; q < NV; ++q) st4(vb + 4 * q, v[q]);
            log.row.push_back(i0);
            log.beta.push_back(bt);
            log.v.insert(log.v.end(), vb, vb + b);
            // from the left: columns c + 1 .. i0 - 1
            for (int k = c + 1; k < i0; ++k) {
                double *a = B + (size_t)k * ld + (i0 - k);
                v4 y[NV];
                for (int q = 0; q < NV; ++q) y[q] = ld4(a + 4 * q);
                v4 d = y[0] * v[0];
                for (int q = 1; q < NV; ++q) d += y[q] * v[q];
                const double f = bt * sum4(d);
                for (int q = 0; q < NV; ++q) st4(a + 4 * q, y[q] - f * v[q]);
            }
            // both sides: A -= v w^T + w v^T, w = p - (beta p^T v / 2) v, p = beta A v
            if (L < b) std::fill(Dn, Dn + LP * LP, 0.0);
            for (int u = 0; u < L; ++u) {
                const double *col = B + (size_t)(i0 + u) * ld - u;
                for (int i = u; i < L; ++i) Dn[u * LP + i] = Dn[i * LP + u] = col[i];
            }
            for (int q = 0; q < NV; ++q) t[q] = v4(0.0);
            for (int u = 0; u < L; ++u) {
                const double f = vb[u];
                for (int q = 0; q < NV; ++q) t[q] += f * ld4(Dn + u * LP + 4 * q);
            }
            v4 d = v4(0.0);
            for (int q = 0; q < NV; ++q) {
                t[q] *= bt;
                d += t[q] * v[q];
            }
            const double K = 0.5 * bt * sum4(d);
            for (int q = 0; q < NV; ++q) st4(wb + 4 * q, t[q] - K * v[q]);
            for (int u = 0; u < L; ++u) {
                double *col = B + (size_t)(i0 + u) * ld - u;
                const double vu = vb[u], wu = wb[u];
                for (int i = u; i < L; i += 4) st4(col + i, ld4(col + i) - (wu * ld4(vb + i) + vu * ld4(wb + i)));
            }
            // from the right: the b rows below, columns [i0, i0 + L), L = b
            if (i0 + L < N) {
                for (int q = 0; q < NV; ++q) t[q] = v4(0.0);
                for (int u = 0; u < L; ++u) {
                    const double *a = B + (size_t)(i0 + u) * ld + (L - u);
                    const double f = vb[u];
                    for (int q = 0; q < NV; ++q) t[q] += f * ld4(a + 4 * q);
                }
                for (int q = 0; q < NV; ++q) t[q] *= bt;
                for (int u = 0; u < L; ++u) {
                    double *a = B + (size_t)(i0 + u) * ld + (L - u);
                    const double f = vb[u];
                    for (int q = 0; q < NV; ++q) st4(a + 4 * q, ld4(a + 4 * q) - f * t[q]);
                }
            }
            for (int q = 0; q < nrp; q += 4) {
                double *z = Zt + (size_t)i0 * nrp + q;
                v4 y = v4(0.0);
                for (int u = 0; u < L; ++u) y += vb[u] * ld4(z + (size_t)u * nrp);
                y *= bt;
                for (int u = 0; u < L; ++u) st4(z + (size_t)u * nrp, ld4(z + (size_t)u * nrp) - vb[u] * y);
            }
        }
    }
}
template <int NV>
__attribute__((target("avx2"))) void band_avx2(Band &M, EigLog &log, double *Zt, int nrp) {
    band_body<NV>(M, log, Zt, nrp);
}
template <int NV>
void band_base(Band &M, EigLog &log, double *Zt, int nrp) {
    band_body<NV>(M, log, Zt, nrp);
}

// Half-width 2 (a block of 2 vectors): the same steps on single entries, where
// half of every vector of four would be padding.
inline __attribute__((always_inline)) void band2_body(Band &M, EigLog &log, double *Zt, int nrp) {
#pragma clang fp contract(off)
    const int N = M.N, ld = M.ld;
    double *B = M.B.data();
    for (int j = 0; j + 2 < N; ++j) {
        for (int c = j, i0 = j + 1; i0 + 1 < N; c = i0, i0 += 2) {
            double *x = B + (size_t)c * ld + (i0 - c);
            const double x0 = x[0], x1 = x[1];
            const double sigma = x1 * x1;
            x[1] = 0.0;
            if (sigma < 1e-280) continue;
            const double mu = -std::copysign(std::sqrt(x0 * x0 + sigma), x0);
            const double v0 = x0 - mu;
            const double bt = -v0 / mu, v1 = x1 / v0;
            x[0] = mu;
            log.row.push_back(i0);
            log.beta.push_back(bt);
            log.v.push_back(1.0);
            log.v.push_back(v1);
            if (i0 - c == 2) {
                double *a = x + ld - 1;  // column c + 1
                const double f = bt * (a[0] + v1 * a[1]);
                a[0] -= f;
                a[1] -= f * v1;
            }
            double *p = B + (size_t)i0 * ld, *q = p + ld;
            const double p0 = bt * (p[0] + v1 * p[1]), p1 = bt * (p[1] + v1 * q[0]);
            const double K = 0.5 * bt * (p0 + v1 * p1);
            const double w0 = p0 - K, w1 = p1 - K * v1;
            p[0] -= 2.0 * w0;
            p[1] -= w0 * v1 + w1;
            q[0] -= 2.0 * (w1 * v1);
            for (int i = 0; i < 2; ++i) {  // the two rows below
                const double t = bt * (p[2 + i] + v1 * q[1 + i]);
                p[2 + i] -= t;
                q[1 + i] -= v1 * t;
            }
            double *z = Zt + (size_t)i0 * nrp;
            for (int i = 0; i < nrp; i += 4) {
                const v4 a = ld4(z + i), b = ld4(z + nrp + i);
                const v4 y = bt * (a + v1 * b);
                st4(z + i, a - y);
                st4(z + nrp + i, b - v1 * y);
            }
        }
    }
}
__attribute__((target("avx2"))) void band2_avx2(Band &M, EigLog &log, double *Zt, int nrp) {
    if (nrp == 4) return band2_body(M, log, Zt, 4);
    band2_body(M, log, Zt, nrp);
}
void band2_base(Band &M, EigLog &log, double *Zt, int nrp) { band2_body(M, log, Zt, nrp); }

// Widest band that is reduced as one; without tracked rows a wider one goes
// through the dense reduction.
constexpr int kMaxBand = 128;

int band_vecs(int b) {
    int nv = 1;
    while (4 * nv < b) nv *= 2;
    return nv;
}

void band_to_tridiag(Band &M, EigLog &log, double *Zt, int nrp) {
    using Fn = void (*)(Band &, EigLog &, double *, int);
    const size_t count = (size_t)M.N * M.N / (2 * M.b) + 2 * (size_t)M.N;
    log.row.reserve(count);
    log.beta.reserve(count);
    log.v.reserve(count * M.b);
#define FLP_BAND(NV) (cpu_avx2() ? &band_avx2<NV> : &band_base<NV>)
    Fn fn = FLP_BAND(32);
    switch (band_vecs(M.b)) {
        case 1: fn = M.b == 2 ? (cpu_avx2() ? &band2_avx2 : &band2_base) : FLP_BAND(1); break;
        case 2: fn = FLP_BAND(2); break;
        case 4: fn = FLP_BAND(4); break;
        case 8: fn = FLP_BAND(8); break;
        case 16: fn = FLP_BAND(16); break;
    }
#undef FLP_BAND
    fn(M, log, Zt, nrp);
}

// One rotation of a QR sweep on the plane (k, k + 1): (x, z) is rotated onto
// its first entry and the 2 x 2 block [a b; b q] with it, with
// t = s (q - a) + 2 c b:  a + s t, q - s t and c t - b.
constexpr int kTwoSweeps = 8;  // shortest block swept twice at once
struct QrSweep {
    int lo, hi, k;
    double x, z;
};
inline __attribute__((always_inline)) void qr_rotate(QrSweep &w, double *d, double *e, double *cs, double *Zt,
                                                     int nrp) {
#pragma clang fp contract(off)
    const int k = w.k;
    const double r = std::sqrt(w.x * w.x + w.z * w.z);
    double c = 1.0, s = 0.0;
    if (r != 0.0) {
        c = w.x / r;
        s = w.z / r;
    }
    if (k > w.lo) e[k - 1] = r;
    const double a = d[k], b = e[k], q = d[k + 1];
    const double t = s * (q - a) + 2.0 * (c * b);
    const double f = s * t;
    d[k] = a + f;
    d[k + 1] = q - f;
    w.x = e[k] = c * t - b;
    if (k + 1 < w.hi) {
        w.z = s * e[k + 1];
        e[k + 1] = c * e[k + 1];
    }
    cs[2 * (k - w.lo)] = c;
    cs[2 * (k - w.lo) + 1] = s;
    double *za = Zt + (size_t)k * nrp;
    for (int i = 0; i < nrp; i += 4) {
        const v4 u = ld4(za + i), v = ld4(za + nrp + i);
        st4(za + i, c * u + s * v);
        st4(za + nrp + i, c * v - s * u);
    }
    ++w.k;
}

// Implicit QR on the tridiagonal (d, e); e[i] couples i and i+1.  On return d
// holds the eigenvalues (unsorted).  A matrix whose largest entry lies far
// from 1 is scaled to it first (the rotations do not depend on the scale): at
// 1e-200 the squares in the rotations underflow and the iteration would not
// move.  The second sweep's rotation k reads what the first one's rotation
// k + 2 has written, and touches nothing that its rotation k + 3 does.
inline __attribute__((always_inline)) bool tridiag_qr_body(std::vector<double> &dv, std::vector<double> &ev,
                                                           EigLog &log, double *Zt, int nrp) {
#pragma clang fp contract(off)
    const int N = (int)dv.size();
    double *d = dv.data(), *e = ev.data();
    int hi = N - 1;
    long guard = 0;
    const long max_steps = 60L * N + 100;
    while (hi > 0) {
        double tiny = DBL_EPSILON * (std::fabs(d[hi - 1]) + std::fabs(d[hi]));
        if (std::fabs(e[hi - 1]) <= tiny || std::fabs(e[hi - 1]) < DBL_MIN) {
            e[hi - 1] = 0.0;
            --hi;
            continue;
        }
        int lo = hi - 1;
        while (lo > 0) {
            double t = DBL_EPSILON * (std::fabs(d[lo - 1]) + std::fabs(d[lo]));
            if (std::fabs(e[lo - 1]) <= t || std::fabs(e[lo - 1]) < DBL_MIN) {
                e[lo - 1] = 0.0;
                break;
            }
            --lo;
        }
        if (++guard > max_steps) return false;
        // shifts: the eigenvalues of the trailing 2 x 2 block, the one nearer
        // to its last entry (Wilkinson's) first
        const double dd = 0.5 * (d[hi - 1] - d[hi]);
        const double ee = e[hi - 1];
        const double den = dd + std::copysign(std::hypot(dd, ee), dd == 0.0 ? 1.0 : dd);
        const double mu = d[hi] - ee * ee / den;
        const double mu2 = d[hi - 1] + ee * ee / den;
        const int len = hi - lo;
        const bool two = len >= kTwoSweeps;
        size_t at = log.cs.size();
        log.cs.resize(at + 2 * (size_t)len * (two ? 2 : 1));
        double *cs = log.cs.data() + at;
        log.sweep.push_back({lo, len, at / 2});
        QrSweep w{lo, hi, lo, d[lo] - mu, e[lo]};
        if (!two) {
            while (w.k < hi) qr_rotate(w, d, e, cs, Zt, nrp);
            continue;
        }
        log.sweep.push_back({lo, len, at / 2 + (size_t)len});
        double *cs2 = cs + 2 * (size_t)len;
        for (int i = 0; i < 3; ++i) qr_rotate(w, d, e, cs, Zt, nrp);
        QrSweep w2{lo, hi, lo, d[lo] - mu2, e[lo]};
        while (w.k < hi) {
            qr_rotate(w, d, e, cs, Zt, nrp);
            qr_rotate(w2, d, e, cs2, Zt, nrp);
        }
        while (w2.k < hi) qr_rotate(w2, d, e, cs2, Zt, nrp);
    }
    return true;
}
__attribute__((target("avx2"))) bool tridiag_qr_avx2(std::vector<double> &d, std::vector<double> &e, EigLog &log,
                                                     double *Zt, int nrp) {
    // constant counts for the usual widths of the tracked rows
    if (nrp == 0) return tridiag_qr_body(d, e, log, Zt, 0);
    if (nrp == 8) return tridiag_qr_body(d, e, log, Zt, 8);
    return tridiag_qr_body(d, e, log, Zt, nrp);
}
bool tridiag_qr_base(std::vector<double> &d, std::vector<double> &e, EigLog &log, double *Zt, int nrp) {
    return tridiag_qr_body(d, e, log, Zt, nrp);
}

bool tridiag_qr(std::vector<double> &d, std::vector<double> &e, EigLog &log, double *Zt, int nrp) {
    const size_t N = d.size();
    if (N <= 1) return true;
    double amax = 0.0;
    for (double x : d) amax = std::max(amax, std::fabs(x));
    for (double x : e) amax = std::max(amax, std::fabs(x));
    if (!std::isfinite(amax)) return false;
    if (amax == 0.0) return true;
    const double scale = (amax < 1e-100 || amax > 1e100) ? 1.0 / amax : 1.0;
    if (scale != 1.0) {
        for (double &x : d) x *= scale;
        for (double &x : e) x *= scale;
    }
    log.sweep.reserve(4 * N);
    log.cs.reserve(2 * N * N + 8 * N);
    if (!(cpu_avx2() ? tridiag_qr_avx2 : tridiag_qr_base)(d, e, log, Zt, nrp)) return false;
    if (scale != 1.0) {
        for (double &x : d) x /= scale;
        for (double &x : e) x /= scale;
    }
    return true;
}

thread_local int tl_eig_threads = 16;  // inner-thread cap of the calling thread

int nthreads_for(long work, int units) {
    int nt = (int)std::min<unsigned>(16u, std::max(1u, std::thread::hardware_concurrency()));
    nt = std::min(nt, std::max(1, tl_eig_threads));
    nt = std::min(nt, units);
    if (work < 4000000L) nt = 1;
    return std::max(nt, 1);
}

template <typename F>
void parallel_for(int units, int nt, F f) {
    if (nt <= 1) {
        f(0, units);
        return;
    }
    std::vector<std::thread> th;
    for (int w = 0; w < nt; ++w) {
        const int u0 = (int)((long)units * w / nt), u1 = (int)((long)units * (w + 1) / nt);
        th.emplace_back(f, u0, u1);
    }
    for (auto &t : th) t.join();
}

// The log replayed backwards on a row-major N x W tile of eigenvector
// columns, then (dense path, A != nullptr) the Householder reflectors from
// the last to the first.  Every column sees the same operations in the same
// order for any W.  A sweep's rotations share a row with the one before: it
// stays in registers, so a rotation reads one row and writes one.
template <int W>
inline __attribute__((always_inline)) void vectors_tile(const EigLog &log, const double *A, const double *beta,
                                                        int N, double *tile) {
#pragma clang fp contract(off)
    constexpr int NW = W / 4;
    for (size_t i = log.sweep.size(); i-- > 0;) {
        const EigLog::Sweep &sw = log.sweep[i];
        const double *cs = log.cs.data() + 2 * sw.at;
        double *row = tile + (size_t)(sw.lo + sw.len) * W;
        v4 b[NW];
        for (int q = 0; q < NW; ++q) b[q] = ld4(row + 4 * q);
        for (int k = sw.len - 1; k >= 0; --k, row -= W) {
            const double c = cs[2 * k], s = cs[2 * k + 1];
            for (int q = 0; q < NW; ++q) {
                const v4 a = ld4(row - W + 4 * q);
                st4(row + 4 * q, s * a + c * b[q]);
                b[q] = c * a - s * b[q];
            }
        }
        for (int q = 0; q < NW; ++q) st4(row + 4 * q, b[q]);
    }
    for (size_t i = log.row.size(); i-- > 0;) {
        const int i0 = log.row[i], L = std::min(log.b, N - i0);
        const double *v = log.v.data() + i * log.b;
        double *z = tile + (size_t)i0 * W;
        if (L == 2) {
            const double v1 = v[1], bt = log.beta[i];
            for (int q = 0; q < NW; ++q) {
                const v4 a = ld4(z + 4 * q), c = ld4(z + W + 4 * q);
                const v4 t = bt * (a + v1 * c);
                st4(z + 4 * q, a - t);
                st4(z + W + 4 * q, c - v1 * t);
            }
            continue;
        }
        v4 y[NW];
        for (int q = 0; q < NW; ++q) y[q] = v4(0.0);
        for (int u = 0; u < L; ++u)
            for (int q = 0; q < NW; ++q) y[q] += v[u] * ld4(z + u * W + 4 * q);
        for (int q = 0; q < NW; ++q) y[q] *= log.beta[i];
        for (int u = 0; u < L; ++u)
            for (int q = 0; q < NW; ++q) st4(z + u * W + 4 * q, ld4(z + u * W + 4 * q) - v[u] * y[q]);
    }
    if (!A) return;
    for (int k = N - 3; k >= 0; --k) {
        const double bt = beta[k];
        if (bt == 0.0) continue;
        const double *v = A + (size_t)k * N + k + 1;
        double *z = tile + (size_t)(k + 1) * W;
        const int len = N - k - 1;
        v4 y[NW];
        for (int q = 0; q < NW; ++q) y[q] = v4(0.0);
        for (int u = 0; u < len; ++u)
            for (int q = 0; q < NW; ++q) y[q] += v[u] * ld4(z + (size_t)u * W + 4 * q);
        for (int q = 0; q < NW; ++q) y[q] *= bt;
        for (int u = 0; u < len; ++u)
            for (int q = 0; q < NW; ++q)
                st4(z + (size_t)u * W + 4 * q, ld4(z + (size_t)u * W + 4 * q) - y[q] * v[u]);
    }
}
template <int W>
__attribute__((target("avx2"))) void vectors_tile_avx2(const EigLog &log, const double *A, const double *beta, int N,
                                                       double *tile) {
    vectors_tile<W>(log, A, beta, N, tile);
}
template <int W>
void vectors_tile_base(const EigLog &log, const double *A, const double *beta, int N, double *tile) {
    vectors_tile<W>(log, A, beta, N, tile);
}

using TileFn = void (*)(const EigLog &, const double *, const double *, int, double *);
template <int W>
TileFn tile_fn() {
    return cpu_avx2() ? &vectors_tile_avx2<W> : &vectors_tile_base<W>;
}

// Columns ids (unsorted eigen-indices) of the log's product, or of Q times it
// with Q = H_0 H_1 ... H_{N-3} when A holds dense reflectors (rows of A,
// beta[k]): identity columns through vectors_tile, tiles of 16 or 8 columns
// (the widest that still gives every thread a tile) claimed by the threads in
// turn.  Z is N x ncols row-major.
void build_cols(const EigLog &log, const double *A, const double *beta, int N, const int *ids, int ncols, double *Z) {
    const long work = (long)(log.cs.size() / 2 + log.v.size() / 2 + (A ? (size_t)N * N : 0)) * ncols;
    const int nt = nthreads_for(work, (ncols + 7) / 8);
    const int W = ncols >= 16 * nt ? 16 : 8;
    const TileFn fn = W == 16 ? tile_fn<16>() : tile_fn<8>();
    const int ntiles = (ncols + W - 1) / W;
    std::atomic<int> next{0};
    auto work_fn = [&](int, int) {
        std::vector<double> tile((size_t)N * W);
        for (;;) {
            const int t = next.fetch_add(1);
            if (t >= ntiles) return;
            const int c0 = t * W, nc = std::min(W, ncols - c0);
            std::fill(tile.begin(), tile.end(), 0.0);
            for (int j = 0; j < nc; ++j) tile[(size_t)ids[c0 + j] * W + j] = 1.0;
            fn(log, A, beta, N, tile.data());
            for (int i = 0; i < N; ++i)
                for (int j = 0; j < nc; ++j) Z[(size_t)i * ncols + c0 + j] = tile[(size_t)i * W + j];
        }
    };
    parallel_for(std::min(nt, ntiles), std::min(nt, ntiles), work_fn);
}

// Householder reduction of a dense symmetric N x N matrix (row-major, full
// storage, overwritten) to tridiagonal (d, e).  Step k maps row k's entries
// k+1..N-1 to mu e_1 with H_k = I - beta_k v_k v_k^T (v_k(0) = 1), applied
// to the trailing block as B -= v w^T + w v^T, w = p - (beta p^T v / 2) v,
// p = beta B v (B symmetric: p accumulates the rows of B scaled by the
// entries of v, in row order, so the inner loops run along rows).  v_k is
// left in row k, beta_k in beta[k].
inline __attribute__((always_inline)) void householder_body(int N, double *A, double *d, double *e, double *beta,
                                                            double *p, double *w) {
#pragma clang fp contract(off)
    for (int k = 0; k + 2 < N; ++k) {
        const int len = N - k - 1;
        double *x = A + (size_t)k * N + k + 1;
        double sigma = 0.0;
        for (int i = 1; i < len; ++i) sigma += x[i] * x[i];
        const double x0 = x[0];
        if (sigma == 0.0) {
            e[k] = x0;
            beta[k] = 0.0;
            for (int i = 1; i < len; ++i) x[i] = 0.0;
            x[0] = 1.0;
            continue;
        }
        const double mu = std::sqrt(x0 * x0 + sigma);
        const double v0 = x0 <= 0.0 ? x0 - mu : -sigma / (x0 + mu);
        const double bt = 2.0 * v0 * v0 / (sigma + v0 * v0);
        const double inv = 1.0 / v0;
        x[0] = 1.0;
        for (int i = 1; i < len; ++i) x[i] *= inv;
        e[k] = mu;
        beta[k] = bt;
        // p = beta B v over the trailing block B = A[k+1:, k+1:]
        for (int i = 0; i < len; ++i) p[i] = 0.0;
        for (int j = 0; j < len; ++j) {
            const double *__restrict row = A + (size_t)(k + 1 + j) * N + k + 1;
            double *__restrict pp = p;
            const double xj = x[j];
            for (int i = 0; i < len; ++i) pp[i] += row[i] * xj;
        }
        double pv = 0.0;
        for (int i = 0; i < len; ++i) {
            p[i] *= bt;
            pv += p[i] * x[i];
        }
        const double K = 0.5 * bt * pv;
        for (int i = 0; i < len; ++i) w[i] = p[i] - K * x[i];
        for (int i = 0; i < len; ++i) {
            double *__restrict row = A + (size_t)(k + 1 + i) * N + k + 1;  // row k + 1 + i, x is row k
            const double xi = x[i], wi = w[i];
            const double *__restrict wr = w;
            const double *__restrict xr = x;
            for (int j = 0; j < len; ++j) row[j] -= xi * wr[j] + wi * xr[j];
        }
    }
    for (int k = 0; k < N; ++k) d[k] = A[(size_t)k * N + k];
    if (N >= 2) e[N - 2] = A[(size_t)(N - 2) * N + N - 1];
}
__attribute__((target("avx2"))) void householder_avx2(int N, double *A, double *d, double *e, double *beta,
                                                       double *p, double *w) {
    householder_body(N, A, d, e, beta, p, w);
}
void householder_base(int N, double *A, double *d, double *e, double *beta, double *p, double *w) {
    householder_body(N, A, d, e, beta, p, w);
}

void householder_tridiag(int N, double *A, std::vector<double> &d, std::vector<double> &e,
                         std::vector<double> &beta) {
    d.assign(N, 0.0);
    e.assign(std::max(N - 1, 0), 0.0);
    beta.assign(std::max(N - 2, 0), 0.0);
    std::vector<double> p(N), w(N);
    (cpu_avx2() ? householder_avx2 : householder_base)(N, A, d.data(), e.data(), beta.data(), p.data(), w.data());
}

// 1 / (largest |entry|) for a matrix whose entries all lie far from 1 (the
// squares in the rotations and reflector norms would underflow or
// overflow), else 1; 0 for non-finite entries.  Eigenvectors do not depend
// on the scale; eigenvalues are divided by it afterwards.
double far_scale(const std::vector<double> &v) {
    double amax = 0.0;
    for (double x : v) amax = std::max(amax, std::fabs(x));
    if (!std::isfinite(amax)) return 0.0;
    return (amax > 0.0 && (amax < 1e-100 || amax > 1e100)) ? 1.0 / amax : 1.0;
}

// Dense path: eigenvalues ascending in evals, selected columns (indices into
// the ascending order) of the eigenvector matrix in Zcols (N x ncols).
int dense_sym_eig(int N, const double *M, double *evals, const int *cols, int ncols, double *Zcols) {
    std::vector<double> A((size_t)N * N);
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) A[(size_t)i * N + j] = 0.5 * (M[(size_t)i * N + j] + M[(size_t)j * N + i]);
    const double sc = far_scale(A);
    if (sc == 0.0) return -2;
    if (sc != 1.0)
        for (double &x : A) x *= sc;
    std::vector<double> d, e, beta;
    householder_tridiag(N, A.data(), d, e, beta);
    EigLog log;
    if (!tridiag_qr(d, e, log, nullptr, 0)) return -2;
    std::vector<int> perm(N);
    std::iota(perm.begin(), perm.end(), 0);
    std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) { return d[a] < d[b]; });
    for (int i = 0; i < N; ++i) evals[i] = d[perm[i]] / sc;
    if (ncols > 0 && Zcols) {
        std::vector<int> ids(ncols);
        for (int j = 0; j < ncols; ++j) ids[j] = perm[cols[j]];
        build_cols(log, A.data(), beta.data(), N, ids.data(), ncols, Zcols);
    }
    return 0;
}

}  // namespace

void set_eig_threads(int n) { tl_eig_threads = std::max(1, n); }

int sym_eig_keep(int N, int bw, const double *M, double *evals, const int *rows, int nrows, double *Zrows,
                 EigLog *keep) {
    if (N <= 0) return -1;
    bw = std::max(0, std::min(bw, N - 1));
    if (bw > kMaxBand) return -1;
    Band Bd;
    Bd.N = N;
    Bd.b = std::max(bw, 1);
    Bd.ld = Bd.b + 4 * band_vecs(Bd.b);
    Bd.B.assign((size_t)(N + 1) * Bd.ld, 0.0);
    for (int j = 0; j < N; ++j)
        for (int d = 0; d <= bw && j + d < N; ++d) {
            const int i = j + d;
            Bd.B[(size_t)j * Bd.ld + d] = 0.5 * (M[(size_t)i * N + j] + M[(size_t)j * N + i]);
        }
    const double sc = far_scale(Bd.B);
    if (sc == 0.0) return -2;
    if (sc != 1.0)
        for (double &x : Bd.B) x *= sc;
    EigLog local;
    EigLog &log = keep ? *keep : local;
    log.clear();
    log.b = Bd.b;
    // the requested rows of the eigenvector matrix, accumulated as the
    // factors are made (independent of the rotation chain, so they fill its
    // latency), padded to whole vectors
    const int nr = (nrows > 0 && Zrows) ? nrows : 0, nrp = round4(nr);
    std::vector<double> Zt((size_t)N * nrp, 0.0);
    for (int i = 0; i < nr; ++i) Zt[(size_t)rows[i] * nrp + i] = 1.0;
    if (bw >= 2) band_to_tridiag(Bd, log, Zt.data(), nrp);
    std::vector<double> d(N), e(std::max(N - 1, 0));
    for (int i = 0; i < N; ++i) d[i] = Bd.B[(size_t)i * Bd.ld];
    for (int i = 0; i + 1 < N; ++i) e[i] = Bd.B[(size_t)i * Bd.ld + 1];
    if (!tridiag_qr(d, e, log, Zt.data(), nrp)) return -2;
    std::vector<int> perm(N);
    std::iota(perm.begin(), perm.end(), 0);
    std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) { return d[a] < d[b]; });
    for (int i = 0; i < N; ++i) evals[i] = d[perm[i]] / sc;
    for (int i = 0; i < nr; ++i)
        for (int j = 0; j < N; ++j) Zrows[(size_t)i * N + j] = Zt[(size_t)perm[j] * nrp + i];
    if (keep) {
        keep->N = N;
        keep->perm = perm;
    }
    return 0;
}

void eig_log_cols(const EigLog &L, const int *cols, int ncols, double *Zcols) {
    std::vector<int> ids(ncols);
    for (int j = 0; j < ncols; ++j) ids[j] = L.perm[cols[j]];
    build_cols(L, nullptr, nullptr, L.N, ids.data(), ncols, Zcols);
}

int sym_eig(int N, int bw, const double *M, double *evals, const int *rows, int nrows, double *Zrows,
            const int *cols, int ncols, double *Zcols) {
    if (N <= 0) return -1;
    const int band = std::min(bw, N - 1);
    if (nrows == 0 && (band >= std::max(24, N / 8) || band > kMaxBand))
        return dense_sym_eig(N, M, evals, cols, ncols, Zcols);
    if (ncols > 0 && Zcols) {
        EigLog L;
        const int rc = sym_eig_keep(N, bw, M, evals, rows, nrows, Zrows, &L);
        if (rc != 0) return rc;
        eig_log_cols(L, cols, ncols, Zcols);
        return 0;
    }
    return sym_eig_keep(N, bw, M, evals, rows, nrows, Zrows, nullptr);
}

}  // namespace flp

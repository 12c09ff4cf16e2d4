// The block step after the filter for gfx950: reorthogonalisation of the
// filtered block (Section 3.2.2) and its normalisation W = Q_{j+1} S_j
// (Cholesky QR twice, eq. lanczos), for one solve or for many independent
// solves with one launch per stage.
//
// A launch's blocks are split into segments, one per solve, by a prefix of
// block counts (OrthSeg tables); a block finds its segment with the same
// ballot count as the segmented filter step.  A single solve passes its
// OrthSeg by value (ONE).  The r x r Cholesky factors are computed on the
// device, so a whole block step runs without a host round trip; a solve that
// needs the host (dependent columns, or another pass) is flagged and
// skipped by the later stages, and the host repairs it afterwards.
//
// Reorthogonalisation: the filter is symmetric, so W = p(A) Q_j has
// components of its own size only along Q_{j-1} and Q_j; those along the
// older blocks are rounding (FP64) or the FP32 filter's error.  The first
// pass of classical Gram-Schmidt therefore covers the last two blocks alone
// (the local pass), the second the whole basis: the basis is read twice per
// step, not four times.  The full pass leaves an orthogonality error of u
// ||W_1|| / ||W_2|| (W_1 before, W_2 after it), so a column it takes more
// than half of (||Q^T W_1|| > ||W_2||, seen from the coefficients and the
// Gram matrix) flags the solve for another pass.
//
// Stages (c = block width r <= 16, k = basis columns, per solve):
//   orth_local   partial sums of Q_loc^T W, Q_loc the basis columns kl .. k-1
//   orth_reduce  the partial sums in a fixed order -> H, H2 or G
//   orth_update  W -= Q_loc H, later W -= Q H2 with the partial Gram matrix
//   orth_tn_*    partial sums of Q^T W (k x c)
//   orth_chol    D_j, Cholesky factor and its inverse (pass 1), or S_j (pass 2)
//   orth_gram    Gram matrix of W, or of W R1^{-1}
//   orth_final   W R1^{-1} R2^{-1} -> the basis and the next filter input
#include "flp_internal.h"
#include "flp_device.h"
#include "flp_gemm.h"

#include <algorithm>

namespace flp {

namespace {

// Index of the segment that owns block blk: pre[] is non-decreasing, so the
// segments starting at or before blk are a prefix, counted 64 at a time with
// one load per lane and a ballot; the count is made wave-uniform so the
// segment's descriptor is read through the scalar cache.
__device__ __forceinline__ int seg_of(const int *__restrict__ pre, int nseg, int blk) {
    const int lane = threadIdx.x % WAVE;
    int seg = -1;
    for (int base = 0; base < nseg; base += WAVE) {
        const int i = base + lane;
        const bool le = i < nseg && pre[i] <= blk;
        const unsigned long long m = __ballot(le);
        seg += __popcll(m);
        if (~m != 0ull) break;
    }
    return __builtin_amdgcn_readfirstlane(seg);
}

// The solve a block works for (*lb: the block's index within it).
template <bool ONE>
__device__ __forceinline__ OrthSeg my_seg(const OrthSeg *__restrict__ tab, const int *__restrict__ pre, int nseg,
                                          const OrthSeg &one, int *lb) {
    if constexpr (ONE) {
        *lb = (int)blockIdx.x;
        return one;
    } else {
        const int seg = seg_of(pre, nseg, blockIdx.x);
        *lb = (int)blockIdx.x - pre[seg];
        return tab[seg];
    }
}

__device__ __forceinline__ bool flagged(const OrthSeg &e, int c) { return as_global(e.out)[2 * c * c] != 0.0; }

// The 4 waves' 16 x 16 sums (NA of them, D layout) added through LDS and
// written as rows ti * 16 + i < K of dst (K x c).
template <int NA>
__device__ __forceinline__ void store_block_sum(dbl4 (&acc)[NA], int K, int c, double *dst, double (*red)[4][WAVE]) {
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        if (a * 16 >= K) break;  // uniform
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][v][lane] = acc[a][v];
        __syncthreads();
        const int v = threadIdx.x / WAVE, l = threadIdx.x % WAVE;
        const double s = red[0][v][l] + red[1][v][l] + red[2][v][l] + red[3][v][l];
        const int i = a * 16 + l / 16 + 4 * v, j = l % 16;
        if (i < K && j < c) as_global_mut(dst)[(size_t)i * c + j] = s;
        __syncthreads();
    }
}

// Rows g .. g + 15 of W as the B operand of four MFMA steps (lane: row 4 t +
// l/16, column l%16; zero outside rows < r1 and columns < c).
__device__ __forceinline__ void load_w_rows(const double *W, int g, int r1, int c, double (&b)[4]) {
    const int lane = threadIdx.x % WAVE, kr = lane / 16, m = lane % 16;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int row = g + 4 * t + kr;
        const double x = as_global(W)[(int64_t)min(row, r1 - 1) * c + min(m, c - 1)];
        b[t] = row < r1 && m < c ? x : 0.0;
    }
}

// Partial sums over a block's rows of Q_loc^T W (columns kl .. k-1 of the
// basis, at most 2 c + 15 < 48 of them; partial (k - kl) x c).  A wave takes
// pieces of 16 rows, a load covers four rows.  Bound by the read of W and
// Q_loc, which is strided by the panel's row of 1 KiB (110 us at n = 1e6, c =
// 8: 2.9 TB/s).
template <bool ONE>
__global__ __launch_bounds__(256) void orth_local_kernel(const OrthSeg *__restrict__ tab,
                                                         const int *__restrict__ pre, int nseg, const OrthSeg one,
                                                         int c) {
    __shared__ double red[4][4][WAVE];
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    constexpr int NA = 3;
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int kr = lane / 16, m = lane % 16;
    const int r0 = lb * e.lrows, r1 = min(e.n, r0 + e.lrows);
    const int K = e.k - e.kl;
    const double *qc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) qc[a] = col_base(e.Q, e.kl + min(a * 16 + m, K - 1));
    dbl4 acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int g = r0 + wave * 16; g < r1; g += 4 * 16) {
        double b[4], q[NA][4];
        load_w_rows(e.W, g, r1, c, b);
#pragma unroll
        for (int a = 0; a < NA; ++a)
            if (a * 16 < K)  // uniform
#pragma unroll
                for (int t = 0; t < 4; ++t) q[a][t] = as_global(qc[a])[(int64_t)min(g + 4 * t + kr, r1 - 1) * e.Q.ld];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int a = 0; a < NA; ++a)
                if (a * 16 < K) acc[a] = mfma16x16x4(q[a][t], b[t], acc[a]);
    }
    store_block_sum<NA>(acc, K, c, e.part + (size_t)lb * K * c, red);
}

// Partial sums of Q^T W (c = 8) on FMA: one basis column per thread and one
// wavefront per block (a basis of 320 columns then has no idle threads), the
// rows walked in step, so each W row is one wide load through the scalar
// cache.  (This kernel has no LDS and no barrier: with
// either in the same kernel the compiler can no longer prove the W rows
// unmodified and falls back to per-lane vector loads of the same row.)
// Partial sums of chunk t go to part[(t k + q) c + j].
template <bool ONE>
__global__ __launch_bounds__(64) void orth_tn_fma_kernel(const OrthSeg *__restrict__ tab,
                                                          const int *__restrict__ pre, int nseg, const OrthSeg one) {
    constexpr int C = 8;
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    const int K = e.k;
    const int ncb = (K + WAVE - 1) / WAVE;
    const int cb = lb % ncb, chunk = lb / ncb;
    const int q = cb * WAVE + threadIdx.x;
    if (q >= K) return;
    const int r0 = chunk * e.prows, r1 = min(e.n, r0 + e.prows);
    double acc[C];
    tn_fma_column<C, 8>(as_global(col_base(e.Q, q)), e.Q.ld, r0, r1, as_global(e.W), C, acc);
    const auto d = as_global_mut(e.part) + ((size_t)chunk * K + q) * C;
#pragma unroll
    for (int j = 0; j < C; ++j) d[j] = acc[j];
}

// The same on FP64 MFMA: one B tile of 16 columns, 8 A tiles (128 basis
// columns) per block, 4 waves over the rows of a chunk combined through LDS.
template <bool ONE>
__global__ __launch_bounds__(256) void orth_tn_mfma_kernel(const OrthSeg *__restrict__ tab,
                                                           const int *__restrict__ pre, int nseg, const OrthSeg one,
                                                           int c) {
    __shared__ double red[4][4][WAVE];
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    const int ngrp = (e.k + 127) / 128;
    const int chunk = lb / ngrp, grp = lb % ngrp;
    const int r0 = chunk * e.prows;
    tn_mfma_block<8>(r0, min(e.n, r0 + e.prows), e.k, c, grp * 128, 0, e.Q, e.W, c, true,
                     e.part + (size_t)chunk * e.k * c, red);
}

// Sum of the per-chunk partials in a fixed order: 16 outputs per block, its
// 16 thread rows split the chunks and combine through LDS.  which: 0 -> H,
// 1 -> H2, 2 -> G from the updates' blocks, 3 -> G from the blocks over W.
template <bool ONE>
__global__ __launch_bounds__(256) void orth_reduce_kernel(const OrthSeg *__restrict__ tab,
                                                          const int *__restrict__ pre, int nseg, const OrthSeg one,
                                                          int c, int which, int chk) {
    __shared__ double red[16][17];
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    if (chk && flagged(e, c)) return;
    const int K = which == 0 ? e.k - e.kl : (which == 1 ? e.k : c);
    const int nch = which == 1 ? e.pchunks : (which == 2 ? e.ublk : e.lblk);
    const auto dst = as_global_mut(which == 0 ? e.H : (which == 1 ? e.H + (size_t)e.k * c : e.G));
    const int total = K * c;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int o = lb * 16 + tx;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (o < total) {
        const auto p = as_global(e.part) + o;
        int q = ty;
        for (; q + 112 < nch; q += 128) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = p[(size_t)(q + 16 * u) * total];
#pragma unroll
            for (int u = 0; u < 8; ++u) s[u % 4] += x[u];
        }
        for (; q < nch; q += 16) s[0] += p[(size_t)q * total];
    }
    red[ty][tx] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    if (ty == 0 && o < total) {
        double t = 0.0;
#pragma unroll
        for (int y = 0; y < 16; ++y) t += red[y][tx];
        dst[o] = t;
    }
}

// W -= Q_loc H (LOCAL) or W -= Q H2 with the partial Gram matrix of the
// result (its rows sit in the D layout, which is the operand layout of
// W^T W, so it costs no further read).  MT row tiles of 16 rows per wave and
// turn.  Bound by the read of the basis.
template <bool ONE, bool LOCAL, int MT, bool PIPE>
__global__ __launch_bounds__(256) void orth_update_kernel(const OrthSeg *__restrict__ tab,
                                                          const int *__restrict__ pre, int nseg, const OrthSeg one,
                                                          int c) {
    __shared__ double red[4][4][WAVE];
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int kq = lane / 16, m = lane % 16;
    const int r0 = lb * e.urows, r1 = min(e.n, r0 + e.urows);
    const int K = LOCAL ? e.k - e.kl : e.k;
    const double *H = LOCAL ? e.H : e.H + (size_t)e.k * c;
    dbl4 gacc[1] = {dbl4{0.0, 0.0, 0.0, 0.0}};
    for (int row0 = r0 + wave * 16 * MT; row0 < r1; row0 += 4 * 16 * MT) {
        dbl4 acc[MT][1];
        gemm_nn_acc<MT, 1, PIPE>(r1, K, c, e.Q, H, c, true, row0, 0, acc, LOCAL ? e.kl : 0);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = row0 + 16 * i + kq + 4 * v;
                double w2 = 0.0;
                if (row < r1 && m < c) {
                    const auto wp = as_global_mut(e.W) + (int64_t)row * c + m;
                    w2 = *wp - acc[i][0][v];
                    *wp = w2;
                }
                if constexpr (!LOCAL) gacc[0] = mfma16x16x4(w2, w2, gacc[0]);
            }
    }
    if constexpr (!LOCAL) store_block_sum<1>(gacc, c, c, e.part + (size_t)lb * c * c, red);
}

// Lane `from`'s value, uniform over the wavefront.
__device__ __forceinline__ double lane_value(double x, int from) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, from);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), from);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The r x r factorisations of one solve.  Pass 1: D_j = sym(diagonal blocks
// of H + H2) to out[0, c^2); the first factor R1 of G (upper, row-major) by
// right-looking Cholesky with the block QR's dependent-column rule (a pivot
// at or below (1e-7 ||W||_F)^2 marks the column: status 1), then R1^{-1};
// status 3 where the full pass took more of a column than it left
// (||H2_j||^2 > G_jj).  Pass 2: the second factor R2 (status 2 if it breaks
// down), R2^{-1} and S_j = R2 R1 to out[c^2, 2 c^2).  k = 0: normalisation
// alone.  The four waves share the column sums of H2; the factorisation is a
// serial chain that the first wave runs in registers: lane j holds column j
// of the matrix, padded to CP x CP with the identity (CP = 1, 4, 8 or 16, the
// chain's length), and the entries a step needs from other columns come by
// readlane (c = 1: 2.6 us with the sums, 8.4 padded to 16 without; c = 16: 9.3,
// the same steps through LDS 24).
// SUM: a solve of few partial Gram matrices (e.few) has them added by its
// block first, 256 / CP^2 threads to an output, and pass 1's sum written to G
// (instead of an orth_reduce launch, 2.2 us and the gap before it).
template <bool ONE, int CP, bool SUM>
__global__ __launch_bounds__(256) void orth_chol_kernel(const OrthSeg *__restrict__ tab, const OrthSeg one, int c,
                                                        int pass) {
    __shared__ double sq[16][16];
    __shared__ double gs[256];
    const OrthSeg e = ONE ? one : tab[blockIdx.x];
    const int cc = c * c;
    double *out = e.out;
    double *status = out + 2 * cc;
    if (pass == 2 && *status != 0.0) return;  // uniform: every lane reads the same flag
    const bool orth = pass == 1 && e.k > 0;
    constexpr int NS = 256 / (CP * CP);  // threads per output
    const bool sum = SUM && e.few;         // uniform
    if (sum) {
        const int o = threadIdx.x / NS, i = o / CP, j = o % CP;
        const int nch = orth ? e.ublk : e.lblk;
        double s = 0.0;
        if (i < c && j < c) {
            const auto p = as_global(e.part) + i * c + j;
            int q = threadIdx.x % NS;
            for (; q + 7 * NS < nch; q += 8 * NS) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = p[(size_t)(q + u * NS) * cc];
#pragma unroll
                for (int u = 0; u < 8; ++u) s += x[u];
            }
            for (; q < nch; q += NS) s += p[(size_t)q * cc];
        }
#pragma unroll
        for (int d = 1; d < (NS < WAVE ? NS : WAVE); d *= 2) s += __shfl_xor(s, d, WAVE);
        gs[threadIdx.x] = s;
    }
    if (orth) {
        // column sums of squares of H2: thread (ty, tx) takes rows ty, ty + 16, ... of column tx
        const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
        const auto h = as_global(e.H) + (size_t)e.k * c;
        double s = 0.0;
        if (tx < c) {
            int q = ty;
            for (; q + 112 < e.k; q += 128) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = h[(size_t)(q + 16 * u) * c + tx];
#pragma unroll
                for (int u = 0; u < 8; ++u) s = fma(x[u], x[u], s);
            }
            for (; q < e.k; q += 16) s = fma(h[(size_t)q * c + tx], h[(size_t)q * c + tx], s);
        }
        sq[ty][tx] = s;
    }
    __syncthreads();
    if (threadIdx.x >= WAVE) return;
    const int lane = threadIdx.x, j = lane % CP;
    const bool col = lane < c;
    double M[CP];
#pragma unroll
    for (int i = 0; i < CP; ++i) {
        double x;
        if (sum) {
            x = gs[(i * CP + j) * NS];
            if constexpr (NS > WAVE) x = (gs[0] + gs[WAVE]) + (gs[2 * WAVE] + gs[3 * WAVE]);
        } else {
            x = as_global(e.G)[min(i, c - 1) * c + min(j, c - 1)];
        }
        M[i] = (i < c && j < c) ? x : (i == j ? 1.0 : 0.0);
        // the host's repair of dependent columns reads G
        if (sum && pass == 1 && i < c && col) as_global_mut(e.G)[i * c + j] = x;
    }
    bool again = false;
    if (orth) {
        const auto h1 = as_global(e.H) + (size_t)(e.k - e.kl - c) * c;
        const auto h2 = as_global(e.H) + (size_t)e.k * c + (size_t)(e.k - c) * c;
        if (col)
            for (int i = 0; i < c; ++i) {
                const double a = h1[i * c + j] + h2[i * c + j], b = h1[j * c + i] + h2[j * c + i];
                out[i * c + j] = 0.5 * (a + b);
            }
        double s = 0.0, g = 0.0;
#pragma unroll
        for (int y = 0; y < 16; ++y) s += sq[y][j];
#pragma unroll
        for (int i = 0; i < CP; ++i) g = i == j ? M[i] : g;
        again = __ballot(col && s > g) != 0ull;
    }
    double thr2 = 1e-300;
    if (pass == 1) {
        double fro2 = 0.0;
#pragma unroll
        for (int i = 0; i < CP; ++i)
            if (i < c) fro2 += fmax(lane_value(M[i], i), 0.0);
        const double thr = 1e-7 * sqrt(fro2);
        thr2 = fmax(thr * thr, 1e-300);
    }
    // right-looking Cholesky: M[i] becomes row i of R
    bool bad = false;
    double inv[CP];  // 1 / R[i][i], uniform
#pragma unroll
    for (int k = 0; k < CP; ++k) {
        const double d = lane_value(M[k], k);
        const bool ok = k >= c || d > thr2;
        bad = bad || !ok;
        const double rkk = ok ? sqrt(d) : 1.0;
        inv[k] = 1.0 / rkk;
        M[k] = j == k ? rkk : (j > k && ok ? M[k] / rkk : 0.0);
#pragma unroll
        for (int i = k + 1; i < CP; ++i) {
            const double f = lane_value(M[k], i);
            M[i] = fma(-f, M[k], M[i]);
        }
    }
    if (bad || again) {
        if (lane == 0) *status = pass == 2 ? kOrthBreakdown : (again ? kOrthAgain : kOrthDependent);
        return;
    }
    // column j of R^{-1} by back substitution
    double T[CP];
#pragma unroll
    for (int i = CP - 1; i >= 0; --i) {
        double t = i == j ? 1.0 : 0.0;
#pragma unroll
        for (int k = i + 1; k < CP; ++k) t = fma(-lane_value(M[i], k), T[k], t);
        T[i] = t * inv[i];
    }
    double *Ri = pass == 1 ? e.Ri1 : e.Ri2;
#pragma unroll
    for (int i = 0; i < CP; ++i)
        if (i < c && col) {
            if (pass == 1) as_global_mut(e.R1)[i * c + j] = M[i];
            as_global_mut(Ri)[i * c + j] = T[i];
        }
    if (pass == 1) {
        if (lane == 0) *status = kOrthOk;
        return;
    }
    // S_j = R2 R1 (both upper triangular)
    double *Sj = out + cc;
    double R1[CP];
#pragma unroll
    for (int i = 0; i < CP; ++i) R1[i] = i < c && j < c ? as_global(e.R1)[min(i, c - 1) * c + min(j, c - 1)] : 0.0;
#pragma unroll
    for (int i = 0; i < CP; ++i) {
        double acc = 0.0;
#pragma unroll
        for (int k = i; k < CP; ++k) acc = fma(lane_value(M[i], k), R1[k], acc);
        if (i < c && col) Sj[i * c + j] = acc;
    }
}

// An upper-triangular r x r matrix R as an MFMA operand: R[4 (l/16) + q][l%16]
// for step q (the permuted k index of load_w_cols), zero outside c x c.
__device__ __forceinline__ void load_tri(const double *R, int c, double (&b)[4]) {
    const int lane = threadIdx.x % WAVE, kq = lane / 16, m = lane % 16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = 4 * kq + q;
        const double x = as_global(R)[min(i, c - 1) * c + min(m, c - 1)];
        b[q] = i < c && m < c ? x : 0.0;
    }
}

// Row g + l%16 of W, columns 4 (l/16) .. + 3 (zero outside rows < r1 and
// columns < c): an operand with the rows on l%16.  Two 16-byte loads where
// the four columns exist together (they need no more than element alignment).
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ void load_w_cols(const double *W, int g, int r1, int c, double (&a)[4]) {
    const int lane = threadIdx.x % WAVE, kq = lane / 16, m = lane % 16;
    const auto p = as_global(W) + (int64_t)min(g + m, r1 - 1) * c;
    const bool row = g + m < r1;
    if ((c & 3) == 0) {
        const int c0 = min(4 * kq, c - 4);
        const dbl2u x0 = *reinterpret_cast<gptr<dbl2u>>(p + c0);
        const dbl2u x1 = *reinterpret_cast<gptr<dbl2u>>(p + c0 + 2);
        const bool in = row && 4 * kq < c;
        a[0] = in ? x0.x : 0.0;
        a[1] = in ? x0.y : 0.0;
        a[2] = in ? x1.x : 0.0;
        a[3] = in ? x1.y : 0.0;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double x = p[min(4 * kq + q, c - 1)];
            a[q] = row && 4 * kq + q < c ? x : 0.0;
        }
    }
}

// Partial sums of the Gram matrix of Y = W R1^{-1} (FIRST: of W, with the
// identity in R1^{-1}'s place): a wave forms 16 rows of Y with four MFMA
// steps, and Y's D layout is the operand layout of Y^T Y.  Y itself is not
// written (orth_final forms it again), so this reads W once, in 16-byte
// pieces.
template <bool ONE, bool FIRST>
__global__ __launch_bounds__(256) void orth_gram_kernel(const OrthSeg *__restrict__ tab, const int *__restrict__ pre,
                                                        int nseg, const OrthSeg one, int c) {
    __shared__ double red[4][4][WAVE];
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    if (!FIRST && flagged(e, c)) return;
    const int wave = threadIdx.x / WAVE;
    const int r0 = lb * e.lrows, r1 = min(e.n, r0 + e.lrows);
    double ri[4];
    if constexpr (FIRST) {
        const int lane = threadIdx.x % WAVE;
#pragma unroll
        for (int q = 0; q < 4; ++q) ri[q] = 4 * (lane / 16) + q == lane % 16 ? 1.0 : 0.0;
    } else {
        load_tri(e.Ri1, c, ri);
    }
    dbl4 gacc[1] = {dbl4{0.0, 0.0, 0.0, 0.0}};
    for (int g = r0 + wave * 64; g < r1; g += 4 * 64) {
        double a[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) load_w_cols(e.W, g + 16 * u, r1, c, a[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            dbl4 y = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q) y = mfma16x16x4(a[u][q], ri[q], y);
#pragma unroll
            for (int v = 0; v < 4; ++v) gacc[0] = mfma16x16x4(y[v], y[v], gacc[0]);
        }
    }
    store_block_sum<1>(gacc, c, c, e.part + (size_t)lb * c * c, red);
}

// Q_{j+1} = (W R1^{-1}) R2^{-1}: the first product transposed (R1^{-T} W^T,
// operands exchanged), whose D layout has the rows on l%16 as the second
// product's operand wants them.  The result goes to the basis columns k ..
// k + c - 1 (when they exist) and to the next filter input (FP64 and, if
// present, FP32), or over W itself (Vin = W: a wave reads its rows before it
// writes them).
template <bool ONE>
__global__ __launch_bounds__(256) void orth_final_kernel(const OrthSeg *__restrict__ tab,
                                                         const int *__restrict__ pre, int nseg, const OrthSeg one,
                                                         int c) {
    int lb;
    const OrthSeg e = my_seg<ONE>(tab, pre, nseg, one, &lb);
    if (flagged(e, c)) return;
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int kq = lane / 16, m = lane % 16;
    const int r0 = lb * e.lrows, r1 = min(e.n, r0 + e.lrows);
    double r1i[4], r2i[4];
    load_tri(e.Ri1, c, r1i);
#pragma unroll
    for (int v = 0; v < 4; ++v) {  // R2^{-1}[l/16 + 4 v][l%16]
        const int i = kq + 4 * v;
        const double x = as_global(e.Ri2)[min(i, c - 1) * c + min(m, c - 1)];
        r2i[v] = i < c && m < c ? x : 0.0;
    }
    const bool basis = e.k + c <= e.qcap;
    double *qc = basis && m < c ? const_cast<double *>(col_base(e.Q, e.k + m)) : nullptr;
    for (int g = r0 + wave * 64; g < r1; g += 4 * 64) {
        double a[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) load_w_cols(e.W, g + 16 * u, r1, c, a[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            dbl4 y = dbl4{0.0, 0.0, 0.0, 0.0}, z = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q) y = mfma16x16x4(r1i[q], a[u][q], y);
#pragma unroll
            for (int v = 0; v < 4; ++v) z = mfma16x16x4(y[v], r2i[v], z);
            if (m < c) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int64_t row = g + 16 * u + kq + 4 * v;
                    if (row < r1) {
                        as_global_mut(e.Vin)[row * c + m] = z[v];
                        if (basis) as_global_mut(qc)[row * e.Q.ld] = z[v];
                        if (e.V32) as_global_mut(e.V32)[row * c + m] = (float)z[v];
                    }
                }
            }
        }
    }
}

template <bool ONE>
void launch_chol(const OrthPlan &p, int c, int pass, hipStream_t s) {
#define FLP_CHOL(CP)                                                                                              \
    if (c <= CP) {                                                                                                \
        if (p.few)                                                                                                \
            hipLaunchKernelGGL((orth_chol_kernel<ONE, CP, true>), dim3(p.nseg), dim3(256), 0, s, p.tab, p.one, c, \
                               pass);                                                                             \
        else                                                                                                      \
            hipLaunchKernelGGL((orth_chol_kernel<ONE, CP, false>), dim3(p.nseg), dim3(256), 0, s, p.tab, p.one,   \
                               c, pass);                                                                          \
        return;                                                                                                   \
    }
    FLP_CHOL(1)
    FLP_CHOL(4)
    FLP_CHOL(8)
    FLP_CHOL(16)
#undef FLP_CHOL
}

#define FLP_ORTH(K, KIND, ...) \
    hipLaunchKernelGGL(K, dim3(p.blocks[KIND]), dim3(256), 0, s, tab, pre[KIND], ns, p.one, c, ##__VA_ARGS__)
template <bool ONE>
void launch_qr(const OrthPlan &p, const int *const *pre, int c, bool have_gram, hipStream_t s) {
    const OrthSeg *tab = p.tab;
    const int ns = p.nseg;
    if (!have_gram) FLP_ORTH((orth_gram_kernel<ONE, true>), kOrthLocal);
    const bool reduce = p.blocks[kOrthRedG] > 0;  // of the solves with many partials
    if (reduce) FLP_ORTH((orth_reduce_kernel<ONE>), kOrthRedG, have_gram ? 2 : 3, 0);
    launch_chol<ONE>(p, c, 1, s);
    FLP_ORTH((orth_gram_kernel<ONE, false>), kOrthLocal);
    if (reduce) FLP_ORTH((orth_reduce_kernel<ONE>), kOrthRedG, 3, 1);
    launch_chol<ONE>(p, c, 2, s);
    FLP_ORTH((orth_final_kernel<ONE>), kOrthLocal);
}

template <bool ONE>
hipError_t launch_all(const OrthPlan &p, int c, hipStream_t s) {
    const OrthSeg *tab = p.tab;
    const int ns = p.nseg;
    const int *pre[kOrthKinds];
    for (int t = 0; t < kOrthKinds; ++t) pre[t] = ONE ? nullptr : p.pre + (size_t)t * ns;
    FLP_ORTH((orth_local_kernel<ONE>), kOrthLocal);
    FLP_ORTH((orth_reduce_kernel<ONE>), kOrthRedL, 0, 0);
    if (p.blocks[kOrthUpd1] > 0) FLP_ORTH((orth_update_kernel<ONE, true, 1, false>), kOrthUpd1);
    if (p.blocks[kOrthUpd] > 0) FLP_ORTH((orth_update_kernel<ONE, true, 4, false>), kOrthUpd);
    if (p.blocks[kOrthFma] > 0)
        hipLaunchKernelGGL((orth_tn_fma_kernel<ONE>), dim3(p.blocks[kOrthFma]), dim3(WAVE), 0, s, tab, pre[kOrthFma],
                           ns, p.one);
    if (p.blocks[kOrthMfma] > 0) FLP_ORTH((orth_tn_mfma_kernel<ONE>), kOrthMfma);
    FLP_ORTH((orth_reduce_kernel<ONE>), kOrthRedH, 1, 0);
    if (p.blocks[kOrthUpd1] > 0) FLP_ORTH((orth_update_kernel<ONE, false, 1, true>), kOrthUpd1);
    if (p.blocks[kOrthUpd] > 0) {
        if (p.upd.tiles == 8)
            FLP_ORTH((orth_update_kernel<ONE, false, 8, false>), kOrthUpd);
        else if (p.upd.ahead)
            FLP_ORTH((orth_update_kernel<ONE, false, 2, true>), kOrthUpd);
        else
            FLP_ORTH((orth_update_kernel<ONE, false, 2, false>), kOrthUpd);
    }
    launch_qr<ONE>(p, pre, c, true, s);
    return hipGetLastError();
#undef FLP_ORTH
}

}  // namespace

RowTiles orth_row_tiles(int n, int k, int c) {
    // a few blocks' worth of rows: one tile per wave, so all of them have work
    if (n < 64 * 512) return {1, true};
    return nn_row_tiles(k, c);
}

namespace {
// wgs: the blocks that the passes over W should take; cap: most doubles of
// partial sums.
void split(OrthSeg &e, int c, RowTiles upd, int wgs, size_t cap, int (&blocks)[kOrthKinds]) {
    const auto up = [](int64_t x, int64_t g) { return (int)((x + g - 1) / g * g); };
    const auto cdiv = [](int64_t x, int64_t y) { return (int)((x + y - 1) / y); };
    const int n = e.n;
    e.lrows = std::max(128, up(cdiv(n, wgs), 64));
    e.lblk = cdiv(n, e.lrows);
    blocks[kOrthLocal] += e.lblk;
    // Few enough partial Gram matrices for one block: at most 32 loads per
    // thread, in rounds of 8, about 3 us; one more launch costs as much.
    const auto gram = [&](int nb) {
        e.few = (int64_t)nb * c * c <= 8192;
        if (!e.few) blocks[kOrthRedG] += cdiv(c * c, 16);
    };
    if (e.k == 0) return gram(e.lblk);  // normalisation alone
    // rows that a block's 4 waves update at once (the local pass takes four tiles for two)
    const int ug = upd.tiles == 1 ? 64 : (upd.tiles == 8 ? 512 : 256);
    e.urows = up(cdiv(n, 2 * wgs), ug);
    e.ublk = cdiv(n, e.urows);
    blocks[upd.tiles == 1 ? kOrthUpd1 : kOrthUpd] += e.ublk;
    gram(std::max(e.lblk, e.ublk));
    blocks[kOrthRedL] += cdiv((int64_t)(e.k - e.kl) * c, 16);
    e.fma = tn_use_fma(e.k, c);
    const int groups = e.fma ? (e.k + WAVE - 1) / WAVE : (e.k + 127) / 128;
    const int grain = e.fma ? 64 : 128;
    e.prows = std::max(grain, up(cdiv(n, std::max(1, (e.fma ? 4 * wgs : 2 * wgs) / groups)), grain));
    if (!e.fma) e.prows = std::max(e.prows, up(cdiv(n, 512), grain));
    while ((size_t)cdiv(n, e.prows) * e.k * c > cap) e.prows *= 2;
    e.pchunks = cdiv(n, e.prows);
    blocks[e.fma ? kOrthFma : kOrthMfma] += e.pchunks * groups;
    blocks[kOrthRedH] += cdiv((int64_t)e.k * c, 16);
}
}  // namespace

void orth_split_single(OrthSeg &e, int c, RowTiles upd, int (&blocks)[kOrthKinds]) {
    split(e, c, upd, 1024, (size_t)32 << 20, blocks);
}

void orth_split_shared(OrthSeg &e, int c, int (&blocks)[kOrthKinds]) {
    // 128 rows to a block as long as that is at most 1024 blocks, and one row
    // tile up to 2^17 rows (ms per batch, one tile / two / by the solve's share
    // of all active solves' entries: one 30^3 matrix, r = 8, FP64 14.6 / 14.8 /
    // 14.4; four of 20^3 .. 40^3, r = 4 36.5 / 38.0 / 37.7, with both tiles
    // among them 39; three of 80^3 .. 100^3, r = 8 604 / 595 / 595)
    split(e, c, e.n < (1 << 17) ? RowTiles{1, true} : kSharedRowTiles, std::min(1024, std::max(16, e.n / 128)),
          (size_t)4 << 20, blocks);
}

size_t orth_part_elems(const OrthSeg &e, int c) {
    size_t m = (size_t)e.lblk * c * c;
    if (e.k > 0) {
        m = std::max(m, (size_t)e.lblk * (e.k - e.kl) * c);
        m = std::max(m, (size_t)e.ublk * c * c);
        m = std::max(m, (size_t)e.pchunks * e.k * c);
    }
    return m;
}

hipError_t launch_seg_orth(const OrthPlan &p, int c, hipStream_t s) {
    if (p.nseg <= 0) return hipSuccess;
    if (c < 1 || c > 16) return hipErrorInvalidValue;
    return p.tab ? launch_all<false>(p, c, s) : launch_all<true>(p, c, s);
}

hipError_t launch_block_qr(const OrthPlan &p, int c, hipStream_t s) {
    if (c < 1 || c > 16 || p.tab || p.nseg != 1) return hipErrorInvalidValue;
    const int *pre[kOrthKinds] = {};
    launch_qr<true>(p, pre, c, false, s);
    return hipGetLastError();
}

}  // namespace flp

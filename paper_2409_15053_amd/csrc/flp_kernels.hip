// Gram-Schmidt and helper kernels of the filtered Lanczos procedure for gfx950 (CDNA4).
//
// * gemm_tn / gemm_nn: the tall-skinny products of the full
//   reorthogonalisation (Section 3.2.2): the update and wide projections on
//   FP64 MFMA (16x16x4), the projection against at most 16 columns on FMA
//   (2 flops per byte: bandwidth-bound either way).
// * small helpers: counter-based normal generator, block copies, residual
//   norms.
#include "flp_internal.h"
#include "flp_device.h"
#include "flp_gemm.h"

#include <algorithm>

namespace flp {

namespace {

template <int NT>
__global__ __launch_bounds__(256) void gemm_tn_partial_kernel(int n, int K, int c, int chunk_rows, int ngroups, DMat A,
                                                              const double *__restrict__ B, int64_t ldb,
                                                              double *__restrict__ partials, bool aligned, bool sym) {
    __shared__ double red[4][4][WAVE];
    const int ntb = (c + 15) / 16;  // B tiles
    // chunk-major and XCD-aware: the blocks of one row chunk (every tile
    // group of the output) run together on one XCD, so the chunk's rows of
    // A and B come from HBM once and from that XCD's L2 for the other groups
    const int L = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = L / ngroups, grp = L % ngroups;
    const int q0 = (grp / ntb) * NT * 16, tb = grp % ntb;
    // symmetric result: a group wholly below the diagonal is not computed
    // (the reduction reads its mirror image); uniform over the block
    if (sym && q0 > tb * 16 + 15) return;
    const int r0 = chunk * chunk_rows;
    tn_mfma_block<NT>(r0, min(n, r0 + chunk_rows), K, c, q0, tb, A, B, ldb, aligned, partials + (size_t)chunk * K * c,
                      red);
}

// Sum of the per-chunk partials in a fixed order (deterministic): each
// block owns 16 outputs; its 16 thread rows split the chunks, eight loads in
// flight each, and combine through LDS (512 chunks of 2560 outputs 7 us; 64
// outputs per block and 4 thread rows took 13).  sym (a square result whose
// partials exist on and above the diagonal only): entry (i, j) below the
// diagonal takes the sums of (j, i).
__global__ __launch_bounds__(256) void reduce_partials_kernel(int nchunks, int total, int c,
                                                              const double *__restrict__ partials,
                                                              double *__restrict__ C, int ldc, bool sym) {
    __shared__ double red[16][17];
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int o = blockIdx.x * 16 + tx;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (o < total) {
        const int i = o / c, j = o % c;
        const double *p = partials + ((sym && i > j) ? j * c + i : o);
        int q = ty;
        for (; q + 112 < nchunks; q += 128) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = p[(size_t)(q + 16 * u) * total];
#pragma unroll
            for (int u = 0; u < 8; ++u) s[u % 4] += x[u];
        }
        for (; q < nchunks; q += 16) s[0] += p[(size_t)q * total];
    }
    red[ty][tx] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    if (ty == 0 && o < total) {
        double t = 0.0;
#pragma unroll
        for (int y = 0; y < 16; ++y) t += red[y][tx];
        C[(size_t)(o / c) * ldc + o % c] = t;
    }
}

// C = beta C + alpha A B (see gemm_nn_rows): one block of 4 waves per
// 4 x 16 MT rows and 16 NT columns, blocks renumbered per XCD.
template <int MT, int NT, bool PIPE>
__global__ __launch_bounds__(256) void gemm_nn_kernel(int n, int K, int c, double alpha, DMat A,
                                                      const double *__restrict__ B, int64_t ldb, double beta,
                                                      double *C, int64_t ldc, bool vec_a) {
    const int nct = (c + 16 * NT - 1) / (16 * NT);
    const int wg = xcd_tile(blockIdx.x, gridDim.x);
    gemm_nn_rows<MT, NT, PIPE>(n, K, c, alpha, A, B, ldb, beta, C, ldc, vec_a, wg / nct, wg % nct);
}

}  // namespace

namespace {

// C partial (K x C) over one chunk of rows without MFMA, for B of exactly
// C columns: thread q owns column q of A and accumulates its C dot products
// with B over the chunk's rows in order.  The B row is the same for the
// whole block (the rows are walked in step), so it is read through the
// scalar cache as one wide load; the A loads of a wave are 64 consecutive
// doubles of one row.  With C <= 16 this product does 2C flops per 8-byte A
// element, far below what the FMA units sustain at HBM speed, so it needs
// no matrix cores.
template <int C, int UNR>
__global__ __launch_bounds__(64) void gemm_tn_fma_kernel(int n, int K, int chunk_rows, DMat A,
                                                          const double *__restrict__ B, int64_t ldb,
                                                          double *__restrict__ partials) {
    const int q = blockIdx.x * WAVE + threadIdx.x;
    if (q >= K) return;  // no block-level synchronisation follows: idle columns leave at once
    const int chunk = blockIdx.y;
    const int r0 = chunk * chunk_rows, r1 = min(n, r0 + chunk_rows);
    double acc[C];
    tn_fma_column<C, UNR>(col_base(A, q), A.ld, r0, r1, B, ldb, acc);
    double *d = partials + ((size_t)chunk * K + q) * C;
#pragma unroll
    for (int j = 0; j < C; ++j) d[j] = acc[j];
}

}  // namespace

// The FMA projection serves B of exactly 8 columns against a basis of at
// least 256 columns; the MFMA kernel's row-parallel layout does better below
// that and at 16 columns, where the thread-per-column kernel's 16 FMAs per
// loaded element hold it back.  Measured at n = 1e6 (TB/s, FMA / MFMA):
// c = 8: K = 128 3.5 / 5.4, 256 5.6 / 5.4, 512 6.0 / 5.5, 768 6.1 / 5.6;
// c = 16: K = 128 2.6 / 5.5, 352 3.8 / 5.0, 768 5.0 / 5.4.
bool tn_use_fma(int K, int c) { return c == 8 && K >= 256; }

TnPlan plan_tn(int n, int K, int c) {
    TnPlan p;
    if (tn_use_fma(K, c)) {
        // FMA path: about 4096 blocks of 64 columns x chunk_rows rows (about
        // 1000-2000 rows each at n = 1e6, the fastest chunking measured), the
        // partial buffer kept near 32M doubles at most
        const int ncb = (K + WAVE - 1) / WAVE;
        int nch = std::max(1, std::min(1024, 4096 / ncb));
        int rows = std::max(64, (n + nch - 1) / nch);
        rows = (rows + 63) / 64 * 64;
        while ((size_t)((n + rows - 1) / rows) * K * c > (size_t)(32u << 20)) rows *= 2;
        p.chunk_rows = rows;
        p.nchunks = (n + rows - 1) / rows;
        p.partial_elems = (size_t)p.nchunks * K * c;
        return p;
    }
    const int ntiles = ((K + 127) / 128) * ((c + 15) / 16);
    // aim for ~2048 blocks in total, at least 128 rows per block, and keep
    // the partial buffer near 32M doubles at most
    int nch = std::min(512, std::max(1, 2048 / std::max(1, ntiles)));
    int rows = (n + nch - 1) / nch;
    rows = std::max(rows, 128);
    size_t per = (size_t)K * c;
    while ((size_t)((n + rows - 1) / rows) * per > (size_t)(32u << 20)) rows *= 2;
    rows = (rows + 127) / 128 * 128;
    p.chunk_rows = rows;
    p.nchunks = (n + rows - 1) / rows;
    p.partial_elems = (size_t)p.nchunks * per;
    return p;
}

hipError_t launch_gemm_tn_partial(const TnPlan &pl, int n, int K, int c, DMat A, const double *B, int64_t ldb,
                                  double *partials, hipStream_t s, bool sym) {
    if (tn_use_fma(K, c)) {
        dim3 grid((K + WAVE - 1) / WAVE, pl.nchunks);
        hipLaunchKernelGGL((gemm_tn_fma_kernel<8, 8>), grid, dim3(WAVE), 0, s, n, K, pl.chunk_rows, A, B, ldb,
                           partials);
        return hipGetLastError();
    }
    // 16-byte A loads need an even leading dimension and panel stride
    const bool aligned = !(A.ld & 1) && !(A.ps & 1) && !(reinterpret_cast<uintptr_t>(A.p) & 15);
    const int nt = K <= 32 ? 2 : (K <= 64 ? 4 : 8);
    const int ngroups = ((K + 16 * nt - 1) / (16 * nt)) * ((c + 15) / 16);
    dim3 grid(pl.nchunks * ngroups);
#define FLP_TN(NT) \
    hipLaunchKernelGGL((gemm_tn_partial_kernel<NT>), grid, dim3(256), 0, s, n, K, c, pl.chunk_rows, ngroups, A, B, ldb, \
                       partials, aligned, sym && K == c)
    if (nt == 2)
        FLP_TN(2);
    else if (nt == 4)
        FLP_TN(4);
    else
        FLP_TN(8);
#undef FLP_TN
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const TnPlan &pl, int K, int c, const double *partials, double *C, int ldc,
                                  hipStream_t s, bool sym) {
    int total = K * c;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((total + 15) / 16), dim3(256), 0, s, pl.nchunks, total, c,
                       partials, C, ldc, sym && K == c);
    return hipGetLastError();
}

// Measured at n = 1e6 (us; two tiles / two with the next group's loads in
// flight / eight): 8 columns, K = 96 171 / 177 / 206, K = 160 285 / 294 / 300,
// K = 320 - / 546 / 578, K = 640 - / 1010 / 1031; 16 columns, K = 160 302 /
// 309 / -, K = 320 - / 591 / 601, K = 720 - / 1185 / 1157; n = 27000, 8
// columns, K = 300: 19 / 16 / -.
RowTiles nn_row_tiles(int k, int c) {
    if (k >= 256 && c <= 8) return {2, true};
    return {k >= 320 ? 8 : 2, false};
}

hipError_t launch_gemm_nn(int n, int K, int c, double alpha, DMat A, const double *B, int64_t ldb, double beta,
                          double *C, int64_t ldc, hipStream_t s) {
    if (n <= 0 || c <= 0) return hipSuccess;
    bool vec_a = (A.ld % 2 == 0) && (A.ps % 2 == 0) && ((reinterpret_cast<uintptr_t>(A.p) & 15) == 0);
    const auto go = [&](auto kernel, int mt, int nt) {
        const int rblocks = (n + 4 * 16 * mt - 1) / (4 * 16 * mt);
        const int nct = (c + 16 * nt - 1) / (16 * nt);
        hipLaunchKernelGGL(kernel, dim3(rblocks * nct), dim3(256), 0, s, n, K, c, alpha, A, B, ldb, beta, C, ldc,
                           vec_a);
    };
    if (c > 16) {
        go(gemm_nn_kernel<2, 4, false>, 2, 4);
    } else {
        const RowTiles t = nn_row_tiles(K, c);
        if (t.tiles == 8)
            go(gemm_nn_kernel<8, 1, false>, 8, 1);
        else if (t.ahead)
            go(gemm_nn_kernel<2, 1, true>, 2, 1);
        else
            go(gemm_nn_kernel<2, 1, false>, 2, 1);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ helpers

namespace {

// Symmetry check, one thread per row: for each stored a_ij, a_ji is looked
// up by binary search in row j (columns sorted) and compared; the count of
// entries without a matching partner goes to *bad (vector atomics).
__global__ void sym_check_kernel(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colind,
                                 const double *__restrict__ val, double tol, unsigned int *bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned int cnt = 0;
    for (int p = rowptr[i]; p < rowptr[i + 1]; ++p) {
        const int j = colind[p];
        if (j < 0 || j >= n) {
            ++cnt;
            continue;
        }
        int lo = rowptr[j], hi = rowptr[j + 1] - 1, found = -1;
        while (lo <= hi) {
            const int mid = (lo + hi) >> 1;
            const int cm = colind[mid];
            if (cm == i) {
                found = mid;
                break;
            }
            if (cm < i)
                lo = mid + 1;
            else
                hi = mid - 1;
        }
        if (found < 0) {
            ++cnt;
            continue;
        }
        const double a = val[p], b = val[found];
        if (fabs(a - b) > tol * fmax(fabs(a), fabs(b))) ++cnt;
    }
    if (cnt) atomicAdd(bad, cnt);
}

__global__ void randn_kernel(int rows, int cols, double *__restrict__ out, int64_t ld, uint64_t seed,
                             uint64_t sid) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t total = (int64_t)rows * cols;
    if (idx >= total) return;
    out[(idx / cols) * ld + idx % cols] = normal_at(seed, sid, (uint64_t)idx);
}

__global__ void copy_block_kernel(int rows, int cols, double scale, const double *__restrict__ src, int64_t lds,
                                  DMat dst, int dcol0, float *__restrict__ dst32, int64_t ldd32) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)rows * cols) return;
    int64_t i = idx / cols;
    int j = (int)(idx % cols);
    double v = scale * src[i * lds + j];
    if (dst.p) {
        int q = dcol0 + j;
        dst.p[(int64_t)(q >> dst.lpw) * dst.ps + i * dst.ld + (q & ((1 << dst.lpw) - 1))] = v;
    }
    if (dst32) dst32[i * ldd32 + j] = (float)v;
}

__global__ void to_float_kernel(int64_t count, const double *__restrict__ src, float *__restrict__ dst) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = (float)src[i];
}

__global__ void scale_kernel(int64_t count, double a, const double *__restrict__ src, double *__restrict__ dst) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = a * src[i];
}

// Column sums over all n rows of (AX - lam X)^2 (RESID) or X Y: part[chunk, j]
// is the sum over the chunk's rows, 64 columns and 4 rows at a time per
// block.  The chunks are short (resid_chunks), because a block is one chain
// of loads whatever its columns: with 1024 rows to a chunk a matrix of 27000
// rows had 27 blocks and took 135 us for 40 columns, 17 now.
template <bool RESID>
__global__ __launch_bounds__(256) void colsum_partial_kernel(int n, int c, const double *__restrict__ P, int64_t ldp,
                                                             const double *__restrict__ X, int64_t ldx,
                                                             const double *__restrict__ lam, int rows_per_chunk,
                                                             double *__restrict__ part) {
    __shared__ double red[256];
    const int chunk = blockIdx.x, j0 = blockIdx.y * 64;
    const int j = j0 + threadIdx.x % 64, rsub = threadIdx.x / 64;
    double s = 0.0;
    if (j < c) {
        const double l = RESID ? lam[j] : 0.0;
        const int64_t r0 = (int64_t)chunk * rows_per_chunk, r1 = min((int64_t)n, r0 + rows_per_chunk);
#pragma unroll 4
        for (int64_t i = r0 + rsub; i < r1; i += 4) {
            const double p = P[i * ldp + j], x = X[i * ldx + j];
            if constexpr (RESID) {
                const double d = p - l * x;
                s = fma(d, d, s);
            } else {
                s = fma(p, x, s);
            }
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < 64 && j < c)
        part[(size_t)chunk * c + j] =
            red[threadIdx.x] + red[threadIdx.x + 64] + red[threadIdx.x + 128] + red[threadIdx.x + 192];
}

// The partials' sum, 16 columns per block and 16 threads to a column, in a
// fixed order; its square root for RESID.
template <bool RESID>
__global__ __launch_bounds__(256) void colsum_final_kernel(int nchunks, int c, const double *__restrict__ part,
                                                           double *__restrict__ out) {
    __shared__ double red[256];
    const int j = blockIdx.x * 16 + threadIdx.x % 16, q0 = threadIdx.x / 16;
    double s = 0.0;
    if (j < c) {
#pragma unroll 4
        for (int q = q0; q < nchunks; q += 16) s += part[(size_t)q * c + j];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < 16 && j < c) {
        double t = 0.0;
        for (int q = 0; q < 16; ++q) t += red[q * 16 + threadIdx.x];
        out[j] = RESID ? sqrt(t) : t;
    }
}

__global__ void transpose_out_kernel(int n, int c, const double *__restrict__ src, int64_t lds,
                                     double *__restrict__ dst) {
    __shared__ double t[32][33];
    int bx = blockIdx.x * 32, by = blockIdx.y * 32;  // bx: rows of src, by: columns
    int tx = threadIdx.x % 32, ty = threadIdx.x / 32;  // 256 threads: ty 0..7
    for (int k = ty; k < 32; k += 8) {
        int i = bx + k, j = by + tx;
        t[k][tx] = (i < n && j < c) ? src[(int64_t)i * lds + j] : 0.0;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {
        int j = by + k, i = bx + tx;
        if (i < n && j < c) dst[(int64_t)j * n + i] = t[tx][k];
    }
}

// dst (row-major n x c, ldd) = src (column-major n x c, ld n): the inverse
// of transpose_out_kernel, tile by tile through LDS.
__global__ void transpose_in_kernel(int n, int c, const double *__restrict__ src, double *__restrict__ dst,
                                    int64_t ldd) {
    __shared__ double t[32][33];
    int bx = blockIdx.x * 32, by = blockIdx.y * 32;  // bx: rows of dst, by: columns
    int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    for (int k = ty; k < 32; k += 8) {
        int j = by + k, i = bx + tx;
        t[tx][k] = (i < n && j < c) ? src[(int64_t)j * n + i] : 0.0;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {
        int i = bx + k, j = by + tx;
        if (i < n && j < c) dst[(int64_t)i * ldd + j] = t[k][tx];
    }
}

}  // namespace

hipError_t launch_sym_check(int n, const int32_t *rowptr, const int32_t *colind, const double *val, double tol,
                            unsigned int *bad, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(sym_check_kernel, dim3((n + 255) / 256), dim3(256), 0, s, n, rowptr, colind, val, tol, bad);
    return hipGetLastError();
}

hipError_t launch_randn(int rows, int cols, double *out, int64_t ld, uint64_t seed, uint64_t sid, hipStream_t s) {
    int64_t total = (int64_t)rows * cols;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(randn_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, rows, cols, out, ld,
                       seed, sid);
    return hipGetLastError();
}

hipError_t launch_copy_block(int rows, int cols, double scale, const double *src, int64_t lds, DMat dst, int dcol0,
                             float *dst32, int64_t ldd32, hipStream_t s) {
    int64_t total = (int64_t)rows * cols;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(copy_block_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, rows, cols, scale,
                       src, lds, dst, dcol0, dst32, ldd32);
    return hipGetLastError();
}

hipError_t launch_to_float(int64_t count, const double *src, float *dst, hipStream_t s) {
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(to_float_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count, src, dst);
    return hipGetLastError();
}

hipError_t launch_scale(int64_t count, double a, const double *src, double *dst, hipStream_t s) {
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(scale_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count, a, src, dst);
    return hipGetLastError();
}

int resid_chunks(int n) { return std::max(1, std::min(1024, (n + 63) / 64)); }

namespace {
template <bool RESID>
hipError_t launch_colsum(int n, int c, const double *P, int64_t ldp, const double *X, int64_t ldx, const double *lam,
                         double *part, int nchunks, double *out, hipStream_t s) {
    if (c <= 0) return hipSuccess;
    const int rpc = (n + nchunks - 1) / nchunks;
    hipLaunchKernelGGL((colsum_partial_kernel<RESID>), dim3(nchunks, (c + 63) / 64), dim3(256), 0, s, n, c, P, ldp, X,
                       ldx, lam, rpc, part);
    hipLaunchKernelGGL((colsum_final_kernel<RESID>), dim3((c + 15) / 16), dim3(256), 0, s, nchunks, c, part, out);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_resid_norms(int n, int c, const double *AX, int64_t ldax, const double *X, int64_t ldx,
                              const double *lam, double *part, int nchunks, double *out, hipStream_t s) {
    return launch_colsum<true>(n, c, AX, ldax, X, ldx, lam, part, nchunks, out, s);
}

hipError_t launch_col_dots(int n, int c, const double *X, int64_t ldx, const double *Y, int64_t ldy, double *part,
                           int nchunks, double *out, hipStream_t s) {
    return launch_colsum<false>(n, c, X, ldx, Y, ldy, nullptr, part, nchunks, out, s);
}

hipError_t launch_transpose_in(int n, int c, const double *src, double *dst, int64_t ldd, hipStream_t s) {
    if (n <= 0 || c <= 0) return hipSuccess;
    dim3 grid((n + 31) / 32, (c + 31) / 32);
    hipLaunchKernelGGL(transpose_in_kernel, grid, dim3(256), 0, s, n, c, src, dst, ldd);
    return hipGetLastError();
}

hipError_t launch_transpose_out(int n, int c, const double *src, int64_t lds, double *dst, hipStream_t s) {
    if (n <= 0 || c <= 0) return hipSuccess;
    dim3 grid((n + 31) / 32, (c + 31) / 32);
    hipLaunchKernelGGL(transpose_out_kernel, grid, dim3(256), 0, s, n, c, src, lds, dst);
    return hipGetLastError();
}

}  // namespace flp

// The bounds estimate's Lanczos run on the device for gfx950 (Section 2.2):
// k steps of single-vector Lanczos, each new vector orthogonalised twice
// against the two before it, for one matrix or for many with one launch per
// stage.
//
// A step is three launches, whatever the number of matrices:
//   lz_spmv    w = A q_j, with the partial sums of q_j . w and q_{j-1} . w
//   lz_pass 1  w -= q_j h_j + q_{j-1} h_{j-1}, partial sums of the second pass
//   lz_pass 2  the same with the second coefficients, partial sums of ||w||^2
// Vectors are kept as the unnormalised z_j = beta_j q_j: the norm of a step is
// known only after its last launch, and the next step scales by 1 / beta_j
// where it reads (A q_j = (A z_j) / beta_j), so no launch is spent on
// normalising or on reducing: every block adds the at most 1024 partial sums
// of the stage before it in the same fixed order.  The step-by-step form
// (projections, updates, reductions and the normalisation as launches of
// their own) took ten.  Bound by launches on small matrices, by the read of A
// on large ones.
#include "flp_internal.h"
#include "flp_device.h"
#include "flp_gather.h"

#include <algorithm>

namespace flp {

namespace {

template <bool ONE>
__device__ __forceinline__ LanczosSeg lz_seg(const LanczosSeg *__restrict__ tab, int nseg, const LanczosSeg &one,
                                             int *lb) {
    if constexpr (ONE) {
        *lb = xcd_tile(blockIdx.x, gridDim.x);
        return one;
    } else {
        const int lane = threadIdx.x % WAVE, blk = (int)blockIdx.x;
        int seg = -1;
        for (int base = 0; base < nseg; base += WAVE) {
            const int i = base + lane;
            const bool le = i < nseg && tab[i].blk0 <= blk;
            const unsigned long long m = __ballot(le);
            seg += __popcll(m);
            if (~m != 0ull) break;
        }
        seg = __builtin_amdgcn_readfirstlane(seg);
        *lb = blk - tab[seg].blk0;
        return tab[seg];
    }
}

// Sum over the block's 256 threads, the same on all of them.
__device__ __forceinline__ double block_sum(double x, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, WAVE);
    __syncthreads();
    if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = x;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// The nb partial sums p[0], p[2], ... of a stage, added by the whole block.
__device__ __forceinline__ double stage_sum(const double *p, int nb, double *red) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < kLanczosBlocks / 256; ++u) {
        const int i = (int)threadIdx.x + 256 * u;
        if (i < nb) s += p[2 * i];
    }
    return block_sum(s, red);
}

__device__ __forceinline__ double inverse(double beta) { return beta > 0.0 ? 1.0 / beta : 0.0; }

// Rows [lb * rows, ...) of a block.
struct LzRows {
    int r0, r1;
};
__device__ __forceinline__ LzRows lz_rows(const LanczosSeg &e, int lb) {
    return LzRows{lb * e.rows, min(e.n, (lb + 1) * e.rows)};
}

// z_0: N(0, 1) entries (the counter-based generator of launch_randn), the
// partial sums of ||z_0||^2, and the Gershgorin interval of the block's rows.
template <bool ONE>
__global__ __launch_bounds__(256) void lz_start_kernel(const LanczosSeg *__restrict__ tab, int nseg,
                                                       const LanczosSeg one) {
    __shared__ double red[4], lo[256], hi[256];
    int lb;
    const LanczosSeg e = lz_seg<ONE>(tab, nseg, one, &lb);
    const LzRows rw = lz_rows(e, lb);
    double s = 0.0, mn = 1e308, mx = -1e308;
    for (int i = rw.r0 + (int)threadIdx.x; i < rw.r1; i += 256) {
        const double z = normal_at(e.seed, 0xB0B0, (uint64_t)i);
        e.z[0][i] = z;
        s = fma(z, z, s);
        double d = 0.0, rad = 0.0;
        for (int p = e.grow[i]; p < e.grow[i + 1]; ++p) {
            if (e.gcol[p] == i)
                d += e.gval[p];
            else
                rad += fabs(e.gval[p]);
        }
        mn = fmin(mn, d - rad);
        mx = fmax(mx, d + rad);
    }
    s = block_sum(s, red);
    lo[threadIdx.x] = mn;
    hi[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            lo[threadIdx.x] = fmin(lo[threadIdx.x], lo[threadIdx.x + w]);
            hi[threadIdx.x] = fmax(hi[threadIdx.x], hi[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        e.part[4 * kLanczosBlocks + 2 * lb] = s;
        e.gersh[2 * lb] = lo[0];
        e.gersh[2 * lb + 1] = hi[0];
    }
}

// Step j: beta_j from the partial norms of the step before (block 0 records
// it), w = (A z_j) / beta_j, partial sums of q_j . w and q_{j-1} . w.
template <bool ONE>
__global__ __launch_bounds__(256) void lz_spmv_kernel(const LanczosSeg *__restrict__ tab, int nseg,
                                                      const LanczosSeg one, int j) {
    __shared__ double red[4];
    int lb;
    const LanczosSeg e = lz_seg<ONE>(tab, nseg, one, &lb);
    if (j >= e.k) return;
    const LzRows rw = lz_rows(e, lb);
    const double beta = sqrt(fmax(stage_sum(e.part + 4 * kLanczosBlocks, e.nb, red), 0.0));
    const double inv = inverse(beta);
    if (lb == 0 && threadIdx.x == 0) e.ab[2 * j] = beta;
    const double ipv = j > 0 ? inverse(e.ab[2 * (j - 1)]) : 0.0;
    const double *z = e.z[j % 3], *zp = e.z[(j + 2) % 3];
    double *w = e.z[(j + 1) % 3];
    const XSource<double, 1, false> xs{z, 1, 0, nullptr, 0, 0, 0u};
    double d0 = 0.0, d1 = 0.0;
    for (int i = rw.r0 + (int)threadIdx.x; i < rw.r1; i += 256) {
        double acc[1] = {0.0};
        if (e.sell) {
            const int o0 = e.rowptr[i / kSellC], o1 = e.rowptr[i / kSellC + 1];
            sell_gather<double, 1, 8, false>(o0 + i % kSellC, (o1 - o0) / kSellC, e.colind, e.val, xs, acc);
        } else {
            row_gather<double, 1, 8, false>(e.rowptr[i], e.rowptr[i + 1], e.colind, e.val, xs, acc);
        }
        const double wi = acc[0] * inv;
        w[i] = wi;
        d0 = fma(z[i] * inv, wi, d0);
        if (j > 0) d1 = fma(zp[i] * ipv, wi, d1);
    }
    d0 = block_sum(d0, red);
    d1 = block_sum(d1, red);
    if (threadIdx.x == 0) {
        e.part[2 * lb] = d0;
        e.part[2 * lb + 1] = d1;
    }
}

// Gram-Schmidt pass (1 or 2) of step j on w = z_{j+1}.  Pass 1 reads its
// coefficients' partial sums from part[0 ..], leaves those of pass 2 in part[2
// kLanczosBlocks ..]; pass 2 leaves ||w||^2 in part[4 kLanczosBlocks ..] and
// records alpha_j, the sum of both passes' coefficients of q_j.
template <bool ONE>
__global__ __launch_bounds__(256) void lz_pass_kernel(const LanczosSeg *__restrict__ tab, int nseg,
                                                      const LanczosSeg one, int j, int pass) {
    __shared__ double red[4];
    int lb;
    const LanczosSeg e = lz_seg<ONE>(tab, nseg, one, &lb);
    if (j >= e.k) return;
    const LzRows rw = lz_rows(e, lb);
    const double *in = e.part + (pass == 1 ? 0 : 2 * kLanczosBlocks);
    const double h0 = stage_sum(in, e.nb, red), h1 = j > 0 ? stage_sum(in + 1, e.nb, red) : 0.0;
    const double inv = inverse(e.ab[2 * j]), ipv = j > 0 ? inverse(e.ab[2 * (j - 1)]) : 0.0;
    if (lb == 0 && threadIdx.x == 0) {
        if (pass == 1)
            e.ab[2 * j + 1] = h0;
        else
            e.ab[2 * j + 1] += h0;
    }
    const double *z = e.z[j % 3], *zp = e.z[(j + 2) % 3];
    double *w = e.z[(j + 1) % 3];
    const double c0 = h0 * inv, c1 = h1 * ipv;
    double d0 = 0.0, d1 = 0.0;
    for (int i = rw.r0 + (int)threadIdx.x; i < rw.r1; i += 256) {
        const double zi = z[i], zpi = j > 0 ? zp[i] : 0.0;
        const double wi = fma(-c1, zpi, fma(-c0, zi, w[i]));
        w[i] = wi;
        if (pass == 1) {
            d0 = fma(zi * inv, wi, d0);
            d1 = fma(zpi * ipv, wi, d1);
        } else {
            d0 = fma(wi, wi, d0);
        }
    }
    d0 = block_sum(d0, red);
    if (pass == 1) d1 = block_sum(d1, red);
    if (threadIdx.x == 0) {
        double *out = e.part + (pass == 1 ? 2 : 4) * kLanczosBlocks;
        out[2 * lb] = d0;
        if (pass == 1) out[2 * lb + 1] = d1;
    }
}

// beta_k and the Gershgorin enclosure: ab[2 k], ab[2 k + 1], ab[2 k + 2].
template <bool ONE>
__global__ __launch_bounds__(256) void lz_final_kernel(const LanczosSeg *__restrict__ tab, const LanczosSeg one) {
    __shared__ double red[4], lo[256], hi[256];
    const LanczosSeg e = ONE ? one : tab[blockIdx.x];
    const double g = stage_sum(e.part + 4 * kLanczosBlocks, e.nb, red);
    double mn = 1e308, mx = -1e308;
    for (int i = threadIdx.x; i < e.nb; i += 256) {
        mn = fmin(mn, e.gersh[2 * i]);
        mx = fmax(mx, e.gersh[2 * i + 1]);
    }
    lo[threadIdx.x] = mn;
    hi[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            lo[threadIdx.x] = fmin(lo[threadIdx.x], lo[threadIdx.x + w]);
            hi[threadIdx.x] = fmax(hi[threadIdx.x], hi[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        e.ab[2 * e.k] = sqrt(fmax(g, 0.0));
        e.ab[2 * e.k + 1] = lo[0];
        e.ab[2 * e.k + 2] = hi[0];
    }
}

template <bool ONE>
hipError_t lz_launch(const LanczosSeg *tab, int nseg, const LanczosSeg &one, int blocks, int kmax, hipStream_t s) {
    hipLaunchKernelGGL((lz_start_kernel<ONE>), dim3(blocks), dim3(256), 0, s, tab, nseg, one);
    for (int j = 0; j < kmax; ++j) {
        hipLaunchKernelGGL((lz_spmv_kernel<ONE>), dim3(blocks), dim3(256), 0, s, tab, nseg, one, j);
        for (int pass = 1; pass <= 2; ++pass)
            hipLaunchKernelGGL((lz_pass_kernel<ONE>), dim3(blocks), dim3(256), 0, s, tab, nseg, one, j, pass);
    }
    hipLaunchKernelGGL((lz_final_kernel<ONE>), dim3(nseg), dim3(256), 0, s, tab, one);
    return hipGetLastError();
}

}  // namespace

void lanczos_split(LanczosSeg &e) {
    const int64_t nb = std::min<int64_t>(kLanczosBlocks, ((int64_t)e.n + 255) / 256);
    e.rows = (int)((((int64_t)e.n + nb - 1) / nb + 255) / 256 * 256);
    e.nb = (e.n + e.rows - 1) / e.rows;
}

hipError_t launch_lanczos(const LanczosSeg *tab, int nseg, const LanczosSeg &one, int blocks, int kmax,
                          hipStream_t s) {
    return tab ? lz_launch<false>(tab, nseg, one, blocks, kmax, s) : lz_launch<true>(nullptr, 1, one, blocks, kmax, s);
}

}  // namespace flp

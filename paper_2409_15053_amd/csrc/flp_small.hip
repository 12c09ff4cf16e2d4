// The Chebyshev filter of a small matrix in one launch (Section 2.2).
//
// The Clenshaw recurrence acts on each column of the block independently, so
// one workgroup can carry one column through all m steps with nothing but
// its own barriers: the matrix stays in its registers (thread t owns rows t,
// t + 1024, ...; W slots of index and value each), the gathered vector
// U_{k+1} in LDS (two buffers, one barrier per step).  The step-by-step form pays a kernel
// launch per step, 3.3-4.1 us each on a matrix of a few thousand rows
// whatever the bytes; here a step costs its LDS gathers and a barrier: 0.25
// us at 400 rows of 5 nonzeros, 0.5 us at 1600 rows, 1.4 us at 3375 rows of 7
// (FP64).  What bounds it is LDS: every nonzero is one gathered read there.
//
// The sums run in the order of cheb_step_kernel's, with the same rounding of
// every operation, so W is bit-identical to the launches it replaces.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "flp_host.h"
#include "flp_device.h"
#include "flp_gather.h"

namespace flp {
namespace {

constexpr int kThreads = 1024;

// Coefficients of the m steps: out = alpha (A X) + beta X + gamma V - Y, V
// from step 1 on, Y from step 2 on (clenshaw_plan); passed by value.
struct SmallCoef {
    int m;
    double alpha0, beta0;        // first step
    double alpha, beta;          // steps between
    double alpha_last, beta_last;
    double gamma[kSmallMaxDegree];
};

// RPT rows per thread, W register slots per row (an even number; longer CSR
// rows read the rest from global memory at every step).  Column indices are
// kept as 16-bit pairs (n <= 1024 RPT < 2^16).  SELL: rowptr holds the slice
// offsets and colind / val the sliced ELL arrays.
template <typename T, int RPT, int W, bool SELL>
__global__ __launch_bounds__(kThreads) void cheb_small_kernel(int n, const int32_t *__restrict__ rowptr,
                                                              const int32_t *__restrict__ colind,
                                                              const T *__restrict__ val,
                                                              const double *__restrict__ V, int ldv,
                                                              double *__restrict__ out, int ldo, SmallCoef co) {
    // V, the thread's own U_{k+1} and U_{k+2} stay in registers where the
    // matrix leaves room (REG), else in LDS with a third ring buffer
    constexpr bool REG = RPT * W * (int)sizeof(T) <= 128;
    constexpr int NB = REG ? 2 : 3;
    __shared__ T x[NB][RPT * kThreads];  // step s reads U_{k+1} in x[s % NB], writes x[(s + 1) % NB]
    __shared__ T vl[REG ? 1 : RPT * kThreads];
    __shared__ double gam[kSmallMaxDegree];
    const int t = (int)threadIdx.x, c = (int)blockIdx.x;
    T a[RPT][W];
    unsigned cols[RPT][W / 2];
    T vr[RPT], u1[RPT], u2[RPT];
    const auto at = [](const T *p, unsigned bytes) { return *(const T *)((const char *)p + bytes); };
    const auto extent = [&](int row, int &base, int &len) {
        if constexpr (SELL) {
            const int o0 = rowptr[row / kSellC];
            base = o0 + row % kSellC;
            len = (rowptr[row / kSellC + 1] - o0) / kSellC;
        } else {
            base = rowptr[row];
            len = rowptr[row + 1] - base;
        }
    };
    if (t < co.m) gam[t] = co.gamma[t];
    // the thread's rows: the first W slots (padded with weight zero on the
    // row's own column) and the column of V
    int w = 1;          // slots the wavefront walks
    bool over = false;  // rows with more than W nonzeros
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = t + q * kThreads, row = min(i, n - 1);
        int base, len;
        extent(row, base, len);
        if (i >= n) len = 0;
        over = over || len > W;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            unsigned cc = (unsigned)row;  // as a byte offset into x below
            a[q][k] = T(0);
            if (k < len) {
                const int p = base + (SELL ? k * kSellC : k);
                cc = (unsigned)colind[p];
                a[q][k] = val[p];
            }
            cc *= (unsigned)sizeof(T);
            if (k & 1)
                cols[q][k / 2] |= cc << 16;
            else
                cols[q][k / 2] = cc;
            if (__ballot(k < len) != 0ull) w = max(w, k + 1);
        }
        const T vi = (T)V[(int64_t)row * ldv + c];
        if constexpr (REG) {
            vr[q] = u1[q] = vi;
            u2[q] = T(0);
        } else {
            vl[i] = vi;
        }
        x[0][i] = vi;
    }
    over = __ballot(over) != 0ull;
    // rows per thread that this wavefront has (uniform)
    const int nq = __builtin_amdgcn_readfirstlane((n - (t / WAVE) * WAVE + kThreads - 1) / kThreads);
    __syncthreads();
    int cur = 0;
    for (int s = 0; s < co.m; ++s) {
        const int nxt = cur == NB - 1 ? 0 : cur + 1, old = NB - cur - nxt;  // old: U_{k+2} of a ring of three
        const T *xs = x[cur];
        const bool last = s == co.m - 1;
        const T alpha = (T)(s == 0 ? co.alpha0 : (last ? co.alpha_last : co.alpha));
        const T beta = (T)(s == 0 ? co.beta0 : (last ? co.beta_last : co.beta));
        const T gamma = (T)gam[s];
        T acc[RPT];
        // the gathers of a wavefront's rows: one body per slot count with all
        // of them in flight where registers allow, else two slots at a time
        // (kept packed by the empty asm: unpacked offsets would be hoisted
        // out of the step loop and spill)
        if constexpr (REG) {
            static_for<1, W + 1>([&](auto N) {
                if (w == decltype(N)::value) {
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        if (q > 0 && q >= nq) continue;  // uniform: no rows here
                        T xv[decltype(N)::value];
#pragma unroll
                        for (int k = 0; k < decltype(N)::value; ++k) {
                            if (k % 2 == 0) asm volatile("" : "+v"(cols[q][k / 2]));
                            xv[k] = at(xs, k % 2 ? cols[q][k / 2] >> 16 : cols[q][k / 2] & 0xffffu);
                        }
                        acc[q] = T(0);
#pragma unroll
                        for (int k = 0; k < decltype(N)::value; ++k) acc[q] = fma(a[q][k], xv[k], acc[q]);
                    }
                }
            });
        } else {
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                if (q > 0 && q >= nq) continue;
                acc[q] = T(0);
#pragma unroll
                for (int k = 0; k < W; k += 2)
                    if (k < w) {
                        asm volatile("" : "+v"(cols[q][k / 2]));
                        const T x0 = at(xs, cols[q][k / 2] & 0xffffu), x1 = at(xs, cols[q][k / 2] >> 16);
                        acc[q] = fma(a[q][k], x0, acc[q]);
                        acc[q] = fma(a[q][k + 1], x1, acc[q]);
                    }
            }
        }
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            if (q > 0 && q >= nq) continue;
            const int i = t + q * kThreads;
            if (over && i < n) {
                int base, len;
                extent(i, base, len);
                for (int k = W; k < len; ++k) {
                    const int p = base + (SELL ? k * kSellC : k);
                    acc[q] = fma(val[p], xs[colind[p]], acc[q]);
                }
            }
            T res;
            if constexpr (REG) {
                res = fma(alpha, acc[q], beta * u1[q]);
                if (s > 0) res = fma(gamma, vr[q], res);
                if (s > 1) res = fma(T(-1), u2[q], res);
                u2[q] = u1[q];
                u1[q] = res;
            } else {
                res = fma(alpha, acc[q], beta * xs[i]);
                if (s > 0) res = fma(gamma, vl[i], res);
                if (s > 1) res = fma(T(-1), x[old][i], res);
            }
            x[nxt][i] = res;
        }
        cur = nxt;
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = t + q * kThreads;
        if (i < n) out[(int64_t)i * ldo + c] = (double)x[cur][i];
    }
}

template <typename T, int RPT, int W>
hipError_t small_launch(const flp_csr *A, const T *val, bool sell, int r, const double *V, int ldv, double *out,
                        int ldo, const SmallCoef &co, hipStream_t s) {
    if (sell)
        hipLaunchKernelGGL((cheb_small_kernel<T, RPT, W, true>), dim3(r), dim3(kThreads), 0, s, A->n, A->rowptr,
                           A->colind, val, V, ldv, out, ldo, co);
    else
        hipLaunchKernelGGL((cheb_small_kernel<T, RPT, W, false>), dim3(r), dim3(kThreads), 0, s, A->n, A->rowptr,
                           A->colind, val, V, ldv, out, ldo, co);
    return hipGetLastError();
}

template <typename T>
hipError_t small_dispatch(int slots, const flp_csr *A, const T *val, bool sell, int r, const double *V, int ldv,
                          double *out, int ldo, const SmallCoef &co, hipStream_t s) {
    const int n = A->n;
#define FLP_SMALL(RPT, W) return small_launch<T, RPT, W>(A, val, sell, r, V, ldv, out, ldo, co, s)
    if (slots == 8) {
        if (n <= kThreads) FLP_SMALL(1, 8);
        if (n <= 2 * kThreads) FLP_SMALL(2, 8);
        if (n <= 3 * kThreads) FLP_SMALL(3, 8);
        if (n <= 4 * kThreads) FLP_SMALL(4, 8);
    } else if (slots == 16) {
        if (n <= kThreads) FLP_SMALL(1, 16);
        if (n <= 2 * kThreads) FLP_SMALL(2, 16);
        if constexpr (sizeof(T) == 4) {
            if (n <= 3 * kThreads) FLP_SMALL(3, 16);
        }
    }
#undef FLP_SMALL
    return hipErrorInvalidValue;
}

}  // namespace

// The line: the matrix has to fit the registers of one workgroup (1024
// threads of 128 registers: up to 4096 rows of at most 8 nonzeros on average,
// 2048 of at most 16, in FP32 3072), and enough steps have to share the cost
// of loading it.  Measured against one launch per step (degree 50 unless
// noted): 1600 rows FP64 33 against 196 us, 3375 rows of 7 FP64 80 against
// 196 (degree 6: 19 against 23) and FP32 70 against 199, 1728 rows of 13
// FP64 70 against 204, 2744 rows of 13 FP32 101 against 200 (degree 5: 27
// against 23); FP32 at 8000 rows of 7 (spilling) 221 against 200.
// The slots are those of the storage that is read (`stored`) where a
// workgroup has room for 16, so that a sliced ELL copy's padded rows stay in
// registers; a copy of more than 5/4 of its slots (AUTO's limit) keeps one
// launch per step, because all the rows of a slice are as long as its longest.
int small_filter_slots(const flp_filter *p, const flp_csr *A, const flp_csr *stored, bool fp32) {
    const int n = A->n;
    if (p->m < 4 || p->m > kSmallMaxDegree) return 0;
    int slots = 0;
    if (A->nnz <= 8 * (int64_t)n) {
        if (n <= 4 * kThreads) slots = stored->nnz > 8 * (int64_t)n && n <= 2 * kThreads ? 16 : 8;
    } else if (A->nnz <= 16 * (int64_t)n && n <= (fp32 ? 3 : 2) * kThreads) {
        if (n <= 2 * kThreads || p->m >= 8) slots = 16;
    }
    const int64_t rows = ((int64_t)n + kSellC - 1) / kSellC * kSellC;
    return 4 * stored->nnz <= 5 * slots * rows + 4 * kSellC ? slots : 0;
}

int launch_small_filter(const flp_filter *p, int slots, const flp_csr *A, const float *val32, bool sell, int r,
                        const double *V, int ldv, double *W, int ldw, bool fp32, hipStream_t s) {
    // the steps' coefficients are the launch plan's
    const auto plan = clenshaw_plan(p, r, V, ldv, W, ldw, nullptr, nullptr, nullptr, fp32);
    SmallCoef co{};
    co.m = (int)plan.size();
    co.alpha0 = plan[0].alpha;
    co.beta0 = plan[0].beta;
    if (co.m > 2) {
        co.alpha = plan[1].alpha;
        co.beta = plan[1].beta;
    }
    co.alpha_last = plan[co.m - 1].alpha;
    co.beta_last = plan[co.m - 1].beta;
    for (int t = 0; t < co.m; ++t) co.gamma[t] = plan[t].gamma;
    if (fp32)
        CK(small_dispatch<float>(slots, A, val32, sell, r, V, ldv, W, ldw, co, s));
    else
        CK(small_dispatch<double>(slots, A, A->val, sell, r, V, ldv, W, ldw, co, s));
    return FLP_OK;
}

}  // namespace flp

// The Chebyshev filter of a small matrix in one launch (Section 2.2).
//
// The Clenshaw recurrence acts on each column of the block independently, so
// one workgroup can carry one column through all m steps with nothing but
// its own barriers: the matrix stays in its registers (thread t owns rows t,
// t + 1024, ...; W slots of index and value each), the gathered vector
// U_{k+1} in LDS (two buffers, one barrier per step).  The step-by-step form pays a kernel
// launch per step, 3.3-4.1 us each on a matrix of a few thousand rows
// whatever the bytes; here a step costs its LDS gathers and a barrier: 0.25
// us at 400 rows of 5 nonzeros, 0.45 us at 1600 rows, 1.1 us at 3375 rows of 7
// (FP64).  What bounds it is LDS: every nonzero is one gathered read there.
//
// The sums run in the order of cheb_step_kernel's, with the same rounding of
// every operation, so W is bit-identical to the launches it replaces.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <type_traits>

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

// x of the lane before, within each 16 lanes (the first gets the last one's).
__device__ __forceinline__ float ring16(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x121, 0xF, 0xF, true));  // row_ror:1
}
__device__ __forceinline__ double ring16(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, 0x121, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), 0x121, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The sum of a CSR row's cnt entries from p on, in order, on 16 lanes (lane of
// 0 .. 15): each reads one entry of 16, the next 16 in flight, and the sum goes
// from lane to lane.  Past the last entry it is read again with weight zero,
// as in row_gather.  The sum is the first lane's.
template <typename T>
__device__ __forceinline__ T row_sum16(int lane, int p, int cnt, const int32_t *__restrict__ colind,
                                       const T *__restrict__ val, const T *xs) {
    T sum = T(0);
    const auto load = [&](int k, int &c, T &a) {
        const int q = p + min(k + lane, cnt - 1);
        c = colind[q];
        const T v = val[q];
        a = k + lane < cnt ? v : T(0);
    };
    int c, cn;
    T a, an;
    load(0, c, a);
    for (int k = 0; k < cnt; k += 16) {
        load(k + 16, cn, an);
        const T xv = xs[c];
#pragma unroll
        for (int j = 0; j < 16; ++j) sum = ring16(fma(a, xv, sum));
        c = cn;
        a = an;
    }
    return sum;
}

// The entries past a row's slots ("tail"): classes by their number.
constexpr int kTailClasses = 7;
__device__ __forceinline__ int tail_limit(int cls) { return cls == 0 ? 0 : 2 << cls; }  // 0, 4, 8, 16, 32, 64
__device__ __forceinline__ int tail_class(int tail) {
    int c = 0;
#pragma unroll
    for (int i = 0; i < kTailClasses - 1; ++i) c += tail > tail_limit(i) ? 1 : 0;
    return c;
}

// RPT rows per thread, W register slots per row (an even number).  Column
// indices are kept as 16-bit pairs (n <= 1024 RPT < 2^16).  SELL: rowptr holds
// the slice offsets and colind / val the sliced ELL arrays.
//
// The entries past the slots are read from memory at every step, by the row's
// own thread, or for CSR rows of long tails by 16 lanes that sum the whole row
// whoever owns it (listed in LDS; the sum meets its owner in the buffer that
// the step writes).  A thread takes about 0.12 us per entry, all the rows of
// the workgroup at once but its RPT one after the other; 16 lanes 0.55 us per
// 16 entries, 64 rows at a time, and 0.9 us in all.  From which tail on rows
// are listed is chosen by these costs.  Measured, us for 30 steps at n = 4000
// (launch per step / here / here with every tail read by the row's thread, an
// entry at a time): one row of 4000 6100 / 2040 / 10100, 8 rows of about 500
// 1070 / 358 / 4060, 64 of 63 362 / 150 / 1200, 256 of 18 229 / 213 / 361,
// half the rows of 13 193 / 153 / 212, row lengths of 6.2 +- 2.3 191 / 162 /
// 168; none 182 / 76 / 80.
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
    constexpr int CAP = SELL ? 1 : RPT * kThreads;
    __shared__ unsigned short list[CAP];  // listed rows: from the front the longest class, from the back the others
    __shared__ unsigned tinfo[RPT * kThreads];  // of a row's tail: first entry, number << 16 (below 2^16 each)
    // any tail at all; the longest; bits of the q that have any; rows listed
    // from the front and from the back; 16-entry pieces of the rows of a class
    enum { ANY, LONGEST, QS, FRONT, BACK, PIECES, COUNTS = PIECES + kTailClasses };
    __shared__ int tails[COUNTS];
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
    if (t < COUNTS) tails[t] = 0;
    // the thread's rows: the first W slots (padded with weight zero on the
    // row's own column) and the column of V
    int w = 1;          // slots the wavefront walks
    unsigned over = 0;  // the thread's rows with tails, a bit each
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = t + q * kThreads, row = min(i, n - 1);
        int base, len;
        extent(row, base, len);
        if (i >= n) len = 0;
        if (len > W) over |= 1u << q;
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
    const bool any_over = __ballot(over != 0u) != 0ull;
    // rows per thread that this wavefront has (uniform)
    const int nq = __builtin_amdgcn_readfirstlane((n - (t / WAVE) * WAVE + kThreads - 1) / kThreads);
    __syncthreads();
    if (any_over) {
        if (t % WAVE == 0) tails[ANY] = 1;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            if (!(over >> q & 1u)) continue;
            int base, len;
            extent(t + q * kThreads, base, len);
            tinfo[t + q * kThreads] = (unsigned)(base + W * (SELL ? kSellC : 1)) | (unsigned)(len - W) << 16;
            if constexpr (!SELL) {
                atomicOr(&tails[QS], 1 << q);
                atomicMax(&tails[LONGEST], len - W);
                atomicAdd(&tails[PIECES + tail_class(len - W)], (len + 15) / 16);
            }
        }
    }
    __syncthreads();
    const bool has_tails = __builtin_amdgcn_readfirstlane(tails[ANY]) != 0;
    unsigned far = 0;  // the thread's listed rows
    int nfront = 0, nlist = 0;
    if constexpr (!SELL) {
        if (has_tails) {
            // costs in ns; the last class is listed always
            int own = 0, best = INT_MAX;
            const int nqs = __popc(tails[QS]);
            for (int c = 0; c < kTailClasses - 1; ++c) {
                int p = 0;
                for (int d = c + 1; d < kTailClasses; ++d) p += tails[PIECES + d];
                const int cost = 120 * nqs * min(tail_limit(c), tails[LONGEST]) + (p > 0 ? 900 + 9 * p : 0);
                if (cost < best) {
                    best = cost;
                    own = tail_limit(c);
                }
            }
            if (any_over) {
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    if (!(over >> q & 1u)) continue;
                    const int tail = (int)(tinfo[t + q * kThreads] >> 16);
                    if (tail <= own) continue;
                    const bool front = tail_class(tail) == kTailClasses - 1;
                    const int at = atomicAdd(&tails[front ? FRONT : BACK], 1);
                    list[front ? at : CAP - 1 - at] = (unsigned short)(t + q * kThreads);
                    far |= 1u << q;
                }
            }
            __syncthreads();
            nfront = __builtin_amdgcn_readfirstlane(tails[FRONT]);
            nlist = nfront + __builtin_amdgcn_readfirstlane(tails[BACK]);
        }
    }
    int cur = 0;
    // the steps, without the code for tails where there are none
    const auto steps = [&](auto TAILS) {
        for (int s = 0; s < co.m; ++s) {
            const int nxt = cur == NB - 1 ? 0 : cur + 1, old = NB - cur - nxt;  // old: U_{k+2} of a ring of three
            const T *xs = x[cur];
            int tt = t;
            asm volatile("" : "+v"(tt));  // nothing of the rows' addresses is kept over the steps
            const bool last = s == co.m - 1;
            const T alpha = (T)(s == 0 ? co.alpha0 : (last ? co.alpha_last : co.alpha));
            const T beta = (T)(s == 0 ? co.beta0 : (last ? co.beta_last : co.beta));
            const T gamma = (T)gam[s];
            if (!SELL && TAILS.value && nlist > 0) {  // uniform over the workgroup
                const int lane = tt % 16;
                for (int l = tt / 16; l < nlist; l += kThreads / 16) {
                    const int i = list[l < nfront ? l : CAP - 1 - (l - nfront)];
                    int base, len;
                    extent(i, base, len);
                    const T sum = row_sum16<T>(lane, base, len, colind, val, xs);
                    if (lane == 0) x[nxt][i] = sum;
                }
                __syncthreads();
            }
            T acc[RPT];
            // the gathers of a wavefront's rows: one body per slot count with
            // all of them in flight where registers allow, else two slots at a
            // time (kept packed by the empty asm: unpacked offsets would be
            // hoisted out of the step loop and spill)
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
                const int i = tt + q * kThreads;
                if (TAILS.value && any_over) {
                    if (far >> q & 1u) {
                        acc[q] = x[nxt][i];
                    } else if (over >> q & 1u) {
                        const unsigned e = tinfo[i];
                        int p = (int)(e & 0xffffu);
                        int k = (int)(e >> 16);
                        constexpr int st = SELL ? kSellC : 1;
                        for (; k > 1; k -= 2, p += 2 * st) {
                            const int c0 = colind[p], c1 = colind[p + st];
                            const T a0 = val[p], a1 = val[p + st];
                            acc[q] = fma(a0, xs[c0], acc[q]);
                            acc[q] = fma(a1, xs[c1], acc[q]);
                        }
                        if (k > 0) acc[q] = fma(val[p], xs[colind[p]], acc[q]);
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
    };
    if (has_tails)
        steps(std::true_type{});
    else
        steps(std::false_type{});
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
// noted): 1600 rows FP64 27 against 196 us, 3375 rows of 7 FP64 63 against
// 196 (degree 6: 19 against 23) and FP32 70 against 199, 1728 rows of 13
// FP64 58 against 204, 2744 rows of 13 FP32 84 against 200 (degree 5: 27
// against 23); FP32 at 8000 rows of 7 (spilling) 221 against 200.
// The slots are those of the storage that is read (`stored`) where a
// workgroup has room for 16, so that a sliced ELL copy's padded rows stay in
// registers.  Every row of its slices is as long as the longest, so a copy
// with a slice wider than 8 entries past the slots keeps one launch per step
// (3 slices of 141 in 4000 rows: 627 us for 30 steps against 378).
int small_filter_slots(const flp_filter *p, const flp_csr *A, const flp_csr *stored, int sell_width, bool fp32) {
    const int64_t n = A->n;
    if (p->m < 4 || p->m > kSmallMaxDegree) return 0;
    int slots = 0;
    if (A->nnz <= 8 * n) {
        if (n <= 4 * kThreads) slots = stored->nnz > 8 * n && n <= 2 * kThreads ? 16 : 8;
    } else if (A->nnz <= 16 * n && n <= (fp32 ? 3 : 2) * kThreads) {
        if (n <= 2 * kThreads || p->m >= 8) slots = 16;
    }
    return sell_width <= slots + 8 ? slots : 0;
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

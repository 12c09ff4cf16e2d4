// First update and second projection of a two-pass Gram-Schmidt in one read
// of the basis (Section 3.2.2's reorthogonalisation, full on both passes):
//   W -= Q H1,   partial sums of H2 = Q^T W
// for a basis Q of K columns and a block W of c <= 16.
#include "flp_internal.h"
#include "flp_device.h"
#include "flp_gemm.h"

#include <algorithm>

namespace flp {

namespace {

typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

// Barrier of LDS accesses alone: global loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A block takes `rows` rows of Q and W, 16 at a time; its NW waves hold the
// K columns of those rows in registers, KT tiles of 16 columns each (lane:
// row l%16, columns 4 (l/16) .. + 3).  Per 16 rows:
//   * every wave multiplies its tiles with its rows of H1 (held in registers
//     throughout); the first wave's W - Q H1 and the others' sums meet in LDS
//     (W is read by the first wave alone and before the barrier, so no read
//     of it is in flight when the rows are written), and every wave takes the
//     result from there in the D layout of the product;
//   * that layout is the operand layout of Q^T W with the rows on l/16; the
//     tiles of Q, which have them on l%16, are transposed through LDS (a
//     wave's own, so without a barrier) and multiplied into the wave's rows
//     of H2, which stay in registers until the end.
// The next 16 rows of Q and W are loaded meanwhile.  One barrier of LDS
// accesses per 16 rows (red is used in turns).  Bound by the read of Q:
// n = 1e6, K = 320, c = 8: 619 us (4.1 TB/s) where the update and the
// projection by themselves take 546 + 473; K = 100: 216 for 176 + 150; n =
// 59319, K = 135, c = 5: 26 for 24 + 16.
template <int NW, int KT>
__global__ __launch_bounds__(64 * NW, 2) void cgs2_fused_kernel(int n, int K, int c, int rows, const DMat Q,
                                                                const double *__restrict__ H, double *W,
                                                                double *__restrict__ part) {
    constexpr int LD = 18;  // doubles per row of a tile in LDS: 16-byte pieces, no bank conflicts
    __shared__ double red[2][NW][4][WAVE];
    __shared__ double tile[NW][KT][16 * LD];
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int kq = lane / 16, m = lane % 16;
    const int r0 = blockIdx.x * rows, r1 = min(n, r0 + rows);
    const int t0 = wave * KT;  // the wave's first tile
    const double *qc[KT];
    double h[KT][4];
    dbl4 acc2[KT];
#pragma unroll
    for (int i = 0; i < KT; ++i) {
        const int kb = 16 * (t0 + i) + 4 * kq;
        qc[i] = col_base(Q, min(kb, (K - 1) & ~3));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double x = as_global(H)[(int64_t)min(kb + q, K - 1) * c + min(m, c - 1)];
            h[i][q] = kb + q < K && m < c ? x : 0.0;
        }
        acc2[i] = dbl4{0.0, 0.0, 0.0, 0.0};
    }
    // columns past K: the last tile's are clamped (their weights are zero and
    // their products discarded), whole tiles past it are skipped
    const auto load_q = [&](int g, double (&a)[KT][4]) {
        const int64_t off = (int64_t)min(g + m, r1 - 1) * Q.ld;
#pragma unroll
        for (int i = 0; i < KT; ++i) {
            const int k0 = 16 * (t0 + i);
            if (k0 + 16 <= K) {  // uniform
                const auto p = as_global(qc[i]) + off;
                const dbl2u x0 = *reinterpret_cast<gptr<dbl2u>>(p);
                const dbl2u x1 = *reinterpret_cast<gptr<dbl2u>>(p + 2);
                a[i][0] = x0.x;
                a[i][1] = x0.y;
                a[i][2] = x1.x;
                a[i][3] = x1.y;
            } else if (k0 < K) {
                const int kb = min(k0 + 4 * kq, (K - 1) & ~3);
#pragma unroll
                for (int q = 0; q < 4; ++q) a[i][q] = as_global(qc[i])[off + min(q, K - 1 - kb)];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) a[i][q] = 0.0;
            }
        }
    };
    const auto load_w = [&](int g, double (&w)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            w[v] = as_global(W)[(int64_t)min(g + kq + 4 * v, r1 - 1) * c + min(m, c - 1)];
    };
    double a[KT][4], w[4] = {};
    load_q(r0, a);
    if (wave == 0) load_w(r0, w);
    for (int g = r0, b = 0; g < r1; g += 16, b ^= 1) {
        double an[KT][4], wn[4] = {};
        load_q(min(g + 16, r1 - 1), an);
        if (wave == 0) load_w(min(g + 16, r1 - 1), wn);
        dbl4 acc = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < KT; ++i) {
            double *t = &tile[wave][i][m * LD + 4 * kq];
            *reinterpret_cast<dbl2 *>(t) = dbl2{a[i][0], a[i][1]};
            *reinterpret_cast<dbl2 *>(t + 2) = dbl2{a[i][2], a[i][3]};
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = mfma16x16x4(a[i][q], h[i][q], acc);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) red[b][wave][v][lane] = wave == 0 ? w[v] - acc[v] : -acc[v];
        lds_barrier();
        double w2[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double s = 0.0;
#pragma unroll
            for (int y = 0; y < NW; ++y) s += red[b][y][v][lane];
            const int row = g + kq + 4 * v;
            w2[v] = row < r1 && m < c ? s : 0.0;
            if (wave == (v & (NW - 1)) && row < r1 && m < c) as_global_mut(W)[(int64_t)row * c + m] = w2[v];
        }
#pragma unroll
        for (int i = 0; i < KT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc2[i] = mfma16x16x4(tile[wave][i][(kq + 4 * v) * LD + m], w2[v], acc2[i]);
#pragma unroll
        for (int i = 0; i < KT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) a[i][q] = an[i][q];
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = wn[v];
    }
    const auto d = as_global_mut(part) + (size_t)blockIdx.x * K * c;
#pragma unroll
    for (int i = 0; i < KT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = 16 * (t0 + i) + kq + 4 * v;
            if (k < K && m < c) d[(size_t)k * c + m] = acc2[i][v];
        }
}

}  // namespace

// Rows per block, whole tiles: two blocks of 256 threads are resident on a
// compute unit where the columns take three tiles per wave or more, four with
// fewer (us with 512 / 1024 blocks: n = 1e6, K = 320 619 / 625, K = 64 209 /
// 152; n = 59319, K = 300 45 / 52).
int cgs2_fused_rows(int n, int K) {
    const int blocks = K > 128 ? 512 : 1024;
    return std::max(16, ((n + blocks - 1) / blocks + 15) / 16 * 16);
}

// Eight waves of five tiles at most: wider bases take the two kernels.  So do
// the narrowest on many rows: four waves share at most two tiles then, and the
// loop's barrier is what they wait for (whole calls, us, two kernels / one: n =
// 1e6, c = 1, K = 8 171 / 226, K = 32 214 / 260; c = 8, K = 8 180 / 231, K = 32
// 280 / 290; c = 16, K = 20 277 / 298; n = 2e5, c = 8, K = 8 74 / 86, K = 32
// 87 / 92; the other side of the line, with the partial sums' reduction of the
// time: n = 1e6, c = 1, K = 36 305 / 294, c = 8, K = 40 380 / 340, c = 16, K =
// 24 329 / 317; n = 1e5, c = 8, K = 8 69 / 70).
bool cgs2_fused_ok(int n, int K, int c) {
    if (c > 16 || K > 640) return false;
    return n <= (1 << 17) || K > (c <= 8 ? 32 : 20);
}

hipError_t launch_cgs2_fused(int n, int K, int c, DMat Q, const double *H, double *W, double *part, hipStream_t s) {
    const int rows = cgs2_fused_rows(n, K), blocks = (n + rows - 1) / rows;
    const int tiles = (K + 15) / 16;
#define FLP_FUSED(NW, KT)                                                                                          \
    if (tiles <= NW * KT) {                                                                                        \
        hipLaunchKernelGGL((cgs2_fused_kernel<NW, KT>), dim3(blocks), dim3(64 * NW), 0, s, n, K, c, rows, Q, H, W, \
                           part);                                                                                  \
        return hipGetLastError();                                                                                  \
    }
    FLP_FUSED(4, 1)
    FLP_FUSED(4, 2)
    FLP_FUSED(4, 3)
    FLP_FUSED(4, 4)
    FLP_FUSED(4, 5)
    FLP_FUSED(8, 3)
    FLP_FUSED(8, 4)
    FLP_FUSED(8, 5)
#undef FLP_FUSED
    return hipErrorInvalidValue;
}

}  // namespace flp

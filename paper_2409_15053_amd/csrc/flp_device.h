// Device-side helpers shared by the filter and the Gram-Schmidt kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace flp {
namespace {

constexpr int WAVE = 64;
constexpr int NXCD = 8;

// Blocks are dispatched round-robin over the 8 XCDs (block b runs on XCD
// b % 8).  Renumber so that each XCD receives one contiguous range of tiles:
// neighbouring rows of the matrix then share that XCD's L2 for the gathered
// vector entries.
__host__ __device__ __forceinline__ int xcd_tile(int b, int G) {
    int q = G / NXCD, rem = G % NXCD;
    int x = b % NXCD, s = b / NXCD;
    return (x < rem) ? x * (q + 1) + s : rem * (q + 1) + (x - rem) * q + s;
}

// Pencil walk over planes of PT consecutive tiles (PT >= NXCD): the tiles
// form Z = G / PT planes (the z-planes of a 3D grid when PT tiles hold one
// N^2 plane of rows) plus a tail.  Each plane is cut into NXCD column ranges
// (pencils); the enumeration takes pencil 0 plane by plane, then pencil 1,
// ..., then the tail in order, and XCD x receives one contiguous stretch of
// it (the positions xcd_tile gives its blocks).  An XCD thus walks its
// pencil through the planes: a row's neighbours in the planes below and
// above (the +-N^2, +-2N^2 columns of a stencil) were gathered by the same
// XCD a few planes earlier, and the few planes of its pencil in flight fit
// that XCD's L2, where the plain row order has a whole plane per XCD step.
// Bijective on [0, G).
__host__ __device__ __forceinline__ int plane_tile(int b, int G, int PT) {
    const int e = xcd_tile(b, G);
    const int Z = G / PT;
    if (PT < NXCD || Z == 0 || e >= Z * PT) return e;
    const int col = e / Z;                    // Z lo(p) <= e < Z lo(p+1)  <=>  lo(p) <= e / Z < lo(p+1)
    const int pc = (NXCD * col + NXCD - 1) / PT, p = pc < NXCD - 1 ? pc : NXCD - 1;
    const int lo = p * PT / NXCD, w = (p + 1) * PT / NXCD - lo;
    const int local = e - Z * lo;
    return (local / w) * PT + lo + local % w;
}

// The tile a block processes.  chunk == 0: xcd_tile (one contiguous range of
// tiles per XCD).  chunk > 0: the tiles are cut into chunks of `chunk`
// consecutive tiles dealt to the XCDs in turn (chunk q on XCD q % 8).
// Blocks dispatched together then cover one contiguous stretch of rows on
// all XCDs at once, so rows far apart in a row's neighbour list (a 3D
// grid's +-plane neighbours) are gathered while still in the shared
// Infinity Cache, and rows up to a chunk apart share an XCD's L2.  The last
// G mod (8 chunk) tiles keep block order.  chunk < 0: plane_tile with planes
// of -chunk matrix rows (rows_per_tile rows per tile).  Bijective on [0, G).
__host__ __device__ __forceinline__ int chunk_tile(int b, int G, int chunk, int rows_per_tile) {
    if (chunk < 0) return plane_tile(b, G, (-chunk + rows_per_tile / 2) / rows_per_tile);
    if (chunk == 0) return xcd_tile(b, G);
    const int span = NXCD * chunk;
    const int full = (G / span) * span;
    if (b >= full) return b;
    const int x = b % NXCD, s = b / NXCD;
    return (s / chunk) * span + x * chunk + s % chunk;
}

// SplitMix64 (Steele, Lea & Flood, OOPSLA 2014): the output function applied
// to a Weyl sequence; used here as a counter-based generator.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// Entry idx of the N(0, 1) sequence (seed, sid): 53-bit uniforms in (0, 1] and
// [0, 1), Box-Muller.
__device__ __forceinline__ double normal_at(uint64_t seed, uint64_t sid, uint64_t idx) {
    const uint64_t key = splitmix64(seed ^ splitmix64(sid));
    const uint64_t u1 = splitmix64(key + 2 * idx), u2 = splitmix64(key + 2 * idx + 1);
    const double a = ((u1 >> 11) + 1) * (1.0 / 9007199254740992.0);
    const double b = (u2 >> 11) * (1.0 / 9007199254740992.0);
    return sqrt(-2.0 * log(a)) * cospi(2.0 * b);
}

// A piece of VEC elements of at most 16 bytes, aligned to its elements only:
// a global access of up to 16 bytes needs no more than 4-byte alignment on
// gfx950, so block widths and leading dimensions that are no multiple of 16
// bytes are read and written in whole pieces too.
template <typename T, int VEC>
struct Vec {
    typedef T type __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
};

// Loads and stores of VEC consecutive elements in pieces of up to 16 bytes.
template <typename T, int VEC>
__device__ __forceinline__ void load_vec(const T *p, T (&v)[VEC]) {
    constexpr int C = VEC * (int)sizeof(T) > 16 ? 16 / (int)sizeof(T) : VEC;
    static_assert(VEC % C == 0, "vector width must be a multiple of 16 bytes");
#pragma unroll
    for (int k = 0; k < VEC / C; ++k) {
        if constexpr (C == 1) {
            v[k] = p[k];
        } else {
            const auto x = *reinterpret_cast<const typename Vec<T, C>::type *>(p + k * C);
#pragma unroll
            for (int j = 0; j < C; ++j) v[k * C + j] = x[j];
        }
    }
}

template <typename T, int VEC>
__device__ __forceinline__ void store_vec(T *p, const T (&v)[VEC]) {
    constexpr int C = VEC * (int)sizeof(T) > 16 ? 16 / (int)sizeof(T) : VEC;
    static_assert(VEC % C == 0, "vector width must be a multiple of 16 bytes");
#pragma unroll
    for (int k = 0; k < VEC / C; ++k) {
        if constexpr (C == 1) {
            p[k] = v[k];
        } else {
            typename Vec<T, C>::type x;
#pragma unroll
            for (int j = 0; j < C; ++j) x[j] = v[k * C + j];
            *reinterpret_cast<typename Vec<T, C>::type *>(p + k * C) = x;
        }
    }
}

// store_vec of a lane's values as the output type.
template <typename T, typename Tout, int VEC>
__device__ __forceinline__ void store_cast(Tout *p, const T (&v)[VEC]) {
    Tout o[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) o[i] = (Tout)v[i];
    store_vec<Tout, VEC>(p, o);
}

}  // namespace
}  // namespace flp

// Launch-shape helpers shared by the kernel sources (internal header).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "fft_tile.h"

namespace ips {

constexpr int NT = 256;

inline bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

inline int len_kind(int N)
{
    int r = N;
    for (int p : {2, 3, 5})
        while (r % p == 0) r /= p;
    return is_pow2(N) ? kPow2 : r == 1 ? kSmooth : kAnyLen;
}

// f(kind) with the kind as a compile-time constant.
template <typename F>
inline void with_kind(int kind, F f)
{
    if (kind == kPow2)
        f(std::integral_constant<int, kPow2>());
    else if (kind == kSmooth)
        f(std::integral_constant<int, kSmooth>());
    else
        f(std::integral_constant<int, kAnyLen>());
}
template <typename F>
inline void by_kind(int N, F f)
{
    with_kind(len_kind(N), f);
}

// As by_kind, powers of two and everything else only.
template <typename F>
inline void by_pow2(int N, F f)
{
    if (is_pow2(N))
        f(std::integral_constant<int, kPow2>());
    else
        f(std::integral_constant<int, kAnyLen>());
}

// The tile helpers address a tile with 32-bit offsets r * rsd + c * csd built
// from 24-bit multiplies (toff): strides below 2^23, extent below 2^31.
inline bool tile_strides_ok(int64_t nrows, int64_t rsd, int64_t ncols, int64_t csd)
{
    const int64_t lim24 = (int64_t)1 << 23, lim31 = ((int64_t)1 << 31) - 1;
    const int64_t ar = rsd < 0 ? -rsd : rsd, ac = csd < 0 ? -csd : csd;
    return ar < lim24 && ac < lim24 && nrows < lim24 && ncols < lim24 && nrows * ar + ncols * ac < lim31;
}

// Raise a kernel's dynamic LDS limit above 64 KiB when a launch needs it.
void set_lds(const void *fn, size_t bytes);

// Blocks of a kernel that fit on the device at once (0 if unknown).
int resident_blocks(const void *fn, int nthreads, size_t lds);

// Transforms longer than kLdsTwMaxN run in blocks of NTB threads whose tile
// holds one complex sequence without row padding (W = 2) and whose twiddles
// are read from the global table (the LDS holds only the tile).
constexpr int NTB = 1024;
constexpr int kLdsTwMaxN = 2048;

inline bool big_fft(int N) { return N > kLdsTwMaxN; }

// f(elements per thread, threads) for the one-block 1D kernels of length N.
template <typename F>
inline hipError_t by_length(int N, F f)
{
    using std::integral_constant;
    if (N <= 4 * NT) return f(integral_constant<int, 4>(), integral_constant<int, NT>());
    if (!big_fft(N)) return f(integral_constant<int, 8>(), integral_constant<int, NT>());
    if (N <= 4 * NTB) return f(integral_constant<int, 4>(), integral_constant<int, NTB>());
    if (N <= 8 * NTB) return f(integral_constant<int, 8>(), integral_constant<int, NTB>());
    return hipErrorInvalidValue;
}

template <typename T>
inline size_t tile_lds(int N, int W)
{
    if (big_fft(N)) return (size_t)N * W * sizeof(T);
    return (size_t)N * sizeof(cx<T>) + (size_t)N * (W + 1) * sizeof(T);
}

// Default width of the register tiles of N rows (0: none).
inline int rt_width(int N)
{
    return N >= 256 && N <= 8192 && is_pow2(N) ? std::max(2, 4096 / N) : 0;
}

// f(RegTile) of the register tile that has N rows and W columns; whether there is
// one: the default width of every power of two from 256 on, and those of WIDER (a sum
// of kWide512, kWide1024: twice the default; kQuad1024: four times), where a kernel
// measured faster so.
enum { kWide512 = 1, kWide1024 = 2, kQuad1024 = 4 };

template <int WIDER, typename F>
inline bool rt_tile(int N, int W, F f)
{
#define IPS_RT(...)                                                     \
    if (RegTile<__VA_ARGS__>::N == N && RegTile<__VA_ARGS__>::W == W) { \
        f(RegTile<__VA_ARGS__>());                                      \
        return true;                                                    \
    }
    IPS_RT(256) IPS_RT(512) IPS_RT(1024) IPS_RT(2048) IPS_RT(4096) IPS_RT(8192)
    if constexpr ((WIDER & kWide512) != 0) IPS_RT(512, 8)
    if constexpr ((WIDER & kWide1024) != 0) IPS_RT(1024, 4)
    if constexpr ((WIDER & kQuad1024) != 0) IPS_RT(1024, 8)
#undef IPS_RT
    return false;
}

// Twiddle table of the transform type: LDS copy (short transforms) or the
// plan's global table (long ones).
template <typename T, bool BIG>
__device__ __forceinline__ const cx<T> *tw_table(unsigned char *smem, const cx<double> *twd,
                                                const cx<float> *twf)
{
    if constexpr (BIG) {
        if constexpr (sizeof(T) == sizeof(float))
            return reinterpret_cast<const cx<T> *>(twf);
        else
            return reinterpret_cast<const cx<T> *>(twd);
    } else {
        return reinterpret_cast<const cx<T> *>(smem);
    }
}

} // namespace ips

// In-register DFTs with compile-time twiddles, used by the four-step FFT
// kernels.  Host-callable as well, so the building blocks can be checked on
// the CPU.
#pragma once

#include <utility>

#include "amap_device.h"

namespace amap {

// ---- compile-time twiddles and in-register DFTs -------------------------------
struct CS {
    double c, s;
};
// cos and sin of 2 pi k / 64 for the first eighth of a turn, rounded to
// double precision (17 digits determine the value).
constexpr double kCos64[9] = {1.0, 0.9951847266721969, 0.9807852804032304, 0.9569403357322088, 0.9238795325112867,
                              0.881921264348355, 0.8314696123025452, 0.773010453362737, 0.7071067811865476};
constexpr double kSin64[9] = {0.0, 0.0980171403295606, 0.19509032201612828, 0.2902846772544624, 0.3826834323650898,
                              0.47139673682599764, 0.5555702330196022, 0.6343932841636455, 0.7071067811865476};
// cos and sin of 2 pi k / R, R a power of two up to 64: the angle mod a
// quarter turn, reflected into its first half, then the quarter's signs, so
// that every value is a correctly rounded one.
constexpr CS cos_sin_2pi(int k, int R) {
    const int k64 = (((k % R) + R) % R) * (64 / R), r = k64 % 16;
    const double c = r <= 8 ? kCos64[r] : kSin64[16 - r], s = r <= 8 ? kSin64[r] : kCos64[16 - r];
    switch (k64 / 16) {
        case 0: return CS{c, s};
        case 1: return CS{-s, c};
        case 2: return CS{-c, -s};
        default: return CS{s, -c};
    }
}

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v / 2); }
constexpr int bitrev(int i, int bits) {
    int r = 0;
    for (int b = 0; b < bits; ++b) r |= ((i >> b) & 1) << (bits - 1 - b);
    return r;
}

// One radix-2 butterfly of a length-LEN stage with twiddle W_LEN^K
// (exp(-2 pi i K/LEN) forward, conjugate inverse); trivial twiddles cost no
// multiplication.  Others take six fused multiply-adds: x' = x + w y as two
// chained FMAs per component, then y' = 2 x - x' (which differs from x - w y
// only by the rounding of x').
template <typename T, bool INV, int LEN, int K>
__host__ __device__ __forceinline__ void bfly(cpx<T>& x, cpx<T>& y) {
    if constexpr (K == 0 || 4 * K == LEN) {
        const cpx<T> t = K == 0 ? y : rot90<T, INV>(y);
        y = x - t;
        x = x + t;
    } else {
        constexpr CS w = cos_sin_2pi(K, LEN);
        const T wr = (T)w.c, wi = INV ? (T)w.s : (T)-w.s;
        const T xr = (T)fma(wr, y.x, (T)fma(-wi, y.y, x.x));
        const T xi = (T)fma(wr, y.y, (T)fma(wi, y.x, x.y));
        y = make_cpx<T>((T)fma((T)2, x.x, -xr), (T)fma((T)2, x.y, -xi));
        x = make_cpx<T>(xr, xi);
    }
}

template <typename T, bool INV, int LEN, int... I>
__host__ __device__ __forceinline__ void dft_stage(cpx<T>* a, std::integer_sequence<int, I...>) {
    (bfly<T, INV, LEN, I % (LEN / 2)>(a[(I / (LEN / 2)) * LEN + I % (LEN / 2)],
                                      a[(I / (LEN / 2)) * LEN + I % (LEN / 2) + LEN / 2]),
     ...);
}

template <typename T, bool INV, int R, int LEN>
__host__ __device__ __forceinline__ void dft_stages(cpx<T>* a) {
    if constexpr (LEN <= R) {
        dft_stage<T, INV, LEN>(a, std::make_integer_sequence<int, R / 2>{});
        dft_stages<T, INV, R, LEN * 2>(a);
    }
}

template <typename T, int R, int... I>
__host__ __device__ __forceinline__ void bitrev_copy(cpx<T>* out, const cpx<T>* in,
                                           std::integer_sequence<int, I...>) {
    ((out[I] = in[bitrev(I, ilog2c(R))]), ...);
}

// In-register DFT of length R (power of two), natural order in and out:
// a[k] <- sum_j a[j] exp(-+2 pi i j k / R).  Unnormalised.
template <typename T, int R, bool INV>
__host__ __device__ __forceinline__ void dft_reg(cpx<T> (&a)[R]) {
    if constexpr (R > 1) {
        cpx<T> b[R];
        bitrev_copy<T, R>(b, a, std::make_integer_sequence<int, R>{});
        dft_stages<T, INV, R, 2>(b);
#pragma unroll
        for (int i = 0; i < R; ++i) a[i] = b[i];
    }
}

}  // namespace amap

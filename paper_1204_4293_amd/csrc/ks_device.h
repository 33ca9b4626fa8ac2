// Device helpers shared by the Kaiser-Squires kernel families: twiddles from
// the table, the strip numbering of the column passes, and the Hermitian
// parts and column packing of the row passes.
#pragma once

#include "amap_device.h"
#include "amap_launch.h"
#include "fft_reg.h"

namespace amap {

// K consecutive values at p (16-byte aligned) through 16-byte loads.
template <typename T, int K>
__device__ __forceinline__ void load16(const T* __restrict__ p, T (&out)[K]) {
    if constexpr (sizeof(T) == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i < K / 4; ++i) {
            const f4 v = reinterpret_cast<const f4*>(p)[i];
            out[4 * i] = v[0]; out[4 * i + 1] = v[1]; out[4 * i + 2] = v[2]; out[4 * i + 3] = v[3];
        }
    } else {
        typedef double d2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < K / 2; ++i) {
            const d2 v = reinterpret_cast<const d2*>(p)[i];
            out[2 * i] = v[0]; out[2 * i + 1] = v[1];
        }
    }
}

__device__ __forceinline__ int signed_freq(int i, int n) { return i < n / 2 ? i : i - n; }

// Reciprocal: the hardware estimate (1 ulp) in single precision, a rounded
// division in double.
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }
// x / den with r = recip(den); in double precision corrected by the
// remainder, so that it carries one rounding like a division.
__device__ __forceinline__ float ratio(float x, float, float r) { return x * r; }
__device__ __forceinline__ double ratio(double x, double den, double r) {
    const double q = x * r;
    return fma(fma(-q, den, x), r, q);
}

// exp(-+2 pi i e / N) from the table of N entries (kTwiddles: the tables of
// 4096, 2048, ... points one after the other, so that a small transform's
// gathers stay in few cache lines).
template <typename T, int LOGN, bool INV>
__device__ __forceinline__ cpx<T> table_twiddle(const cpx<T>* __restrict__ tw, int e) {
    const cpx<T> w = tw[2 * kMaxN - (2 << LOGN) + (e & ((1 << LOGN) - 1))];
    return INV ? make_cpx(w.x, -w.y) : w;
}

// exp(-+2 pi i base k / N) for k = 1 .. K-1, passed to f(k, w) in increasing
// k: five table reads (base times 1, 2, 4, 8, 16) and one complex product
// per power, w(k) = w(k without its lowest set bit) * w(lowest set bit), so
// each power carries at most four roundings and only a few are live at once.
template <typename T, int LOGN, bool INV, int K, typename Fn>
__device__ __forceinline__ void twiddle_powers(const cpx<T>* __restrict__ tw, int base, Fn&& f) {
    static_assert(K <= 64, "at most 64 powers");
    constexpr int NB = K <= 2 ? 1 : (K <= 4 ? 2 : (K <= 8 ? 3 : (K <= 16 ? 4 : (K <= 32 ? 5 : 6))));
    cpx<T> p[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) p[b] = table_twiddle<T, LOGN, INV>(tw, base << b);
    cpx<T> w[K];
#pragma unroll
    for (int k = 1; k < K; ++k) {
        const int low = k & -k, rest = k - low;
        const int bit = __builtin_ctz(low);
        w[k] = rest ? cmul(w[rest], p[bit]) : p[bit];
        f(k, w[k]);
    }
}

// Strip s and map b of the column kernels' workgroup.  With xcd = 1,
// workgroups are renumbered so that consecutive strips of a map run on one
// XCD (the hardware deals workgroups out to the eight XCDs in turn): strips
// whose row segments share a cache line then meet in one L2 instead of each
// XCD fetching the whole line.  xcd = 2, for realisations that all read one
// input larger than the L2s: as 1, but all maps of a strip before the next
// strip, so that the input's lines are fetched once for all of them.
__device__ __forceinline__ void strip_of(int xcd, int& s, int& b) {
    s = blockIdx.x;
    b = blockIdx.y;
    const int nx = gridDim.x;
    const int total = nx * gridDim.y;
    if (xcd) {
        // XCD k runs workgroups k, k + 8, ..: one more where total is no multiple of 8
        const int l = blockIdx.x + nx * blockIdx.y, k = l & 7;
        const int v = k * (total >> 3) + min(k, total & 7) + (l >> 3);
        if (xcd == 2) {
            b = v % (int)gridDim.y;
            s = v / (int)gridDim.y;
        } else {
            s = v % nx;
            b = v / nx;
        }
    }
}
// Orders the LDS accesses of one wavefront (the lanes of one transform).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Twice the Hermitian part of K at k, from a = K(k) and b = K(-k): of K
// itself (kappa_E) or of -i K (b_mode: kappa_B).
template <typename T>
__device__ __forceinline__ cpx<T> hermitian(const cpx<T>& a, const cpx<T>& b, bool b_mode) {
    return b_mode ? make_cpx(a.y + b.y, b.x - a.x) : make_cpx(a.x + b.x, a.y - b.y);
}

// The value of the other lane of a lane pair (2i, 2i + 1).
__device__ __forceinline__ float lane_swap1(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_swap1(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0xB1, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0xB1, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// The packed value of a lane pair's columns (x even in the even lane, x + 1
// in the odd): own = h(y, x) of this lane.  The even lane returns z(y, x/2),
// the odd one z(-y, x/2); for the rows 0 and n/2 in one (`self`), whose
// h are real and imaginary part of own, z(0, x/2) and z(n/2, x/2).
template <typename T>
__device__ __forceinline__ cpx<T> pack_columns(const cpx<T>& own, bool odd, bool self) {
    const T ox = lane_swap1(own.x), oy = lane_swap1(own.y);
    if (self) return odd ? make_cpx(oy, own.y) : make_cpx(own.x, ox);
    return odd ? make_cpx(ox + own.y, own.x - oy) : make_cpx(own.x - oy, own.y + ox);
}

// The passes of large transforms (ks_fft3.hip).
template <typename T, int LOGN, bool CROP> hipError_t launch_ks3_fwd(const KsArgs<T>& a);
template <typename T, int LOGN, bool CROP> hipError_t launch_ks3_rows(const KsArgs<T>& a);
template <typename T, int LOGN, bool CROP> hipError_t launch_ks3_inv(const KsArgs<T>& a);

}  // namespace amap

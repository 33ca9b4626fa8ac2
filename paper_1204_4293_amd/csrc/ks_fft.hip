// Kaiser-Squires inversion on the GPU: a two-dimensional complex FFT with the
// spectral multiply by conj(D(k)) fused between the forward and inverse
// transforms along x.
//
// Pass structure for one n x n map (columns first, so that the row pass sees
// whole spectral rows and can apply the KS kernel between its forward and
// inverse transforms):
//   P1  column strips:  (g1 + i g2) [optionally rotated by Philox phases]
//                       -> forward FFT along y             -> C
//   P2  rows y, -y:     forward FFT along x, multiply by conj(D)/n^2,
//                       Hermitian part, inverse FFT along x, two columns
//                       packed into one                    -> half of C
//   P3  column strips:  inverse FFT along y -> two columns of kappa_E
// A strip is W adjacent columns, so every HBM access is a W-element row
// segment; a row pass reads whole rows and writes their left halves.
//
// Fields that are zero outside an ny x nx rectangle at the grid's origin
// (CROP) are read and written at their own size: P1 takes only the strips
// the field reaches, P2 reads and writes only those columns, P3 writes only
// the field's rows.
//
// Each length-N transform is a four-step FFT with N = N1 * N2: every thread
// holds N1 (then N2) values in registers and runs a radix-2 DFT on them with
// compile-time twiddles, the inter-step twiddles come from a table, and one
// LDS exchange separates the two steps.  Along x a transform's N2 threads
// sit in one wavefront, so the exchange needs no workgroup barrier, and the
// inverse transform starts from the forward output exactly as each thread
// holds it.  Transforms whose per-thread DFTs would fill the register file,
// and row passes from 128 points, run the three-step kernels of ks_fft3.hip.
#include "ks_device.h"

namespace amap {

// Four-step factors: N = N1 * N2, N1 = N2 or 2 N2.
template <int LOGN>
struct FS {
    static constexpr int N = 1 << LOGN;
    static constexpr int N1 = 1 << ((LOGN + 1) / 2);
    static constexpr int N2 = 1 << (LOGN / 2);
    static constexpr int RR = N1 / N2;
};

// Threads and LDS of the four-step column kernels: strips of W columns, N2
// threads per column; WREQ (if smaller) narrows the strip so that a small
// batch still spreads over many workgroups.  A strip's N x W values pass
// through LDS in PH phases of N / PH rows (loads) and N1 / PH first-step
// outputs (exchange).
//   forward (FWD): up to 16 columns and 512 threads.  Where a thread's
//     first-step DFT fits half the register file (FP32, N1 <= 32) the
//     phases keep LDS at 64 KiB and the kernel is built for two workgroups
//     per CU; otherwise LDS is held to 128 KiB at one workgroup per CU;
//   inverse: as many columns (up to 16) as 128 KiB of LDS holds in one
//     phase.  Its first step loads straight from memory and keeps many
//     values in flight, so neither a register cap nor narrower phases pay.
template <typename T, int LOGN, bool FWD, int WREQ = 0>
struct Strip4 {
    static constexpr int N = 1 << LOGN, N1 = FS<LOGN>::N1, N2 = FS<LOGN>::N2;
    static constexpr int CPX = (int)sizeof(cpx<T>);
    static constexpr int WT = 512 / N2 > 16 ? 16 : 512 / N2;
    static constexpr int WL = (128 * 1024 / CPX) / N > 16 ? 16 : (128 * 1024 / CPX) / N;
    static constexpr int WMAX = FWD ? WT : WL;
    static constexpr int W = (WREQ > 0 && WREQ < WMAX) ? WREQ : WMAX;
    static constexpr int NT = W * N2;
    static constexpr bool TWO = FWD && sizeof(T) == 4 && N1 <= 32 && NT >= 256;
    static constexpr int CAP = TWO ? 64 * 1024 : 128 * 1024;
    static constexpr int BYTES = N * W * CPX;
    static constexpr int PH0 = BYTES <= CAP ? 1 : BYTES / CAP;
    static constexpr int PH = PH0 > N1 ? N1 : PH0;
    static constexpr int LDS = N * W / PH;  // complex values
    static constexpr int MINW = TWO ? 2 * NT / 256 : 1;  // waves per SIMD for two workgroups
    static_assert(N1 % PH == 0, "phases split the first-step index evenly");
};
template <typename T, int LOGN, int WREQ = 0>
using StripF = Strip4<T, LOGN, true, WREQ>;
template <typename T, int LOGN, int WREQ = 0>
using StripI = Strip4<T, LOGN, false, WREQ>;

// Exchange region of one row: forward [N1][N2+1], inverse [N2][N1+1].
template <int LOGN>
constexpr int row4_elems() {
    constexpr int N1 = FS<LOGN>::N1, N2 = FS<LOGN>::N2;
    return (N1 * (N2 + 1)) > (N2 * (N1 + 1)) ? (N1 * (N2 + 1)) : (N2 * (N1 + 1));
}

// ---- P1: load shears (optionally rotate), forward FFT along y (four-step) -------
// CROP: the shears are ny x nx, row-major, zero outside; only the strips they
// reach run.
template <typename T, int LOGN, bool ROTATE, bool CROP, int WREQ>
__global__ void __launch_bounds__((StripF<T, LOGN, WREQ>::NT), (StripF<T, LOGN, WREQ>::MINW))
k_ks_cols_fwd(const T* __restrict__ g1, const T* __restrict__ g2, long long g_stride,
              const long long* __restrict__ g1_off, const long long* __restrict__ g2_off,
              cpx<T>* __restrict__ C, uint64_t seed, uint64_t r0, const cpx<T>* __restrict__ tw,
              int xcd, int ny, int nx) {
    using F = FS<LOGN>;
    using S = StripF<T, LOGN, WREQ>;
    constexpr int N = F::N, N1 = F::N1, N2 = F::N2, W = S::W, NT = S::NT, PH = S::PH;
    constexpr int ROWS = N / PH, K = N1 / PH;  // rows and first-step indices per phase
    __shared__ cpx<T> buf[S::LDS];
    int sx, b;
    strip_of(xcd, sx, b);
    const int x0 = sx * W;
    const T* a1 = g1 + (g1_off ? g1_off[b] : (long long)b * g_stride);
    const T* a2 = g2 + (g2_off ? g2_off[b] : (long long)b * g_stride);
    constexpr int G = 16 / (int)sizeof(T);  // values per 16-byte load
    const int c = threadIdx.x % W, t = threadIdx.x / W;
    // row y = N2 n1 + t of column c goes to a[n1]; phase p stages rows
    // p ROWS .. (p+1) ROWS - 1, i.e. n1 = p K .. (p+1) K - 1
    cpx<T> a[N1];
#pragma unroll
    for (int p = 0; p < PH; ++p) {
        const int y0 = p * ROWS;
        if (CROP && y0 >= ny) {  // rows outside the field
#pragma unroll
            for (int n1 = 0; n1 < K; ++n1) a[p * K + n1] = make_cpx((T)0, (T)0);
            continue;
        }
        if (p > 0) __syncthreads();  // the previous phase's reads are done
        if constexpr (CROP) {
            const int wv = nx - x0 < W ? nx - x0 : W;              // the field's columns and
            const int yv = ny - y0 < ROWS ? ny - y0 : ROWS;        // rows in this phase
            if (ROTATE && (wv < W || yv < ROWS)) {
                for (int e = threadIdx.x; e < ROWS * W; e += NT) buf[e] = make_cpx((T)0, (T)0);
                __syncthreads();
            }
            if constexpr (ROTATE) {
                // Philox blocks cover 8 pixels in flat order: a row segment
                // meets up to W / 8 + 1 of them
                constexpr int OCT = (W + 6) / 8 + 1;
                const uint64_t r = r0 + b;
                for (int o = threadIdx.x; o < yv * OCT; o += NT) {
                    const int yl = o / OCT;
                    const int f0 = (y0 + yl) * nx + x0;            // flat index of the segment
                    const int oct = (f0 >> 3) + (o - yl * OCT);
                    if (8 * oct >= f0 + wv) continue;
                    T gp[8], gq[8];  // on their way while the block is drawn
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int f = min(max(8 * oct + i, f0), f0 + wv - 1);
                        gp[i] = a1[f];
                        gq[i] = a2[f];
                    }
                    uint32_t u[8];
                    philox_block_u32(seed, r, (uint64_t)oct, u);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int f = 8 * oct + i;
                        if (f < f0 || f >= f0 + wv) continue;
                        rotate_by_u32(u[i], gp[i], gq[i]);
                        buf[yl * W + (f - f0)] = make_cpx(gp[i], gq[i]);
                    }
                }
            } else {
                constexpr int ITER = ROWS * W / NT, U = ITER < 8 ? ITER : 8;  // U loads on their way at a time
                static_assert(ROWS * W % NT == 0 && ITER % U == 0, "a phase's values spread evenly over the threads");
                for (int i0 = 0; i0 < ITER; i0 += U) {
                    cpx<T> v[U];
#pragma unroll
                    for (int i = 0; i < U; ++i) {
                        const int e = threadIdx.x + (i0 + i) * NT, yl = e / W, cc = e % W;
                        const bool in = yl < yv && cc < wv;
                        const int gi = in ? (y0 + yl) * nx + x0 + cc : y0 * nx + x0;
                        v[i] = make_cpx(a1[gi], a2[gi]);
                        if (!in) v[i] = make_cpx((T)0, (T)0);
                    }
#pragma unroll
                    for (int i = 0; i < U; ++i) buf[threadIdx.x + (i0 + i) * NT] = v[i];
                }
            }
        } else if constexpr (ROTATE) {
            // one Philox block covers 8 consecutive pixels of a row
            static_assert(W % 8 == 0, "a segment is whole blocks");
            constexpr int OCT_PER_ROW = W / 8;
            const uint64_t r = r0 + b;
            for (int o = threadIdx.x; o < ROWS * OCT_PER_ROW; o += NT) {
                const int yl = o / OCT_PER_ROW, y = y0 + yl;
                const int cx = (o % OCT_PER_ROW) * 8;
                const int xa = x0 + cx;
                const uint64_t pix = (uint64_t)y * N + xa;
                uint32_t u[8];
                philox_block_u32(seed, r, pix >> 3, u);
                T gp[8], gq[8];
                load16<T, 8>(a1 + (long long)y * N + xa, gp);
                load16<T, 8>(a2 + (long long)y * N + xa, gq);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    rotate_by_u32(u[i], gp[i], gq[i]);
                    buf[yl * W + cx + i] = make_cpx(gp[i], gq[i]);
                }
            }
        } else {
            // G consecutive columns of a row per load
            for (int e = threadIdx.x; e < ROWS * (W / G); e += NT) {
                const int yl = e / (W / G), cc = (e % (W / G)) * G;
                const long long gi = (long long)(y0 + yl) * N + x0 + cc;
                T gp[G], gq[G];
                load16<T, G>(a1 + gi, gp);
                load16<T, G>(a2 + gi, gq);
#pragma unroll
                for (int i = 0; i < G; ++i) buf[yl * W + cc + i] = make_cpx(gp[i], gq[i]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int n1 = 0; n1 < K; ++n1) a[p * K + n1] = buf[(N2 * n1 + t) * W + c];
    }
    dft_reg<T, N1, false>(a);
    twiddle_powers<T, LOGN, false, N1>(tw, t, [&](int k1, const cpx<T>& w) { a[k1] = cmul(a[k1], w); });
    cpx<T>* out = C + (long long)b * N * N + x0 + c;
    // exchange phase q: first-step outputs k1 = q K .. (q+1) K - 1, then the
    // second step over n2 for each (k1, column) of the phase
#pragma unroll
    for (int q = 0; q < PH; ++q) {
        __syncthreads();  // LDS free
#pragma unroll
        for (int kl = 0; kl < K; ++kl) buf[(kl * N2 + t) * W + c] = a[q * K + kl];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < (K + N2 - 1) / N2; ++r) {
            const int kl = t + N2 * r;
            if (K % N2 == 0 || kl < K) {
                cpx<T> v[N2];
#pragma unroll
                for (int n2 = 0; n2 < N2; ++n2) v[n2] = buf[(kl * N2 + n2) * W + c];
                dft_reg<T, N2, false>(v);
                const int k1 = q * K + kl;
#pragma unroll
                for (int k2 = 0; k2 < N2; ++k2) store_stream(&out[(long long)(k1 + N1 * k2) * N], v[k2]);
            }
        }
    }
}

// ---- P2: rows: forward FFT along x, multiply by conj(D)/n^2, inverse (four-step) -
// The forward transform of one row for the N2 lanes t of a line, with E its
// exchange region: on return b[r][k2] holds the row's transform at
// frequency k1 + N1 k2, k1 = t + N2 r.  CROP: the row is zero from x = nx on
// (and not read there).
template <typename T, int LOGN, bool CROP>
__device__ __forceinline__ void ks_row_spectrum(const cpx<T>* __restrict__ row, int t, cpx<T>* E,
                                                const cpx<T>* __restrict__ tw,
                                                cpx<T> (&b)[FS<LOGN>::RR][FS<LOGN>::N2], int nx) {
    using F = FS<LOGN>;
    constexpr int N1 = F::N1, N2 = F::N2, RR = F::RR;
    cpx<T> a[N1];
    // forward, step 1: DFT_N1 over n1 of x[N2 n1 + t]
#pragma unroll
    for (int n1 = 0; n1 < N1; ++n1)
        a[n1] = !CROP || N2 * n1 + t < nx ? row[N2 * n1 + t] : make_cpx((T)0, (T)0);
    dft_reg<T, N1, false>(a);
    E[t] = a[0];
    twiddle_powers<T, LOGN, false, N1>(tw, t, [&](int k1, const cpx<T>& w) {
        E[k1 * (N2 + 1) + t] = cmul(a[k1], w);
    });
    wave_lds_sync();
    // forward, step 2: DFT_N2 over n2 -> X[k1 + N1 k2], k1 = t + N2 r
#pragma unroll
    for (int r = 0; r < RR; ++r) {
#pragma unroll
        for (int n2 = 0; n2 < N2; ++n2) b[r][n2] = E[(t + N2 * r) * (N2 + 1) + n2];
        dft_reg<T, N2, false>(b[r]);
    }
}

// b (laid out as ks_row_spectrum leaves it, spectral row y) times
// conj(D)/(SCALE_DEN n^2), with D = [(m1^2 - m2^2) + 2 i nu m1 m2] / (m1^2 + m2^2).
    // Every integer here is exact in T (|m| <= n/2, so m1^2 + m2^2 < 2^24),
    // so the arithmetic runs in T without integer multiplies; 1 / max(den, 1)
    // gives D(0) = 0 because both numerators vanish there.  The imaginary
    // part is 0 on the Nyquist row and column.  The frequency index is
    // t + c with c = N2 r + N1 k2 a multiple of N2 and t < N2, so it lies
    // below n/2 exactly when c does: m1 is t plus a constant.
template <typename T, int LOGN, int SCALE_DEN>
__device__ __forceinline__ void ks_multiply(cpx<T> (&b)[FS<LOGN>::RR][FS<LOGN>::N2], int y, int t) {
    using F = FS<LOGN>;
    constexpr int N = F::N, N1 = F::N1, N2 = F::N2, RR = F::RR;
    const T scale = (T)1 / ((T)N * (T)N * (T)SCALE_DEN);
    const int m2i = signed_freq(y, N);
    const T m2 = (T)m2i, m2sq = m2 * m2;
    const T two_m2 = m2i == -N / 2 ? (T)0 : (T)2 * m2;
    const T tf = (T)t;
#pragma unroll
    for (int r = 0; r < RR; ++r) {
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) {
            const int c = N2 * r + N1 * k2;
            const T m1 = tf + (T)(c < N / 2 ? c : c - N);
            const T m1sq = m1 * m1;
            const T den = fmax(m1sq + m2sq, (T)1), q = recip(den);
            const T dr = scale * ratio(m1sq - m2sq, den, q);
            const T di = (c == N / 2 && t == 0) ? (T)0 : scale * ratio(m1 * two_m2, den, q);
            const cpx<T> v = b[r][k2];
            b[r][k2] = cmul(v, make_cpx(dr, -di));
        }
    }
}

// P2 packed.  kappa_E is the inverse transform of the Hermitian part
// H(k) = [K(k) + conj(K(-k))]/2 of the spectrum K (kappa_B that of
// [K(k) - conj(K(-k))]/2i).  Transformed back along x, H gives complex rows
// h(ky, x) with h(-ky, x) = conj(h(ky, x)): half of them carry everything,
// and since kappa_E is real, columns 2c and 2c+1 can share one inverse
// transform along y, of z(ky, c) = h(ky, 2c) + i h(ky, 2c+1) (real part:
// column 2c, imaginary part: column 2c+1).  So a map's packed spectrum is
// n x n/2 (the left half of its rows; kappa_B's, where wanted, takes the
// right half), and without kappa_B the row pass writes and the inverse
// column pass reads half of the full spectrum.  kappa_E does not depend on
// whether kappa_B is wanted.
//
// A unit takes spectral rows y and -y: two lines run the forward transform
// and the multiply and leave their spectral rows in LDS in natural frequency
// order (-k is the mirrored address).  H(y, .) is then transformed back by
// all 2 N2 lanes of the unit (the lanes of row y, then those of row -y):
// the low half holds the even-indexed and the high half the odd-indexed
// inputs of each length-N2 and length-N1 DFT of the four-step inverse, and
// one radix-2 step across the halves completes them.  Neighbouring lanes end
// with neighbouring columns: the even lane forms z(y, .), the odd one
// z(-y, .), over the first halves of the rows they read.  Rows 0 and n/2
// are their own mirrors; their h are real and share one transform as real
// and imaginary part.
template <typename T, int LOGN>
struct RowHalf {
    static constexpr int N2 = FS<LOGN>::N2, N = 1 << LOGN;
    static constexpr int U0 = 64 / (2 * N2);  // one wavefront: small maps spread over more CUs
    static constexpr int UNITS = U0 > N / 2 ? N / 2 : U0;  // row pairs per workgroup
    static constexpr int NT = UNITS * 2 * N2;
};

// Exchange across the halves of a group of 2 H lanes (H a power of two, the
// group aligned to 2 H): afterwards a low lane holds (its d, its partner's
// d) and a high lane (its partner's s, its s) in (d, s).
template <int H>
__device__ __forceinline__ void half_swap_u32(uint32_t& d, uint32_t& s, bool hi) {
    const uint32_t got = (uint32_t)__shfl_xor((int)(hi ? d : s), H);
    if (hi) d = got;
    else s = got;
}
template <int H, typename T>
__device__ __forceinline__ void half_swap(T& d, T& s, bool hi) {
    if constexpr (sizeof(T) == 4) {
        uint32_t a = __builtin_bit_cast(uint32_t, d), b = __builtin_bit_cast(uint32_t, s);
        half_swap_u32<H>(a, b, hi);
        d = __builtin_bit_cast(T, a);
        s = __builtin_bit_cast(T, b);
    } else {
        const uint64_t a = __builtin_bit_cast(uint64_t, d), b = __builtin_bit_cast(uint64_t, s);
        uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b, bh = (uint32_t)(b >> 32);
        half_swap_u32<H>(al, bl, hi);
        half_swap_u32<H>(ah, bh, hi);
        d = __builtin_bit_cast(T, ((uint64_t)ah << 32) | al);
        s = __builtin_bit_cast(T, ((uint64_t)bh << 32) | bl);
    }
}

// Radix-2 step of an inverse length-2M DFT across a lane pair, from the
// half-length DFTs E (low lane) and O (high lane) after half_swap: the lane
// of half h forms X[I + h M/2] = E + w O and X[I + h M/2 + M] = E - w O with
// w = exp(2 pi i (I + h M/2) / 2M), which is i times the low lane's twiddle.
template <typename T, int L, int I>
__device__ __forceinline__ void pair_bfly(cpx<T>& e, cpx<T>& o, bool hi) {
    constexpr CS w = cos_sin_2pi(I, L);
    const T wr = hi ? (T)-w.s : (T)w.c;
    const T wi = hi ? (T)w.c : (T)w.s;
    const T xr = fma(wr, o.x, fma(-wi, o.y, e.x));
    const T xi = fma(wr, o.y, fma(wi, o.x, e.y));
    o = make_cpx<T>(fma((T)2, e.x, -xr), fma((T)2, e.y, -xi));
    e = make_cpx<T>(xr, xi);
}
template <typename T, int M, int H, int... I>
__device__ __forceinline__ void pair_bflies(cpx<T> (&v)[M], bool hi, std::integer_sequence<int, I...>) {
    constexpr int Q = M / 2;
    ((half_swap<H>(v[I].x, v[Q + I].x, hi), half_swap<H>(v[I].y, v[Q + I].y, hi)), ...);
    (pair_bfly<T, 2 * M, I>(v[I], v[Q + I], hi), ...);
}
// Inverse DFT of length 2M over a lane pair (l, l + H): the low lane holds
// inputs 0, 2, .., the high lane 1, 3, .. (M each, in order).  On return the
// lane of half h holds outputs i + h M/2 in v[i] and i + h M/2 + M in
// v[M/2 + i], i < M/2.
template <typename T, int M, int H>
__device__ __forceinline__ void pair_dft_inv(cpx<T> (&v)[M], bool hi) {
    static_assert(M >= 2, "at least two values per lane");
    dft_reg<T, M, true>(v);
    pair_bflies<T, M, H>(v, hi, std::make_integer_sequence<int, M / 2>{});
}
// The output index held in v[j] by the lane of half h after pair_dft_inv.
template <int M>
__device__ __forceinline__ constexpr int pair_out(int j, int h) {
    return j < M / 2 ? j + h * (M / 2) : j - M / 2 + h * (M / 2) + M;
}

// ks_multiply for a lane pair (t, t + N2) holding spectral rows y0 (low
// half) and -y0 (high half), 0 < y0 < n/2, at the same frequencies.  conj(D)
// of row -y0 is the conjugate of that of row y0, so each half evaluates it,
// with y0's sign, at half of the frequencies (the low half at k2 < N2/2,
// the high half at k2 + N2/2) and the halves exchange the values; passing
// (V, -V) for the imaginary part hands each half its own row's sign.  The
// factors are those ks_multiply computes, value for value (the sign changes
// are exact).
template <typename T, int LOGN, int SCALE_DEN>
__device__ __forceinline__ void ks_multiply_pair(cpx<T> (&b)[FS<LOGN>::RR][FS<LOGN>::N2], int y0, int t,
                                                 bool hi) {
    using F = FS<LOGN>;
    constexpr int N = F::N, N1 = F::N1, N2 = F::N2, RR = F::RR, HALF = N2 / 2;
    const T scale = (T)1 / ((T)N * (T)N * (T)SCALE_DEN);
    const T m2 = (T)y0, m2sq = m2 * m2, two_m2 = (T)2 * m2;
    // the high half's frequency index is t + c + n/2 with c = N2 r + N1 k2 < n/2,
    // so its m1 is t - n/2 + c
    const T tb = (T)t - (hi ? (T)(N / 2) : (T)0);
    const auto apply = [](cpx<T>& v, T dr, T di) {
        v = cmul(v, make_cpx(dr, -di));
    };
#pragma unroll
    for (int r = 0; r < RR; ++r) {
#pragma unroll
        for (int k2 = 0; k2 < HALF; ++k2) {
            const int c = N2 * r + N1 * k2;
            const T m1 = tb + (T)c;
            const T m1sq = m1 * m1;
            const T den = fmax(m1sq + m2sq, (T)1), q = recip(den);
            T dr_lo = scale * ratio(m1sq - m2sq, den, q), dr_hi = dr_lo;
            // the Nyquist column n/2 is the high half's c = 0 at t = 0
            const T v = (c == 0 && hi && t == 0) ? (T)0 : scale * ratio(m1 * two_m2, den, q);
            T di_lo = v, di_hi = -v;
            half_swap<N2>(dr_lo, dr_hi, hi);
            half_swap<N2>(di_lo, di_hi, hi);
            apply(b[r][k2], dr_lo, di_lo);
            apply(b[r][k2 + HALF], dr_hi, di_hi);
        }
    }
}

template <typename T, int LOGN, bool WANT_B, bool CROP>
__global__ void __launch_bounds__((RowHalf<T, LOGN>::NT))
k_ks_rows_half(cpx<T>* __restrict__ C, const cpx<T>* __restrict__ tw, int nx) {
    using F = FS<LOGN>;
    using RP = RowHalf<T, LOGN>;
    constexpr int N = F::N, N1 = F::N1, N2 = F::N2, RR = F::RR, EX = row4_elems<LOGN>();
    constexpr int M2 = N2 / 2, M1 = N1 / 2;  // values per lane in the two inverse steps
    // a unit (2 N2 lanes, aligned) lies in one wavefront, so wave-level
    // ordering covers its exchanges and its cross-lane steps
    static_assert(2 * N2 <= 64, "a unit must lie in one wavefront");
    static_assert(N2 >= 4, "at least two values per lane and half");
    // the exchange of the inverse takes the spectra's place, or, where
    // kappa_B is formed from them afterwards, a region of its own
    constexpr int REG = WANT_B ? 3 : 2;
    __shared__ cpx<T> ex[RP::UNITS * REG * EX];
    const int line = threadIdx.x / N2, t = threadIdx.x % N2;
    const int u = line >> 1, h = line & 1;  // h: row y (0) or -y (1)
    const bool hi = h != 0;
    const int q = blockIdx.x * RP::UNITS + u;
    const int r0 = q, r1 = q == 0 ? N / 2 : N - q;
    cpx<T>* map = C + (long long)blockIdx.y * N * N;
    {
        const int y = hi ? r1 : r0;
        cpx<T>* E = ex + (u * REG + h) * EX;
        cpx<T> b[RR][N2];
        ks_row_spectrum<T, LOGN, CROP>(map + (long long)y * N, t, E, tw, b, nx);
        // times conj(D), carrying the 1/2 of H; rows 0 and n/2 are not a
        // conjugate pair
        if (q != 0) ks_multiply_pair<T, LOGN, 2>(b, r0, t, hi);
        else ks_multiply<T, LOGN, 2>(b, y, t);
        wave_lds_sync();  // the forward exchange's reads are done
#pragma unroll
        for (int r = 0; r < RR; ++r)
#pragma unroll
            for (int k2 = 0; k2 < N2; ++k2) E[t + N2 * r + N1 * k2] = b[r][k2];
    }
    // inter-step twiddles exp(2 pi i k1 m / N) for this lane's k1 and m
    cpx<T> w[RR][M2];
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
        for (int j = 0; j < M2; ++j) w[r][j] = table_twiddle<T, LOGN, true>(tw, (t + N2 * r) * pair_out<M2>(j, h));
    wave_lds_sync();  // the unit's two spectral rows are in LDS
    // H at k1 = t + N2 r, k2 = 2 j + h (the spectra carry the 1/2)
    const cpx<T>* Ka = ex + (u * REG) * EX;
    const cpx<T>* Kb = ex + (u * REG + 1) * EX;
    cpx<T>* E = ex + (u * REG + (WANT_B ? 2 : 0)) * EX;  // the unit's exchange region
    const bool odd = (t & 1) != 0;
#pragma unroll
    for (int f = 0; f < (WANT_B ? 2 : 1); ++f) {  // kappa_E, kappa_B
        cpx<T> z[RR][M2];
#pragma unroll
        for (int r = 0; r < RR; ++r)
#pragma unroll
            for (int j = 0; j < M2; ++j) {
                const int kx = t + N2 * r + N1 * (2 * j + h), mk = (N - kx) & (N - 1);
                if (q != 0) {
                    z[r][j] = hermitian(Ka[kx], Kb[mk], f != 0);
                } else {  // H_0 + i H_{n/2}
                    const cpx<T> ha = hermitian(Ka[kx], Ka[mk], f != 0), hb = hermitian(Kb[kx], Kb[mk], f != 0);
                    z[r][j] = make_cpx(ha.x - hb.y, ha.y + hb.x);
                }
            }
        // step 1: DFT_N2 over k2 for each k1 held, then the twiddle
#pragma unroll
        for (int r = 0; r < RR; ++r) {
            pair_dft_inv<T, M2, N2>(z[r], hi);
#pragma unroll
            for (int j = 0; j < M2; ++j) z[r][j] = cmul(z[r][j], w[r][j]);
        }
        wave_lds_sync();  // the reads of the spectra are done
#pragma unroll
        for (int r = 0; r < RR; ++r)
#pragma unroll
            for (int j = 0; j < M2; ++j) E[pair_out<M2>(j, h) * (N1 + 1) + t + N2 * r] = z[r][j];
        wave_lds_sync();
        // step 2: DFT_N1 over k1 for m = t -> h(y, t + N2 n)
        cpx<T> v[M1];
#pragma unroll
        for (int j = 0; j < M1; ++j) v[j] = E[t * (N1 + 1) + 2 * j + h];
        pair_dft_inv<T, M1, N2>(v, hi);
        cpx<T>* out = map + (long long)(odd ? r1 : r0) * N + f * (N / 2) + (t >> 1);
#pragma unroll
        for (int j = 0; j < M1; ++j) {
            const cpx<T> z = pack_columns(v[j], odd, q == 0);
            const int xc = (N2 / 2) * pair_out<M1>(j, h);  // column pair, from t / 2
            if (!CROP || 2 * (xc + (t >> 1)) < nx) out[xc] = z;
        }
    }
}

// ---- P3: inverse FFT along y (four-step), two columns a transform -----------------
// Column c < n/2 of the packed spectra becomes columns 2c (real part) and
// 2c + 1 (imaginary part) of kappa_E, column n/2 + c those of kappa_B.  The
// grid has `strips` strips for each of them.  CROP: ny x nx outputs.
template <typename T, int LOGN, bool CROP, int WREQ>
__global__ void __launch_bounds__((StripI<T, LOGN, WREQ>::NT), (StripI<T, LOGN, WREQ>::MINW))
k_ks_cols_inv(const cpx<T>* __restrict__ C, T* __restrict__ kE, T* __restrict__ kB,
              long long out_stride, const long long* __restrict__ kE_off, const cpx<T>* __restrict__ tw,
              int xcd, int strips, int ny, int nx) {
    using F = FS<LOGN>;
    using S = StripI<T, LOGN, WREQ>;
    constexpr int N = F::N, N1 = F::N1, N2 = F::N2, W = S::W, PH = S::PH, K = N1 / PH;
    __shared__ cpx<T> buf[S::LDS];
    int sx, b;
    strip_of(xcd, sx, b);
    const bool second = sx >= strips;  // kappa_B
    const int c = threadIdx.x % W, t = threadIdx.x / W;
    const int col = (second ? sx - strips : sx) * W + c;
    const cpx<T>* in = C + (long long)b * N * N + (second ? N / 2 : 0) + col;
    cpx<T> a[N1];
#pragma unroll
    for (int n1 = 0; n1 < N1; ++n1) a[n1] = in[(long long)(N2 * n1 + t) * N];
    dft_reg<T, N1, true>(a);
    twiddle_powers<T, LOGN, true, N1>(tw, t, [&](int k1, const cpx<T>& w) { a[k1] = cmul(a[k1], w); });
    const int os = CROP ? nx : N;  // output row
    T* o = (second ? kB + (long long)b * out_stride
                   : kE + (kE_off ? kE_off[b] : (long long)b * out_stride)) + 2 * col;
    // exchange in PH phases of K first-step outputs each, as the forward pass
#pragma unroll
    for (int q = 0; q < PH; ++q) {
        if (q > 0) __syncthreads();  // the previous phase's reads are done
#pragma unroll
        for (int kl = 0; kl < K; ++kl) buf[(kl * N2 + t) * W + c] = a[q * K + kl];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < (K + N2 - 1) / N2; ++r) {
            const int kl = t + N2 * r;
            if (K % N2 == 0 || kl < K) {
                cpx<T> v[N2];
#pragma unroll
                for (int n2 = 0; n2 < N2; ++n2) v[n2] = buf[(kl * N2 + n2) * W + c];
                dft_reg<T, N2, true>(v);
                const int k1 = q * K + kl;
#pragma unroll
                for (int k2 = 0; k2 < N2; ++k2) {
                    const int y = k1 + N1 * k2;
                    if constexpr (CROP) {
                        if (y >= ny) continue;
                        if (2 * col < nx) o[(long long)y * os] = v[k2].x;
                        if (2 * col + 1 < nx) o[(long long)y * os + 1] = v[k2].y;
                    } else {
                        *reinterpret_cast<cpx<T>*>(o + (long long)y * os) = v[k2];
                    }
                }
            }
        }
    }
}

// ---- host launchers ------------------------------------------------------------
// Strips as wide as leave a launch ~512 workgroups (cols columns of each of
// `maps` maps), from wmax down to 4 columns (n = 256 and up: narrower maps
// are small at any width).  Rotating strips draw random blocks of 8 pixels,
// a strip of four each block twice and, in a cropped field, up to two for
// four pixels: they stay at 8 columns and leave 128 workgroups.  Measured
// (us of all noise passes, float, 4 / 8 / 16 columns): 512^2 x 8 realisations 85 / 73 /
// 74; 1024^2 x 2: 101 / 92 / 94, x 4: 142 / 121 / 120; 1000^2 field x 2: 139 /
// 129 / 133, x 4: 210 / 188 / 181.
static int strip_width(int n, int cols, long long maps, int wmax, bool rotate) {
    const int least = rotate ? 8 : 4;
    int w = wmax;
    while (n >= 256 && w > least && (cols + w - 1) / w * maps < (rotate ? 128 : 512)) w /= 2;
    return w;
}

// Which forward passes of a size run in four steps at all (ks_fwd): rotating
// ones but for 4096 points, others but for 2048.
template <int LOGN>
constexpr bool fwd4_rotates() { return LOGN < 12; }
template <int LOGN>
constexpr bool fwd4_plain() { return LOGN != 11; }

template <typename T, int LOGN, bool CROP, int WREQ>
static hipError_t cols_fwd_w(const KsArgs<T>& a) {
    constexpr int N = 1 << LOGN;
    using S = StripF<T, LOGN, WREQ>;
    const int nx = CROP ? a.nx : N, ny = CROP ? a.ny : N;
    const dim3 g((nx + S::W - 1) / S::W, a.batch);
    // XCD grouping where strips read row segments narrower than a 128-byte
    // line, except for a shared input (noise realisations), whose lines each
    // XCD's strips keep in its L2 as they are dealt out (grouped by strip it
    // measured 4 to 6% slower at 1024^2 and 2048^2)
    const bool shared_in = a.g_stride == 0 && !a.g1_off && a.batch > 1;
    const int xcd = (!shared_in && S::W * (int)sizeof(T) < 128) ? 1 : 0;
    if constexpr (fwd4_rotates<LOGN>() && WREQ >= 8) {
        if (a.rotate) {
            AMAP_LAUNCH("ks_cols_fwd_rotate", a.stream,
                        k_ks_cols_fwd<T, LOGN, true, CROP, WREQ><<<g, S::NT, 0, a.stream>>>(
                            a.g1, a.g2, a.g_stride, a.g1_off, a.g2_off, a.C, a.seed, a.r0, a.tw, xcd, ny, nx));
            return hipGetLastError();
        }
    }
    if constexpr (fwd4_plain<LOGN>()) {
        if (!a.rotate) {
            AMAP_LAUNCH("ks_cols_fwd", a.stream,
                        k_ks_cols_fwd<T, LOGN, false, CROP, WREQ><<<g, S::NT, 0, a.stream>>>(
                            a.g1, a.g2, a.g_stride, a.g1_off, a.g2_off, a.C, a.seed, a.r0, a.tw, xcd, ny, nx));
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;
}

template <typename T, int LOGN, bool CROP, int WREQ>
static hipError_t cols_inv_w(const KsArgs<T>& a) {
    constexpr int N = 1 << LOGN, W = WREQ < N / 2 ? WREQ : N / 2;
    using S = StripI<T, LOGN, W>;
    const int nx = CROP ? a.nx : N, ny = CROP ? a.ny : N;
    const int strips = ((nx + 1) / 2 + S::W - 1) / S::W;
    const int xcd = 2 * S::W * (int)sizeof(T) < 128 ? 1 : 0;
    AMAP_LAUNCH(a.rotate ? "ks_cols_inv_noise" : "ks_cols_inv", a.stream,
                k_ks_cols_inv<T, LOGN, CROP, W><<<dim3(strips * (a.kB ? 2 : 1), a.batch), S::NT, 0, a.stream>>>(
                    a.C, a.kE, a.kB, a.out_stride, a.kE_off, a.tw, xcd, strips, ny, nx));
    return hipGetLastError();
}

// Which passes run the three-step kernels: by size, type, cropping and
// rotation, never by the number of maps, since the two kinds of transform
// round differently and a map's values may not depend on which maps share
// its launch.  Their 16 values per thread leave room for four wavefronts per
// SIMD where the four-step kernels hold 32 or 64 values and run one or two;
// the four-step kernels need one exchange less and give the forward pass
// 16-column strips (128-byte row segments) up to 2048 points.  Measured (us,
// four-step / three-step, float):
//   row pass:      512^2: 11.6 / 7.1; 1024^2 x 128: 374 / 323; 2048^2 x 32:
//                  614 / 392; 128^2 x 200: 16.1 / 16.4; 256^2 x 200: 35 / 44,
//                  but all passes of one map, whose row pass takes as long as
//                  one unit: 128^2 12.5 / 11.4, 256^2 double 14.6 / 13.4, with
//                  kappa_B, whose inverse runs beside kappa_E's, 16.3 / 13.7
//   inverse pass:  1024^2 x 128: 222 / 248; 2048^2 x 32: 303 / 257;
//                  4096^2 x 8: 672 / 360
//   forward pass:  rotating, 1024^2 x 128: 315 / 400; 2048^2 x 32: 430 / 488;
//                  4096^2 x 8: 998 / 816
//                  2048^2, one map: 41 / 21, two: 46 / 38, four: 68 / 80, eight:
//                  154 / 158, twenty-five: 397 / 448; one of 4096^2: 112 / 129
//                  rotating, 1000 x 1000 in 2048^2 x 15: 154 / 131
// Double precision from 1024 points (whose per-thread DFTs would not fit the
// registers) has three-step kernels only.
template <typename T, int LOGN, bool CROP>
constexpr bool fwd3_always() { return sizeof(T) == 8 ? LOGN >= 10 : CROP && LOGN >= 11; }
template <typename T, int LOGN>
constexpr bool rows3() { return LOGN >= 7; }
template <typename T, int LOGN>
constexpr bool inv3() { return LOGN >= (sizeof(T) == 8 ? 10 : 11); }

template <typename T, int LOGN, bool CROP>
static hipError_t ks_fwd(const KsArgs<T>& a) {
    if constexpr (fwd3_always<T, LOGN, CROP>()) {
        return launch_ks3_fwd<T, LOGN, CROP>(a);
    } else {
        if constexpr (!fwd4_rotates<LOGN>()) {
            if (a.rotate) return launch_ks3_fwd<T, LOGN, CROP>(a);
        }
        if constexpr (!fwd4_plain<LOGN>()) {
            if (!a.rotate) return launch_ks3_fwd<T, LOGN, CROP>(a);
        }
        constexpr int N = 1 << LOGN, WF = StripF<T, LOGN>::W;
        const int w = strip_width(N, CROP ? a.nx : N, a.batch, WF, a.rotate);
        if constexpr (WF >= 16) {
            if (w == 16) return cols_fwd_w<T, LOGN, CROP, 16>(a);
        }
        if constexpr (WF >= 8) {
            if (w == 8) return cols_fwd_w<T, LOGN, CROP, 8>(a);
        }
        return cols_fwd_w<T, LOGN, CROP, 4>(a);
    }
}

template <typename T, int LOGN, bool CROP>
static hipError_t ks_rows(const KsArgs<T>& a) {
    if constexpr (rows3<T, LOGN>()) {
        return launch_ks3_rows<T, LOGN, CROP>(a);
    } else {
        constexpr int N = 1 << LOGN;
        using RP = RowHalf<T, LOGN>;
        const int nx = CROP ? a.nx : N;
        const dim3 g((N / 2) / RP::UNITS, a.batch);
        if (a.kB)
            AMAP_LAUNCH(a.rotate ? "ks_rows_noise" : "ks_rows", a.stream,
                        k_ks_rows_half<T, LOGN, true, CROP><<<g, RP::NT, 0, a.stream>>>(a.C, a.tw, nx));
        else
            AMAP_LAUNCH(a.rotate ? "ks_rows_noise" : "ks_rows", a.stream,
                        k_ks_rows_half<T, LOGN, false, CROP><<<g, RP::NT, 0, a.stream>>>(a.C, a.tw, nx));
        return hipGetLastError();
    }
}

template <typename T, int LOGN, bool CROP>
static hipError_t ks_inv(const KsArgs<T>& a) {
    if constexpr (inv3<T, LOGN>()) {
        return launch_ks3_inv<T, LOGN, CROP>(a);
    } else {
        constexpr int N = 1 << LOGN, WI = StripI<T, LOGN>::W;
        const int w = strip_width(N, CROP ? (a.nx + 1) / 2 : N / 2, a.batch, WI, false);
        if constexpr (WI >= 16) {
            if (w == 16) return cols_inv_w<T, LOGN, CROP, 16>(a);
        }
        if constexpr (WI >= 8) {
            if (w == 8) return cols_inv_w<T, LOGN, CROP, 8>(a);
        }
        return cols_inv_w<T, LOGN, CROP, 4>(a);
    }
}

template <typename T, int LOGN, bool CROP>
static hipError_t ks_launch_n(const KsArgs<T>& a) {
    hipError_t e = ks_fwd<T, LOGN, CROP>(a);
    if (e == hipSuccess) e = ks_rows<T, LOGN, CROP>(a);
    return e == hipSuccess ? ks_inv<T, LOGN, CROP>(a) : e;
}

template <typename T, bool CROP>
static hipError_t ks_launch_size(const KsArgs<T>& a) {
    switch (a.logn) {
        case 4: return ks_launch_n<T, 4, CROP>(a);
        case 5: return ks_launch_n<T, 5, CROP>(a);
        case 6: return ks_launch_n<T, 6, CROP>(a);
        case 7: return ks_launch_n<T, 7, CROP>(a);
        case 8: return ks_launch_n<T, 8, CROP>(a);
        case 9: return ks_launch_n<T, 9, CROP>(a);
        case 10: return ks_launch_n<T, 10, CROP>(a);
        case 11: return ks_launch_n<T, 11, CROP>(a);
        case 12: return ks_launch_n<T, 12, CROP>(a);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_ks(const KsArgs<T>& a) {
    const int N = 1 << a.logn;
    if (a.logn < 4 || a.logn > kMaxLogN || a.batch < 1) return hipErrorInvalidValue;
    const bool crop = a.ny > 0;
    if (crop && (a.nx < 1 || a.ny > N || a.nx > N)) return hipErrorInvalidValue;
    return crop && (a.ny < N || a.nx < N) ? ks_launch_size<T, true>(a) : ks_launch_size<T, false>(a);
}

template hipError_t launch_ks<float>(const KsArgs<float>&);
template hipError_t launch_ks<double>(const KsArgs<double>&);

}  // namespace amap

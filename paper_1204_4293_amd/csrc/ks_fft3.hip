// Kaiser-Squires passes in three steps (row pass from 128 points, column
// passes from 2048 or, in double precision, 1024), with the pass structure,
// the layouts and the CROP fields of ks_fft.hip.
//
// A length-N transform is a three-step FFT, N = X * X * R3 with X = 16 (rows
// up to 512 points: 8): L = N / X threads hold X values each.  With
// n = L n1 + R3 n2 + n3 and k = k1 + X k2 + X^2 k3,
//   step 1: DFT_X over n1, times W_{X^2}^(n2 k1);        thread (n2, n3)
//   step 2: DFT_X over n2, times W_N^(n3 (k1 + X k2));   thread (k1, n3)
//   step 3: DFT_R3 over n3;                              thread u = k mod L
// Thread t starts with the elements t + L m and ends with the frequencies
// t + L m (m < X), so an inverse transform starts from a forward one's
// output as it lies.  Between the steps the values go through LDS, real
// parts first, then imaginary parts: an exchange takes half the LDS of the
// data, so that twice as many columns or workgroups fit a CU.  A two-step
// transform holds 64 (32) values per thread: at 4096 points one workgroup of
// two wavefronts per SIMD fills the register file and runs its loads,
// butterflies and stores one after another.
#include "ks_device.h"

namespace amap {

template <int LOGN, int RX = 16>
struct F3 {
    static constexpr int N = 1 << LOGN, L = N / RX, R3 = N / (RX * RX), S3 = RX / R3;
    static_assert((RX == 16 || RX == 8) && R3 >= 2 && R3 <= RX, "three steps of RX, RX and 2 to RX");
    // exchange buffer of W interleaved lines, elements of T; the row padding
    // spreads the lanes of one access over the banks
    static constexpr int P1(int W) { return W == 1 ? R3 : 0; }
    static constexpr int P2(int W) { return W == 1 ? 64 / R3 : 1; }
    static constexpr int elems(int W) {
        return (RX * (L + P1(W)) > R3 * (RX * RX + P2(W)) ? RX * (L + P1(W)) : R3 * (RX * RX + P2(W))) * W;
    }
};

// Waits for a workgroup of one wavefront, or for all of its wavefronts.
template <bool WAVE>
__device__ __forceinline__ void f3_sync() {
    if constexpr (WAVE) wave_lds_sync();
    else __syncthreads();
}

// Steps 1 and 2 of thread t's line: DFT and twiddle.  A twiddle is a table
// value or the product of two: 15 (16) reads, most of them different in every
// lane, took the row pass of 4096^2 floats 779 us against 440, and cost the
// float columns 1 to 4%.  Four reads a step differ from lane to lane; with
// one (step 2: products of three) the row passes took as long or longer
// (1024^2 x 128: 337 us, now 320; 2048^2 x 32: 409, now 393) and the errors of
// kappa and sigma were 4 to 10% larger.
template <typename T, int LOGN, bool INV, int RX>
__device__ __forceinline__ void f3_step1(cpx<T> (&a)[RX], int t, const cpx<T>* __restrict__ tw) {
    constexpr int LOG2X = RX == 16 ? 8 : 6;  // of the RX^2 points of the first two steps
    const int n2 = t / F3<LOGN, RX>::R3;
    dft_reg<T, RX, INV>(a);
    cpx<T> v[4];  // powers 1, 2, 3
#pragma unroll
    for (int j = 1; j < 4; ++j) v[j] = table_twiddle<T, LOG2X, INV>(tw, n2 * j);
#pragma unroll
    for (int i = 0; i < RX / 4; ++i) {
        cpx<T> base{};
        if (i) {
            base = table_twiddle<T, LOG2X, INV>(tw, n2 * 4 * i);
            a[4 * i] = cmul(a[4 * i], base);
        }
#pragma unroll
        for (int j = 1; j < 4; ++j) a[4 * i + j] = cmul(a[4 * i + j], i ? cmul(base, v[j]) : v[j]);
    }
}
template <typename T, int LOGN, bool INV, int RX>
__device__ __forceinline__ void f3_step2(cpx<T> (&a)[RX], int t, const cpx<T>* __restrict__ tw) {
    constexpr int R3 = F3<LOGN, RX>::R3;
    const int k1 = t / R3, n3 = t % R3;
    dft_reg<T, RX, INV>(a);
    // W_N^(n3 (k1 + 4 RX i)) W_N^(RX n3 j), k2 = 4 i + j
    cpx<T> v[4];
#pragma unroll
    for (int j = 1; j < 4; ++j) v[j] = table_twiddle<T, LOGN, INV>(tw, RX * n3 * j);
#pragma unroll
    for (int i = 0; i < RX / 4; ++i) {
        const cpx<T> base = table_twiddle<T, LOGN, INV>(tw, n3 * (k1 + 4 * RX * i));
        a[4 * i] = cmul(a[4 * i], base);
#pragma unroll
        for (int j = 1; j < 4; ++j) a[4 * i + j] = cmul(a[4 * i + j], cmul(base, v[j]));
    }
}
// Step 3: the S3 DFTs of length R3; a[s R3 + n3] in, a[m] at frequency
// t + L m out.
template <typename T, int LOGN, bool INV, int RX>
__device__ __forceinline__ void f3_step3(cpx<T> (&a)[RX]) {
    constexpr int R3 = F3<LOGN, RX>::R3, S3 = F3<LOGN, RX>::S3;
    cpx<T> o[RX];
#pragma unroll
    for (int s = 0; s < S3; ++s) {
        cpx<T> v[R3];
#pragma unroll
        for (int i = 0; i < R3; ++i) v[i] = a[s * R3 + i];
        dft_reg<T, R3, INV>(v);
#pragma unroll
        for (int i = 0; i < R3; ++i) o[s + S3 * i] = v[i];
    }
#pragma unroll
    for (int m = 0; m < RX; ++m) a[m] = o[m];
}

// The three steps in double precision with RX = 16, as radix-4 passes whose
// inputs are multiplied by table twiddles: pass p joins four transforms of
// 4^p points.  Two passes make a step (the third of 8 points ends in radix
// 2), so that no step needs twiddles after its DFT.  27 to 31 table values a
// thread, none of them a product, and fewer multiplications than a DFT_16 of
// radix-2 butterflies and its twiddles: kappa's rms error at 1024^2 (2048^2)
// is 4.2e-16 (4.4e-16), 5.6e-16 (6.2e-16) with those, and the rotating forward
// pass of 1024^2 x 16 (2048^2 x 8) takes 95 us (329), 114 (372) with those.
template <typename T, bool INV>
__device__ __forceinline__ void radix4(cpx<T>& a0, cpx<T>& a1, cpx<T>& a2, cpx<T>& a3) {
    const cpx<T> s0 = a0 + a2, d0 = a0 - a2, s1 = a1 + a3, d1 = rot90<T, INV>(a1 - a3);
    a0 = s0 + s1;
    a1 = d0 + d1;
    a2 = s0 - s1;
    a3 = d0 - d1;
}
// DFT_16 as two radix-4 passes over a[j]: in, j = 4 u + v; out, k = q + 4 r.
// w1(u) (u = 1..3) multiplies the inputs of the first pass, w2(v, q) (v =
// 1..3) those of the second.
template <typename T, bool INV, typename W1, typename W2>
__device__ __forceinline__ void radix4_pair(cpx<T> (&a)[16], W1&& w1, W2&& w2) {
#pragma unroll
    for (int u = 1; u < 4; ++u) w1(u, a[4 * u], a[4 * u + 1], a[4 * u + 2], a[4 * u + 3]);
#pragma unroll
    for (int v = 0; v < 4; ++v) radix4<T, INV>(a[v], a[4 + v], a[8 + v], a[12 + v]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int v = 1; v < 4; ++v) w2(v, q, a[4 * q + v]);
        radix4<T, INV>(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
    }
    // a[4 q + r] holds k = q + 4 r
    cpx<T> o[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) o[k] = a[4 * (k % 4) + k / 4];
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = o[k];
}
struct W16Table {  // exp(-2 pi i k / 16)
    double c[10], s[10];
    constexpr W16Table() : c(), s() {
        for (int k = 0; k < 10; ++k) {
            const CS w = cos_sin_2pi(k, 16);
            c[k] = w.c;
            s[k] = -w.s;
        }
    }
};
template <typename T, bool INV>
__device__ __forceinline__ void radix4_step1(cpx<T> (&a)[16]) {
    constexpr W16Table w;
    radix4_pair<T, INV>(
        a, [](int, cpx<T>&, cpx<T>&, cpx<T>&, cpx<T>&) {},
        [&](int v, int q, cpx<T>& x) {
            if (v * q == 4) x = rot90<T, INV>(x);
            else if (q != 0) x = cmul(x, make_cpx((T)w.c[v * q], (T)(INV ? -w.s[v * q] : w.s[v * q])));
        });
}
template <typename T, int LOGN, bool INV>
__device__ __forceinline__ void radix4_step2(cpx<T> (&a)[16], int t, const cpx<T>* __restrict__ tw) {
    const int k1 = t / F3<LOGN>::R3;
    radix4_pair<T, INV>(
        a,
        [&](int u, cpx<T>& x0, cpx<T>& x1, cpx<T>& x2, cpx<T>& x3) {
            const cpx<T> w = table_twiddle<T, 6, INV>(tw, u * k1);
            x0 = cmul(x0, w); x1 = cmul(x1, w); x2 = cmul(x2, w); x3 = cmul(x3, w);
        },
        [&](int v, int q, cpx<T>& x) { x = cmul(x, table_twiddle<T, 8, INV>(tw, v * (k1 + 16 * q))); });
}
// The S3 DFTs of length R3 of frequencies K = t + L s.
template <typename T, int LOGN, bool INV>
__device__ __forceinline__ void radix4_step3(cpx<T> (&a)[16], int t, const cpx<T>* __restrict__ tw) {
    constexpr int R3 = F3<LOGN>::R3, S3 = F3<LOGN>::S3, L = F3<LOGN>::L;
    if constexpr (R3 == 16) {
        radix4_pair<T, INV>(
            a,
            [&](int u, cpx<T>& x0, cpx<T>& x1, cpx<T>& x2, cpx<T>& x3) {
                const cpx<T> w = table_twiddle<T, LOGN - 2, INV>(tw, u * t);
                x0 = cmul(x0, w); x1 = cmul(x1, w); x2 = cmul(x2, w); x3 = cmul(x3, w);
            },
            [&](int v, int q, cpx<T>& x) { x = cmul(x, table_twiddle<T, LOGN, INV>(tw, v * (t + 256 * q))); });
    } else {
        constexpr int V = R3 / 4;  // n3 = V u + v: a radix-4 pass over u, for V = 2 one of radix 2 over v
        static_assert(V == 1 || V == 2, "third steps of 4, 8 or 16 points");
        cpx<T> o[16];
#pragma unroll
        for (int s = 0; s < S3; ++s) {
            const int K = t + L * s;
            cpx<T> z[V][4];
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int u = 0; u < 4; ++u) z[v][u] = a[s * R3 + V * u + v];
#pragma unroll
            for (int u = 1; u < 4; ++u) {
                const cpx<T> w = table_twiddle<T, LOGN - V + 1, INV>(tw, u * K);
#pragma unroll
                for (int v = 0; v < V; ++v) z[v][u] = cmul(z[v][u], w);
            }
#pragma unroll
            for (int v = 0; v < V; ++v) radix4<T, INV>(z[v][0], z[v][1], z[v][2], z[v][3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (V == 1) {
                    o[s + S3 * q] = z[0][q];
                } else {
                    const cpx<T> y = cmul(z[1][q], table_twiddle<T, LOGN, INV>(tw, K + 256 * q));
                    o[s + S3 * q] = z[0][q] + y;
                    o[s + S3 * (q + 4)] = z[0][q] - y;
                }
            }
        }
#pragma unroll
        for (int m = 0; m < 16; ++m) a[m] = o[m];
    }
}

// Addresses of the two exchanges in a buffer of W interleaved lines (line
// c): element j of thread t, written after and read before a step.
template <int LOGN, int W, int RX>
struct Ex3 {
    using F = F3<LOGN, RX>;
    static __device__ __forceinline__ int w1(int t, int j) { return (j * (F::L + F::P1(W)) + t) * W; }
    static __device__ __forceinline__ int r1(int t, int j) {
        return ((t / F::R3) * (F::L + F::P1(W)) + F::R3 * j + t % F::R3) * W;
    }
    static __device__ __forceinline__ int w2(int t, int j) {
        return ((t % F::R3) * (RX * RX + F::P2(W)) + t / F::R3 + RX * j) * W;
    }
    static __device__ __forceinline__ int r2(int t, int j) {
        return ((j % F::R3) * (RX * RX + F::P2(W)) + t + F::L * (j / F::R3)) * W;
    }
};

// One exchange of the ITEMS items a thread holds (thread indices t0 + i DT of
// line buf of W): real parts, then imaginary parts.
template <typename T, int LOGN, int W, int ITEMS, bool SECOND, bool WAVE, int DT, int RX>
__device__ __forceinline__ void f3_exchange(cpx<T> (&a)[ITEMS][RX], T* buf, int t0) {
    using E = Ex3<LOGN, W, RX>;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        f3_sync<WAVE>();  // earlier reads of the buffer are done
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int j = 0; j < RX; ++j) {
                const int t = t0 + i * DT;
                buf[SECOND ? E::w2(t, j) : E::w1(t, j)] = part ? a[i][j].y : a[i][j].x;
            }
        f3_sync<WAVE>();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int j = 0; j < RX; ++j) {
                const int t = t0 + i * DT;
                const T v = buf[SECOND ? E::r2(t, j) : E::r1(t, j)];
                if (part) a[i][j].y = v;
                else a[i][j].x = v;
            }
    }
}

// The whole transform of the items a thread holds.
template <typename T, int LOGN, int W, int ITEMS, bool INV, bool WAVE, int DT, int RX = 16>
__device__ __forceinline__ void f3_transform(cpx<T> (&a)[ITEMS][RX], T* buf, int t0, const cpx<T>* __restrict__ tw) {
    constexpr bool R4 = sizeof(T) == 8 && RX == 16;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if constexpr (R4) radix4_step1<T, INV>(a[i]);
        else f3_step1<T, LOGN, INV, RX>(a[i], t0 + i * DT, tw);
    }
    f3_exchange<T, LOGN, W, ITEMS, false, WAVE, DT, RX>(a, buf, t0);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if constexpr (R4) radix4_step2<T, LOGN, INV>(a[i], t0 + i * DT, tw);
        else f3_step2<T, LOGN, INV, RX>(a[i], t0 + i * DT, tw);
    }
    f3_exchange<T, LOGN, W, ITEMS, true, WAVE, DT, RX>(a, buf, t0);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if constexpr (R4) radix4_step3<T, LOGN, INV>(a[i], t0 + i * DT, tw);
        else f3_step3<T, LOGN, INV, RX>(a[i]);
    }
}

// Column strips: W columns, ITEMS items of 16 values per thread.
template <typename T, int LOGN, int W, int ITEMS_>
struct Strip3 {
    static constexpr int L = F3<LOGN>::L;
    static constexpr int ITEMS = ITEMS_;
    static constexpr int NT = W * L / ITEMS, DT = L / ITEMS;
    static constexpr int ELEMS = F3<LOGN>::elems(W);
    // workgroups of at most 512 threads share a CU in pairs where their LDS allows
    static constexpr int MINW = NT >= 1024 ? 4 : (2 * ELEMS * (int)sizeof(T) <= 160 * 1024 ? 2 * NT / 256 : NT / 256);
};

// ---- P1 ---------------------------------------------------------------------------
template <typename T, int LOGN, int W, int IT, bool ROTATE, bool CROP>
__global__ void __launch_bounds__((Strip3<T, LOGN, W, IT>::NT), (Strip3<T, LOGN, W, IT>::MINW))
k3_cols_fwd(const T* __restrict__ g1, const T* __restrict__ g2, long long g_stride,
            const long long* __restrict__ g1_off, const long long* __restrict__ g2_off,
            cpx<T>* __restrict__ C, uint64_t seed, uint64_t r0, const cpx<T>* __restrict__ tw, int xcd,
            int ny, int nx) {
    using S = Strip3<T, LOGN, W, IT>;
    constexpr int N = 1 << LOGN, L = S::L, ITEMS = S::ITEMS, DT = S::DT;
    __shared__ T buf[S::ELEMS];
    int sx, b;
    strip_of(xcd, sx, b);
    const int x0 = sx * W;
    const int c = threadIdx.x % W, t0 = threadIdx.x / W;
    const T* a1 = g1 + (g1_off ? g1_off[b] : (long long)b * g_stride);
    const T* a2 = g2 + (g2_off ? g2_off[b] : (long long)b * g_stride);
    const int rs = CROP ? nx : N;  // input row
    const bool colin = !CROP || x0 + c < nx;
    cpx<T> a[ITEMS][16];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int y = t0 + i * DT + L * m;
            const bool in = colin && (!CROP || y < ny);
            const int f = y * rs + x0 + c;
            a[i][m] = in ? make_cpx(a1[f], a2[f]) : make_cpx((T)0, (T)0);
        }
    if constexpr (ROTATE) {
        // The W lanes of a row segment share its Philox blocks: each lane
        // draws those of every W-th row and hands the words round through LDS
        // (lanes of one wavefront).  A segment lies in one block of 8 pixels
        // (flat order), or, in a field of any width, in two.
        constexpr int BPR = CROP ? 2 : 1, RW = 8 * BPR;
        static_assert(W <= 8, "a segment meets at most two blocks");
        // words of a lane group, padded (where that fits) to spread the groups over the banks
        constexpr int PAD = (S::NT / W) * (W * RW + 8) * 4 <= S::ELEMS * (int)sizeof(T) ? 8 : 0;
        constexpr int GS = W * RW + PAD;
        static_assert((S::NT / W) * GS * 4 <= S::ELEMS * (int)sizeof(T), "words fit the exchange buffer");
        uint32_t* words = reinterpret_cast<uint32_t*>(buf) + (threadIdx.x / W) * GS;
        const uint64_t r = r0 + b;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int m0 = 0; m0 < 16; m0 += W) {
                wave_lds_sync();  // the previous words are read
                const int f = (t0 + i * DT + L * (m0 + c)) * rs + x0;
#pragma unroll
                for (int k = 0; k < BPR; ++k) {
                    uint32_t u[8];
                    philox_block_u32(seed, r, (uint64_t)((f >> 3) + k), u);
#pragma unroll
                    for (int q = 0; q < 8; ++q) words[c * RW + 8 * k + q] = u[q];
                }
                wave_lds_sync();
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    const int fj = (t0 + i * DT + L * (m0 + j)) * rs + x0;
                    cpx<T>& v = a[i][m0 + j];
                    rotate_by_u32(words[j * RW + (fj & 7) + c], v.x, v.y);
                }
            }
    }
    f3_transform<T, LOGN, W, ITEMS, false, false, DT>(a, buf + c, t0, tw);
    cpx<T>* out = C + (long long)b * N * N + x0 + c;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
#pragma unroll
        for (int m = 0; m < 16; ++m) store_stream(&out[(long long)(t0 + i * DT + L * m) * N], a[i][m]);
}

// ---- P2 ---------------------------------------------------------------------------
// A unit (spectral rows y and -y, or 0 and n/2) takes 2 L threads, one unit
// per workgroup or as many as fill a wavefront: half i of the threads
// transforms its row and multiplies it by conj(D);
// half 0 then forms kappa_E's Hermitian row y from the two (row -y mirrored)
// and transforms it back, while half 1's wavefronts only keep the barriers
// company, or, with WANT_B, do the same for kappa_B's row -y.  (Both rows in
// one thread's registers spilled 300 to 900 bytes a lane.)  Built for four
// wavefronts per SIMD in single precision, which costs a few spilled values
// and is worth them (4096^2 x 8: 420 us; 714 at three wavefronts, 454 at four,
// with other twiddles).
template <int LOGN, int RX>
struct Rows3 {
    static constexpr int L = F3<LOGN, RX>::L;
    static constexpr int UNITS = 2 * L < 64 ? 64 / (2 * L) : 1;
    static constexpr int NT = UNITS * 2 * L;
    // a row's exchange buffer, padded so that the rows of a wavefront fall on different banks
    static constexpr int ELEMS = F3<LOGN, RX>::elems(1) + (L < 64 ? L : 0);
};
template <typename T, int LOGN, int RX, bool WANT_B, bool CROP>
__global__ void __launch_bounds__((Rows3<LOGN, RX>::NT), (sizeof(T) == 4 ? 4 : 2))
k3_rows(cpx<T>* __restrict__ C, const cpx<T>* __restrict__ tw, int nx) {
    using S = Rows3<LOGN, RX>;
    constexpr int N = 1 << LOGN, L = S::L, ELEMS = S::ELEMS;
    constexpr bool WAVE = L <= 64;       // a row's threads lie in one wavefront
    constexpr bool UNIT = 2 * L <= 64;   // and so do a unit's
    __shared__ T buf[S::UNITS * 2 * ELEMS];
    int half = (int)threadIdx.x / L % 2;  // uniform in a wavefront unless a row takes part of one
    if constexpr (L >= 64) half = __builtin_amdgcn_readfirstlane(half);
    const int t = threadIdx.x % L, q = blockIdx.x * S::UNITS + (int)threadIdx.x / (2 * L);
    const int r0 = q, r1 = q == 0 ? N / 2 : N - q;
    T* mine = buf + ((int)threadIdx.x / (2 * L) * 2 + half) * ELEMS;
    const T* other = buf + ((int)threadIdx.x / (2 * L) * 2 + 1 - half) * ELEMS;
    cpx<T>* map = C + (long long)blockIdx.y * N * N;
    cpx<T> a[1][RX];
    {
        const cpx<T>* row = map + (long long)(half ? r1 : r0) * N;
#pragma unroll
        for (int m = 0; m < RX; ++m) a[0][m] = !CROP || t + L * m < nx ? row[t + L * m] : make_cpx((T)0, (T)0);
    }
    f3_transform<T, LOGN, 1, 1, false, WAVE, 0, RX>(a, mine, t, tw);
    // times conj(D)/(2 n^2), D = [(m1^2 - m2^2) + 2 i nu m1 m2] / (m1^2 + m2^2):
    // the imaginary part vanishes on the Nyquist row and column and changes
    // sign from row y to -y; 1 / max(den, 1) gives D(0) = 0
    {
        const T scale = (T)1 / ((T)N * (T)N * (T)2);
        const T m2 = q == 0 ? (half ? (T)(N / 2) : (T)0) : (half ? (T)-q : (T)q);
        const T m2sq = m2 * m2, two_m2 = q == 0 ? (T)0 : (T)2 * m2;
#pragma unroll
        for (int m = 0; m < RX; ++m) {
            const T m1 = (T)t + (T)(m < RX / 2 ? L * m : L * m - N);
            const T m1sq = m1 * m1;
            const T den = fmax(m1sq + m2sq, (T)1), r = recip(den);
            const T dr = scale * ratio(m1sq - m2sq, den, r);
            const T di = (m == RX / 2 && t == 0) ? (T)0 : scale * ratio(m1 * two_m2, den, r);
            const cpx<T> v = a[0][m];
            a[0][m] = cmul(v, make_cpx(dr, -di));
        }
    }
    // H of this half's mode from its own K(k) and the mirrored K(-k), which
    // lies in the other row or (q = 0) in the row itself
    const bool b_mode = half != 0;
    if (q != 0) {
#pragma unroll
        for (int part = 0; part < 2; ++part) {  // one component at a time, in place
            f3_sync<UNIT>();
#pragma unroll
            for (int m = 0; m < RX; ++m) mine[t + L * m] = part ? a[0][m].y : a[0][m].x;
            f3_sync<UNIT>();
            if (b_mode && !WANT_B) continue;
#pragma unroll
            for (int m = 0; m < RX; ++m) {
                const T v = other[(N - t - L * m) & (N - 1)];
                cpx<T>& k = a[0][m];
                if (!b_mode) {
                    if (part) k.y -= v;
                    else k.x += v;
                } else {
                    if (part) k = make_cpx(k.y + v, k.x);
                    else k.x = v - k.x;
                }
            }
        }
    } else {  // Z = H_0 + i H_{n/2}: each half hands the other's mode over
        cpx<T> v[RX];
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            f3_sync<UNIT>();
#pragma unroll
            for (int m = 0; m < RX; ++m) mine[t + L * m] = part ? a[0][m].y : a[0][m].x;
            f3_sync<UNIT>();
#pragma unroll
            for (int m = 0; m < RX; ++m) {
                const T w = mine[(N - t - L * m) & (N - 1)];
                if (part) v[m].y = w;
                else v[m].x = w;
            }
        }
#pragma unroll
        for (int m = 0; m < RX; ++m) {
            const cpx<T> keep = hermitian(a[0][m], v[m], b_mode);
            v[m] = hermitian(a[0][m], v[m], !b_mode);
            a[0][m] = keep;
        }
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            f3_sync<UNIT>();
#pragma unroll
            for (int m = 0; m < RX; ++m) mine[t + L * m] = part ? v[m].y : v[m].x;
            f3_sync<UNIT>();
#pragma unroll
            for (int m = 0; m < RX; ++m) {
                const T w = other[t + L * m];
                if (part) v[m].y = w;
                else v[m].x = w;
            }
        }
#pragma unroll
        for (int m = 0; m < RX; ++m) {
            const cpx<T> h0 = b_mode ? v[m] : a[0][m], h1 = b_mode ? a[0][m] : v[m];
            a[0][m] = make_cpx(h0.x - h1.y, h0.y + h1.x);
        }
    }
    if constexpr (WAVE) f3_sync<UNIT>();  // the other half's reads are done (else the transform's barriers tell)
    if (!WANT_B && half != 0) {
        // the barriers of the other half's transform
        if constexpr (!WAVE) {
#pragma unroll
            for (int k = 0; k < 8; ++k) __syncthreads();
        }
        return;
    }
    f3_transform<T, LOGN, 1, 1, true, WAVE, 0, RX>(a, mine, t, tw);
    // the even lane's row of each pair of columns is the row transformed (y
    // for kappa_E, -y for kappa_B), the odd lane's its mirror
    const bool odd = (t & 1) != 0;
    const bool up = q == 0 || half == 0;
    cpx<T>* out = map + (long long)(odd == up ? r1 : r0) * N + (half ? N / 2 : 0) + (t >> 1);
#pragma unroll
    for (int m = 0; m < RX; ++m) {
        const cpx<T> v = pack_columns(a[0][m], odd, q == 0);
        if (!CROP || 2 * ((t >> 1) + (L / 2) * m) < nx) out[(L / 2) * m] = v;
    }
}

// ---- P3 ---------------------------------------------------------------------------
template <typename T, int LOGN, int W, int IT, bool CROP>
__global__ void __launch_bounds__((Strip3<T, LOGN, W, IT>::NT), (Strip3<T, LOGN, W, IT>::MINW))
k3_cols_inv(const cpx<T>* __restrict__ C, T* __restrict__ kE, T* __restrict__ kB, long long out_stride,
            const long long* __restrict__ kE_off, const cpx<T>* __restrict__ tw, int xcd, int strips, int ny,
            int nx) {
    using S = Strip3<T, LOGN, W, IT>;
    constexpr int N = 1 << LOGN, L = S::L, ITEMS = S::ITEMS, DT = S::DT;
    __shared__ T buf[S::ELEMS];
    int sx, b;
    strip_of(xcd, sx, b);
    const bool second = sx >= strips;  // kappa_B
    const int c = threadIdx.x % W;
    int t0 = threadIdx.x / W;
    const int col = (second ? sx - strips : sx) * W + c;
    const cpx<T>* in = C + (long long)b * N * N + (second ? N / 2 : 0) + col;
    cpx<T> a[ITEMS][16];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
#pragma unroll
        for (int m = 0; m < 16; ++m) a[i][m] = in[(long long)(t0 + i * DT + L * m) * N];
    f3_transform<T, LOGN, W, ITEMS, true, false, DT>(a, buf + c, t0, tw);
    if constexpr (sizeof(T) == 8) {
        // every value complete, and no address formed, before the first store:
        // left free, the compiler moves the last butterflies into the stores'
        // conditions and their addresses ahead of the loads, and spills (4096^2:
        // 60 us, 104 so; a 2000 x 2000 field with kappa_B in 2048^2: 34, 62)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int m = 0; m < 16; ++m) asm volatile("" : "+v"(a[i][m].x), "+v"(a[i][m].y));
        asm volatile("" : "+v"(t0));
    }
    const int os = CROP ? nx : N;
    T* o = (second ? kB + (long long)b * out_stride
                   : kE + (kE_off ? kE_off[b] : (long long)b * out_stride)) + 2 * col;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int y = t0 + i * DT + L * m;
            if constexpr (CROP) {
                if (y < ny && 2 * col < nx) o[(long long)y * os] = a[i][m].x;
                if (y < ny && 2 * col + 1 < nx) o[(long long)y * os + 1] = a[i][m].y;
            } else {
                *reinterpret_cast<cpx<T>*>(o + (long long)y * os) = a[i][m];
            }
        }
}

// ---- host launchers ----------------------------------------------------------------
// Sizes whose rotating forward pass runs in four steps (ks_fft.hip).
template <typename T, int LOGN, bool CROP>
constexpr bool fwd3_plain() { return sizeof(T) == 4 && LOGN == 11 && !CROP; }

template <typename T, int LOGN, bool CROP, int W, int IT>
static hipError_t fwd3(const KsArgs<T>& a) {
    constexpr int N = 1 << LOGN;
    using S = Strip3<T, LOGN, W, IT>;
    const int nx = CROP ? a.nx : N, ny = CROP ? a.ny : N;
    const dim3 g((nx + W - 1) / W, a.batch);
    // realisations of one input: all of a strip's on one XCD (4096^2 float, 8
    // realisations: 816 us, 1129 strip by strip)
    const bool shared_in = a.g_stride == 0 && !a.g1_off && a.batch > 1;
    const int xcd = shared_in ? 2 : 1;
    if constexpr (!fwd3_plain<T, LOGN, CROP>()) {
        if (a.rotate) {
            AMAP_LAUNCH("ks_cols_fwd_rotate", a.stream,
                        k3_cols_fwd<T, LOGN, W, IT, true, CROP><<<g, S::NT, 0, a.stream>>>(
                            a.g1, a.g2, a.g_stride, a.g1_off, a.g2_off, a.C, a.seed, a.r0, a.tw, xcd, ny, nx));
            return hipGetLastError();
        }
    }
    if (a.rotate) return hipErrorInvalidValue;
    AMAP_LAUNCH("ks_cols_fwd", a.stream,
                k3_cols_fwd<T, LOGN, W, IT, false, CROP><<<g, S::NT, 0, a.stream>>>(
                    a.g1, a.g2, a.g_stride, a.g1_off, a.g2_off, a.C, a.seed, a.r0, a.tw, xcd, ny, nx));
    return hipGetLastError();
}

template <typename T, int LOGN, bool CROP, int W, int IT>
static hipError_t inv3(const KsArgs<T>& a) {
    constexpr int N = 1 << LOGN;
    using S = Strip3<T, LOGN, W, IT>;
    const int nx = CROP ? a.nx : N, ny = CROP ? a.ny : N;
    const int strips = ((nx + 1) / 2 + W - 1) / W;
    AMAP_LAUNCH(a.rotate ? "ks_cols_inv_noise" : "ks_cols_inv", a.stream,
                k3_cols_inv<T, LOGN, W, IT, CROP><<<dim3(strips * (a.kB ? 2 : 1), a.batch), S::NT, 0, a.stream>>>(
                    a.C, a.kE, a.kB, a.out_stride, a.kE_off, a.tw, 1, strips, ny, nx));
    return hipGetLastError();
}

// Strips of eight columns keep the spectrum's row segments at 64 bytes (128 in
// double precision); four-column strips only where eight would leave CUs
// idle, or 4096 doubles would not fit.  Measured (us, 8 / 4 columns): float
// 4096^2 x 8: 816 / 2267; double 1024^2 x 16: 95 / 145, one map 18.2 / 16.0;
// double 2048^2 x 8: 329 / 409, one map 32 / 40.  Two items per thread in
// single precision, one where the launch is small (2048^2, one map: 20.4
// against 22.1).  Maps of 2048^2 floats take sixteen columns, four items per
// thread, from one workgroup per CU on (us, 8 / 16 columns: one map 21 / 30,
// two 40 / 38, four 104 / 80, eight 194 / 158, twenty-five 504 / 448; not grouped
// by XCD, where two strips share a line of the input, 514).  None of this
// changes a map's values: strips and items only spread the same transforms.
template <typename T, int LOGN, bool CROP>
hipError_t launch_ks3_fwd(const KsArgs<T>& a) {
    const long long wgs = ((CROP ? a.nx : 1 << LOGN) + 7) / 8 * (long long)a.batch;
    if constexpr (fwd3_plain<T, LOGN, CROP>()) {
        return wgs < 512 ? fwd3<T, LOGN, CROP, 8, 1>(a) : fwd3<T, LOGN, CROP, 16, 4>(a);
    } else if constexpr (sizeof(T) == 4) {
        if constexpr (LOGN < 12) {
            if (wgs <= 512) return fwd3<T, LOGN, CROP, 8, 1>(a);
        }
        return fwd3<T, LOGN, CROP, 8, 2>(a);
    } else if constexpr (LOGN == 12) {
        return fwd3<T, LOGN, CROP, 4, 1>(a);
    } else {
        if (wgs < 256) return fwd3<T, LOGN, CROP, 4, 1>(a);
        return fwd3<T, LOGN, CROP, 8, 1>(a);
    }
}

// Eight values per thread up to 512 points: twice the lanes of sixteen, half
// the work of each (512^2, all KS passes, us, 16 / 8 values: float 19.0 / 16.8,
// double 23.0 / 20.6; 200 realisations' noise passes 721 / 707, 1409 / 1378).
// Rows of 128 points take two units per wavefront (200 maps: 16.4 us, 23.1 with
// one unit of 32 threads per workgroup).
template <typename T, int LOGN, bool CROP>
hipError_t launch_ks3_rows(const KsArgs<T>& a) {
    constexpr int N = 1 << LOGN, RX = LOGN <= 9 ? 8 : 16;
    using S = Rows3<LOGN, RX>;
    const int nx = CROP ? a.nx : N;
    const dim3 g(N / 2 / S::UNITS, a.batch);
    if (a.kB)
        AMAP_LAUNCH(a.rotate ? "ks_rows_noise" : "ks_rows", a.stream,
                    k3_rows<T, LOGN, RX, true, CROP><<<g, S::NT, 0, a.stream>>>(a.C, a.tw, nx));
    else
        AMAP_LAUNCH(a.rotate ? "ks_rows_noise" : "ks_rows", a.stream,
                    k3_rows<T, LOGN, RX, false, CROP><<<g, S::NT, 0, a.stream>>>(a.C, a.tw, nx));
    return hipGetLastError();
}

// The packed columns are pairs, so a strip of four writes eight columns of
// kappa.  Measured (us, 8 / 4 columns): float 4096^2 x 8: 400 / 360; float
// 2048^2 x 32 (two items): 257 / -; double, where one map counts for more than
// many: 1024^2 11.4 / 9.7, x 16: 56 / 66; 2048^2 22.9 / 18.7, x 8: 131 / 136.
template <typename T, int LOGN, bool CROP>
hipError_t launch_ks3_inv(const KsArgs<T>& a) {
    if constexpr (sizeof(T) == 4 && LOGN < 12) return inv3<T, LOGN, CROP, 8, 2>(a);
    else return inv3<T, LOGN, CROP, 4, 1>(a);
}

#define AMAP_KS3(T, LOGN, CROP)                                            \
    template hipError_t launch_ks3_fwd<T, LOGN, CROP>(const KsArgs<T>&);   \
    template hipError_t launch_ks3_rows<T, LOGN, CROP>(const KsArgs<T>&);  \
    template hipError_t launch_ks3_inv<T, LOGN, CROP>(const KsArgs<T>&);
AMAP_KS3(float, 11, false) AMAP_KS3(float, 11, true)
AMAP_KS3(float, 12, false) AMAP_KS3(float, 12, true)
AMAP_KS3(double, 10, false) AMAP_KS3(double, 10, true)
AMAP_KS3(double, 11, false) AMAP_KS3(double, 11, true)
AMAP_KS3(double, 12, false) AMAP_KS3(double, 12, true)
#undef AMAP_KS3
#define AMAP_KS3_ROWS(T, LOGN)                                             \
    template hipError_t launch_ks3_rows<T, LOGN, false>(const KsArgs<T>&); \
    template hipError_t launch_ks3_rows<T, LOGN, true>(const KsArgs<T>&);
AMAP_KS3_ROWS(float, 7) AMAP_KS3_ROWS(float, 8) AMAP_KS3_ROWS(float, 9) AMAP_KS3_ROWS(float, 10)
AMAP_KS3_ROWS(double, 7) AMAP_KS3_ROWS(double, 8) AMAP_KS3_ROWS(double, 9)
#undef AMAP_KS3_ROWS

}  // namespace amap

// Brute-force aperture mass from the tangential shear (eq:shearmap), the
// comparison method whose O(n^2 cut^2) cost the starlet removes (Sec. 5.1).
//
// M(x) = -sum_d [ Q(|d|) cos2phi_d g1(x+d) + Q(|d|) sin2phi_d g2(x+d) ]
// over the integer offsets 0 < |d|^2 <= cut^2.  The weight of g1 is even in
// dy and that of g2 odd, so the rows y + dy and y - dy share their weights:
//
//   M(x, y) = -sum_{dy >= 0} sum_dx [ wc(dx, dy) S_dy(x + dx, y)
//                                     + ws(dx, dy) D_dy(x + dx, y) ],
//   S_dy = g1(y + dy) + g1(y - dy),  D_dy = g2(y + dy) - g2(y - dy)
//
// (wc halved at dy = 0, where ws = 0).  A row of S and D costs two additions
// per column and is used by all 2 h + 1 taps of its row offset, so the sum
// takes half the multiply-adds of the plain one.
//
// A wavefront computes P consecutive outputs per lane: 64 P outputs of one
// row (maps narrower than that put several rows in one wavefront).  Per row
// offset it loads the rows y +- dy of both components (a row ahead, into
// registers), leaves S and D in its own LDS rows and walks the taps in groups
// of four dx: one new 4-vector of S and of D from LDS and the group's eight
// weights from the scalar cache (dy is uniform across the wavefront) for
// 8 P fused multiply-adds.  The first and last group of a row skip the taps
// outside the disc (a zero weight would carry a NaN or an infinity there into
// the sum).  No barrier: a wavefront reads only what it wrote.  SPLIT wavefronts of a
// workgroup take the row offsets of one segment in turn and add up in a
// fixed order at the end.  The kernel is bound by the multiply-adds: 1024^2,
// cut 64, float in 411 us, i.e. 27 GFLOP done (half of the plain sum's 54) at
// 66 TFLOP/s of the 78.6 that unpacked FP32 instructions reach.  A ring of
// input rows shared by the workgroup without the pairing of rows took 991 us,
// and 292 us against 123 at cut 32; maps under 512 px, which had no staging,
// took 1.8 ms at 256^2, cut 64, against 45 us.
//
// The weights are tabulated on the device in the same stream (a table built
// on the host cost four uploads and a stream synchronisation, 50 us a call).
#include "amap_device.h"
#include "amap_host.h"
#include "amap_launch.h"

namespace amap {

// Weights of row offset dy = blockIdx.y (0 .. R) at dx = 4 k - R4 + q, group
// k, tap q: Q cos 2phi at [8 k + q], Q sin 2phi at [8 k + 4 + q] of the row's
// 8 ng values, zero outside |d|^2 <= c2; half[dy]: the largest |dx| inside
// (-1: none).  Evaluated in double precision, rounded once.
template <typename T>
__global__ void __launch_bounds__(64)
k_direct_taps(int filter, double theta, double fparam, double c2, int R, int R4, int ng,
              int* __restrict__ half, T* __restrict__ gtab) {
    const int dy = blockIdx.y;
    const int e = blockIdx.x * 64 + threadIdx.x;
    if (e == 0) {
        int h = -1;
        for (int dx = 0; dx <= R && (double)(dx * dx + dy * dy) <= c2; ++dx) h = dx;
        half[dy] = h;
    }
    if (e >= 4 * ng) return;
    const int dx = e - R4;
    const double r2 = (double)(dx * dx + dy * dy);
    double wc = 0.0, ws = 0.0;
    if (r2 <= c2 && r2 != 0.0) {
        const double q = direct_filter_Q(filter, sqrt(r2), theta, fparam);
        wc = q * (double)(dx * dx - dy * dy) / r2;
        ws = q * 2.0 * (double)dx * (double)dy / r2;
        if (dy == 0) wc *= 0.5;  // S_0 is 2 g1
    }
    T* row = gtab + ((long long)dy * ng + e / 4) * 8 + e % 4;
    row[0] = (T)wc;
    row[4] = (T)ws;
}

template <typename T>
struct Vec4 { T e[4]; };
// p is 16-byte aligned
template <typename T>
__device__ __forceinline__ Vec4<T> ld4(const T* p) {
    if constexpr (sizeof(T) == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 v = *reinterpret_cast<const f4*>(p);
        return Vec4<T>{{v[0], v[1], v[2], v[3]}};
    } else {
        typedef double d2 __attribute__((ext_vector_type(2)));
        const d2 a = *reinterpret_cast<const d2*>(p), b = *reinterpret_cast<const d2*>(p + 2);
        return Vec4<T>{{a[0], a[1], b[0], b[1]}};
    }
}
template <typename T>
__device__ __forceinline__ void st4(T* p, const Vec4<T>& r) {
    if constexpr (sizeof(T) == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<f4*>(p) = f4{r.e[0], r.e[1], r.e[2], r.e[3]};
    } else {
        typedef double d2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<d2*>(p) = d2{r.e[0], r.e[1]};
        *reinterpret_cast<d2*>(p + 2) = d2{r.e[2], r.e[3]};
    }
}

// The 4 x P taps of one group: dx = dx0 + q (q < 4) for outputs i < P, from
// the windows v of S and u of D (P + 4 values from dx0 on); w holds the
// group's four Q cos 2phi and four Q sin 2phi.  EDGE: only the taps lo <= q
// <= hi (uniform across the wavefront), which lie inside the disc.
template <typename T, int P, bool EDGE>
__device__ __forceinline__ void direct_group(T (&acc)[P], const T* __restrict__ w, const Vec4<T> (&v)[P / 4 + 1],
                                             const Vec4<T> (&u)[P / 4 + 1], int lo, int hi) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (EDGE && (q < lo || q > hi)) continue;
        const T wc = w[q], ws = w[4 + q];
#pragma unroll
        for (int i = 0; i < P; ++i)
            acc[i] = fma(wc, v[(i + q) / 4].e[(i + q) % 4], fma(ws, u[(i + q) / 4].e[(i + q) % 4], acc[i]));
    }
}

// Wavefronts of a workgroup: SPLIT of them per segment, at least four.
constexpr int direct_waves(int split) { return split > 4 ? split : 4; }
constexpr int kDirectPF = 3;     // 4-vectors of a staged row prefetched per lane

// Elements of one wavefront's S and D rows.
__host__ __device__ inline int direct_lds_elems(int tw, int rows, int R4) {
    return rows * 2 * (tw + 2 * R4 + 8);
}

template <typename T, int P, int SPLIT>
__global__ void __launch_bounds__(64 * direct_waves(SPLIT))
k_map_direct_rows(const T* __restrict__ g1, const T* __restrict__ g2, int logn, int R, int R4,
                  const int* __restrict__ half, const T* __restrict__ gtab, T* __restrict__ out) {
    constexpr int SEGS = direct_waves(SPLIT) / SPLIT, PV = P / 4;
    extern __shared__ __align__(16) unsigned char direct_smem[];
    const int n = 1 << logn, m = n - 1;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int part = wave % SPLIT;
    const int tw = n < 64 * P ? n : 64 * P;          // outputs of a row in one wavefront
    const int lpr = tw / P, rows = 64 / lpr;         // lanes per row, rows per wavefront
    const int ntx = n / tw;
    const int seg = blockIdx.x * SEGS + wave / SPLIT;
    const int sub = lane / lpr, li = lane - sub * lpr;
    const int x0 = (seg % ntx) * tw, y = (seg / ntx) * rows + sub;
    const int SW = tw + 2 * R4 + 8;                  // staged row width, a multiple of 4
    const int nvec = SW / 4, ng = R4 / 2 + 1;
    T* S = reinterpret_cast<T*>(direct_smem) + wave * direct_lds_elems(tw, rows, R4) + sub * 2 * SW;
    T* Dr = S + SW;
    T acc[P];
#pragma unroll
    for (int i = 0; i < P; ++i) acc[i] = (T)0;
    // rows y +- dy of both components at staged vector c
    Vec4<T> pa[kDirectPF], pb[kDirectPF], qa[kDirectPF], qb[kDirectPF];
    auto fetch = [&](int dy, int c, Vec4<T>& a, Vec4<T>& b, Vec4<T>& d, Vec4<T>& e) {
        const int col = (x0 - R4 + 4 * c) & m;
        const long long up = (long long)((y + dy) & m) * n + col, dn = (long long)((y - dy) & m) * n + col;
        a = ld4(g1 + up); b = ld4(g1 + dn);
        d = ld4(g2 + up); e = ld4(g2 + dn);
    };
    auto stage = [&](int c, const Vec4<T>& a, const Vec4<T>& b, const Vec4<T>& d, const Vec4<T>& e) {
        Vec4<T> s, t;
#pragma unroll
        for (int q = 0; q < 4; ++q) { s.e[q] = a.e[q] + b.e[q]; t.e[q] = d.e[q] - e.e[q]; }
        st4(S + 4 * c, s);
        st4(Dr + 4 * c, t);
    };
    auto prefetch = [&](int dy) {
#pragma unroll
        for (int k = 0; k < kDirectPF; ++k) {
            const int c = li + k * lpr;
            if (c < nvec) fetch(dy, c, pa[k], pb[k], qa[k], qb[k]);
        }
    };
    prefetch(part <= R ? part : R);
    for (int dy = part; dy <= R; dy += SPLIT) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");  // the last row's reads are done
#pragma unroll
        for (int k = 0; k < kDirectPF; ++k) {
            const int c = li + k * lpr;
            if (c < nvec) stage(c, pa[k], pb[k], qa[k], qb[k]);
        }
        for (int c = li + kDirectPF * lpr; c < nvec; c += lpr) {
            Vec4<T> a, b, d, e;
            fetch(dy, c, a, b, d, e);
            stage(c, a, b, d, e);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        if (dy + SPLIT <= R) prefetch(dy + SPLIT);
        const int h = half[dy];
        if (h < 0) continue;
        const T* r1 = S + P * li + R4;
        const T* r2 = Dr + P * li + R4;
        const T* wrow = gtab + ((long long)dy * ng + R4 / 4) * 8;
        const int gb = -((h + 3) >> 2), ge = h >> 2;  // groups dx0 = 4 g cover [-h, h]
        // the window of group g is the PV + 1 4-vectors from 4 g on
        Vec4<T> v[PV + 1], u[PV + 1];
#pragma unroll
        for (int k = 0; k < PV; ++k) {
            v[k] = ld4(r1 + 4 * (gb + k));
            u[k] = ld4(r2 + 4 * (gb + k));
        }
        // the first and the last group of the row may reach out of the disc
        const auto edge = [&](int g) {
            v[PV] = ld4(r1 + 4 * (g + PV));
            u[PV] = ld4(r2 + 4 * (g + PV));
            direct_group<T, P, true>(acc, wrow + g * 8, v, u, -h - 4 * g, h - 4 * g);
#pragma unroll
            for (int k = 0; k < PV; ++k) { v[k] = v[k + 1]; u[k] = u[k + 1]; }
        };
        edge(gb);
        int g = gb + 1;
        for (; g + PV < ge; g += PV + 1) {
            // PV + 1 groups per iteration: the window is renamed, not moved
#pragma unroll
            for (int s = 0; s < PV + 1; ++s) {
                v[(s + PV) % (PV + 1)] = ld4(r1 + 4 * (g + s + PV));
                u[(s + PV) % (PV + 1)] = ld4(r2 + 4 * (g + s + PV));
                Vec4<T> vv[PV + 1], uu[PV + 1];
#pragma unroll
                for (int k = 0; k < PV + 1; ++k) {
                    vv[k] = v[(s + k) % (PV + 1)];
                    uu[k] = u[(s + k) % (PV + 1)];
                }
                direct_group<T, P, false>(acc, wrow + (g + s) * 8, vv, uu, 0, 3);
            }
        }
        for (; g < ge; ++g) {
            v[PV] = ld4(r1 + 4 * (g + PV));
            u[PV] = ld4(r2 + 4 * (g + PV));
            direct_group<T, P, false>(acc, wrow + g * 8, v, u, 0, 3);
#pragma unroll
            for (int k = 0; k < PV; ++k) { v[k] = v[k + 1]; u[k] = u[k + 1]; }
        }
        if (gb < ge) edge(ge);
    }
    if constexpr (SPLIT > 1) {
        __syncthreads();  // every wavefront is done with its rows
        T* red = reinterpret_cast<T*>(direct_smem);  // [SEGS][SPLIT - 1][P][64]
        T* mine = red + ((wave / SPLIT) * (SPLIT - 1)) * P * 64 + lane;
        if (part > 0) {
#pragma unroll
            for (int i = 0; i < P; ++i) mine[((part - 1) * P + i) * 64] = acc[i];
        }
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int p = 0; p < SPLIT - 1; ++p)
#pragma unroll
            for (int i = 0; i < P; ++i) acc[i] += mine[(p * P + i) * 64];
    }
    T* o = out + (long long)y * n + x0 + P * li;
#pragma unroll
    for (int k = 0; k < PV; ++k)
        st4(o + 4 * k, Vec4<T>{{-acc[4 * k], -acc[4 * k + 1], -acc[4 * k + 2], -acc[4 * k + 3]}});
}

size_t direct_workspace_bytes(int R, size_t elem) {
    const int R4 = (R + 3) / 4 * 4, ng = R4 / 2 + 1;
    const size_t halves = ((size_t)(R + 1) * sizeof(int) + 255) & ~(size_t)255;
    return halves + (size_t)(R + 1) * ng * 8 * elem;
}

template <typename T, int P, int SPLIT>
static hipError_t launch_direct_rows(int logn, const T* g1, const T* g2, int R, int R4, const int* half,
                                     const T* gtab, T* out, hipStream_t s) {
    const int n = 1 << logn, tw = n < 64 * P ? n : 64 * P, rows = 64 * P / tw;
    constexpr int WAVES = direct_waves(SPLIT);
    const int segs = (n / tw) * (n / rows), per = WAVES / SPLIT;
    size_t elems = (size_t)WAVES * direct_lds_elems(tw, rows, R4);
    if (elems < (size_t)WAVES * P * 64) elems = (size_t)WAVES * P * 64;
    const size_t lds = elems * sizeof(T);
    if (n % rows != 0 || segs % per != 0 || lds > 128 * 1024) return hipErrorInvalidConfiguration;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_map_direct_rows<T, P, SPLIT>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    AMAP_LAUNCH("map_direct", s,
                k_map_direct_rows<T, P, SPLIT><<<segs / per, 64 * WAVES, lds, s>>>(
                    g1, g2, logn, R, R4, half, gtab, out));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_map_direct(int logn, const T* g1, const T* g2, int filter, double theta, double fparam,
                             double cut, void* ws, T* out, hipStream_t s) {
    const int n = 1 << logn;
    const int R = (int)cut, R4 = (R + 3) / 4 * 4, ng = R4 / 2 + 1;
    int* half = static_cast<int*>(ws);
    T* gtab = reinterpret_cast<T*>(static_cast<char*>(ws) + (((size_t)(R + 1) * sizeof(int) + 255) & ~(size_t)255));
    AMAP_LAUNCH("direct_taps", s,
                k_direct_taps<T><<<dim3((4 * ng + 63) / 64, R + 1), 64, 0, s>>>(filter, theta, fparam, cut * cut,
                                                                               R, R4, ng, half, gtab));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // Wavefronts per segment (SPLIT): maps from 512 px have a segment per 512
    // outputs, so 4 fill the chip from 512 x 512 on (1024^2, cut 32, float:
    // 126 us with 4, 151 with 1, 157 with 8; 512^2: 44, 135, 46); narrower
    // maps have at most 256 segments of 256 outputs and take as many as a
    // workgroup holds (256^2, cut 64, float: 45 us with 16, 56 with 8, 94 with
    // 4; double: 106, 83, 133: 16 wavefronts of doubles leave one workgroup
    // per CU and spill).
    if (n >= 512) return launch_direct_rows<T, 8, 4>(logn, g1, g2, R, R4, half, gtab, out, s);
    return launch_direct_rows<T, 4, sizeof(T) == 4 ? 16 : 8>(logn, g1, g2, R, R4, half, gtab, out, s);
}

template hipError_t launch_map_direct<float>(int, const float*, const float*, int, double, double, double,
                                             void*, float*, hipStream_t);
template hipError_t launch_map_direct<double>(int, const double*, const double*, int, double, double, double,
                                              void*, double*, hipStream_t);

}  // namespace amap

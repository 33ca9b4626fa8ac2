// Fields with edges and of any size: the starlet cascade under periodic,
// mirror or zero boundary rules (0, 1, 2), the running statistics of noise
// realisations (Sec. 1, Sec. 5.1: Welford's update in double, then sigma and
// S/N), and peak counts with neighbours taken through the edge rule
// (Sec. 2.2).
//
// The a trous cascade is that of Sec. 3 (B3 taps (1,4,6,4,1)/16 at dilation
// 2^(j-1), row pass along x then column pass along y, w_j = c_{j-1} - c_j);
// the paper leaves edges open, so the rule is the caller's: periodic (index
// mod n), mirror (whole-sample symmetric: reflection about the first and
// last samples, period 2(n-1)) or zero outside the field, applied to
// c_{j-1} on each axis at every step.  One thread per output pixel; the
// taps of interior pixels are contiguous rows, so the loads coalesce.
#include <hip/hip_runtime.h>

#include "amap_device.h"
#include "amap_launch.h"

namespace amap {

namespace {

// i mapped into [0, n) by the rule; -1 for a sample outside (zero rule).
__device__ __forceinline__ int bc_index(int i, int n, int mode) {
    if (i >= 0 && i < n) return i;
    if (mode == 0) {
        const int k = i % n;
        return k < 0 ? k + n : k;
    }
    if (mode == 1) {
        const int p = 2 * (n - 1);
        int k = i % p;
        if (k < 0) k += p;
        return k < n ? k : p - k;
    }
    return -1;
}

template <typename T>
__device__ __forceinline__ T b3(T a0, T a1, T a2, T a3, T a4) {
    return (T)0.0625 * (a0 + a4) + (T)0.25 * (a1 + a3) + (T)0.375 * a2;
}

// r[y][x] = sum_t h_t c[y][x + (t-2) d]; grid (ceil(nx/256), ny, maps),
// map z at c + z c_stride and r + z r_stride
template <typename T>
__global__ void __launch_bounds__(256)
k_bc_row(const T* __restrict__ c, T* __restrict__ r, int nx, int d, int mode, long long c_stride,
         long long r_stride) {
    const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y;
    if (x >= nx) return;
    c += blockIdx.z * c_stride;
    r += blockIdx.z * r_stride;
    const T* row = c + (long long)y * nx;
    T v[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        const int i = bc_index(x + (t - 2) * d, nx, mode);
        v[t] = i < 0 ? (T)0 : row[i];
    }
    r[(long long)y * nx + x] = b3(v[0], v[1], v[2], v[3], v[4]);
}

// c_next[y][x] = sum_t h_t r[y + (t-2) d][x], w = c_prev - c_next.  c_prev
// and c_next may be the same array: each thread reads and writes only its
// own pixel of them.  grid (ceil(nx/256), ny, maps); map z's w and c_next
// at + z pl_stride
template <typename T>
__global__ void __launch_bounds__(256)
k_bc_col(const T* __restrict__ r, const T* c_prev, T* __restrict__ w, T* c_next, int ny, int nx,
         int d, int mode, long long r_stride, long long cp_stride, long long pl_stride) {
    const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y;
    if (x >= nx) return;
    r += blockIdx.z * r_stride;
    c_prev += blockIdx.z * cp_stride;
    w += blockIdx.z * pl_stride;
    c_next += blockIdx.z * pl_stride;
    T v[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        const int i = bc_index(y + (t - 2) * d, ny, mode);
        v[t] = i < 0 ? (T)0 : r[(long long)i * nx + x];
    }
    const long long o = (long long)y * nx + x;
    const T cn = b3(v[0], v[1], v[2], v[3], v[4]);
    const T cp = c_prev[o];
    w[o] = cp - cn;
    c_next[o] = cn;
}

// One smoothing step at dilation d as a tile: kBcTW consecutive columns by
// kBcTH rows of one residue class ry (mod d) of the rows, y = ry + d (M0 + m).
// Taps of the column pass then stay in the class (the edge rule maps each
// tap row on its own, so the tile simply loads the mapped rows), and the
// tile stages kBcTH + 4 rows of kBcTW + 4d columns of c_{j-1} once: the row
// pass runs in LDS on all of them, the column pass on the kBcTH middle rows,
// and w_j = c_{j-1} - c_j and c_j are written (c_j to a buffer apart from
// c_{j-1}, whose halo other tiles still read).  grid (column tiles,
// d * row-tile count, maps); dynamic LDS (kBcTH + 4)(kBcTW + 4d + kBcTW) T,
// under 64 KiB up to dilation bc_max_d.
constexpr int kBcTW = 64, kBcTH = 16;
template <typename T>
constexpr int bc_max_d() { return sizeof(T) == 4 ? 128 : 64; }
template <typename T>
__global__ void __launch_bounds__(256)
k_bc_scale_tile(const T* __restrict__ c_prev, T* __restrict__ w, T* __restrict__ c_next, int ny,
                int nx, int d, int mode, long long cp_stride, long long cn_stride, long long w_stride) {
    extern __shared__ unsigned char lds_raw[];
    T* reg = reinterpret_cast<T*>(lds_raw);            // [kBcTH + 4][RW]
    const int RW = kBcTW + 4 * d;
    T* rr = reg + (kBcTH + 4) * RW;                    // [kBcTH + 4][kBcTW]
    const int x0 = blockIdx.x * kBcTW;
    const int ry = blockIdx.y % d, M0 = (blockIdx.y / d) * kBcTH;
    c_prev += blockIdx.z * cp_stride;
    c_next += blockIdx.z * cn_stride;
    w += blockIdx.z * w_stride;
    // stage: region row m is c_{j-1} row bc(ry + d (M0 + m - 2)), region
    // column i is column bc(x0 - 2d + i)
    for (int e = threadIdx.x; e < (kBcTH + 4) * RW; e += 256) {
        const int m = e / RW, i = e - m * RW;
        const int yy = bc_index(ry + d * (M0 + m - 2), ny, mode);
        const int xx = bc_index(x0 - 2 * d + i, nx, mode);
        reg[e] = (yy < 0 || xx < 0) ? (T)0 : c_prev[(long long)yy * nx + xx];
    }
    __syncthreads();
    // row pass on every staged row
    for (int e = threadIdx.x; e < (kBcTH + 4) * kBcTW; e += 256) {
        const int m = e / kBcTW, i = e - m * kBcTW;
        const T* g = reg + m * RW + i;
        rr[e] = b3(g[0], g[d], g[2 * d], g[3 * d], g[4 * d]);
    }
    __syncthreads();
    // column pass on the middle rows
    for (int e = threadIdx.x; e < kBcTH * kBcTW; e += 256) {
        const int m = e / kBcTW, i = e - m * kBcTW;
        const int y = ry + d * (M0 + m), x = x0 + i;
        if (y >= ny || x >= nx) continue;
        const T* g = rr + m * kBcTW + i;
        const T cn = b3(g[0], g[kBcTW], g[2 * kBcTW], g[3 * kBcTW], g[4 * kBcTW]);
        const T cp = reg[(m + 2) * RW + 2 * d + i];
        const long long o = (long long)y * nx + x;
        w[o] = cp - cn;
        c_next[o] = cn;
    }
}

// Welford's update with realisations r0 .. r0+nb-1 in order, the b-th's
// values at w + b w_stride (realisation 0 writes M and M2 unread).
template <typename T>
__global__ void __launch_bounds__(256)
k_welford_bc(const T* __restrict__ w, long long w_stride, int nb, double* __restrict__ M,
             double* __restrict__ M2, long long count, int r0) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    double m = r0 == 0 ? 0.0 : M[i], m2 = r0 == 0 ? 0.0 : M2[i];
    for (int b = 0; b < nb; ++b) {
        const double v = (double)w[b * w_stride + i];
        const int r = r0 + b;
        if (r == 0) {
            m = v;
            m2 = 0.0;
            continue;
        }
        const double d = v - m, mn = m + d / (double)(r + 1);
        m2 = m2 + d * (v - mn);
        m = mn;
    }
    M[i] = m;
    M2[i] = m2;
}

template <typename T>
__global__ void __launch_bounds__(256)
k_sigma_snr_bc(const double* __restrict__ M2, int R, const T* __restrict__ w_signal, T* __restrict__ sigma,
               T* __restrict__ snr, long long count) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const double sg = sqrt(M2[i] / (double)(R - 1));
    sigma[i] = (T)sg;
    if (snr) snr[i] = sg > 0.0 ? (T)((double)w_signal[i] / sg) : (T)0;
}

// Whether pixel idx of value v is a strict 8-neighbour maximum under the
// edge rule (0 outside under the zero rule) and, with a mask, it and every
// neighbour inside the field are observed.  Every load is issued before the
// first test, so a candidate costs one memory latency.
template <typename T, bool MASK>
__device__ __forceinline__ bool bc_peak(const T* __restrict__ p, const unsigned char* __restrict__ mask,
                                        int idx, T v, int ny, int nx, int mode) {
    const int y = idx / nx, x = idx - y * nx;
    int yy[3], xx[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        yy[d] = bc_index(y + d - 1, ny, mode);
        xx[d] = bc_index(x + d - 1, nx, mode);
    }
    T q[9];
    unsigned char ok[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const bool in = yy[k / 3] >= 0 && xx[k % 3] >= 0;
        const int at = in ? yy[k / 3] * nx + xx[k % 3] : idx;
        q[k] = p[at];
        q[k] = in ? q[k] : (T)0;
        if (MASK) ok[k] = mask[at];  // outside the field: the pixel's own byte, tested anyway
    }
    bool pk = true;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        if (k != 4) pk = pk & (v > q[k]);
        if (MASK) pk = pk & (ok[k] != 0);
    }
    return pk;
}

// Strict 8-neighbour maxima above thr of ny x nx planes, neighbours taken
// through the edge rule; grid (blocks, nplanes) of 256 threads.  Pixels are
// walked in flat order (the values before a plane's first 16-byte boundary
// and after its last by the first block), four vectors per thread in flight,
// and only a pixel above thr splits its index and looks at its neighbours.
// A block's count gathers in LDS and is added once.  Bound by the read of
// the planes: six 1000^2 float planes with a mask in 15 us (51 us one pixel at
// a time, each neighbour loaded after the test of the one before).
template <typename T, bool MASK>
__global__ void __launch_bounds__(256)
k_count_peaks_bc(const T* __restrict__ planes, const unsigned char* __restrict__ mask, int ny,
                 int nx, int mode, double thr, long long* __restrict__ counts) {
    __shared__ unsigned int block_count;
    if (threadIdx.x == 0) block_count = 0u;
    constexpr int G = 16 / (int)sizeof(T), U = 4;
    typedef T vec __attribute__((ext_vector_type(G)));
    const int npix = ny * nx;
    const T* p = planes + (long long)blockIdx.y * npix;
    const int head0 = (int)((-(reinterpret_cast<uintptr_t>(p) / sizeof(T))) & (G - 1));
    const int head = head0 < npix ? head0 : npix;
    const int nvec = (npix - head) / G;
    const vec* pv = reinterpret_cast<const vec*>(p + head);
    unsigned int npk = 0;
    const int stride = gridDim.x * 256;
    for (int i0 = blockIdx.x * 256 + threadIdx.x; i0 < nvec; i0 += U * stride) {
        vec v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * stride;
            v[u] = pv[i < nvec ? i : i0];
        }
        unsigned int found = 0u;  // bit u G + c: a pixel above thr
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < G; ++c)
                found |= ((double)v[u][c] > thr && i0 + u * stride < nvec ? 1u : 0u) << (u * G + c);
        while (found) {  // one copy of the test: unrolled over the pixels it outgrew the instruction cache
            const int k = __builtin_ctz(found);
            found &= found - 1u;
            const int idx = head + (i0 + (k / G) * stride) * G + k % G;
            npk += bc_peak<T, MASK>(p, mask, idx, p[idx], ny, nx, mode) ? 1u : 0u;
        }
    }
    if (blockIdx.x == 0) {  // the ends outside whole vectors: fewer than 2 G values
        const int tail0 = head + nvec * G, ends = head + npix - tail0;
        if ((int)threadIdx.x < ends) {
            const int idx = (int)threadIdx.x < head ? (int)threadIdx.x : tail0 + (int)threadIdx.x - head;
            const T v = p[idx];
            if ((double)v > thr) npk += bc_peak<T, MASK>(p, mask, idx, v, ny, nx, mode) ? 1u : 0u;
        }
    }
    __syncthreads();  // block_count is zeroed
    if (npk) atomicAdd(&block_count, npk);
    __syncthreads();
    if (threadIdx.x == 0 && block_count)
        atomicAdd((unsigned long long*)&counts[blockIdx.y], (unsigned long long)block_count);
}

// Shear of a masked field: both components kept where the mask byte is
// non-zero and zeroed where the pixel is missing; four pixels per thread
// (count a multiple of 4, buffers 256-byte aligned), in place allowed.
template <typename T>
__global__ void __launch_bounds__(256)
k_mask_shear(const T* g1, const T* g2, const unsigned char* __restrict__ mask, T* o1, T* o2,
             long long quads) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= quads) return;
    const uchar4 m = reinterpret_cast<const uchar4*>(mask)[i];
    const unsigned char mm[4] = {m.x, m.y, m.z, m.w};
    T a[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { a[k] = g1[4 * i + k]; b[k] = g2[4 * i + k]; }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        o1[4 * i + k] = mm[k] ? a[k] : (T)0;
        o2[4 * i + k] = mm[k] ? b[k] : (T)0;
    }
}

// The last count % 4 pixels.
template <typename T>
__global__ void k_mask_shear_tail(const T* g1, const T* g2, const unsigned char* __restrict__ mask,
                                  T* o1, T* o2, long long first, long long count) {
    const long long i = first + threadIdx.x;
    if (i >= count) return;
    const T a = g1[i], b = g2[i];
    o1[i] = mask[i] ? a : (T)0;
    o2[i] = mask[i] ? b : (T)0;
}

}  // namespace

template <typename T>
hipError_t launch_count_peaks_bc(int ny, int nx, int nplanes, int mode, const T* planes,
                                 const unsigned char* mask, double thr, long long* counts,
                                 hipStream_t s) {
    hipError_t e = launch_zero_i64(counts, nplanes, s);
    if (e != hipSuccess) return e;
    // four vectors per thread, at most 256 blocks (adds) per counter
    const long long per = 256ll * 4 * (16 / (long long)sizeof(T));
    long long b = ((long long)ny * nx + per - 1) / per;
    const dim3 grid((unsigned)(b > 256 ? 256 : b), nplanes);
    if (mask)
        AMAP_LAUNCH("count_peaks_bc", s,
                    k_count_peaks_bc<T, true><<<grid, 256, 0, s>>>(planes, mask, ny, nx, mode, thr, counts));
    else
        AMAP_LAUNCH("count_peaks_bc", s,
                    k_count_peaks_bc<T, false><<<grid, 256, 0, s>>>(planes, mask, ny, nx, mode, thr, counts));
    return hipGetLastError();
}
template hipError_t launch_count_peaks_bc<float>(int, int, int, int, const float*, const unsigned char*,
                                                 double, long long*, hipStream_t);
template hipError_t launch_count_peaks_bc<double>(int, int, int, int, const double*, const unsigned char*,
                                                  double, long long*, hipStream_t);

template <typename T>
hipError_t launch_mask_shear(long long count, const T* g1, const T* g2, const unsigned char* mask,
                             T* o1, T* o2, hipStream_t s) {
    const long long quads = count / 4;
    if (quads > 0)
        AMAP_LAUNCH("mask_shear", s,
                    k_mask_shear<T><<<(unsigned)((quads + 255) / 256), 256, 0, s>>>(g1, g2, mask, o1, o2,
                                                                                   quads));
    if (count % 4)
        AMAP_LAUNCH("mask_shear", s,
                    k_mask_shear_tail<T><<<1, 4, 0, s>>>(g1, g2, mask, o1, o2, 4 * quads, count));
    return hipGetLastError();
}
template hipError_t launch_mask_shear<float>(long long, const float*, const float*, const unsigned char*,
                                             float*, float*, hipStream_t);
template hipError_t launch_mask_shear<double>(long long, const double*, const double*,
                                              const unsigned char*, double*, double*, hipStream_t);

template <typename T>
hipError_t launch_starlet_bc(int ny, int nx, int J, int mode, const T* image, T* planes, T* tmp,
                             int maps, long long image_stride, long long planes_stride, hipStream_t s) {
    const long long plane = (long long)ny * nx;
    T* coarse = planes + (long long)(J - 1) * plane;
    // scales 1 .. jt (dilation <= bc_max_d) run as tiles, alternating their
    // c_j between tmp and the coarse plane so that c_jt lands in the coarse
    // plane; the later scales run a row and a column pass in place there
    int jt = 0;
    while (jt + 1 < J && (1 << jt) <= bc_max_d<T>()) ++jt;
    const T* c_prev = image;
    long long cp_stride = image_stride;
    for (int j = 1; j <= jt; ++j) {
        const int d = 1 << (j - 1);
        const bool to_coarse = ((jt - j) & 1) == 0;
        T* dst = to_coarse ? coarse : tmp;
        const long long dst_stride = to_coarse ? planes_stride : plane;
        const int rows = (ny + d - 1) / d;  // rows of the largest residue class
        const int row_tiles = (rows + kBcTH - 1) / kBcTH;
        const dim3 grid((nx + kBcTW - 1) / kBcTW, d * row_tiles, maps);
        const size_t lds = (size_t)(kBcTH + 4) * (kBcTW + 4 * d + kBcTW) * sizeof(T);
        AMAP_LAUNCH("starlet_bc_tile", s,
                    k_bc_scale_tile<T><<<grid, 256, lds, s>>>(c_prev, planes + (long long)(j - 1) * plane,
                                                              dst, ny, nx, d, mode, cp_stride, dst_stride,
                                                              planes_stride));
        c_prev = dst;
        cp_stride = dst_stride;
    }
    const dim3 grid((nx + 255) / 256, ny, maps);
    for (int j = jt + 1; j < J; ++j) {
        const int d = 1 << (j - 1);
        AMAP_LAUNCH("starlet_bc_row", s,
                    k_bc_row<T><<<grid, 256, 0, s>>>(c_prev, tmp, nx, d, mode, cp_stride, plane));
        AMAP_LAUNCH("starlet_bc_col", s,
                    k_bc_col<T><<<grid, 256, 0, s>>>(tmp, c_prev, planes + (long long)(j - 1) * plane,
                                                     coarse, ny, nx, d, mode, plane, cp_stride,
                                                     planes_stride));
        c_prev = coarse;
        cp_stride = planes_stride;
    }
    return hipGetLastError();
}
static unsigned blocks256(long long count) { return (unsigned)((count + 255) / 256); }

template <typename T>
hipError_t launch_welford_bc(const T* w, long long w_stride, int nb, double* M, double* M2,
                             long long count, int r0, hipStream_t s) {
    AMAP_LAUNCH("welford_bc", s,
                k_welford_bc<T><<<blocks256(count), 256, 0, s>>>(w, w_stride, nb, M, M2, count, r0));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_sigma_snr_bc(const double* M2, int R, const T* w_signal, T* sigma, T* snr,
                               long long count, hipStream_t s) {
    AMAP_LAUNCH("sigma_snr_bc", s,
                k_sigma_snr_bc<T><<<blocks256(count), 256, 0, s>>>(M2, R, w_signal, sigma, snr, count));
    return hipGetLastError();
}

#define AMAP_BOUNDED_NOISE(T)                                                                            \
    template hipError_t launch_welford_bc<T>(const T*, long long, int, double*, double*, long long, int, \
                                             hipStream_t);                                               \
    template hipError_t launch_sigma_snr_bc<T>(const double*, int, const T*, T*, T*, long long, hipStream_t);
AMAP_BOUNDED_NOISE(float)
AMAP_BOUNDED_NOISE(double)
#undef AMAP_BOUNDED_NOISE

template hipError_t launch_starlet_bc<float>(int, int, int, int, const float*, float*, float*, int,
                                             long long, long long, hipStream_t);
template hipError_t launch_starlet_bc<double>(int, int, int, int, const double*, double*, double*, int,
                                              long long, long long, hipStream_t);
}  // namespace amap

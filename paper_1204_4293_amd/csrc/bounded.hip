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
// c_{j-1} on each axis at every step.  A step runs as LDS tiles up to a
// dilation of bc_max_d, beyond it as a row and a column pass with one thread
// per output pixel.
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
// own pixel of them.  grid (ceil(nx/256), ny, maps); map z's w
// at + z w_stride, its c_next at + z cn_stride
template <typename T>
__global__ void __launch_bounds__(256)
k_bc_col(const T* __restrict__ r, const T* c_prev, T* __restrict__ w, T* c_next, int ny, int nx,
         int d, int mode, long long r_stride, long long cp_stride, long long w_stride, long long cn_stride) {
    const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y;
    if (x >= nx) return;
    r += blockIdx.z * r_stride;
    c_prev += blockIdx.z * cp_stride;
    w += blockIdx.z * w_stride;
    c_next += blockIdx.z * cn_stride;
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

// One smoothing step at dilation d as a tile: 64 columns by kBcTH rows of one
// residue class ry (mod d) of the rows, y = ry + d (M0 + m).  Taps of the
// column pass then stay in the class (the edge rule maps each tap row on its
// own, so the tile simply loads the mapped rows), and the tile stages
// kBcTH + 4 rows of 64 + 4d columns of c_{j-1} once: the row pass runs in LDS
// on all of them, the column pass on the kBcTH middle rows, and c_j goes to a
// buffer apart from c_{j-1}, whose halo other tiles still read.  A lane
// keeps one column: it stages column chunks of 64, so the edge rule is worked
// out once per chunk and row (uniform), not per value, and its wavefront owns
// kBcTH / 4 consecutive output rows, a sliding window down the column.
//
// NOISE: the tile takes nb realisations in turn, the next one's values on
// their way (in registers) while the current one is filtered, and keeps
// Welford's mean and squared deviations of its pixels in registers (double):
// w_j goes nowhere.  They continue from M and M2 unless r0 = 0 and end there,
// or, with the last realisation (r0 + nb = R), as sigma and S/N.  Else
// (signal): blockIdx.z is the map, w_j = c_{j-1} - c_j is stored.
//
// Bound by memory traffic (8 bytes a pixel, scale and realisation, and the
// halos through L2).  16 realisations of a 1000 x 1000 float field, one
// scale: 57 us (d <= 16) to 75 (d = 32), where storing w_j and a pass for the
// statistics took 109; one map: 6.5 to 9.5 us, 9.5 with the edge rule worked
// out per value.
// grid (column tiles, d * row tiles, maps or 1); dynamic LDS
// (kBcTH + 4)(64 + 4d + 64) T, under 64 KiB up to dilation bc_max_d.  KC:
// column chunks of a staged row.
constexpr int kBcTH = 16;
template <typename T>
constexpr int bc_max_d() { return sizeof(T) == 4 ? 128 : 64; }

template <typename T>
struct BcArgs {
    const T* c_prev;
    T* c_next;  // null (NOISE): the last scale
    T* w;       // signal: w_j
    int ny, nx, d, mode;
    long long cp_stride, cn_stride, w_stride;  // per map or realisation
    // NOISE
    int nb, r0, R;
    double *M, *M2;
    const T* w_signal;
    T *sigma, *snr;
};

template <typename T, bool NOISE, int KC>
__global__ void __launch_bounds__(256)
k_bc_scale(BcArgs<T> a) {
    constexpr int ROWS = kBcTH + 4, RPW = ROWS / 4, OPW = kBcTH / 4;  // staged and output rows per wavefront
    extern __shared__ unsigned char lds_raw[];
    T* reg = reinterpret_cast<T*>(lds_raw);  // [ROWS][RW]
    const int d = a.d, RW = 64 + 4 * d;
    T* rr = reg + ROWS * RW;                 // [ROWS][64]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int x0 = blockIdx.x * 64;
    const int ry = blockIdx.y % d, M0 = (blockIdx.y / d) * kBcTH;
    const long long plane = (long long)a.ny * a.nx;
    // this lane's staged columns and its wavefront's staged rows (-1: 0)
    int col[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int i = lane + 64 * k;
        col[k] = i < RW ? bc_index(x0 - 2 * d + i, a.nx, a.mode) : -1;
    }
    int row[RPW];
#pragma unroll
    for (int q = 0; q < RPW; ++q) row[q] = bc_index(ry + d * (M0 + wave + 4 * q - 2), a.ny, a.mode);
    // owned pixels: column x of OPW rows
    const int x = x0 + lane;
    const auto out_row = [&](int k) { return ry + d * (M0 + OPW * wave + k); };
    T v[RPW][KC];
    const auto fetch = [&](const T* src) {
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const T* p = src + (long long)(row[q] < 0 ? 0 : row[q]) * a.nx;
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const T t = p[col[k] < 0 ? 0 : col[k]];
                v[q][k] = row[q] < 0 || col[k] < 0 ? (T)0 : t;
            }
        }
    };
    double mean[OPW], m2[OPW];
    if constexpr (NOISE) {
#pragma unroll
        for (int k = 0; k < OPW; ++k) {
            const int y = out_row(k);
            const bool in = a.r0 > 0 && y < a.ny && x < a.nx;
            mean[k] = in ? a.M[(long long)y * a.nx + x] : 0.0;
            m2[k] = in ? a.M2[(long long)y * a.nx + x] : 0.0;
        }
    }
    const int maps = NOISE ? a.nb : 1;
    const long long first = NOISE ? 0 : blockIdx.z;
    fetch(a.c_prev + first * a.cp_stride);
    for (int b = 0; b < maps; ++b) {
        const long long map = first + b;
        __syncthreads();  // the previous map's reads of the tile are done
#pragma unroll
        for (int q = 0; q < RPW; ++q)
#pragma unroll
            for (int k = 0; k < KC; ++k)
                if (lane + 64 * k < RW) reg[(wave + 4 * q) * RW + lane + 64 * k] = v[q][k];
        if (NOISE && b + 1 < maps) fetch(a.c_prev + (map + 1) * a.cp_stride);
        __syncthreads();
        // row pass on every staged row
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const T* g = reg + (wave + 4 * q) * RW + lane;
            rr[(wave + 4 * q) * 64 + lane] = b3(g[0], g[d], g[2 * d], g[3 * d], g[4 * d]);
        }
        __syncthreads();
        // column pass on this wavefront's output rows
        T win[OPW + 4];
#pragma unroll
        for (int k = 0; k < OPW + 4; ++k) win[k] = rr[(OPW * wave + k) * 64 + lane];
        const double inv = NOISE ? 1.0 / (double)(a.r0 + b + 1) : 0.0;
#pragma unroll
        for (int k = 0; k < OPW; ++k) {
            const int y = out_row(k);
            const T cn = b3(win[k], win[k + 1], win[k + 2], win[k + 3], win[k + 4]);
            const T wv = reg[(OPW * wave + k + 2) * RW + 2 * d + lane] - cn;
            const bool in = y < a.ny && x < a.nx;
            const long long o = (long long)y * a.nx + x;
            if (in && (!NOISE || a.c_next)) a.c_next[map * a.cn_stride + o] = cn;
            if constexpr (NOISE) {
                const double dl = (double)wv - mean[k];
                mean[k] = fma(dl, inv, mean[k]);
                m2[k] = fma(dl, (double)wv - mean[k], m2[k]);
            } else {
                if (in) a.w[map * a.w_stride + o] = wv;
            }
        }
    }
    if constexpr (NOISE) {
        const bool last = a.r0 + a.nb == a.R;
#pragma unroll
        for (int k = 0; k < OPW; ++k) {
            const int y = out_row(k);
            if (y >= a.ny || x >= a.nx) continue;
            const long long o = (long long)y * a.nx + x;
            if (last) {
                const double sg = sqrt(m2[k] / (double)(a.R - 1));
                a.sigma[o] = (T)sg;
                if (a.snr) a.snr[o] = sg > 0.0 ? (T)((double)a.w_signal[o] / sg) : (T)0;
            } else {
                a.M[o] = mean[k];
                a.M2[o] = m2[k];
            }
        }
    }
}

// Welford's update of one or more scales (blockIdx.y) with realisations
// r0 .. r0+nb-1 in order, the b-th's detail plane at w + b w_stride, scale by
// scale w_scale apart: the arithmetic of k_bc_scale's.  Realisation 0 starts
// from nothing, the last one (r0 + nb = R) ends as sigma and S/N.
template <typename T>
__global__ void __launch_bounds__(256)
k_bc_stats(const T* __restrict__ w, long long w_stride, long long w_scale, int nb, int r0, int R,
           double* __restrict__ M, double* __restrict__ M2, const T* __restrict__ w_signal, T* __restrict__ sigma,
           T* __restrict__ snr, long long count) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const long long o = blockIdx.y * count + i;
    w += blockIdx.y * w_scale + i;
    double mean = 0.0, m2 = 0.0;
    if (r0 > 0) {
        mean = M[o];
        m2 = M2[o];
    }
    constexpr int U = 8;  // values on their way at a time
    for (int b0 = 0; b0 < nb; b0 += U) {
        T v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = w[(b0 + k < nb ? b0 + k : nb - 1) * w_stride];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (b0 + k >= nb) break;
            const double inv = 1.0 / (double)(r0 + b0 + k + 1);
            const double dl = (double)v[k] - mean;
            mean = fma(dl, inv, mean);
            m2 = fma(dl, (double)v[k] - mean, m2);
        }
    }
    if (r0 + nb < R) {
        M[o] = mean;
        M2[o] = m2;
        return;
    }
    const double sg = sqrt(m2 / (double)(R - 1));
    sigma[o] = (T)sg;
    if (snr) snr[o] = sg > 0.0 ? (T)((double)w_signal[o] / sg) : (T)0;
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

// One scale as a tile launch over `maps` maps (signal) or a.nb realisations.
template <typename T, bool NOISE, int KC>
static hipError_t launch_bc_scale_kc(const BcArgs<T>& a, int maps, hipStream_t s) {
    const int rows = (a.ny + a.d - 1) / a.d;  // rows of the largest residue class
    const int row_tiles = (rows + kBcTH - 1) / kBcTH;
    const dim3 grid((a.nx + 63) / 64, a.d * row_tiles, NOISE ? 1 : maps);
    const size_t lds = (size_t)(kBcTH + 4) * (64 + 4 * a.d + 64) * sizeof(T);
    if (64 + 4 * a.d > 64 * KC || lds > 64 * 1024) return hipErrorInvalidConfiguration;
    AMAP_LAUNCH(NOISE ? "noise_bc_tile" : "starlet_bc_tile", s, k_bc_scale<T, NOISE, KC><<<grid, 256, lds, s>>>(a));
    return hipGetLastError();
}
template <typename T, bool NOISE>
static hipError_t launch_bc_scale(const BcArgs<T>& a, int maps, hipStream_t s) {
    if (a.d <= 16) return launch_bc_scale_kc<T, NOISE, 2>(a, maps, s);
    if (a.d <= 32) return launch_bc_scale_kc<T, NOISE, 3>(a, maps, s);
    if (a.d <= 64) return launch_bc_scale_kc<T, NOISE, 5>(a, maps, s);
    return launch_bc_scale_kc<T, NOISE, 9>(a, maps, s);
}

int bc_tile_scales(int J, size_t elem) {
    int jt = 0;
    while (jt + 1 < J && (1 << jt) <= (elem == 4 ? bc_max_d<float>() : bc_max_d<double>())) ++jt;
    return jt;
}

template <typename T>
hipError_t launch_starlet_bc(int ny, int nx, int J, int mode, const T* image, T* planes, T* tmp,
                             int maps, long long image_stride, long long planes_stride, hipStream_t s) {
    const long long plane = (long long)ny * nx;
    T* coarse = planes + (long long)(J - 1) * plane;
    // scales 1 .. jt run as tiles, alternating their c_j between tmp and the
    // coarse plane so that c_jt lands in the coarse plane; the later scales
    // run a row and a column pass in place there
    const int jt = bc_tile_scales(J, sizeof(T));
    BcArgs<T> a{};
    a.c_prev = image;
    a.cp_stride = image_stride;
    a.ny = ny; a.nx = nx; a.mode = mode; a.w_stride = planes_stride;
    for (int j = 1; j <= jt; ++j) {
        const bool to_coarse = ((jt - j) & 1) == 0;
        a.d = 1 << (j - 1);
        a.c_next = to_coarse ? coarse : tmp;
        a.cn_stride = to_coarse ? planes_stride : plane;
        a.w = planes + (long long)(j - 1) * plane;
        const hipError_t e = launch_bc_scale<T, false>(a, maps, s);
        if (e != hipSuccess) return e;
        a.c_prev = a.c_next;
        a.cp_stride = a.cn_stride;
    }
    const dim3 grid((nx + 255) / 256, ny, maps);
    for (int j = jt + 1; j < J; ++j) {
        const int d = 1 << (j - 1);
        AMAP_LAUNCH("starlet_bc_row", s,
                    k_bc_row<T><<<grid, 256, 0, s>>>(a.c_prev, tmp, nx, d, mode, a.cp_stride, plane));
        AMAP_LAUNCH("starlet_bc_col", s,
                    k_bc_col<T><<<grid, 256, 0, s>>>(tmp, a.c_prev, planes + (long long)(j - 1) * plane,
                                                     coarse, ny, nx, d, mode, plane, a.cp_stride,
                                                     planes_stride, planes_stride));
        a.c_prev = coarse;
        a.cp_stride = planes_stride;
    }
    return hipGetLastError();
}

// Whether a field's realisations run side by side, their details stored, and
// the statistics are taken in a pass of their own: where a scale's tiles are
// few workgroups per CU, one realisation after the other in a tile takes
// about 3 us each, however small the field.  Seven scales, apart / in the
// tiles, us: 250^2 x 16 realisations (64 tiles) 81 / 277; 500^2 x 16 (256)
// 174 / 317; 940 x 221 x 7 (236) 133 / 202; 700^2 x 16 (484) 371 / 421; 850^2
// x 16 (756) 534 / 491; 1000^2 x 16 (1008) 617 / 516; in double precision 700^2
// 600 / 672, 850^2 858 / 752.
static bool bc_noise_apart(int ny, int nx) {
    return (long long)((nx + 63) / 64) * ((ny + kBcTH - 1) / kBcTH) < 600;
}
int bc_noise_details(int ny, int nx, int J, size_t elem) {
    const int jt = bc_tile_scales(J, elem);
    return bc_noise_apart(ny, nx) ? jt : jt < J - 1 ? 1 : 0;
}

template <typename T>
hipError_t launch_noise_bc(int ny, int nx, int J, int mode, T* kappa, T* tmp, T* row, T* wpl, int nb, int r0,
                           int R, double* M, double* M2, const T* w_signal, T* sigma, T* snr, hipStream_t s) {
    const long long plane = (long long)ny * nx;
    const int jt = bc_tile_scales(J, sizeof(T));
    const bool kept = bc_noise_apart(ny, nx);
    BcArgs<T> a{};
    a.ny = ny; a.nx = nx; a.mode = mode; a.nb = nb; a.r0 = r0; a.R = R;
    a.cp_stride = a.cn_stride = a.w_stride = plane;
    T* cur = kappa;
    T* nxt = tmp;
    const auto stats = [&](int j, int scales) {  // of scales j .. j + scales - 1, their details in wpl
        const long long o = (long long)(j - 1) * plane;
        AMAP_LAUNCH("noise_bc_stats", s,
                    k_bc_stats<T><<<dim3((unsigned)((plane + 255) / 256), scales), 256, 0, s>>>(
                        wpl, plane, nb * plane, nb, r0, R, M + o, M2 + o, w_signal ? w_signal + o : nullptr,
                        sigma + o, snr ? snr + o : nullptr, plane));
    };
    for (int j = 1; j < J; ++j) {
        const long long o = (long long)(j - 1) * plane;
        if (j <= jt) {
            a.d = 1 << (j - 1);
            a.c_prev = cur;
            a.c_next = kept || j + 1 < J ? nxt : nullptr;
            a.w = kept ? wpl + (j - 1) * nb * plane : nullptr;
            a.M = M + o; a.M2 = M2 + o;
            a.w_signal = w_signal ? w_signal + o : nullptr;
            a.sigma = sigma + o;
            a.snr = snr ? snr + o : nullptr;
            const hipError_t e = kept ? launch_bc_scale<T, false>(a, nb, s) : launch_bc_scale<T, true>(a, 1, s);
            if (e != hipSuccess) return e;
            T* t = cur; cur = nxt; nxt = t;
            if (kept && j == jt) stats(1, jt);
            continue;
        }
        // larger dilations: row and column passes in place, then the update
        const int d = 1 << (j - 1);
        const dim3 grid((nx + 255) / 256, ny, nb);
        AMAP_LAUNCH("starlet_bc_row", s, k_bc_row<T><<<grid, 256, 0, s>>>(cur, row, nx, d, mode, plane, plane));
        AMAP_LAUNCH("starlet_bc_col", s,
                    k_bc_col<T><<<grid, 256, 0, s>>>(row, cur, wpl, cur, ny, nx, d, mode, plane, plane, plane,
                                                     plane));
        stats(j, 1);
    }
    return hipGetLastError();
}

template hipError_t launch_noise_bc<float>(int, int, int, int, float*, float*, float*, float*, int, int, int,
                                           double*, double*, const float*, float*, float*, hipStream_t);
template hipError_t launch_noise_bc<double>(int, int, int, int, double*, double*, double*, double*, int, int,
                                            int, double*, double*, const double*, double*, double*, hipStream_t);
template hipError_t launch_starlet_bc<float>(int, int, int, int, const float*, float*, float*, int,
                                             long long, long long, hipStream_t);
template hipError_t launch_starlet_bc<double>(int, int, int, int, const double*, double*, double*, int,
                                              long long, long long, hipStream_t);
}  // namespace amap

// Noise statistics, S/N and peak counts (Sec. 1: sigma from the variance of
// randomised reconstructions, S = M_ap / sigma; Sec. 2.2: peak counts), and
// the Philox phase stream behind the randomisation.
#include "amap_device.h"
#include "amap_launch.h"

namespace amap {

// Index of pixel idx's statistics for scale j under `lay`: for every stage
// on sub-grids that has started by scale j, the pixel's place in the
// current block (the whole plane, then one sub-grid of the stage before)
// goes to that block's sub-grid order for the stage's d.
__device__ __forceinline__ long long stat_index(long long idx, int logn, int j, const StatLayout& lay) {
    long long s = idx;
    int dprev = 0;
    for (int k = 0; k < lay.count && lay.j0[k] <= j; ++k) {
        const int d = lay.j0[k] - 1, lm = logn - dprev;
        const long long mask = (1ll << (2 * lm)) - 1;
        s = (s & ~mask) | subgrid_index(s & mask, lm, d - dprev);
        dprev = d;
    }
    return s;
}

template <typename T>
__global__ void __launch_bounds__(256)
k_noise_finalize(const double* __restrict__ M2, int R, int J, int logn, StatLayout lay,
                 const T* __restrict__ planes_signal, T* __restrict__ sigma, T* __restrict__ snr) {
    const long long n2 = 1ll << (2 * logn);
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n2) return;
    for (int j = 0; j < J - 1; ++j) {
        const long long e = (long long)j * n2 + idx;
        double var = M2[(long long)j * n2 + stat_index(idx, logn, j + 1, lay)] /
                     (double)(R - 1);
        var = var > 0.0 ? var : 0.0;
        const T sg = (T)sqrt(var);
        sigma[e] = sg;
        if (snr) snr[e] = sg > (T)0 ? planes_signal[e] / sg : (T)0;
    }
}

// sigma and S/N of scale blockIdx.y + 1 from the partials of every batch and
// group, merged in order.  A block takes 2^logcp pixels (a row segment, or
// whole rows) and walks them in the order their statistics lie in memory: on
// sub-grids of d, the pixels of one residue mod d after the other, so that a
// wavefront reads runs and not a line per lane; sigma goes through LDS (a
// row padded by one per d pixels, against bank conflicts) into row order for
// the stores.  The merge weights are worked out once per block.  Bound by its
// reads (8 bytes a partial): 4096^2, J = 9, four batches, 1.2 ms; one lane
// per pixel in row order took 3.2.
template <typename T, typename A>
__global__ void __launch_bounds__(256)
k_noise_finalize_parts(const A* __restrict__ part, NoiseParts np, int R, int B, int logn, int logcp,
                       StatLayout lay, const T* __restrict__ planes_signal, T* __restrict__ sigma,
                       T* __restrict__ snr) {
    extern __shared__ __align__(16) unsigned char fin_smem[];
    const long long n2 = 1ll << (2 * logn);
    const int j = blockIdx.y;
    const int G = np.groups[j];
    const int total = (R + B - 1) / B * G;  // partials: batch by batch, group by group
    double* f = reinterpret_cast<double*>(fin_smem);  // nb / nt of each
    double* h = f + total;                            // na nb / nt
    T* sg = reinterpret_cast<T*>(h + total);
    for (int k = threadIdx.x; k < total; k += 256) {
        const int b = k / G, g = k - b * G;
        const int bb = R - b * B < B ? R - b * B : B;
        const int q = bb / G, r = bb - q * G;  // group g holds q (+ 1 if g < r) realisations
        const double nb = (double)(q + (g < r ? 1 : 0)), na = (double)(b * B + g * q + (g < r ? g : r));
        f[k] = nb / (na + nb);  // the first group of a batch is never empty
        h[k] = na * f[k];
    }
    __syncthreads();
    int ld = 0;  // log2 of the scale's sub-grid stride
    for (int k = 0; k < lay.count && lay.j0[k] <= j + 1; ++k) ld = lay.j0[k] - 1;
    const int logwx = logn < logcp ? logn : logcp, logper = logwx - ld;
    const int wx = 1 << logwx, per = 1 << logper, pitch = wx + per;
    const long long px0 = (long long)blockIdx.x << logcp;
    const A* base = part + np.off[j];
    const long long gs = (long long)np.ns[j] * 2 * n2;  // elements per group
    // pixel e of the block in memory order: where its partials lie and where its sigma goes in LDS
    const auto locate = [&](int e, int& at) {
        const int row = e >> logwx, i = e & (wx - 1);
        const int xx = i & (per - 1), x = (i >> logper) + (xx << ld);
        at = row * pitch + x + xx;
        return base + stat_index(px0 + ((long long)row << logwx) + x, logn, j + 1, lay);
    };
    const auto finish = [&](double m2, int at) {
        double var = m2 / (double)(R - 1);
        var = var > 0.0 ? var : 0.0;
        sg[at] = (T)sqrt(var);
    };
    const int npx = 1 << logcp;
    if (total == 1) {
        constexpr int U = 4;  // pixels in flight
        for (int e0 = threadIdx.x; e0 < npx; e0 += U * 256) {
            A v[U];
            int at[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e0 + u * 256 < npx) v[u] = locate(e0 + u * 256, at[u])[n2];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e0 + u * 256 < npx) finish((double)v[u], at[u]);
        }
    } else {
        for (int e0 = threadIdx.x; e0 < npx; e0 += 2 * 256) {
            // two pixels, four partials of each in flight (npx is 256 or even)
            const bool two = e0 + 256 < npx;
            int at[2];
            const A* p[2];
            p[0] = locate(e0, at[0]);
            p[1] = locate(two ? e0 + 256 : e0, at[1]);
            const A* q[2] = {p[0], p[1]};  // partial k, and its batch's first
            double mean[2] = {0.0, 0.0}, m2[2] = {0.0, 0.0};
            int g = 0;
            for (int k0 = 0; k0 < total; k0 += 4) {
                A mb[4][2], qb[4][2];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        if (k0 + u < total) {
                            mb[u][c] = q[c][0];
                            qb[u][c] = q[c][n2];
                        }
                        q[c] += gs;
                    }
                    if (++g == G) {
                        g = 0;
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            p[c] += np.block;
                            q[c] = p[c];
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (k0 + u >= total) continue;
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const double d = (double)mb[u][c] - mean[c];
                        mean[c] += d * f[k0 + u];
                        m2[c] += (double)qb[u][c] + d * d * h[k0 + u];
                    }
                }
            }
            finish(m2[0], at[0]);
            if (two) finish(m2[1], at[1]);
        }
    }
    __syncthreads();
    const long long o = (long long)j * n2 + px0;
    for (int e = threadIdx.x; e < (1 << logcp); e += 256) {
        const int row = e >> logwx, x = e & (wx - 1);
        const T v = sg[row * pitch + x + (x >> ld)];
        sigma[o + e] = v;
        if (snr) snr[o + e] = v > (T)0 ? planes_signal[o + e] / v : (T)0;
    }
}

__global__ void k_zero_i64(long long* p, long long count) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0;
}

// Strict 8-neighbour maxima above thr, periodic.  grid (blocks, nplanes) of
// 1024 threads: each block takes chunks of 4096 pixels of its plane in turn (every thread
// four consecutive pixels of a row, n >= 16, so they share the row) and
// loads a neighbourhood only if one of its pixels is above thr.  The block's
// count gathers in LDS and reaches the plane's counter by one atomic add:
// device-wide adds to one address serialise, so there are few of them.
template <typename T>
__global__ void __launch_bounds__(1024)
k_count_peaks(const T* __restrict__ snr, int logn, double thr, long long* __restrict__ counts) {
    __shared__ unsigned int block_count;
    if (threadIdx.x == 0) block_count = 0u;
    const int n = 1 << logn, m = n - 1;
    const long long n2 = (long long)n * n;
    const T* p = snr + (long long)blockIdx.y * n2;
    unsigned int npk = 0;
    for (long long idx = ((long long)blockIdx.x * 1024 + threadIdx.x) * 4; idx < n2;
         idx += (long long)gridDim.x * 4096) {
        const int x = (int)(idx & m), y = (int)(idx >> logn);
        T r[3][6];  // rows y-1, y, y+1 at columns x-1 .. x+4
#pragma unroll
        for (int i = 0; i < 4; ++i) r[1][1 + i] = p[idx + i];
        bool cand[4], any = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            cand[i] = (double)r[1][1 + i] > thr;
            any = any || cand[i];
        }
        if (!any) continue;
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
            const T* row = p + (long long)((y + dy) & m) * n;
            r[dy + 1][0] = row[(x - 1) & m];
            r[dy + 1][5] = row[(x + 4) & m];
            if (dy != 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) r[dy + 1][1 + i] = row[x + i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const T v = r[1][1 + i];
            bool pk = cand[i];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    if (a != 1 || b != 1) pk = pk & (v > r[a][i + b]);
            npk += pk ? 1u : 0u;
        }
    }
    __syncthreads();  // block_count is zeroed
    if (npk) atomicAdd(&block_count, npk);
    __syncthreads();
    if (threadIdx.x == 0 && block_count)
        atomicAdd((unsigned long long*)&counts[blockIdx.y], (unsigned long long)block_count);
}

// Histogram of peak heights (Sec. 2.2): pixels that are strict 8-neighbour
// maxima of sign*value, periodic, binned by h = sign*value into nbins equal
// bins over [lo, lo + nbins*width); the bin is floor((h - lo) / width) in
// double.  A thread takes four columns of kHistRows rows: it loads their
// window (a 4-vector and two edge values per row) before any test, keeps one
// bit per peak, then bins its peaks one at a time, so a wavefront divides as
// often as its busiest lane has peaks (reading heights again from L1) and
// not once per pixel.  Counts gather in LDS and are added to hist once per
// block and bin; grid (blocks, nplanes), blocks striding over the plane.
// Bound by the loads: six 1024^2 float planes, 40 bins in 11 us (24.5 us with
// nine loads per pixel, one pixel at a time).
constexpr int kHistRows = 8, kHistNT = 256;
template <typename T>
__global__ void __launch_bounds__(kHistNT)
k_peak_hist(const T* __restrict__ planes, int logn, int sign, double lo, double width, int nbins,
            long long* __restrict__ hist) {
    extern __shared__ unsigned int bins[];
    for (int b = threadIdx.x; b < nbins; b += kHistNT) bins[b] = 0u;
    __syncthreads();
    constexpr int K = kHistRows;
    static_assert(4 * K == 32, "one bit per pixel of a thread");
    const int n = 1 << logn, m = n - 1;
    const long long n2 = (long long)n * n;
    const T* p = planes + (long long)blockIdx.y * n2;
    const int lc = logn - 2;                          // log2 vector columns
    const int items = (n / K) << lc;                  // (strip of K rows, vector column)
    for (int it = blockIdx.x * kHistNT + threadIdx.x; it < items; it += gridDim.x * kHistNT) {
        const int x = (it & ((1 << lc) - 1)) * 4, y0 = (it >> lc) * K;
        T r[K + 2][6];  // rows y0 - 1 .. y0 + K at columns x - 1 .. x + 4
#pragma unroll
        for (int a = 0; a < K + 2; ++a) {
            const T* row = p + (long long)((y0 + a - 1) & m) * n;
            r[a][0] = row[(x - 1) & m];
#pragma unroll
            for (int b = 0; b < 4; ++b) r[a][1 + b] = row[x + b];
            r[a][5] = row[(x + 4) & m];
        }
        if (sign < 0) {
#pragma unroll
            for (int a = 0; a < K + 2; ++a)
#pragma unroll
                for (int b = 0; b < 6; ++b) r[a][b] = -r[a][b];
        }
        unsigned int found = 0u;
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const T v = r[a + 1][b + 1];
                bool pk = true;
#pragma unroll
                for (int da = 0; da < 3; ++da)
#pragma unroll
                    for (int db = 0; db < 3; ++db)
                        if (da != 1 || db != 1) pk = pk & (v > r[a + da][b + db]);
                found |= (pk ? 1u : 0u) << (4 * a + b);
            }
        while (found) {
            const int k = __builtin_ctz(found);
            found &= found - 1u;
            const T v = p[(long long)(y0 + (k >> 2)) * n + x + (k & 3)];
            const double b = floor(((double)(sign > 0 ? v : -v) - lo) / width);
            if (b >= 0.0 && b < (double)nbins) atomicAdd(&bins[(int)b], 1u);
        }
    }
    __syncthreads();
    long long* out = hist + (long long)blockIdx.y * nbins;
    for (int b = threadIdx.x; b < nbins; b += kHistNT)
        if (bins[b]) atomicAdd((unsigned long long*)&out[b], (unsigned long long)bins[b]);
}

// ---- plane moments: deterministic two-pass reductions in double -----------------
// Sum of a block's 256 values (fixed order: wave shuffles, then the waves).
__device__ __forceinline__ double block_sum256(double v, double* sh) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    const double t = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return t;
}

// Sum of a plane's nb partials by a block of 256 threads (fixed order).
__device__ __forceinline__ double fold256(const double* __restrict__ part, int nb, double* sh) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) v += part[b];
    return block_sum256(v, sh);
}

// Pass 1: per-block sums of a plane (grid (nb, nplanes)) into part; pass 2
// (CENTRAL): every block folds those nb sums to the plane's mean (they come
// from L2; a launch of their own took 3 us), then its sums of (x - mean)^k, k = 2, 3, 4, into
// cpart [3][nplanes][nb].  Both passes are bound by their reads of the planes.
template <typename T, bool CENTRAL>
__global__ void __launch_bounds__(256)
k_moment_part(const T* __restrict__ planes, long long n2, double* __restrict__ part,
              double* __restrict__ cpart) {
    __shared__ double sh[4];
    constexpr int G = 16 / (int)sizeof(T);  // n2 is a multiple of 256
    typedef T vec __attribute__((ext_vector_type(G)));
    const int pl = blockIdx.y, nb = gridDim.x;
    const vec* p = reinterpret_cast<const vec*>(planes + (long long)pl * n2);
    const long long nv = n2 / G;
    double* mine = part + (long long)pl * nb;
    const long long stride = (long long)nb * 256;
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    // the first vectors are on their way while the mean is folded
    constexpr int U = 4;
    vec v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i + u * stride < nv ? p[i + u * stride] : vec(0);
    const double mu = CENTRAL ? fold256(mine, nb, sh) / (double)n2 : 0.0;
    double s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (;;) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u * stride >= nv) continue;
#pragma unroll
            for (int c = 0; c < G; ++c) {
                const double d = (double)v[u][c] - mu;
                if (CENTRAL) {
                    const double d2 = d * d;
                    s1 += d2;
                    s2 += d2 * d;
                    s3 += d2 * d2;
                } else {
                    s1 += d;
                }
            }
        }
        i += U * stride;
        if (i >= nv) break;
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = i + u * stride < nv ? p[i + u * stride] : vec(0);
    }
    const double t1 = block_sum256(s1, sh);
    if (!CENTRAL) {
        if (threadIdx.x == 0) mine[blockIdx.x] = t1;
        return;
    }
    const double t2 = block_sum256(s2, sh);
    const double t3 = block_sum256(s3, sh);
    if (threadIdx.x == 0) {
        const long long o = (long long)pl * nb + blockIdx.x;
        const long long ps = (long long)gridDim.y * nb;
        cpart[o] = t1;
        cpart[ps + o] = t2;
        cpart[2 * ps + o] = t3;
    }
}

// Folds the nb partials of each plane (one block per plane, fixed order):
// the mean and m2, m3, m4 into out4[4 * plane ...].
__global__ void __launch_bounds__(256)
k_moment_fold(const double* __restrict__ part, const double* __restrict__ cpart, int nb, long long n2,
              double* __restrict__ out4) {
    __shared__ double sh[4];
    const int pl = blockIdx.x, np = gridDim.x;
    const long long stride = (long long)np * nb, o = (long long)pl * nb;
    const double mu = fold256(part + o, nb, sh);
    double mk[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) mk[k] = fold256(cpart + k * stride + o, nb, sh);
    if (threadIdx.x == 0) {
        out4[4 * pl] = mu / (double)n2;
#pragma unroll
        for (int k = 0; k < 3; ++k) out4[4 * pl + 1 + k] = mk[k] / (double)n2;
    }
}

// Thread t writes the eight 32-bit values of Philox block t.
__global__ void __launch_bounds__(256)
k_phase_u32(int logn, uint64_t seed, uint64_t r, uint32_t* __restrict__ out) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long n2 = 1ll << (2 * logn);
    if (8 * t >= n2) return;
    uint32_t u[8];
    philox_block_u32(seed, r, (uint64_t)t, u);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[8 * t + i] = u[i];
}

static unsigned blocks_for(long long count) { return (unsigned)((count + 255) / 256); }
// Blocks per plane for the peak histogram: one per kHistNT items, at most 128
// or, for few planes, enough for 1024 blocks in all (each block adds its
// non-empty bins to the plane's, so there are few of them).
static unsigned hist_blocks(long long n2, int nplanes) {
    const long long items = n2 / (4 * kHistRows);
    long long b = (items + kHistNT - 1) / kHistNT;
    const long long most = 1024 / nplanes > 128 ? 1024 / nplanes : 128;
    return (unsigned)(b > most ? most : b);
}
// Blocks per plane for the peak count: chunks of 4096 pixels, at most 64
// blocks (so at most 64 atomic adds per plane's counter).
static unsigned peak_blocks(long long n2) {
    const long long chunks = (n2 + 4095) / 4096;
    return (unsigned)(chunks < 64 ? chunks : 64);
}

template <typename T>
hipError_t launch_noise_finalize(int logn, int J, int R, const double* M2,
                                 const T* planes_signal, T* sigma, T* snr, hipStream_t s,
                                 const StatLayout& layout) {
    const long long n2 = 1ll << (2 * logn);
    if (layout.count < 0 || layout.count > 16) return hipErrorInvalidValue;
    for (int k = 0; k < layout.count; ++k)  // stage starts inside [1, J), increasing
        if (layout.j0[k] < 1 || layout.j0[k] >= J || (k > 0 && layout.j0[k] <= layout.j0[k - 1]))
            return hipErrorInvalidValue;
    AMAP_LAUNCH("noise_finalize", s,
                k_noise_finalize<T><<<blocks_for(n2), 256, 0, s>>>(M2, R, J, logn, layout,
                                                                   planes_signal, sigma, snr));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_noise_finalize_parts(int logn, int J, int R, int B, const NoiseParts& parts,
                                       const void* part, const T* planes_signal, T* sigma, T* snr,
                                       hipStream_t s, const StatLayout& layout) {
    if (!parts.ok || J - 1 > kMaxScales || B < 1 || layout.count < 0 || layout.count > 16)
        return hipErrorInvalidValue;
    // pixels per block: 2048 (8 per thread), fewer while that leaves the chip
    // short of blocks, 256 at least; a segment holds whole strides of the
    // sub-grids
    int logcp = 11;
    while (logcp > 8 && ((J - 1) << (2 * logn)) >> logcp < 8192) --logcp;
    int ld = 0, most = 0;
    for (int k = 0; k < layout.count; ++k) ld = layout.j0[k] - 1;
    if (logcp < ld) logcp = ld;
    if (logcp > 2 * logn || ld > logn) return hipErrorInvalidValue;
    for (int j = 0; j < J - 1; ++j) most = parts.groups[j] > most ? parts.groups[j] : most;
    const long long total = (long long)((R + B - 1) / B) * most;
    if (total < 1 || total > kMaxMerge) return hipErrorInvalidValue;
    const size_t lds = (size_t)total * 2 * sizeof(double) + (2ull << logcp) * sizeof(T);
    AMAP_LAUNCH("noise_finalize", s,
                k_noise_finalize_parts<T, T><<<dim3(1u << (2 * logn - logcp), J - 1), 256, lds, s>>>(
                    static_cast<const T*>(part), parts, R, B, logn, logcp, layout, planes_signal, sigma, snr));
    return hipGetLastError();
}

hipError_t launch_zero_i64(long long* p, long long count, hipStream_t s) {
    if (count > 0) AMAP_LAUNCH("zero", s, k_zero_i64<<<blocks_for(count), 256, 0, s>>>(p, count));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_count_peaks(int logn, int nplanes, const T* snr, double thr, long long* counts,
                              hipStream_t s) {
    const long long n2 = 1ll << (2 * logn);
    hipError_t e = launch_zero_i64(counts, nplanes, s);
    if (e != hipSuccess) return e;
    AMAP_LAUNCH("count_peaks", s,
                k_count_peaks<T><<<dim3(peak_blocks(n2), nplanes), 1024, 0, s>>>(snr, logn, thr, counts));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_peak_hist(int logn, int nplanes, const T* planes, int sign, double lo,
                            double width, int nbins, long long* hist, hipStream_t s) {
    const long long n2 = 1ll << (2 * logn);
    hipError_t e = launch_zero_i64(hist, (long long)nplanes * nbins, s);
    if (e != hipSuccess) return e;
    AMAP_LAUNCH("peak_hist", s,
                k_peak_hist<T><<<dim3(hist_blocks(n2, nplanes), nplanes), kHistNT, nbins * sizeof(unsigned int), s>>>(
                    planes, logn, sign, lo, width, nbins, hist));
    return hipGetLastError();
}

int moment_blocks(int logn) {
    const long long n2 = 1ll << (2 * logn);
    const long long nb = n2 / (256 * 16);  // sixteen values per thread or more
    return (int)(nb < 1 ? 1 : (nb > 256 ? 256 : nb));  // few enough blocks to run at once
}

template <typename T>
hipError_t launch_plane_moments(int logn, int nplanes, const T* planes, double* part, double* out4,
                                hipStream_t s) {
    const long long n2 = 1ll << (2 * logn);
    const int nb = moment_blocks(logn);
    double* cpart = part + (long long)nplanes * nb;
    AMAP_LAUNCH("moments_mean", s,
                k_moment_part<T, false><<<dim3(nb, nplanes), 256, 0, s>>>(planes, n2, part, cpart));
    AMAP_LAUNCH("moments_central", s,
                k_moment_part<T, true><<<dim3(nb, nplanes), 256, 0, s>>>(planes, n2, part, cpart));
    AMAP_LAUNCH("moments_fold", s, k_moment_fold<<<nplanes, 256, 0, s>>>(part, cpart, nb, n2, out4));
    return hipGetLastError();
}

hipError_t launch_phase_u32(int logn, uint64_t seed, uint64_t r, uint32_t* out, hipStream_t s) {
    const long long n2 = 1ll << (2 * logn);
    AMAP_LAUNCH("phase_u32", s, k_phase_u32<<<blocks_for(n2 / 8), 256, 0, s>>>(logn, seed, r, out));
    return hipGetLastError();
}

template hipError_t launch_noise_finalize<float>(int, int, int, const double*, const float*, float*,
                                                 float*, hipStream_t, const StatLayout&);
template hipError_t launch_noise_finalize<double>(int, int, int, const double*, const double*,
                                                  double*, double*, hipStream_t, const StatLayout&);
template hipError_t launch_noise_finalize_parts<float>(int, int, int, int, const NoiseParts&, const void*,
                                                       const float*, float*, float*, hipStream_t,
                                                       const StatLayout&);
template hipError_t launch_noise_finalize_parts<double>(int, int, int, int, const NoiseParts&, const void*,
                                                        const double*, double*, double*, hipStream_t,
                                                        const StatLayout&);
template hipError_t launch_count_peaks<float>(int, int, const float*, double, long long*, hipStream_t);
template hipError_t launch_count_peaks<double>(int, int, const double*, double, long long*, hipStream_t);
template hipError_t launch_peak_hist<float>(int, int, const float*, int, double, double, int, long long*,
                                            hipStream_t);
template hipError_t launch_peak_hist<double>(int, int, const double*, int, double, double, int,
                                             long long*, hipStream_t);
template hipError_t launch_plane_moments<float>(int, int, const float*, double*, double*, hipStream_t);
template hipError_t launch_plane_moments<double>(int, int, const double*, double*, double*, hipStream_t);

}  // namespace amap

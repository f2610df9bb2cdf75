// Small utility kernels: fills, copies with pinned-slot masking, model statistics
// (deterministic two-stage reduction) and the non-finite check.
#pragma once

#include "common.h"

namespace fd3d {

constexpr int kReduceBlocks = 512;
constexpr int kReduceThreads = 256;
constexpr int kStats = 6;  // vp_max, vs_min(mu>0), rho_min, mu_min, m2_min, bad

template <typename T>
__global__ void __launch_bounds__(256) fill_zero(T *__restrict__ p, long n)
{
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x)
        p[q] = T(0);
}

// dst = src for up to nine field-shaped arrays, 0 at the pinned slots of components with half
// offsets (sx, sy, sz) (all 0: a plain copy).  Each side has its own row and plane strides (a
// node array: nx, nx ny; a field of the interleaved-rows layout: 9 nx, 9 nx ny).  One launch,
// blockIdx.y the array; V samples (16 bytes where the rows allow it) per access and 32-bit
// index arithmetic: the nine fields of 256^3 rows, FP32, 220 us (5.5 TB/s) against 608 us in nine
// launches of one sample per access and 64-bit divisions, whose arithmetic bounded it.
template <typename T> struct FieldCopy {
    T *dst;
    const T *src;
    int sx, sy, sz;
};
template <typename T> struct FieldCopies {
    FieldCopy<T> f[9];
    long dsy, dsz, ssy, ssz;
    int nx, ny, nz;
};

template <typename T, int V> __global__ void __launch_bounds__(256) copy_fields(FieldCopies<T> a)
{
    typedef T vec __attribute__((ext_vector_type(V)));
    const FieldCopy<T> f = a.f[blockIdx.y];
    const unsigned per = (unsigned)a.nx / V, n = per * (unsigned)a.ny * (unsigned)a.nz;
    for (unsigned q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const unsigned row = q / per, c = q - row * per, k = row / (unsigned)a.ny, j = row - k * (unsigned)a.ny;
        vec v = *(const vec *)(f.src + (V * c + a.ssy * j + a.ssz * k));
        if ((int)j > a.ny - 1 - f.sy || (int)k > a.nz - 1 - f.sz) v = vec(T(0));
        if (f.sx && c == per - 1) v[V - 1] = T(0);
        *(vec *)(f.dst + (V * c + a.dsy * j + a.dsz * k)) = v;
    }
}

// Contiguous copy of n 16-byte words (checkpoints).
static __global__ void __launch_bounds__(256) copy_block(float4 *__restrict__ dst, const float4 *__restrict__ src, long n)
{
    for (long q = blockIdx.x * 256L + threadIdx.x; q < n; q += (long)gridDim.x * 256) dst[q] = src[q];
}

// Zero at the pinned slots of the velocity components stored in the slots of a segment: slot m
// holds its components in the three arrays from seg + (m / 3) group + 3 (m mod 3) fstep (bytes).
// The rest of a slot is written before it is read, so nothing else needs a fill (the whole
// segment's took 0.8 of the 62 ms of a 40-step gradient at 256^3).
template <typename T>
__global__ void __launch_bounds__(256) zero_pinned(char *seg, size_t group, size_t fstep, int nx, int ny, int nz, long sy, long sz)
{
    const int m = blockIdx.y / 3, c = blockIdx.y % 3;
    T *f = (T *)(seg + (size_t)(m / 3) * group + (size_t)(3 * (m % 3) + c) * fstep);
    const int na = c == 0 ? ny : nx, nb = c == 2 ? ny : nz;  // the two other axes
    for (int q = blockIdx.x * 256 + threadIdx.x; q < na * nb; q += gridDim.x * 256) {
        const int b = q / na, a = q - b * na;
        const long at = c == 0 ? (nx - 1) + sy * a + sz * b : (c == 1 ? a + sy * (ny - 1) + sz * b : a + sy * b + sz * (nz - 1));
        f[at] = T(0);
    }
}

// Medium given on a coarse node grid c[mz][my][mx], sampled trilinearly at every node of
// the simulation grid f[nz][ny][nx] (Sec. 2.2.1); both grids span the same box, so node i
// sits at coarse coordinate i (m - 1) / (n - 1).  Weights and sums in double.
__device__ __forceinline__ void coarse_axis(int i, int n, int m, int &lo, int &hi, double &t)
{
    const double q = n > 1 ? i * ((double)(m - 1) / (double)(n - 1)) : 0.0;
    lo = (int)floor(q);
    lo = lo < m - 2 ? lo : (m - 2 > 0 ? m - 2 : 0);
    hi = lo + 1 < m - 1 ? lo + 1 : m - 1;
    t = q - lo;
}

template <typename T>
__global__ void __launch_bounds__(256) upsample_trilinear(const T *__restrict__ c, int mx, int my, int mz,
                                                          T *__restrict__ f, int nx, int ny, int nz)
{
    const long n = (long)nx * ny * nz;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x) {
        const int i = (int)(q % nx);
        const int j = (int)((q / nx) % ny);
        const int k = (int)(q / ((long)nx * ny));
        int x0, x1, y0, y1, z0, z1;
        double tx, ty, tz;
        coarse_axis(i, nx, mx, x0, x1, tx);
        coarse_axis(j, ny, my, y0, y1, ty);
        coarse_axis(k, nz, mz, z0, z1, tz);
        const int zs[2] = {z0, z1}, ys[2] = {y0, y1}, xs[2] = {x0, x1};
        const double wz[2] = {1.0 - tz, tz}, wy[2] = {1.0 - ty, ty}, wx[2] = {1.0 - tx, tx};
        double v = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b)
                for (int d = 0; d < 2; ++d)
                    v += wz[a] * wy[b] * wx[d] * (double)c[xs[d] + (long)mx * (ys[b] + (long)my * zs[a])];
        f[q] = (T)v;
    }
}

__device__ __forceinline__ double dmin(double a, double b) { return a < b ? a : b; }
__device__ __forceinline__ double dmax(double a, double b) { return a > b ? a : b; }

// Per-block partial statistics of the model, written to part[block][kStats].
template <typename T>
__global__ void __launch_bounds__(kReduceThreads) model_stats(const T *__restrict__ lam, const T *__restrict__ mu,
                                                              const T *__restrict__ rho, long n, double *__restrict__ part)
{
    __shared__ double sh[kStats][kReduceThreads];
    double vpmax = 0.0, vsmin = 1e300, rmin = 1e300, mmin = 1e300, m2min = 1e300, bad = 0.0;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x) {
        const double l = (double)lam[q], m = (double)mu[q], r = (double)rho[q];
        if (!isfinite(l) || !isfinite(m) || !isfinite(r)) { bad = 1.0; continue; }
        rmin = dmin(rmin, r);
        mmin = dmin(mmin, m);
        m2min = dmin(m2min, l + 2.0 * m);
        if (r > 0.0 && l + 2.0 * m > 0.0) vpmax = dmax(vpmax, sqrt((l + 2.0 * m) / r));
        if (r > 0.0 && m > 0.0) vsmin = dmin(vsmin, sqrt(m / r));
    }
    const int t = threadIdx.x;
    sh[0][t] = vpmax; sh[1][t] = vsmin; sh[2][t] = rmin; sh[3][t] = mmin; sh[4][t] = m2min; sh[5][t] = bad;
    __syncthreads();
    for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
        if (t < w) {
            sh[0][t] = dmax(sh[0][t], sh[0][t + w]);
            for (int s = 1; s < 5; ++s) sh[s][t] = dmin(sh[s][t], sh[s][t + w]);
            sh[5][t] = dmax(sh[5][t], sh[5][t + w]);
        }
        __syncthreads();
    }
    if (t < kStats) part[blockIdx.x * kStats + t] = sh[t][0];
}

// Combines the partials, a statistic per wave-sized group of threads (one thread that read
// them all in turn took 140 us).
static __global__ void __launch_bounds__(kStats * 64) stats_final(const double *__restrict__ part, int nblocks,
                                                                  double *__restrict__ out)
{
    const int s = threadIdx.x / 64, lane = threadIdx.x % 64;
    const bool top = s == 0 || s == 5;  // vp_max and bad are maxima, the others minima
    double r = top ? 0.0 : 1e300;
    for (int b = lane; b < nblocks; b += 64) {
        const double v = part[b * kStats + s];
        r = top ? dmax(r, v) : dmin(r, v);
    }
    for (int w = 32; w > 0; w >>= 1) {
        const double v = __shfl_down(r, w);
        r = top ? dmax(r, v) : dmin(r, v);
    }
    if (lane == 0) out[s] = r;
}

// flag[0] = 1 if any of the nine fields holds a non-finite value (written only then).
template <typename T>
__global__ void __launch_bounds__(256) finite_check(Grid<T> G, int *__restrict__ flag)
{
    const long n = (long)G.nx * G.ny * G.nz;
    bool bad = false;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x) {
        const int i = (int)(q % G.nx);
        const int j = (int)((q / G.nx) % G.ny);
        const int k = (int)(q / ((long)G.nx * G.ny));
        const long p = i + G.sy * j + G.sz * k;
        for (int c = 0; c < NFIELD; ++c) bad |= !isfinite(G.f[c][p]);
    }
    if (bad) flag[0] = 1;
}

} // namespace fd3d

// Row kernels: one thread per cell, one row of cells per wave, every neighbour straight from
// global memory (no LDS plane, barrier or z sweep).  The passes of the cell variant, and of
// the default choice on grids whose working set stays in the Infinity Cache.
//
// What bounds them.  On small grids a SIMD holds only a few waves and a pass lasts as long as
// one wave's chain of dependent steps, so the chain is kept short: a wave's row j and plane k
// are uniform, so row and plane offsets (and whether they lie in the grid) are scalar, the
// lane adds its column, and a sample outside the grid reads 0 through the buffer descriptor's
// range check; no load sits behind a branch, and all loads of a cell are in flight together.
// On grids of some million cells the fabric behind the L2s bounds them: neighbouring rows and
// planes are dealt to one XCD in an order that keeps them in its L2, and the L2s then miss the
// compulsory bytes only (42 + 12 B per cell in the velocity pass and 46 + 24 in the stress pass
// at 128^3, FP32, by the counters, of 40 + 12 and 44 + 24).
// Grids larger than the cache belong to the tile sweeps, whose long streams HBM serves
// faster.  Forward step (both passes, receivers included), FP32, MI355X, us, against the best
// tile sweep and the one-thread-per-cell kernels with a bounds test per load (vel_cell):
//   grid             rows    tile sweep   vel_cell / stress_cell
//   32^3              6.9       14.5        15.1
//   64^3             10.3       19.5        19.4
//   149 x 101 x 87   31.0       40.7        73.9
//   128^3            35.9       45.7        69.8   (7.0 TB/s of 120 B per cell)
//   192 x 192 x 128  88.7       94.3
//   256^3           448        364
#pragma once

#include "fwd_tile.h"

namespace fd3d {

// Work of a row launch: blocks of 256 threads, 1 << lbx (64, 128 or 256) columns by 256 >> lbx
// rows of one plane.  The grid is cut into ns strips of rps row blocks along y and nslab slabs
// of np planes along z; a piece (strip of a slab) is walked plane by plane.  Each of the 8 XCDs
// takes the cpx pieces [x cpx, (x + 1) cpx), one after the other.
struct RowMap {
    int ntx;  // column blocks
    int lbx;
    int rps;
    int ns, nslab, np, cpx;

    // blocks of one plane of a piece, and planes of an XCD's pieces
    __host__ __device__ int tiles() const { return rps * ntx; }
    __host__ __device__ int planes() const { return np * cpx; }
};

// Cell of a lane; row and plane are uniform over its wave.  k = nz: no work.
struct RowPos {
    int i, j, k;
};

// Cell of a lane in block y of plane k of a strip.
__device__ __forceinline__ RowPos row_cell(const RowMap &rm, int strip, int y, int k)
{
    int tx = 0;
    if (rm.ntx > 1) {
        tx = y % rm.ntx;
        y /= rm.ntx;
    }
    const int t = threadIdx.x;
    const int row = __builtin_amdgcn_readfirstlane(t >> rm.lbx);
    return {(tx << rm.lbx) + (t & ((1 << rm.lbx) - 1)), (strip * rm.rps + y) * (256 >> rm.lbx) + row, k};
}

// Block (x, y, z) of a launch: XCD x, block y of a plane, plane z of the XCD's pieces
// (reverse: from the last).
__device__ __forceinline__ RowPos row_pos(const RowMap &rm, int nz, int x, int y, int z, bool reverse)
{
    int piece = x * rm.cpx;
    if (reverse) z = rm.planes() - 1 - z;
    if (rm.cpx > 1) {
        const int c = z / rm.np;
        z -= c * rm.np;
        piece += c;
    }
    int strip = piece, slab = 0;
    if (rm.nslab > 1) {
        slab = rm.ns > 1 ? piece / rm.ns : piece;
        strip = piece - slab * rm.ns;
    }
    return row_cell(rm, strip, y, strip < rm.ns && slab < rm.nslab ? slab * rm.np + z : nz);
}

// Byte offsets of a wave's samples in the window of its plane: column i + d (per lane), row
// j + a and plane k + c (uniform).  Columns outside the grid get kOOB, rows and planes kSkip
// (see Window): an offset with any of them is out of range.  Lanes past the last column leave at
// once (they may wrap into the window): their loads took as long as the others' (149 x 101 x 87:
// 34.0 us a step with them, 32.2 without; 330 x 70 x 60: 33.1 and 32.3; no change at 128^3).
template <typename T> struct RowOffsets {
    Window w;
    int i, j, k, nx, ny, nz;
    unsigned rb;  // bytes per row

    __device__ __forceinline__ RowOffsets(const Grid<T> &G, const RowPos &p)
        : w(window<T>(p.k, p.k + 1, G.nz, G.sz)), i(p.i), j(p.j), k(p.k), nx(G.nx), ny(G.ny), nz(G.nz),
          rb((unsigned)G.sy * (unsigned)sizeof(T))
    {
    }
    __device__ __forceinline__ unsigned operator()(int d, int a, int c) const
    {
        const unsigned x = (unsigned)(i + d), y = (unsigned)(j + a), z = (unsigned)(k + c);
        const unsigned row = (y < (unsigned)ny ? y * rb : kSkip) + (z < (unsigned)nz ? (z - (unsigned)w.b0) * w.pb : kSkip);
        return (x < (unsigned)nx ? x * (unsigned)sizeof(T) : kOOB) + row;
    }
    __device__ __forceinline__ T get(rsrc_t f, int d, int a, int c) const { return ld<T>(f, (*this)(d, a, c)); }
    // z neighbour c of a stress sample; with the free surface the samples above k = 0 are odd
    // images (HALF: SXZ, SYZ, -f[-1 - k]; else SZZ, -f[-k])
    template <bool FS, bool HALF> __device__ __forceinline__ T getz(rsrc_t f, int c) const
    {
        const int kk = k + c;
        if (FS && kk < 0) return -get(f, 0, 0, (HALF ? -1 - kk : -kk) - k);
        return get(f, 0, 0, c);
    }
};

// Stress samples around a cell that the divergences of the velocity pass take.
template <typename T> struct SigmaTaps {
    T xx0, xxp1, xxp2, xxm1;
    T xy0, xyym1, xyyp1, xyym2, xyxm1, xyxp1, xyxm2;
    T yy0, yyp1, yyp2, yym1;
    T xz0, xzxm1, xzxp1, xzxm2, xzm1, xzp1, xzm2;
    T yz0, yzym1, yzyp1, yzym2, yzm1, yzp1, yzm2;
    T zz0, zzp1, zzp2, zzm1;
};

// s: the six stress fields (xx, yy, zz, xy, xz, yz).
template <bool FS, typename T>
__device__ __forceinline__ SigmaTaps<T> load_sigma(const T *const *s, const RowOffsets<T> &o)
{
    const rsrc_t xx = wfield(s[0], o.w), yy = wfield(s[1], o.w), zz = wfield(s[2], o.w);
    const rsrc_t xy = wfield(s[3], o.w), xz = wfield(s[4], o.w), yz = wfield(s[5], o.w);
    SigmaTaps<T> t;
    t.xx0 = o.get(xx, 0, 0, 0); t.xxp1 = o.get(xx, 1, 0, 0); t.xxp2 = o.get(xx, 2, 0, 0); t.xxm1 = o.get(xx, -1, 0, 0);
    t.xy0 = o.get(xy, 0, 0, 0); t.xyym1 = o.get(xy, 0, -1, 0); t.xyyp1 = o.get(xy, 0, 1, 0); t.xyym2 = o.get(xy, 0, -2, 0);
    t.xyxm1 = o.get(xy, -1, 0, 0); t.xyxp1 = o.get(xy, 1, 0, 0); t.xyxm2 = o.get(xy, -2, 0, 0);
    t.yy0 = o.get(yy, 0, 0, 0); t.yyp1 = o.get(yy, 0, 1, 0); t.yyp2 = o.get(yy, 0, 2, 0); t.yym1 = o.get(yy, 0, -1, 0);
    t.xz0 = o.get(xz, 0, 0, 0); t.xzxm1 = o.get(xz, -1, 0, 0); t.xzxp1 = o.get(xz, 1, 0, 0); t.xzxm2 = o.get(xz, -2, 0, 0);
    t.yz0 = o.get(yz, 0, 0, 0); t.yzym1 = o.get(yz, 0, -1, 0); t.yzyp1 = o.get(yz, 0, 1, 0); t.yzym2 = o.get(yz, 0, -2, 0);
    t.xzm1 = o.template getz<FS, true>(xz, -1); t.xzp1 = o.template getz<FS, true>(xz, 1); t.xzm2 = o.template getz<FS, true>(xz, -2);
    t.yzm1 = o.template getz<FS, true>(yz, -1); t.yzp1 = o.template getz<FS, true>(yz, 1); t.yzm2 = o.template getz<FS, true>(yz, -2);
    t.zz0 = o.get(zz, 0, 0, 0); t.zzp1 = o.template getz<FS, false>(zz, 1);
    t.zzp2 = o.template getz<FS, false>(zz, 2); t.zzm1 = o.template getz<FS, false>(zz, -1);
    return t;
}

// Divergences of the stress at the three velocity samples (o2: second order along z).
template <typename T>
__device__ __forceinline__ void divergence(const SigmaTaps<T> &t, const bool o2[3], T rdx, T rdy, T rdz, T d[3])
{
    d[0] = dstag(t.xxp1, t.xx0, t.xxp2, t.xxm1, rdx) + dstag(t.xy0, t.xyym1, t.xyyp1, t.xyym2, rdy)
         + dz_or_o2(o2[0], t.xz0, t.xzm1, t.xzp1, t.xzm2, rdz);
    d[1] = dstag(t.xy0, t.xyxm1, t.xyxp1, t.xyxm2, rdx) + dstag(t.yyp1, t.yy0, t.yyp2, t.yym1, rdy)
         + dz_or_o2(o2[1], t.yz0, t.yzm1, t.yzp1, t.yzm2, rdz);
    d[2] = dstag(t.xz0, t.xzxm1, t.xzxp1, t.xzxm2, rdx) + dstag(t.yz0, t.yzym1, t.yzyp1, t.yzym2, rdy)
         + dz_or_o2(o2[2], t.zzp1, t.zz0, t.zzp2, t.zzm1, rdz);
}

// Velocity samples around a cell that the strain rates of the stress pass take.
template <typename T> struct VelTaps {
    T x0, xm1, xp1, xm2, xyp1, xyp2, xym1, xzp1, xzp2, xzm1;
    T y0, ym1, yp1, ym2, yxp1, yxp2, yxm1, yzp1, yzp2, yzm1;
    T z0, zm1, zp1, zm2, zxp1, zxp2, zxm1, zyp1, zyp2, zym1;
};

template <typename T> __device__ __forceinline__ VelTaps<T> load_velocity(const T *const *v, const RowOffsets<T> &o)
{
    const rsrc_t vx = wfield(v[0], o.w), vy = wfield(v[1], o.w), vz = wfield(v[2], o.w);
    VelTaps<T> t;
    t.x0 = o.get(vx, 0, 0, 0); t.xm1 = o.get(vx, -1, 0, 0); t.xp1 = o.get(vx, 1, 0, 0); t.xm2 = o.get(vx, -2, 0, 0);
    t.xyp1 = o.get(vx, 0, 1, 0); t.xyp2 = o.get(vx, 0, 2, 0); t.xym1 = o.get(vx, 0, -1, 0);
    t.xzp1 = o.get(vx, 0, 0, 1); t.xzp2 = o.get(vx, 0, 0, 2); t.xzm1 = o.get(vx, 0, 0, -1);
    t.y0 = o.get(vy, 0, 0, 0); t.ym1 = o.get(vy, 0, -1, 0); t.yp1 = o.get(vy, 0, 1, 0); t.ym2 = o.get(vy, 0, -2, 0);
    t.yxp1 = o.get(vy, 1, 0, 0); t.yxp2 = o.get(vy, 2, 0, 0); t.yxm1 = o.get(vy, -1, 0, 0);
    t.yzp1 = o.get(vy, 0, 0, 1); t.yzp2 = o.get(vy, 0, 0, 2); t.yzm1 = o.get(vy, 0, 0, -1);
    t.z0 = o.get(vz, 0, 0, 0); t.zm1 = o.get(vz, 0, 0, -1); t.zp1 = o.get(vz, 0, 0, 1); t.zm2 = o.get(vz, 0, 0, -2);
    t.zxp1 = o.get(vz, 1, 0, 0); t.zxp2 = o.get(vz, 2, 0, 0); t.zxm1 = o.get(vz, -1, 0, 0);
    t.zyp1 = o.get(vz, 0, 1, 0); t.zyp2 = o.get(vz, 0, 2, 0); t.zym1 = o.get(vz, 0, -1, 0);
    return t;
}

template <typename T> struct Strain {
    T xx, yy, zz, xy, xz, yz;
};

// Strain rates; l, m: lambda and mu of the node (free surface only).
template <bool FS, bool VAC, typename T>
__device__ __forceinline__ Strain<T> strain(const VelTaps<T> &t, const Grid<T> &G, const SurfacePlanes &sp, int k, T l, T m)
{
    const T rdx = G.rdx, rdy = G.rdy, rdz = G.rdz;
    Strain<T> e;
    e.xx = dstag(t.x0, t.xm1, t.xp1, t.xm2, rdx);
    e.yy = dstag(t.y0, t.ym1, t.yp1, t.ym2, rdy);
    if (FS && k == 0) e.zz = -l / (l + T(2) * m) * (e.xx + e.yy);
    else if (FS && k == 1) e.zz = (t.z0 - t.zm1) * rdz;
    else e.zz = dz_or_o2(VAC && o2_int(sp.n, k), t.z0, t.zm1, t.zp1, t.zm2, rdz);
    e.xy = dstag(t.xyp1, t.x0, t.xyp2, t.xym1, rdy) + dstag(t.yxp1, t.y0, t.yxp2, t.yxm1, rdx);
    const T dzvx = dz_or_o2((FS && k == 0) || (VAC && o2_half(sp.x, k)), t.xzp1, t.x0, t.xzp2, t.xzm1, rdz);
    e.xz = dzvx + dstag(t.zxp1, t.z0, t.zxp2, t.zxm1, rdx);
    const T dzvy = dz_or_o2((FS && k == 0) || (VAC && o2_half(sp.y, k)), t.yzp1, t.y0, t.yzp2, t.yzm1, rdz);
    e.yz = dzvy + dstag(t.zyp1, t.z0, t.zyp2, t.zym1, rdy);
    return e;
}

// mu (or its perturbation) at a node and its means at the three shear points beside it.
template <typename T> struct ShearMeans {
    T m, xy, xz, yz;
};

template <typename T> __device__ __forceinline__ ShearMeans<T> shear_means(const T *mu, const RowOffsets<T> &o)
{
    const rsrc_t f = wfield(mu, o.w);
    const T m = o.get(f, 0, 0, 0), mx = o.get(f, 1, 0, 0), my = o.get(f, 0, 1, 0), mxy = o.get(f, 1, 1, 0);
    const T mz = o.get(f, 0, 0, 1), mxz = o.get(f, 1, 0, 1), myz = o.get(f, 0, 1, 1);
    return {m, ((m + mx) + (my + mxy)) / T(4), ((m + mx) + (mz + mxz)) / T(4), ((m + my) + (mz + myz)) / T(4)};
}

// Damping factors of a lane's column, row and plane at integer and half positions.
template <typename T> struct Damping {
    T xi, xh, yi, yh, zi, zh;

    __device__ __forceinline__ Damping(const Grid<T> &G, const RowPos &p)
    {
        xi = G.g[0][0][p.i];
        xh = G.g[0][1][p.i];
        yi = sload(G.g[1][0], p.j);
        yh = sload(G.g[1][1], p.j);
        zi = sload(G.g[2][0], p.k);
        zh = sload(G.g[2][1], p.k);
    }
};

// Whether the wave's row holds a tap of source component comp (uniform).
template <typename T> __device__ __forceinline__ bool row_has_tap(const Inject<T> &s, int comp, const RowPos &p)
{
    return (unsigned)(p.j - s.j0[comp]) < 2u && (unsigned)(p.k - s.k0[comp]) < 2u;
}

// (V) at a lane's cell, same arithmetic per sample as vel_tile_body; modes kFwd, kFwdSave,
// kAdjA, kBornV.
template <typename T, bool FS, int MODE, bool VAC>
__device__ __forceinline__ void vel_row_body(const Grid<T> &G, const Inject<T> &src, int n, const RowPos &p,
                                             const TileIO<T> &io)
{
    constexpr bool born = MODE == kBornV, adj = MODE == kAdjA;
    if (p.k >= G.nz || p.j >= G.ny || p.i >= G.nx) return;
    const RowOffsets<T> o(G, p);
    const unsigned own = o(0, 0, 0);
    const SigmaTaps<T> t = load_sigma<FS, T>(G.f + SXX, o);
    SigmaTaps<T> q;
    if constexpr (born) q = load_sigma<false, T>(io.pin, o);
    const rsrc_t rho = wfield(G.rho, o.w);
    const T r0 = ld<T>(rho, own), rb[3] = {o.get(rho, 1, 0, 0), o.get(rho, 0, 1, 0), o.get(rho, 0, 0, 1)};
    T e0 = T(0), eb[3] = {}, v0[3], w0[3] = {}, s0[3] = {}, g0[3] = {};
    if constexpr (born) {
        const rsrc_t dr = wfield(io.acc[0], o.w);
        e0 = ld<T>(dr, own);
        eb[0] = o.get(dr, 1, 0, 0);
        eb[1] = o.get(dr, 0, 1, 0);
        eb[2] = o.get(dr, 0, 0, 1);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v0[c] = ld<T>(wfield(G.f[VX + c], o.w), own);
        if constexpr (born) w0[c] = ld<T>(wfield(io.out[c], o.w), own);
        if constexpr (adj) {
            s0[c] = ld<T>(wfield(io.vst[c], o.w), own);
            g0[c] = ld<T>(wfield(io.acc[c], o.w), own);
        }
    }
    const Damping<T> D(G, p);
    const SurfacePlanes sp = VAC ? surface_planes(G, p.i, p.j) : SurfacePlanes{0, 0, 0};
    const T dt = G.dt;
    const bool o2[3] = {VAC && o2_int(sp.x, p.k), VAC && o2_int(sp.y, p.k), VAC && o2_half(sp.n, p.k)};
    const bool none[3] = {false, false, false};
    T d[3], pd[3];
    divergence(t, o2, G.rdx, G.rdy, G.rdz, d);
    if constexpr (born) divergence(q, none, G.rdx, G.rdy, G.rdz, pd);
    const bool taps = !adj && src.on &&
                      (row_has_tap(src, VX, p) || row_has_tap(src, VY, p) || row_has_tap(src, VZ, p));
    const T s = taps ? sload(src.wavelet, n) : T(0);
    const T g[3] = {D.xh * D.yi * D.zi, D.xi * D.yh * D.zi, D.xi * D.yi * D.zh};
    const unsigned so[3] = {p.i <= G.nx - 2 ? own : kOOB, p.j <= G.ny - 2 ? own : kOOB, p.k <= G.nz - 2 ? own : kOOB};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if constexpr (adj) {
            const T re = (r0 + rb[c]) * T(0.5);
            const T dd = dt * d[c];
            st(wfield(G.f[VX + c], o.w), so[c], (g[c] * (v0[c] * re - dd)) * buoy(r0, rb[c]));
            st(wfield(io.acc[c], o.w), so[c], g0[c] - (s0[c] * re) * dd);
        } else {
            const T b = buoy(r0, rb[c]);
            T cf = T(0);
            if (taps) cf = coef_of(src, VX + c, tap_of(src, VX + c, p.i, p.j, p.k));
            T v = v0[c] + dt * b * d[c];
            if (taps) v += b * cf * s;
            v = v * g[c];
            st(wfield(MODE == kFwdSave ? G.save[VX + c] : G.f[VX + c], o.w), so[c], v);
            if constexpr (born) {  // the source term, then the perturbation's own update
                const T db = -(b * b) * ((e0 + eb[c]) * T(0.5));
                T add = dt * db * d[c];
                if (taps) add += db * cf * s;
                const T pv = w0[c] + add;
                const T w = pv + dt * b * pd[c];
                st(wfield(io.out[c], o.w), so[c], w * g[c]);
            }
        }
    }
}

// (S) at a lane's cell, same arithmetic per sample as stress_tile_body; modes kFwd, kAdjM,
// kAdjB, kBornS.
template <typename T, bool FS, int MODE, bool VAC>
__device__ __forceinline__ void stress_row_body(const Grid<T> &G, const Inject<T> &src, int n, const RowPos &p,
                                                const TileIO<T> &io)
{
    constexpr bool born = MODE == kBornS, adjm = MODE == kAdjM, adjb = MODE == kAdjB;
    if (p.k >= G.nz || p.j >= G.ny || p.i >= G.nx) return;
    const RowOffsets<T> o(G, p);
    const unsigned own = o(0, 0, 0);
    const VelTaps<T> t = load_velocity<T>(G.f + VX, o);
    VelTaps<T> q;
    if constexpr (born) q = load_velocity<T>(io.pin, o);
    if constexpr (adjm) q = load_velocity<T>(io.y, o);
    T s0[6], b0[6] = {}, a0[5] = {};
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        s0[c] = ld<T>(wfield(G.f[SXX + c], o.w), own);
        if constexpr (born) b0[c] = ld<T>(wfield(io.out[c], o.w), own);
        if (adjm && c < 5) a0[c < 5 ? c : 0] = ld<T>(wfield(io.acc[c < 5 ? c : 0], o.w), own);
    }
    T l = T(0), dl = T(0);
    ShearMeans<T> m{}, dm{};
    if constexpr (!adjb) {
        l = ld<T>(wfield(G.lam, o.w), own);
        m = shear_means<T>(G.mu, o);
    }
    if constexpr (born) {
        dl = ld<T>(wfield(io.acc[0], o.w), own);
        dm = shear_means<T>(io.acc[1], o);
    }
    const Damping<T> D(G, p);
    const SurfacePlanes sp = VAC ? surface_planes(G, p.i, p.j) : SurfacePlanes{0, 0, 0};
    const SurfacePlanes flat{0, 0, 0};
    const T dt = G.dt, mm = m.m;
    const Strain<T> e = strain<FS, VAC>(t, G, sp, p.k, l, mm);
    const T gn = D.xi * D.yi * D.zi;
    const T g[6] = {gn, gn, gn, D.xh * D.yh * D.zi, D.xh * D.yi * D.zh, D.xi * D.yh * D.zh};
    const bool ix = p.i <= G.nx - 2, jy = p.j <= G.ny - 2, kz = p.k <= G.nz - 2;
    const unsigned so[6] = {own, own, own, ix && jy ? own : kOOB, ix && kz ? own : kOOB, jy && kz ? own : kOOB};
    if constexpr (adjb) {  // A_s <- G_s A_s - dt E(Y)
        const T ev[6] = {e.xx, e.yy, e.zz, e.xy, e.xz, e.yz};
#pragma unroll
        for (int c = 0; c < 6; ++c) st(wfield(G.f[SXX + c], o.w), so[c], g[c] * s0[c] - dt * ev[c]);
    } else if constexpr (adjm) {
        // the adjoint stress update of the step after, stored and taken as this step's A_s
        const Strain<T> y = strain<false, false>(q, G, flat, p.k, l, mm);
        const T yv[6] = {y.xx, y.yy, y.zz, y.xy, y.xz, y.yz};
        T a[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            a[c] = g[c] * s0[c] - dt * yv[c];
            st(wfield(G.f[SXX + c], o.w), so[c], a[c]);
        }
        // gradients of C and X = C T with T = G_s A_s
        const T txx = gn * a[0], tyy = gn * a[1], tzz = gn * a[2];
        const T trT = (txx + tyy) + tzz;
        st(wfield(io.acc[0], o.w), own, a0[0] + dt * ((e.xx + e.yy) + e.zz) * trT);
        st(wfield(io.acc[1], o.w), own, a0[1] + dt * T(2) * ((e.xx * txx + e.yy * tyy) + e.zz * tzz));
        st(wfield(io.out[0], o.w), own, l * trT + T(2) * mm * txx);
        st(wfield(io.out[1], o.w), own, l * trT + T(2) * mm * tyy);
        st(wfield(io.out[2], o.w), own, l * trT + T(2) * mm * tzz);
        const T txy = g[3] * a[3], txz = g[4] * a[4], tyz = g[5] * a[5];
        st(wfield(io.acc[2], o.w), so[3], a0[2] + dt * e.xy * txy);
        st(wfield(io.acc[3], o.w), so[4], a0[3] + dt * e.xz * txz);
        st(wfield(io.acc[4], o.w), so[5], a0[4] + dt * e.yz * tyz);
        st(wfield(io.out[3], o.w), so[3], m.xy * txy);
        st(wfield(io.out[4], o.w), so[4], m.xz * txz);
        st(wfield(io.out[5], o.w), so[5], m.yz * tyz);
    } else {
        const T tr = e.xx + e.yy + e.zz;
        T nxx = s0[0] + dt * (l * tr + T(2) * mm * e.xx);
        T nyy = s0[1] + dt * (l * tr + T(2) * mm * e.yy);
        T nzz = s0[2] + dt * (l * tr + T(2) * mm * e.zz);
        T nxy = s0[3] + dt * m.xy * e.xy;
        T nxz = s0[4] + dt * m.xz * e.xz;
        T nyz = s0[5] + dt * m.yz * e.yz;
        if (src.on && (row_has_tap(src, SXX, p) || row_has_tap(src, SXY, p) || row_has_tap(src, SXZ, p) ||
                       row_has_tap(src, SYZ, p))) {
            const T s = sload(src.wavelet, n);
            const int ta = tap_of(src, SXX, p.i, p.j, p.k);
            nxx += coef_of(src, SXX, ta) * s;
            nyy += coef_of(src, SYY, ta) * s;
            nzz += coef_of(src, SZZ, ta) * s;
            nxy += coef_of(src, SXY, tap_of(src, SXY, p.i, p.j, p.k)) * s;
            nxz += coef_of(src, SXZ, tap_of(src, SXZ, p.i, p.j, p.k)) * s;
            nyz += coef_of(src, SYZ, tap_of(src, SYZ, p.i, p.j, p.k)) * s;
        }
        st(wfield(G.f[SXX], o.w), own, nxx * gn);
        st(wfield(G.f[SYY], o.w), own, nyy * gn);
        st(wfield(G.f[SZZ], o.w), own, (FS && p.k == 0) ? T(0) : nzz * gn);
        st(wfield(G.f[SXY], o.w), so[3], nxy * g[3]);
        st(wfield(G.f[SXZ], o.w), so[4], nxz * g[4]);
        st(wfield(G.f[SYZ], o.w), so[5], nyz * g[5]);
        if constexpr (born) {
            // the perturbation's stress term (no damping, no source), then its own update
            const T bxx = b0[0] + dt * (dl * tr + T(2) * dm.m * e.xx);
            const T byy = b0[1] + dt * (dl * tr + T(2) * dm.m * e.yy);
            const T bzz = b0[2] + dt * (dl * tr + T(2) * dm.m * e.zz);
            const T bxy = b0[3] + dt * dm.xy * e.xy, bxz = b0[4] + dt * dm.xz * e.xz, byz = b0[5] + dt * dm.yz * e.yz;
            const Strain<T> pe = strain<false, false>(q, G, flat, p.k, l, mm);
            const T ptr = pe.xx + pe.yy + pe.zz;
            const T pxx = bxx + dt * (l * ptr + T(2) * mm * pe.xx);
            const T pyy = byy + dt * (l * ptr + T(2) * mm * pe.yy);
            const T pzz = bzz + dt * (l * ptr + T(2) * mm * pe.zz);
            const T pxy = bxy + dt * m.xy * pe.xy;
            const T pxz = bxz + dt * m.xz * pe.xz;
            const T pyz = byz + dt * m.yz * pe.yz;
            st(wfield(io.out[0], o.w), own, pxx * gn);
            st(wfield(io.out[1], o.w), own, pyy * gn);
            st(wfield(io.out[2], o.w), own, pzz * gn);
            st(wfield(io.out[3], o.w), so[3], pxy * g[3]);
            st(wfield(io.out[4], o.w), so[4], pxz * g[4]);
            st(wfield(io.out[5], o.w), so[5], pyz * g[5]);
        }
    }
}

// ---------------------------------------------------------------------------------
// Single-grid launches: grid (8, rm.tiles(), rm.planes()), which the hardware deals round robin
// over the 8 XCDs along x.  The stress pass walks the planes backwards, from where the velocity
// pass ended.  Its blocks before the last rm.planes() along z sample receivers: a receiver takes
// two dependent loads from the far side of the L2s, and sampled by the last blocks it outlasted
// the cells (us a step, last / first: 64^3, 16 receivers 13.0 / 11.8; 149 x 101 x 87, 256
// receivers 35.2 / 31.3; 128^3, 256 receivers 41.1 / 37.4).
template <typename T, bool FS, int MODE, bool VAC>
__global__ void __launch_bounds__(256) vel_row(Grid<T> G, Inject<T> src, int n, RowMap rm)
{
    vel_row_body<T, FS, MODE, VAC>(G, src, n, row_pos(rm, G.nz, blockIdx.x, blockIdx.y, blockIdx.z, false), TileIO<T>{});
}

// Receiver work item of this thread in the blocks before the planes.
__device__ __forceinline__ int row_receiver()
{
    return (((int)blockIdx.z * (int)gridDim.y + (int)blockIdx.y) * 8 + (int)blockIdx.x) * 256 + (int)threadIdx.x;
}

template <typename T, bool FS, bool VAC>
__global__ void __launch_bounds__(256) stress_row(Grid<T> G, Inject<T> src, int n, RowMap rm, RecJob<T> rec)
{
    const int z = (int)blockIdx.z - ((int)gridDim.z - rm.planes());
    if (z < 0) {
        const int q = row_receiver();
        if (q < rec.nq) sample_receiver(rec, q, n);
        return;
    }
    stress_row_body<T, FS, kFwd, VAC>(G, src, n, row_pos(rm, G.nz, blockIdx.x, blockIdx.y, z, true), TileIO<T>{});
}

// Adjoint and Born passes.
template <typename T, int MODE>
__global__ void __launch_bounds__(256) vel_row_io(Grid<T> G, Inject<T> src, int n, RowMap rm, TileIO<T> io)
{
    constexpr bool up = vel_sweeps_up<MODE>();
    const RowPos p = row_pos(rm, G.nz, blockIdx.x, blockIdx.y, blockIdx.z, up);
    vel_row_body<T, false, MODE, false>(G, src, n, p, io);
}

template <typename T, int MODE>
__global__ void __launch_bounds__(256) stress_row_io(Grid<T> G, Inject<T> src, int n, RowMap rm, TileIO<T> io, RecJob<T> rec,
                                                     RecJob<T> prec)
{
    const int z = (int)blockIdx.z - ((int)gridDim.z - rm.planes());
    if (z < 0) {
        const int q = row_receiver();
        if (q < rec.nq) sample_receiver(rec, q, n);
        else if (q - rec.nq < prec.nq) sample_receiver(prec, q - rec.nq, n);
        return;
    }
    constexpr bool up = stress_sweeps_up<MODE>();
    const RowPos p = row_pos(rm, G.nz, blockIdx.x, blockIdx.y, z, up);
    stress_row_body<T, false, MODE, false>(G, src, n, p, io);
}

// ---------------------------------------------------------------------------------
// Many grids in one launch: the blocks of all shots form one list (shot by shot, strip by
// strip, plane by plane), cut into 8 equal runs, one per XCD.  Block b takes entry b / 8 of the
// run of XCD b mod 8 (the passes that walk backwards count from the last).  Runs rather than 8
// slabs of every shot: four shots of 96 x 80 x 72, forward step 56.4 us
// against 57.6; 40 x 50 x 60 by six: 30.3 against 31.3 (both before the search below).
// A block finds its shot by a binary search through the scalar cache: a table of the bases in
// LDS, as the persistent tile launches keep one, costs every block a load, a barrier and a scan
// before its first sample (six shots of 96 x 80 x 72 80.2 us a step with it, 76.1 without; one
// of 149 x 101 x 87 37.2 and 34.1; one of 128^3 41.3 and 39.4).
struct ShotRows {  // a shot's blocks, and the first of them in the list
    RowMap rm;
    int base;
};

template <typename T>
__device__ __forceinline__ const ShotFwd<T> &row_shot(const ShotFwd<T> *shots, const ShotRows *rows, int nshot, int total,
                                                      int block, bool reverse, RowPos &p)
{
    const int per = (total + 7) / 8, q = block >> 3;
    const int at = (block & 7) * per + (reverse ? per - 1 - q : q);
    const int l = at < total ? at : total - 1;  // past the last block: no work (below)
    int s = 0;
    for (int e = nshot; e - s > 1;) {
        const int m = (s + e) >> 1;
        if (sload(&rows[m].base, 0) <= l) s = m;
        else e = m;
    }
    const ShotFwd<T> &d = shots[s];
    const RowMap rm = rows[s].rm;
    const int b = l - rows[s].base, strip = rm.ns > 1 ? b / (rm.tiles() * rm.np) : 0, r = b - strip * rm.tiles() * rm.np;
    const int z = r / rm.tiles();
    p = row_cell(rm, strip, r - z * rm.tiles(), at < total ? z : d.G.nz);
    return d;
}

template <typename T, bool FS, int MODE, bool VAC>
__global__ void __launch_bounds__(256) vel_row_multi(const ShotFwd<T> *__restrict__ shots,
                                                     const ShotRows *__restrict__ rows, int nshot, int total, int n)
{
    RowPos p;
    const ShotFwd<T> &d = row_shot(shots, rows, nshot, total, (int)blockIdx.x, vel_sweeps_up<MODE>(), p);
    const Grid<T> G = d.G;
    const Inject<T> src = d.src;
    const TileIO<T> io = d.io;
    vel_row_body<T, FS, MODE, VAC>(G, src, n, p, io);
}

template <typename T, bool FS, int MODE, bool VAC>
__global__ void __launch_bounds__(256) stress_row_multi(const ShotFwd<T> *__restrict__ shots,
                                                        const ShotRows *__restrict__ rows, int nshot, int total, int n,
                                                        RecMulti<T> rec)
{
    const int block = (int)blockIdx.x - ((int)gridDim.x - rec.wgs);  // receivers first (a multiple of 8 blocks)
    if (block < 0) {
        __shared__ int s_base[kMaxShots];
        sample_batch_receivers(rec, s_base, n, (int)blockIdx.x);
        return;
    }
    RowPos p;
    const ShotFwd<T> &d = row_shot(shots, rows, nshot, total, block, stress_sweeps_up<MODE>(), p);
    const Grid<T> G = d.G;
    const Inject<T> src = d.src;
    const TileIO<T> io = d.io;
    stress_row_body<T, FS, MODE, VAC>(G, src, n, p, io);
}

} // namespace fd3d

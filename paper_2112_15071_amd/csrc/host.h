// Host side of the fd3d library (C ABI of include/fd3d.h): the context, its workspace
// layout and the helpers the translation units share.
//
//   runtime.hip   contexts, options, workspace layout, model check, damping profiles,
//                 source and receiver staging, state access, the allocation-free entry
//   forward.hip   the step loop (Sec. 2.2 update order), kernel selection and its tuner
//   gradient.hip  checkpointed discrete adjoint and the FWI gradient
//   batch.hip     batches of shots, persistent launches, graphs, the batched gradient
//                 (batch_plan.h: which kernels its launches run, in which order)
//   born.hip      tangent-linear (Born) forward
#pragma once

#include "fd3d.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "common.h"
#include "fwd_cell.h"
#include "fwd_tile.h"
#include "row.h"
#include "adj_cell.h"
#include "util_kernels.h"

namespace fd3d {

// Message of the last failed call on this thread (fd3d_last_error).
extern thread_local std::string g_err;

// Records msg as the thread's last error and returns code.
int fail(int code, const std::string &msg);

#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) return fail(FD3D_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

constexpr size_t kAlign = 256;
constexpr int kDefaultMaxRec = 4096;

inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

inline size_t rectap_bytes(int tsize) { return 8 * sizeof(int) + 8 * (size_t)tsize; }

// Workspace layout (byte offsets).  Two copies of the state: the fused step reads one and
// writes the other.  The fields are stored in one of two forms:
//  * separate arrays: each field x fastest and unpadded, padded to 4 KiB plus a 1 KiB
//    skew so that the nine streams of a pass do not start on the same HBM channel; the
//    model arrays are the caller's;
//  * interleaved rows: one block of kRows rows per (y, z) row index, row q holding field q
//    ([nz][ny][kRows][nx]), so that the rows of the nine fields a tile reads lie side by
//    side; the model is copied once into a block of the same shape (rows 0-2: lam, mu,
//    rho; rows 3-5: a Born perturbation), so every array of a pass has the same strides.
// A group of nine fields (a state copy, the adjoint state, a checkpoint, ...) is one block
// of interleaved rows, or nine padded arrays.
constexpr int kRows = 9;

struct Layout {
    bool rows;              // interleaved rows
    size_t field[2][NFIELD];
    size_t model;           // interleaved rows without a coarse medium: the model block
    size_t prof[3][2];
    size_t src;     // source coefficients [NFIELD][8]
    size_t rec;
    size_t colors;  // receiver order grouped by colour (tap-disjoint sets), int[max_rec]
    size_t part;
    size_t stats;
    size_t flag;
    size_t total;
    size_t field_bytes;     // bytes of one field's samples
    size_t fstep;           // bytes from one field of a group to the next
    size_t group;           // bytes of a group of up to nine fields
};

// Workspace layout of a grid under the given options (field storage chosen by opts.layout).
Layout layout_of(int nx, int ny, int nz, const fd3d_opts &o);

int check_opts(const fd3d_opts *o);
fd3d_opts default_opts();

inline int max_rec_of(const fd3d_opts &o) { return o.max_receivers > 0 ? o.max_receivers : kDefaultMaxRec; }

// The medium arrays are a coarse grid read by trilinear samples (opts.coarse).
inline bool coarse_on(const fd3d_opts &o) { return o.coarse[0] > 0; }

} // namespace fd3d

// A context (fd3d_create): one grid, its model and options, its workspace layout, the
// host staging of sources and receivers, the kernel choice and the gradient state.
struct fd3d_ctx {
    int n[3];
    int nt;
    int tsize;
    double dx, dy, dz, dt;  // spacing per axis (m), time step (s)
    fd3d_opts opts;
    const void *lam, *mu, *rho;
    char *ws;
    size_t ws_bytes;
    fd3d::Layout L;
    double info[4];
    std::vector<unsigned char> prof_host;  // typed profiles, kept for the async upload
    std::vector<unsigned char> src_host;   // source coefficients, kept for the async upload
    std::vector<unsigned char> rec_host;   // receiver descriptors, kept for the async upload
    std::vector<int> color_host;           // receivers grouped by colour, kept for the async upload
    std::vector<int> color_off;            // colour c holds color_host[color_off[c] .. color_off[c+1])
    std::vector<unsigned char> src_dev;    // source coefficients now in the workspace
    std::vector<double> rec_dev;           // receiver positions whose descriptors are in the workspace
    bool rec_dev_valid;                    // rec_dev describes the workspace's descriptors
    hipEvent_t staged;     // marks the end of the uploads from the host staging buffers;
                           // null in a context that must create no HIP objects (its call
                           // synchronises the stream before the buffers are released)
    bool staged_pending;
    // optional per-kernel timing of the step loop
    int prof_on;
    std::vector<hipEvent_t> prof_ev;  // pairs: [2*q] before, [2*q+1] after launch q
    std::vector<int> prof_pass;       // pass of launch q
    int prof_used;
    // kernel selection for the step loop
    int variant;  // FD3D_KERNEL_CELL, FD3D_KERNEL_TILE or FD3D_KERNEL_FUSED
    int cur;      // state copy holding the current state (0 or 1)
    int tile_x;   // columns of a tile (64, 128, 256)
    int tile_y;   // rows of a tile (4, 8, 16)
    int zchunk;   // z planes per workgroup sweep
    long window;  // largest buffer window (kMaxWindowBytes; less to reach larger planes' kernels)
    bool auto_kernel;  // nothing selected yet: each operation picks rows or sweeps (kernels_of)
    bool tuned;        // the variant is the forward tuner's: the other operations still pick
    // gradient state: checkpoints written by fd3d_forward_ckpt into a caller workspace
    const char *grad_ws;
    int grad_k;
    int grad_ready;
    int adj_done;  // an adjoint has run on grad_ws since its checkpointed forward
    int grad_y;    // the last adjoint was the tiled one: the adjoint velocity is held as Y
};

namespace fd3d {

template <typename T> Grid<T> make_grid(const fd3d_ctx *c)
{
    Grid<T> G;
    G.nx = c->n[0];
    G.ny = c->n[1];
    G.nz = c->n[2];
    G.sy = c->L.rows ? (long)kRows * G.nx : G.nx;
    G.sz = G.sy * G.ny;
    G.dt = (T)c->dt;
    G.rdx = (T)(1.0 / c->dx);
    G.rdy = (T)(1.0 / c->dy);
    G.rdz = (T)(1.0 / c->dz);
    G.ks = c->opts.vacuum_top;
    G.ksmap = (const int *)c->opts.vacuum_map;
    for (int a = 0; a < 3; ++a) {
        G.cm[a] = coarse_on(c->opts) ? c->opts.coarse[a] : 0;
        G.cs[a] = G.cm[a] ? (T)((double)(G.cm[a] - 1) / (double)(c->n[a] - 1)) : T(0);
    }
    if (c->L.model) {  // the model's copy in interleaved rows
        G.lam = (const T *)(c->ws + c->L.model);
        G.mu = (const T *)(c->ws + c->L.model + c->L.fstep);
        G.rho = (const T *)(c->ws + c->L.model + 2 * c->L.fstep);
    } else {
        G.lam = (const T *)c->lam;
        G.mu = (const T *)c->mu;
        G.rho = (const T *)c->rho;
    }
    for (int f = 0; f < NFIELD; ++f) G.f[f] = (T *)(c->ws + c->L.field[c->cur][f]);
    for (int a = 0; a < 3; ++a)
        for (int h = 0; h < 2; ++h) G.g[a][h] = (const T *)(c->ws + c->L.prof[a][h]);
    for (int f = 0; f < NFIELD; ++f) G.save[f] = nullptr;
    return G;
}

// The current state copy.  (The other one needs no fill: the fused step that writes it stores
// every sample.)
template <typename T> void zero_fields(fd3d_ctx *c, hipStream_t st)
{
    fill_zero<T><<<2048, 256, 0, st>>>((T *)(c->ws + c->L.field[c->cur][0]), (long)(c->L.group / sizeof(T)));
}

// Strided copies of `count` field-shaped arrays (1 .. 9) between node arrays (x fastest,
// unpadded) and the workspace's field storage; comp0 >= 0: array q is component comp0 + q, its
// pinned slots zeroed.
template <typename T>
void copy_arrays(const fd3d_ctx *c, int count, T *const *dst, bool dst_fields, const T *const *src, bool src_fields,
                 int comp0, hipStream_t st)
{
    const long nx = c->n[0], ny = c->n[1];
    const long fsy = c->L.rows ? kRows * nx : nx;
    FieldCopies<T> a;
    a.dsy = dst_fields ? fsy : nx;
    a.ssy = src_fields ? fsy : nx;
    a.dsz = a.dsy * ny;
    a.ssz = a.ssy * ny;
    a.nx = c->n[0];
    a.ny = c->n[1];
    a.nz = c->n[2];
    constexpr int V = 16 / (int)sizeof(T);
    bool wide = nx % V == 0;  // rows of whole 16-byte words, aligned
    for (int q = 0; q < 9; ++q) {
        const int p = q < count ? q : 0;
        FieldCopy<T> &f = a.f[q];
        f.dst = dst[p];
        f.src = src[p];
        f.sx = f.sy = f.sz = 0;
        if (comp0 >= 0) {
            f.sx = stag(comp0 + p, 0);
            f.sy = stag(comp0 + p, 1);
            f.sz = stag(comp0 + p, 2);
        }
        wide = wide && (uintptr_t)f.dst % 16 == 0 && (uintptr_t)f.src % 16 == 0;
    }
    const dim3 g(1024, count);
    if (wide) copy_fields<T, V><<<g, 256, 0, st>>>(a);
    else copy_fields<T, 1><<<g, 256, 0, st>>>(a);
}

// The current state zeroed, for either element type.
void zero_fields_any(fd3d_ctx *c, hipStream_t st);

// Builds the source (tap boxes into inj) and the receiver descriptors and colours, and
// uploads them from the context's host staging buffers (after the previous call's
// uploads from those buffers are done).  Defined for float and double.
template <typename T>
int stage_inputs(fd3d_ctx *c, const fd3d_source *src, Inject<T> &inj, int nrec, const double *rec_pos,
                 hipStream_t st);

// Event pair around one launch when timing is on.
struct Timer {
    fd3d_ctx *c;
    hipStream_t st;
    void begin(int pass)
    {
        if (!c->prof_on) return;
        const int q = c->prof_used;
        if ((size_t)(2 * q + 2) > c->prof_ev.size()) {
            hipEvent_t a = nullptr, b = nullptr;
            (void)hipEventCreate(&a);
            (void)hipEventCreate(&b);
            c->prof_ev.push_back(a);
            c->prof_ev.push_back(b);
            c->prof_pass.push_back(pass);
        }
        c->prof_pass[q] = pass;
        (void)hipEventRecord(c->prof_ev[2 * q], st);
    }
    void end()
    {
        if (!c->prof_on) return;
        (void)hipEventRecord(c->prof_ev[2 * c->prof_used + 1], st);
        ++c->prof_used;
    }
};

inline TileMap tile_map(const fd3d_ctx *c)
{
    TileMap tm;
    tm.ntx = (c->n[0] + c->tile_x - 1) / c->tile_x;
    tm.nty = (c->n[1] + c->tile_y - 1) / c->tile_y;
    tm.zc = c->zchunk;
    tm.nzc = (c->n[2] + c->zchunk - 1) / c->zchunk;
    return tm;
}

// Supported tile shapes: 64x{4,8,16}, 128x{4,8}, 256x4 (FP64: 64x{4,8}, 128x4).
inline bool tile_supported(int tsize, int tx, int ty)
{
    if (tsize == 8) return (tx == 64 && (ty == 4 || ty == 8)) || (tx == 128 && ty == 4);
    return (tx == 64 && (ty == 4 || ty == 8 || ty == 16)) || (tx == 128 && (ty == 4 || ty == 8)) ||
           (tx == 256 && ty == 4);
}

// Calls f(TX, TY) with the tile shape as integral constants (64x8 for a shape that is
// not compiled for T).
template <typename T, typename F> decltype(auto) with_tile(int tx, int ty, F &&f)
{
    using X64 = std::integral_constant<int, 64>;
    using X128 = std::integral_constant<int, 128>;
    using X256 = std::integral_constant<int, 256>;
    using Y4 = std::integral_constant<int, 4>;
    using Y8 = std::integral_constant<int, 8>;
    using Y16 = std::integral_constant<int, 16>;
    const int key = tx * 100 + ty;
    if constexpr (sizeof(T) == 8) {
        switch (key) {
        case 6404: return f(X64{}, Y4{});
        case 12804: return f(X128{}, Y4{});
        default: return f(X64{}, Y8{});
        }
    } else {
        switch (key) {
        case 6404: return f(X64{}, Y4{});
        case 6416: return f(X64{}, Y16{});
        case 12804: return f(X128{}, Y4{});
        case 12808: return f(X128{}, Y8{});
        case 25604: return f(X256{}, Y4{});
        default: return f(X64{}, Y8{});
        }
    }
}

// Passes of a step.  Forward: velocity, stress.  Adjoint step (reverse order of the
// forward step): stress-A (C gradients, X = C G_s A_s), velocity-A (A_v update, b
// gradient, Y = G_v A_v / rho_eff), stress-B (A_s update from Y); the tiled adjoint runs
// stress-B of step n+1 and stress-A of step n as one pass, stress-M, and a last stress-B
// after step 0.  The velocity pass also comes in a variant for the gradient's segment
// recompute: the tile kernels write v^{n+1/2} through the grid's save pointers instead of
// over v^{n-1/2}, the cell kernel writes it to both.
enum Pass { kPassVel = 0, kPassStress = 1, kPassStressA, kPassVelA, kPassStressB, kPassVelSave, kPassStressM };

// Tile and fused sweeps address a window of at most zchunk + 8 planes (and at most the
// grid's nz) through one buffer descriptor per field, of at most 1 GiB (fd3d_limit_window).
inline bool window_ok(const fd3d_ctx *c, int zc)
{
    const long rows = c->L.rows ? kRows : 1, planes = std::min(zc + 8, c->n[2]);
    return planes * rows * (long)c->n[0] * (long)c->n[1] * (long)c->tsize <= c->window;
}

// Tile workgroups of NT threads that the device runs at once: the tile kernels' registers
// allow 16 waves a CU in FP32 (80 to 128 VGPRs), 12 in FP64.
inline long tile_slots(int tsize, int nt)
{
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    return (long)std::max(1, (tsize == 8 ? 12 : 16) / (nt / 64)) * cus;
}

inline long tile_columns(const fd3d_ctx *c, int tx, int ty)
{
    return (long)((c->n[0] + tx - 1) / tx) * ((c->n[1] + ty - 1) / ty);
}

// Depth of a grid's sweeps in a launch of depth zc: its planes cut evenly into sweeps of at
// most zc planes (at least 4, and within one window).
inline int sweep_depth(const fd3d_ctx *c, int zc)
{
    const int nz = c->n[2], cuts = (nz + zc - 1) / zc;
    int d = std::max(4, (nz + cuts - 1) / cuts);
    while (d > 4 && !window_ok(c, d)) d = std::max(4, d / 2);
    return d;
}

// Depth of a launch of sweeps by workgroups of nt threads over ns grids, of cols(q) columns of
// tiles each, and its cost (1e300: no sweep fits one window).  The workgroups run in rounds of
// as many as the chip holds; for one to three rounds, the least depth that needs no more of them.
// A sweep of zc planes costs about zc + 14 planes' time (its z halo and the z queues' first loads).
template <typename S, typename F> double launch_depth(int ns, S &&shot, F &&cols, int nt, int &zc)
{
    int nz = 4;
    for (int q = 0; q < ns; ++q) nz = std::max(nz, shot(q)->n[2]);
    const long slots = tile_slots(shot(0)->tsize, nt);
    double best = 1e300;
    for (int r = 1; r <= 3; ++r) {
        int lo = 4, hi = nz;
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            long sweeps = 0;
            for (int q = 0; q < ns; ++q) sweeps += cols(q) * ((shot(q)->n[2] + mid - 1) / mid);
            if (sweeps <= r * slots) hi = mid;
            else lo = mid + 1;
        }
        long sweeps = 0;
        int deepest = 0;
        bool fits = true;
        for (int q = 0; q < ns; ++q) {
            const int d = sweep_depth(shot(q), lo);
            fits = fits && window_ok(shot(q), d);
            deepest = std::max(deepest, d);
            sweeps += cols(q) * ((shot(q)->n[2] + d - 1) / d);
        }
        const double cost = (double)((sweeps + slots - 1) / slots) * (deepest + 14) * slots * nt;
        if (fits && cost < best) {
            best = cost;
            zc = lo;
        }
    }
    return best;
}

// Tile shape and depth of a launch of sweeps over ns grids with nothing selected (zc = 0: none
// fits one window): the least cost.  FP32 rows of 64 columns (256 bytes) cost 1.3 of a wider
// tile's, the lanes past a row's end included; wide tiles win ties, with a coarse medium (whose
// grids mostly stay in the cache) narrow ones, at the same cost.  Over 66 launches beyond the cache
// (forward, Born, gradient, batches; FP32) this comes to 0.8 % of the fastest of all shapes and
// depths on average, over 57 in FP64 to 2.6 % (1 % where the sweeps are the default).  Us per step, a fixed 64- or 32-plane
// sweep of the tile as wide as the rows / all shapes at par, 20 waves a CU, zc + 3, a batch always
// in one round / this: forward 230^3 346 / 355 / 286, 230 x 300 x 260 535 / 571 / 429; Born 230^3
// 797 / 831 / 626; gradient 230^3 1820 / 1832 / 1375; gradients of four shots of 160 x 150 x 100
// 1455 / 1599 / 1032, of three of 260 x 200 x 150 3951 / 4740 / 3020; batch of four 160 x 300 x 260
// 1320 / 1438 / 1223; coarse 64^3 88 / 30 / 21.
struct Sweep {
    int tx, ty, zc;
};
template <typename S> Sweep choose_sweep(int ns, S &&shot)
{
    static const int shapes[][2] = {{256, 4}, {128, 8}, {64, 16}, {128, 4}, {64, 8}, {64, 4}};
    const int ts = shot(0)->tsize;
    const bool coarse = coarse_on(shot(0)->opts);
    Sweep s{64, 8, 0};
    double best = 1e300;
    for (int k = 0; k < 6; ++k) {
        const int tx = shapes[coarse ? 5 - k : k][0], ty = shapes[coarse ? 5 - k : k][1];
        if (!tile_supported(ts, tx, ty)) continue;
        int zc = 0;
        const double cost = launch_depth(ns, shot, [&](int q) { return tile_columns(shot(q), tx, ty); }, tx * ty, zc) *
                            (ts == 4 && !coarse && tx == 64 ? 1.3 : 1.0);
        if (cost < best) {
            best = cost;
            s = {tx, ty, zc};
        }
    }
    return s;
}

// Work of a row launch over a grid.  Blocks as wide as the rows, of the width that leaves the
// fewest lanes idle (the widest of equals; 149 x 101 x 87: 32.2 us a step with 64 columns, 35.6
// with 256).  Grids whose planes are small are cut into 8 slabs of planes, one per XCD: the few
// planes that neighbouring cells share stay in its 4 MiB L2 (64^3: 10.3 us against 10.3 in 8
// strips and 14.1 in 4).  Larger planes are cut into strips of at most 32 rows instead (256 x 256
// x 72: 76.5 us against 111 in slabs; 200 x 150: 57 against 58, 256 x 128: 67 either way).
constexpr long kSlabPlaneBytes = 128 << 10;
// A launch over many shots (list) cuts its list of blocks into runs by itself: strips only.
inline RowMap row_map(const fd3d_ctx *c, bool list = false)
{
    const int nx = c->n[0], ny = c->n[1], nz = c->n[2];
    RowMap rm;
    rm.lbx = 8;
    for (int l = 7; l >= 6; --l) {
        auto padded = [&](int b) { return ((nx + (1 << b) - 1) >> b) << b; };
        if (padded(l) < padded(rm.lbx)) rm.lbx = l;
    }
    rm.ntx = (nx + (1 << rm.lbx) - 1) >> rm.lbx;
    const int rows = 256 >> rm.lbx, blocks = (ny + rows - 1) / rows;
    if ((long)nx * ny * c->tsize <= kSlabPlaneBytes) {
        rm.nslab = 8;
        rm.ns = 1;
    } else {
        rm.nslab = 1;
        rm.ns = std::min(blocks, (std::max(8, (ny + 31) / 32) + 7) / 8 * 8);
    }
    rm.rps = (blocks + rm.ns - 1) / rm.ns;
    rm.ns = (blocks + rm.rps - 1) / rm.rps;
    if (list) rm.nslab = 1;
    rm.np = (nz + rm.nslab - 1) / rm.nslab;
    rm.cpx = (rm.ns * rm.nslab + 7) / 8;
    return rm;
}

// Largest grid of blocks along y and z.
constexpr int kMaxGridYZ = 65535;

// Grid of a row launch that also samples nq receiver items; none (x = 0) when those do not fit
// beside the planes.
inline dim3 row_grid(const RowMap &rm, int nq = 0)
{
    const long per = 8L * rm.tiles() * 256, z = rm.planes() + (nq + per - 1) / per;
    return z <= kMaxGridYZ ? dim3(8, rm.tiles(), (unsigned)z) : dim3(0, 1, 1);
}

// The row kernels address the planes around a cell (at most 9) through one buffer descriptor
// per field, and deal tiles and planes out along y and z of a grid of blocks; the cell variant of
// a context whose planes are too large for the one or too many for the other (16 x 4096 x 4200:
// 128 strips of 4200 planes over 8 XCDs) runs the kernels with a bounds test per load.
inline bool rows_ok(const fd3d_ctx *c)
{
    if (!window_ok(c, 1)) return false;
    const RowMap rm = row_map(c);
    return rm.tiles() <= kMaxGridYZ && (long)rm.np * rm.cpx <= kMaxGridYZ;
}

// Those kernels take a plane along z and four rows along y of a grid of blocks.
inline bool cells_ok(const fd3d_ctx *c) { return c->n[2] <= kMaxGridYZ && (c->n[1] + 3) / 4 <= kMaxGridYZ; }

// Kernels of an operation that steps `arrays` cell-sized arrays: rows, tile sweeps, or the
// kernels with a bounds test per load (cells).  A selected variant decides, one that the tuner
// found for the forward, which alone it timed; with nothing selected, the size (RowSize).
// FP32 rows run while the arrays stay in the Infinity Cache.  Measured on both sides of the limit
// (MI355X, us per step, rows / best tile sweep): the forward's 12 arrays at 192 x 192 x 128 (226
// MB) 89 / 94, 72 x 256 x 220 (195 MB, few lanes filled) 105 / 101 and 256 x 256 x 96 (302 MB) 156
// / 133; Born's 24 at 128^3 (201 MB) 74 / 94, 33 x 256 x 256 (208 MB) 112 / 120 and 192 x 160 x 128
// (377 MB) 210 / 185; the adjoint's 29 at 149 x 101 x 87 (152 MB) 147 / 167, 128^3 (243 MB) 201 /
// 202 and 192 x 160 x 128 (456 MB) 380 / 369 (whole gradients).
// FP64 rows hold twice the registers, which halves the waves in flight, and from some 400 thousand
// lanes on (idle ones past a row's end included) the sweeps are as fast in every operation, where
// the rows fill their lanes from 660 thousand.  Forward, Born, gradient, rows / best sweep, in
// thousands of lanes: 48 x 80 x 64 (328) 20 / 25, 37 / 41, 78 / 91; 72 x 56 x 56 (401) 25 / 25, 44 /
// 42, 93 / 93; 90 x 60 x 60 (461) 28 / 26, 51 / 47, 107 / 101; 120 x 64 x 64 (524, 94 % filled) 30
// / 30, 54 / 59, 121 / 119; 128 x 80 x 64 (655, all) 35 / 37, 66 / 69, 147 / 145; 88 x 88 x 80 (991)
// 44 / 39, 82 / 73, 176 / 157; 110 x 100 x 96 (1229, 86 %) 58 / 52, 114 / 102, 275 / 224; batches'
// forward: two of 64^3 (524, all) 33 / 33, six of 40^3 (614, 63 %) 37 / 34.
constexpr int kForwardArrays = 12, kBornArrays = 24, kAdjointArrays = 29;
constexpr double kRowBytes32 = 230.0 * 1024 * 1024, kRowLanes64 = 400e3, kFullRowLanes64 = 660e3;
struct RowSize {  // of the row launches of one operation over some grids
    double bytes = 0.0, cells = 0.0, lanes = 0.0;

    void add(const fd3d_ctx *c, int arrays)
    {
        const RowMap rm = row_map(c);
        const double rows = (double)c->n[1] * c->n[2];
        cells += rows * c->n[0];
        lanes += rows * (rm.ntx << rm.lbx);
        bytes += rows * c->n[0] * arrays * c->tsize;
    }
    bool pays(int tsize) const
    {
        return tsize == 8 ? lanes <= (cells >= 0.9 * lanes ? kFullRowLanes64 : kRowLanes64) : bytes <= kRowBytes32;
    }
};
enum class Kern { rows, tiles, cells };
inline bool unselected(const fd3d_ctx *c, int arrays) { return c->auto_kernel || (c->tuned && arrays != kForwardArrays); }
inline Kern kernels_of(const fd3d_ctx *c, int arrays)
{
    if (!unselected(c, arrays))
        return c->variant != FD3D_KERNEL_CELL ? Kern::tiles : rows_ok(c) ? Kern::rows : Kern::cells;
    if (coarse_on(c->opts)) return Kern::tiles;
    RowSize size;
    size.add(c, arrays);
    return size.pays(c->tsize) && rows_ok(c) ? Kern::rows : Kern::tiles;
}

// Default tile shape and sweep depth (choose_sweep).  False when no sweep fits one window.
inline bool default_tiles(fd3d_ctx *c)
{
    const Sweep s = choose_sweep(1, [c](int) { return c; });
    c->tile_x = s.tx;
    c->tile_y = s.ty;
    c->zchunk = s.zc > 0 ? sweep_depth(c, s.zc) : 4;
    return s.zc > 0;
}

// Cache policy of a context's single-grid tile launches: the model arrays and the
// gradient's stored velocities and accumulators are streamed (non-temporal) when the
// grid's working set, nine fields and three model arrays, exceeds the 256 MB Infinity
// Cache.  Below that the whole working set can stay cached from step to step, and
// streaming would evict the model.
constexpr double kInfinityCacheBytes = 256.0 * 1024 * 1024;
inline bool stream_model(const fd3d_ctx *c)
{
    if (coarse_on(c->opts)) return false;  // the coarse medium is small and stays cached
    return 12.0 * (double)c->n[0] * (double)c->n[1] * (double)c->n[2] * (double)c->tsize > kInfinityCacheBytes;
}

// One forward pass (velocity, stress or their storing variants); defined for float and double,
// with and without free surface.  rec (stress passes of the forward only): the step's receiver
// sampling, carried by the row or tile launch or launched after the cell kernel.
template <typename T, bool FS>
void launch_pass(const fd3d_ctx *c, Kern kern, const Grid<T> &G, const Inject<T> &inj, int n, int pass, hipStream_t st,
                 const RecJob<T> &rec = RecJob<T>{});

// The receiver sampling of a grid's velocity (none when nrec is 0).
template <typename T> RecJob<T> rec_job(const T *vx, const T *vy, const T *vz, const RecTap<T> *taps, int nrec,
                                        int nt, T *traces)
{
    RecJob<T> r{};
    if (nrec <= 0) return r;
    r.v[0] = vx;
    r.v[1] = vy;
    r.v[2] = vz;
    r.taps = taps;
    r.traces = traces;
    r.nq = 3 * nrec;
    r.nt = nt;
    return r;
}

// One forward step: velocity pass, then the stress pass, which samples the receivers.
template <typename T, bool FS>
void step(fd3d_ctx *c, Kern kern, const Grid<T> &G, const Inject<T> &inj, int n, int nrec, const RecTap<T> *taps,
          T *traces, hipStream_t st, Timer &tm);

// Fused tile shapes: FP32 64x4 and 64x8, FP64 64x4.
bool fused_supported(const fd3d_ctx *c, int tx, int ty);

// Gradient workspace (byte offsets): adjoint state, staggered-point gradient
// accumulators, the tiled adjoint's intermediate fields, checkpoints every k steps, the
// stored velocities of one k-step segment, a copy of the segment's checkpoint (the cell
// adjoint's v^{n-1/2} of the segment's first step), and the residual buffer of
// fd3d_gradient.
// Every group of fields has the layout of the context's state (one block of interleaved
// rows, or padded arrays): field q of a group at q * fstep.
struct GradLayout {
    size_t fstep;   // bytes from one field of a group to the next
    size_t group;   // bytes of a group of nine fields
    size_t adj;     // 9 fields: A_v, A_s
    size_t acc;     // 8 fields: gl, gm, g_mu_xy, g_mu_xz, g_mu_yz, g_bx, g_by, g_bz
    size_t scr;     // 9 fields: X = C G_s A_s (6, stress layout), Y = G_v A_v / rho_eff (3)
    size_t ckpt;    // nseg groups: state at the start of steps 0, k, 2k, ...
    size_t seg;     // ceil(k/3) groups: v^{n+1/2} of three steps of a segment per group
    size_t prev;    // one group: a copy of the segment's checkpoint (cell adjoint)
    size_t res;     // residual [max_rec][3][nt]
    size_t misfit;  // one T
    size_t total;
    int nseg, k;
};

// Gradient workspace layout for checkpoints every k steps.
GradLayout make_grad_layout(const fd3d_ctx *c, int k);

// Stored v^{n+1/2} of step m of a segment (m < k): fields 3 (m mod 3) .. +2 of group m / 3.
inline char *seg_slot(char *gws, const GradLayout &GL, int m)
{
    return gws + GL.seg + (size_t)(m / 3) * GL.group + (size_t)(3 * (m % 3)) * GL.fstep;
}

// v^{n-1/2} of segment step m: the previous step's stored v^{n+1/2}, or for m = 0 the
// velocity fields of the copy of the segment's checkpoint.
inline char *prev_velocity(char *gws, const GradLayout &GL, int m)
{
    return m > 0 ? seg_slot(gws, GL, m - 1) : gws + GL.prev;
}

// The nt-step forward of a context (checkpoints into gws with GL); float and double.
template <typename T>
int forward_impl(fd3d_ctx *c, const fd3d_source *src, int nrec, const double *rec_pos, void *traces, int flags,
                 hipStream_t st, char *gws = nullptr, const GradLayout *GL = nullptr);

template <typename T> AdjGrid<T> make_adj(char *gws, const GradLayout &GL)
{
    AdjGrid<T> A;
    for (int f = 0; f < NFIELD; ++f) A.a[f] = (T *)(gws + GL.adj + f * GL.fstep);
    T *acc[8];
    for (int q = 0; q < 8; ++q) acc[q] = (T *)(gws + GL.acc + q * GL.fstep);
    A.gl = acc[0];
    A.gm = acc[1];
    for (int q = 0; q < 3; ++q) {
        A.gs[q] = acc[2 + q];
        A.gb[q] = acc[5 + q];
    }
    for (int q = 0; q < 3; ++q) A.vst[q] = A.vprev[q] = nullptr;
    return A;
}

// The stored velocities of segment step m for the one-thread-per-cell adjoint (the tiled
// adjoint reads v^{n+1/2} only).
template <typename T> void set_stored_velocity(AdjGrid<T> &A, char *gws, const GradLayout &GL, int m)
{
    const char *slot = seg_slot(gws, GL, m), *prev = prev_velocity(gws, GL, m);
    for (int q = 0; q < 3; ++q) {
        A.vst[q] = (const T *)(slot + q * GL.fstep);
        A.vprev[q] = (const T *)(prev + q * GL.fstep);
    }
}

// Fields of the three tiled adjoint passes of segment step m: grids (f[] re-pointed) and
// tile outputs.  The tiled adjoint holds Y = G_v A_v / rho_eff (intermediate fields 6-8)
// in place of A_v.
template <typename T> struct AdjTiles {
    Grid<T> g[3];     // stress-A (or stress-M), velocity-A, stress-B
    TileIO<T> io[3];
};

template <typename T> AdjTiles<T> adj_tiles(const Grid<T> &G, char *gws, const GradLayout &GL, int m)
{
    auto fld = [&](size_t base, int q) { return (T *)(gws + base + q * GL.fstep); };
    const char *slot = seg_slot(gws, GL, m);
    AdjTiles<T> P;
    for (int p = 0; p < 3; ++p) {
        P.g[p] = G;
        for (int f = 0; f < NFIELD; ++f) P.g[p].save[f] = nullptr;
        std::memset(&P.io[p], 0, sizeof P.io[p]);
    }
    for (int q = 0; q < 3; ++q) {
        P.g[0].f[VX + q] = (T *)(slot + q * GL.fstep);  // stored v^{n+1/2}
        P.g[1].f[VX + q] = fld(GL.scr, 6 + q);            // Y
        P.g[2].f[VX + q] = fld(GL.scr, 6 + q);
        P.io[1].acc[q] = fld(GL.acc, 5 + q);              // g_b
        P.io[1].vst[q] = (const T *)(slot + q * GL.fstep);
        P.io[0].y[q] = fld(GL.scr, 6 + q);                // Y of the step after (stress-M)
    }
    for (int q = 0; q < 6; ++q) {
        P.g[0].f[SXX + q] = fld(GL.adj, SXX + q);  // A_s
        P.g[1].f[SXX + q] = fld(GL.scr, q);        // X
        P.g[2].f[SXX + q] = fld(GL.adj, SXX + q);
        P.io[0].out[q] = fld(GL.scr, q);
    }
    for (int q = 0; q < 5; ++q) P.io[0].acc[q] = fld(GL.acc, q);  // gl, gm, g_mu_xy, g_mu_xz, g_mu_yz
    return P;
}

// What the tiled adjoint's residual injection of segment step m updates.
template <typename T> TapAdjoint<T> tap_adjoint(const Grid<T> &G, char *gws, const GradLayout &GL, int m)
{
    const AdjTiles<T> P = adj_tiles<T>(G, gws, GL, m);
    TapAdjoint<T> A;
    for (int q = 0; q < 3; ++q) {
        A.y[q] = P.g[1].f[VX + q];
        A.gb[q] = P.io[1].acc[q];
        A.vst[q] = P.io[1].vst[q];
    }
    A.rho = G.rho;
    for (int a = 0; a < 3; ++a)
        for (int h = 0; h < 2; ++h) A.g[a][h] = G.g[a][h];
    A.sy = G.sy;
    A.sz = G.sz;
    return A;
}

// The tiled adjoint's last term of the gradient of b, from the initial velocity (the
// velocity fields of checkpoint 0) and the first step's Y.
template <typename T> void launch_gb_initial(const Grid<T> &G, const AdjGrid<T> &A, char *gws, const GradLayout &GL,
                                             hipStream_t st)
{
    auto v0 = [&](int q) { return (const T *)(gws + GL.ckpt + q * GL.fstep); };
    auto y = [&](int q) { return (const T *)(gws + GL.scr + (6 + q) * GL.fstep); };
    const dim3 blk(64, 4, 1), grd((G.nx + 63) / 64, (G.ny + 3) / 4, G.nz);
    gb_initial_velocity<T><<<grd, blk, 0, st>>>(G, v0(0), v0(1), v0(2), y(0), y(1), y(2), A.gb[0], A.gb[1], A.gb[2]);
}

// Zero the adjoint state, accumulators and intermediate fields, and the segment's stored
// velocities at the pinned staggered positions, which are never stored and must read 0.
template <typename T> void zero_grad_fields(const Grid<T> &G, char *gws, const GradLayout &GL, hipStream_t st)
{
    fill_zero<T><<<2048, 256, 0, st>>>((T *)(gws + GL.adj), (long)((GL.ckpt - GL.adj) / sizeof(T)));
    for (int m0 = 0; m0 < GL.k; m0 += 3 * 4096) {  // whole groups, at most the largest grid of blocks
        const int slots = std::min(GL.k - m0, 3 * 4096);
        zero_pinned<T><<<dim3(16, 3 * slots), 256, 0, st>>>(seg_slot(gws, GL, m0), GL.group, GL.fstep, G.nx, G.ny, G.nz,
                                                            G.sy, G.sz);
    }
}

// Copies the nine fields of a group (of the state, or a checkpoint) with the pads between them.
inline void copy_group(const fd3d_ctx *c, char *dst, const char *src, hipStream_t st)
{
    copy_block<<<2048, 256, 0, st>>>((float4 *)dst, (const float4 *)src, (long)(c->L.group / 16));
}

// Validates a caller's gradient workspace for checkpoints every k steps.
int check_gws(const fd3d_ctx *ctx, void *gws, size_t gws_bytes, int k);

} // namespace fd3d

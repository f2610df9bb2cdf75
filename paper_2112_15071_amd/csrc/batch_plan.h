// Batches on the host: the batch, and which kernels its launches run in which order.
//
// Schedules.  Lockstep: every launch covers every shot, and the shots advance one step
// at a time together.  Cache-blocked groups: the shots, taken from the smallest working
// set (nine fields and three model arrays) to the largest, are cut into runs whose
// working sets add up to at most a given number of bytes; one group runs all its nt
// steps (one launch per pass over the group's shots) before the next group starts.
// Sized to the last-level (Infinity) cache, a group's fields stay resident from one step
// to the next.  Shots are independent, so both schedules give every shot the same result
// bit for bit.
#pragma once

#include "host.h"

namespace fd3d {

// Shots at positions [s0, s0 + ns) of the batch's schedule order, stepped by one launch
// per pass: their work items and receiver components (counted from the group's first),
// the persistent grid size and the tile shapes of the launch (tx2 = 0: one shape).
struct BatchGroup {
    int s0, ns, tiles, recs, wgs;
    int tx, ty, tx2, ty2;
    int vac;  // some shot of the group has a vacuum surface
    int zc;   // depth of the launch for shots with nothing selected (0: each shot's own)
    int every_zc;  // depth of every shot, selected or not (0: the above)
    int rtiles;              // row kernels: their blocks
    const ShotRows *rows;    // and the shots' shares of them (null: tile kernels)
    int ntp;  // cache policy of the group's forward passes (see group_streams)
};

} // namespace fd3d

struct fd3d_batch {
    int nshot;
    std::vector<fd3d_ctx *> ctx;
    int tsize, nt, fs;
    char *ws;
    size_t ws_bytes;
    size_t off_fwd, off_rec, off_rows;
    int tile_x, tile_y, wgs_req;
    int tile2_x, tile2_y;  // optional second tile shape (same workgroup size), 0: none
    bool tiles_set;        // the caller or the tuner selected the batch's tile shapes
    size_t group_bytes;    // 0: lockstep; otherwise the cache-blocked group budget
    bool sched_set;        // the caller or the tuner selected the schedule
    int grad_x, grad_y, grad_z;  // tile shape and depth of the gradient's sweeps (x < 0: as the
                                 // batch's tiles are set; 0: the library's choice; z 0: whole depth)
    std::vector<fd3d::BatchGroup> groups;
    std::vector<int> order;  // shot at each position of the descriptor arrays
    std::vector<unsigned char> fwd_host, rec_host;
    std::vector<fd3d::ShotRows> rows_host;
    hipEvent_t staged;
    bool staged_pending;
    hipStream_t cap;
    std::vector<unsigned char> grad_host;  // batched-gradient descriptors, kept for the async upload
    hipGraph_t graph;
    hipGraphExec_t gexec;
    bool graph_valid;
    long graph_key;
};

namespace fd3d {

// Two contexts whose batched passes read the same model arrays: the caller's, in place,
// or one copy in interleaved rows (see share_model).
inline bool shares_model(const fd3d_ctx *a, const fd3d_ctx *b)
{
    return a->L.rows == b->L.rows && (a->lam == b->lam || a->mu == b->mu || a->rho == b->rho);
}

// Streaming (non-temporal) policy for the forward passes of a group of contexts, as
// stream_model for one grid: FP32, the group's working sets add up to more than the
// Infinity Cache, and no two of its shots share a model array (a shared model is re-read
// by the other shots' tiles of the same launch).
inline bool group_streams(const fd3d_ctx *const *ctx, int ns)
{
    if (ns < 1 || ctx[0]->tsize != 4) return false;
    double bytes = 0.0;
    for (int q = 0; q < ns; ++q) {
        bytes += 12.0 * (double)ctx[q]->n[0] * (double)ctx[q]->n[1] * (double)ctx[q]->n[2] * (double)ctx[q]->tsize;
        for (int r = 0; r < q; ++r)
            if (shares_model(ctx[q], ctx[r])) return false;
    }
    return bytes > kInfinityCacheBytes;
}

// The batch's own tile shapes as one group covering every shot (counts not filled in).
inline BatchGroup whole_batch(const fd3d_batch *b)
{
    BatchGroup g{};
    g.s0 = 0;
    g.ns = b->nshot;
    g.tx = b->tile_x;
    g.ty = b->tile_y;
    g.tx2 = b->tile2_x;
    g.ty2 = b->tile2_y;
    g.ntp = group_streams(b->ctx.data(), b->nshot);
    return g;
}

// Tile map of one shot of a launch, and whether it uses the launch's second tile shape
// (when that covers its rows with fewer idle columns).
inline TileMap shot_tiles(const BatchGroup &b, const fd3d_ctx *c, int &alt)
{
    int tx = b.tx, ty = b.ty;
    alt = 0;
    if (b.tx2 > 0) {
        const int pad1 = (c->n[0] + tx - 1) / tx * tx, pad2 = (c->n[0] + b.tx2 - 1) / b.tx2 * b.tx2;
        if (pad2 < pad1) {
            alt = 1;
            tx = b.tx2;
            ty = b.ty2;
        }
    }
    TileMap tm;
    tm.ntx = (c->n[0] + tx - 1) / tx;
    tm.nty = (c->n[1] + ty - 1) / ty;
    tm.zc = b.every_zc > 0 ? std::min(b.every_zc, std::max(4, c->n[2]))
            : c->auto_kernel && b.zc > 0 ? sweep_depth(c, b.zc) : c->zchunk;
    tm.nzc = (c->n[2] + tm.zc - 1) / tm.zc;
    return tm;
}

// Sweeps of a launch over ns shots of which some have no kernel selected: their common depth,
// and unless the batch's tile shapes are selected, the launch's shape (choose_sweep).
template <typename C> void fit_sweeps(BatchGroup &g, int ns, bool tiles_set, C &&shot)
{
    bool any = false;
    for (int q = 0; q < ns; ++q) any = any || shot(q)->auto_kernel;
    if (!any) return;
    int zc = 0;
    if (tiles_set) {
        auto cols = [&](int q) {
            int alt = 0;
            const TileMap tm = shot_tiles(g, shot(q), alt);
            return (long)tm.ntx * tm.nty;
        };
        if (launch_depth(ns, shot, cols, g.tx * g.ty, zc) < 1e300) g.zc = zc;
        return;
    }
    const Sweep s = choose_sweep(ns, shot);
    if (s.zc == 0) return;
    g.tx = s.tx;
    g.ty = s.ty;
    g.tx2 = g.ty2 = 0;
    g.zc = s.zc;
}

// Whether a launch over these shots runs the row kernels: when neither the batch has tile shapes
// selected nor a shot a tile or fused kernel, and all shots' arrays (`arrays` each) together are of
// a size that the row kernels are for (kernels_of).  In lockstep, us per step, rows / fastest sweep,
// forward and gradient: six shots of 40 x 50 x 60 28.0 / 30.8 and 111 / 127, twelve 53.2 / 52.0 and
// 208 / 209, seven of 64^3 44.4 / 50.5 and 190 / 193, three of 100 x 90 x 70 (92 and 222 MB) 46.7 /
// 50.7 and 220 / 212, two of 128 x 96 x 80 39.3 / 48.0 and 180 / 191, four (forward only, 189 MB)
// 77.9 / 84.6.
inline bool batch_rows(bool tiles_set, const fd3d_ctx *const *ctx, int ns, int arrays)
{
    if (tiles_set) return false;
    RowSize size;
    if (ns == 1 && arrays == kForwardArrays) return kernels_of(ctx[0], arrays) == Kern::rows;
    for (int q = 0; q < ns; ++q) {
        const fd3d_ctx *c = ctx[q];
        if (!rows_ok(c) || (!unselected(c, arrays) && c->variant != FD3D_KERNEL_CELL)) return false;
        size.add(c, arrays);
    }
    return size.pays(ctx[0]->tsize);
}

// Where the batch workspace holds the shots' row maps.
inline const ShotRows *batch_row_maps(const fd3d_batch *b) { return (const ShotRows *)(b->ws + b->off_rows); }

// Kernels of the batched gradient, which steps every shot in each launch: the group of its adjoint
// passes and recompute (gr.rows: row kernels), and whether its forward runs rows.
inline bool gradient_group(const fd3d_batch *b, BatchGroup &gr)
{
    const bool tiles = b->grad_x != 0 && (b->grad_x > 0 || b->tiles_set);
    auto shot = [&](int q) { return b->ctx[q]; };
    gr = whole_batch(b);
    if (b->grad_x > 0) {
        gr.tx = b->grad_x;
        gr.ty = b->grad_y;
        gr.tx2 = gr.ty2 = 0;
        gr.every_zc = b->grad_z > 0 ? b->grad_z : 1 << 30;
    } else if (batch_rows(tiles, b->ctx.data(), b->nshot, kAdjointArrays)) {
        gr.rows = batch_row_maps(b);
    } else {
        fit_sweeps(gr, b->nshot, tiles, shot);
    }
    return batch_rows(tiles, b->ctx.data(), b->nshot, kForwardArrays);
}

// Working set of one shot in the step loop: nine fields and the three model arrays.
inline size_t shot_footprint(const fd3d_ctx *c) { return (size_t)12 * c->n[0] * c->n[1] * c->n[2] * c->tsize; }

// Groups of the batch's schedule and their kernels: rows (batch_rows) or sweeps.  The sweeps of a
// cache-blocked group whose shots all have the tile kernel selected, or are tuned, with one shape of
// their own use that shape; the others the batch's selected shapes, or without those
// what fits the shots with nothing selected (fit_sweeps).
inline void make_groups(fd3d_batch *b)
{
    b->groups.clear();
    b->order.resize(b->nshot);
    for (int s = 0; s < b->nshot; ++s) b->order[s] = s;
    BatchGroup all = whole_batch(b);
    // with neither schedule nor tile shapes selected, groups that stay in the Infinity Cache
    // (one shot per group where a shot alone exceeds it): three shots of 128^3 112 us per step against
    // 120 in lockstep, two each of 128^3, 192 x 192 x 128 and 256 x 256 x 128 584 against 716
    const size_t budget = b->sched_set || b->tiles_set ? b->group_bytes : (size_t)kRowBytes32;
    if (budget == 0) {
        if (batch_rows(b->tiles_set, b->ctx.data(), b->nshot, kForwardArrays)) all.rows = batch_row_maps(b);
        else fit_sweeps(all, b->nshot, b->tiles_set, [&](int q) { return b->ctx[q]; });
        b->groups.push_back(all);
        return;
    }
    std::stable_sort(b->order.begin(), b->order.end(),
                     [&](int x, int y) { return shot_footprint(b->ctx[x]) < shot_footprint(b->ctx[y]); });
    auto ctx_at = [&](int p) { return b->ctx[b->order[p]]; };
    int s = 0;
    while (s < b->nshot) {
        BatchGroup g = all;
        g.s0 = s;
        size_t bytes = shot_footprint(ctx_at(s));
        int e = s + 1;
        while (e < b->nshot && bytes + shot_footprint(ctx_at(e)) <= budget) bytes += shot_footprint(ctx_at(e++));
        g.ns = e - s;
        std::vector<const fd3d_ctx *> members;
        for (int q = s; q < e; ++q) members.push_back(ctx_at(q));
        g.ntp = group_streams(members.data(), g.ns);
        if (batch_rows(b->tiles_set, members.data(), g.ns, kForwardArrays)) g.rows = batch_row_maps(b) + g.s0;
        const fd3d_ctx *c0 = ctx_at(s);
        auto tiled = [](const fd3d_ctx *c) {
            return !c->auto_kernel && (c->variant == FD3D_KERNEL_TILE || (c->variant == FD3D_KERNEL_CELL && c->tuned));
        };
        bool same = tiled(c0);
        for (int q = s + 1; q < e && same; ++q)
            same = tiled(ctx_at(q)) && ctx_at(q)->tile_x == c0->tile_x && ctx_at(q)->tile_y == c0->tile_y;
        if (same && tile_supported(b->tsize, c0->tile_x, c0->tile_y)) {
            g.tx = c0->tile_x;
            g.ty = c0->tile_y;
            g.tx2 = g.ty2 = 0;
        }
        if (!g.rows) fit_sweeps(g, g.ns, b->tiles_set, [&](int q) { return ctx_at(s + q); });
        b->groups.push_back(g);
        s = e;
    }
}

// Whether the batch's sequence is captured into a graph when asked; a longer one is launched step by
// step.  Groups multiply the two launches per step of lockstep.  A graph of 64000 launches costs 0.12
// s and 114 MB of host memory to build, and its replays take as long as the single launches (eight
// shots of 64^3, 4000 steps 0.341 s either way; of 128 x 128 x 96 1.002 and 0.993 s); building one
// of 256000 ended the process with a segmentation fault.
constexpr long kMaxGraphLaunches = 65536;
inline bool graph_fits(const fd3d_batch *b) { return 2L * b->nt * (long)b->groups.size() <= kMaxGraphLaunches; }

} // namespace fd3d

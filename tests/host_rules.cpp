// Prints what the library's host rules choose; built and read by test_host_rules_cpu.py.
// One question per line of stdin: "sweep <tsize> <coarse> <nx ny nz> ..." asks for the tile
// shape and depth of a launch over the grids, "rows <tsize> <coarse> <nx ny nz> [<receiver items> 1 1]" whether
// the row kernels take a grid, the map of their launch and its grid of blocks,
// "groups <tsize> 0 <tile_x> <tile_y> <group MiB> {<nx ny nz> <kernel> 0 0}..." the groups of a batch:
// tile_x 0: no tile shapes selected, group MiB -1: no schedule, kernel: -1 none or FD3D_KERNEL_*
// (tiles of 64 x 16), 10 more: the tuner's; answers shots, rows, tile_x, tile_y of each group.
// "graph <tsize> 0 <steps> 0 <group MiB> {as groups}..." whether a batch's sequence is captured.
// "kern <tsize> <coarse> 0 0 0 <nx ny nz> <kernel> 0 0" what forward, Born and adjoint run
// (0 rows, 1 sweeps, 2 kernels with a bounds test per load).  "tuner <tsize> 0 <nx ny nz>" runs
// fd3d_autotune where there is no device, so that it fails, and prints its return code and
// whether the context still has nothing selected.
#include "batch_plan.h"

#include <cstdio>
#include <iostream>
#include <sstream>

static fd3d_ctx grid(int nx, int ny, int nz, int tsize, int coarse)
{
    fd3d_ctx c{};
    c.n[0] = nx;
    c.n[1] = ny;
    c.n[2] = nz;
    c.tsize = tsize;
    c.window = fd3d::kMaxWindowBytes;
    c.opts.coarse[0] = c.opts.coarse[1] = c.opts.coarse[2] = coarse;
    // the library's automatic layout (interleaved rows when the whole depth fits one window)
    c.L.rows = 9.0 * nx * ny * nz * tsize <= (double)fd3d::kMaxWindowBytes;
    return c;
}

int main()
{
    for (std::string line; std::getline(std::cin, line);) {
        std::istringstream in(line);
        std::string what;
        int ts, cm, nx, ny, nz;
        in >> what >> ts >> cm;
        std::vector<fd3d_ctx> g;
        int tx = 0, ty = 0, mib = 0;
        const bool select = what == "groups" || what == "kern" || what == "graph";
        if (select) in >> tx >> ty >> mib;
        while (in >> nx >> ny >> nz) {
            g.push_back(grid(nx, ny, nz, ts, cm));
            if (!select) continue;
            int kernel, a, b;
            in >> kernel >> a >> b;
            fd3d_ctx &c = g.back();
            c.auto_kernel = kernel < 0;
            c.tuned = kernel >= 10;
            c.variant = kernel >= 10 ? kernel - 10 : kernel;
            c.tile_x = 64;
            c.tile_y = 16;
            c.zchunk = 32;
        }
        if (what == "sweep") {
            const fd3d::Sweep s = fd3d::choose_sweep((int)g.size(), [&](int q) { return &g[q]; });
            std::printf("%d %d", s.tx, s.ty);
            for (auto &c : g) std::printf(" %d", s.zc ? fd3d::sweep_depth(&c, s.zc) : 0);
            std::printf("\n");
        } else if (what == "groups" || what == "graph") {
            const bool graph = what == "graph";
            const int steps = tx;
            if (graph) tx = 0;
            fd3d_batch b{};
            char ws = 0;
            b.nshot = (int)g.size();
            for (auto &c : g) b.ctx.push_back(&c);
            b.tsize = ts;
            b.ws = &ws;  // row maps: an address to compare with null
            b.tile_x = tx ? tx : 64;
            b.tile_y = tx ? ty : 8;
            b.tiles_set = tx > 0;
            b.sched_set = mib >= 0;
            b.group_bytes = mib > 0 ? (size_t)mib << 20 : 0;
            fd3d::make_groups(&b);
            if (graph) {
                b.nt = steps;
                std::printf("%d\n", (int)fd3d::graph_fits(&b));
                continue;
            }
            for (const fd3d::BatchGroup &r : b.groups) std::printf("%d %d %d %d ", r.ns, (int)(r.rows != nullptr), r.tx, r.ty);
            std::printf("\n");
        } else if (what == "kern") {
            for (int a : {fd3d::kForwardArrays, fd3d::kBornArrays, fd3d::kAdjointArrays})
                std::printf("%d ", (int)fd3d::kernels_of(&g[0], a));
            std::printf("\n");
        } else if (what == "tuner") {
            int n = 0;
            if (hipGetDeviceCount(&n) == hipSuccess && n > 0) return 1;  // no workspace to run on
            g[0].auto_kernel = true;
            const int rc = fd3d_autotune(&g[0], 1, nullptr, nullptr, nullptr);
            std::printf("%d %d\n", rc, (int)g[0].auto_kernel);
        } else if (what == "rows") {
            const fd3d::RowMap r = fd3d::row_map(&g[0]);
            const dim3 b = fd3d::row_grid(r, g.size() > 1 ? g[1].n[0] : 0);
            std::printf("%d %d %d %d %d %d %d %d %d %u %u %u\n", (int)fd3d::rows_ok(&g[0]), r.lbx, r.ntx, r.rps, r.ns, r.nslab,
                        r.np, r.cpx, r.tiles(), b.x, b.y, b.z);
        }
    }
}

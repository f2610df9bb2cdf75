"""The host's launch rules, asked on the CPU: host_rules.cpp is compiled against the library's
own csrc/host.h (host pass only, no device needed) and answers one question per line."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    from paper_2112_15071_amd import build as B

    exe = str(tmp_path_factory.mktemp("host_rules") / "host_rules")
    subprocess.run([B.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-std=c++17", "-O1", "-w",
                    "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, os.path.join(ROOT, "tests", "host_rules.cpp"),
                    "-o", exe, "-x", "none", B.LIB, "-Wl,-rpath," + os.path.dirname(B.LIB)], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
        rows = [[int(v) for v in r.split()] for r in out.splitlines()]
        assert len(rows) == len(lines)
        return rows

    return run


# Launches with nothing selected that a narrow tile or one round of whole-depth sweeps made
# slower than a fixed sweep of the tile as wide as the rows; the shape and depth measured fastest
# on MI355X (or within 2 % of it).
SWEEPS = [("4 0", [(230, 230, 230)], (256, 4, 58)), ("4 0", [(230, 300, 260)], (256, 4, 87)),
          ("4 0", [(256, 256, 256)], (256, 4, 64)), ("4 0", [(300, 300, 200)], (128, 8, 100)),
          ("4 0", [(260, 260, 260)], (64, 16, 87)), ("4 0", [(200, 180, 160)], (256, 4, 32)),
          ("4 0", [(160, 150, 100)] * 4, (64, 16, 50)), ("4 0", [(260, 200, 150)] * 3, (128, 8, 150)),
          ("4 0", [(230, 230, 230)] * 2, (256, 4, 115)),
          ("4 1", [(64, 64, 64)], (64, 4, 4)), ("4 1", [(192, 192, 128)], (64, 4, 19)),
          ("8 0", [(120, 112, 104)], (128, 4, 12)), ("8 0", [(150, 150, 100)], (64, 8, 25))]


def test_default_sweeps(ask):
    lines = [f"sweep {k[0]} {9 * int(k[2])} " + " ".join("%d %d %d" % g for g in grids) for k, grids, _ in SWEEPS]
    for (k, grids, want), got in zip(SWEEPS, ask(lines)):
        assert tuple(got[:3]) == want, (k, grids, got)


def test_default_sweeps_stay_within_the_limits(ask):
    """Over all sizes (uneven launches included): a supported shape, depths of 4 planes up, and
    windows (depth + 8 planes, at most the grid's) within 1 GiB, also where planes are so large
    that only short sweeps fit."""
    import random

    rng = random.Random(3)
    sizes = lambda: tuple(int(round(4 * 2 ** rng.uniform(0, 9.5))) for _ in range(3))
    cases = [(ts, [sizes() for _ in range(rng.choice([1, 1, 2, 5]))]) for _ in range(300) for ts in (4, 8)]
    cases = [(ts, [g for g in gs if g[0] * g[1] * g[2] < 2 ** 30] or [(4, 4, 4)]) for ts, gs in cases]
    cases += [(4, [(4096, 4096, 24)]), (4, [(8192, 3000, 60)]), (8, [(4096, 2048, 100)])]
    shapes = {4: {(64, 4), (64, 8), (64, 16), (128, 4), (128, 8), (256, 4)}, 8: {(64, 4), (64, 8), (128, 4)}}
    rows = ask([f"sweep {ts} 0 " + " ".join("%d %d %d" % g for g in gs) for ts, gs in cases])
    for (ts, gs), r in zip(cases, rows):
        assert tuple(r[:2]) in shapes[ts], (ts, gs, r)
        for (nx, ny, nz), zc in zip(gs, r[2:]):
            rows_of = 9 if 9 * nx * ny * nz * ts <= 2 ** 30 else 1
            plane = rows_of * nx * ny * ts
            if zc == 0:  # no sweep: not even one of 4 planes fits
                assert min(12, nz) * plane > 2 ** 30, (ts, gs, r)
            else:
                assert zc >= 4 and min(zc + 8, nz) * plane <= 2 ** 30, (ts, gs, r)


def test_row_launches_fit_the_grid_of_blocks(ask):
    """A row launch covers every row and plane and stays within 65535 blocks along y and z, or the
    row kernels refuse the grid: tall grids of many strips (16 x 4096 x 4200: 16 pieces of 4200
    planes per XCD), long thin ones, and random ones.  Receivers that do not fit beside the planes
    are left to a launch of their own (x = 0)."""
    import random

    rng = random.Random(5)
    grids = [(16, 4096, 4200), (16, 4096, 4095), (4, 4, 600000), (4, 100000, 1000), (2000000, 4, 4), (64, 64, 64),
             (149, 101, 87), (7, 6, 5), (300, 130, 12)]
    for _ in range(400):
        g = tuple(int(round(4 * 2 ** rng.uniform(0, 17))) for _ in range(3))
        if g[0] * g[1] * g[2] < 2 ** 31 - 1:
            grids.append(g)
    rows = ask([f"rows 4 0 {x} {y} {z}" for x, y, z in grids])
    seen = {True: 0, False: 0}
    for (nx, ny, nz), (ok, lbx, ntx, rps, ns, nslab, np_, cpx, tiles, bx, by, bz) in zip(grids, rows):
        assert ntx << lbx >= nx and ns * rps * (256 >> lbx) >= ny and nslab * np_ >= nz and 8 * cpx >= ns * nslab
        assert tiles == rps * ntx
        if ok:
            assert (bx, by, bz) == (8, tiles, np_ * cpx) and by <= 65535 and bz <= 65535, (nx, ny, nz)
        seen[bool(ok)] += 1
    assert not rows[0][0] and rows[1][0] and not rows[2][0]
    assert seen[True] > 100 and seen[False] > 10
    # 64^3 (8 planes per XCD, 16 tiles): 32768 items per layer of blocks
    per = 8 * 16 * 256
    few, most, many = ask([f"rows 4 0 64 64 64 {q} 1 1" for q in (1, per * (65535 - 8), per * (65535 - 8) + 1)])
    assert few[9:] == [8, 16, 9] and most[9:] == [8, 16, 65535] and many[9] == 0


CELL, TILE, NONE, TUNED_CELL, TUNED_TILE = 0, 1, -1, 10, 11
SMALL, OTHER = (64, 64, 64), (96, 80, 72)  # 12 and 25 MiB of fields and model


def groups(ask, tiles, mib, shots, ts=4):
    line = f"groups {ts} 0 {tiles[0]} {tiles[1]} {mib} " + " ".join("%d %d %d %d 0 0" % (*g, k) for g, k in shots)
    r = ask([line])[0]
    return [tuple(r[i:i + 4]) for i in range(0, len(r), 4)]


@pytest.mark.parametrize("kernel", [NONE, CELL])
def test_selected_batch_tiles_exclude_the_rows(ask, kernel):
    """Row kernels only where the batch has no tile shapes selected, in lockstep (0) and in
    groups (16 MiB: one shot each; 64: both); with shapes selected, those, except where a group's
    shots have a tile of their own selected."""
    shots = [(SMALL, kernel), (OTHER, kernel)]
    for mib in (-1, 0, 16, 64):
        assert all(rows for _, rows, _, _ in groups(ask, (0, 0), mib, shots)), mib
        n = 2 if mib == 16 else 1
        assert [g[1:] for g in groups(ask, (128, 8), mib, shots)] == [(0, 128, 8)] * n, mib
    own = [(SMALL, TILE), (OTHER, kernel)]
    assert [g[1:] for g in groups(ask, (128, 8), 16, own)] == [(0, 64, 16), (0, 128, 8)]
    assert [g[1:] for g in groups(ask, (128, 8), 64, own)] == [(0, 128, 8)]


def test_kernels_of_an_operation(ask):
    """With nothing selected every operation goes by the size of its arrays, with a kernel
    selected by that, and with a tuned one only the forward by that."""
    rows, sweeps = 0, 1
    cases = [((64, 64, 64), NONE, [rows] * 3), ((160, 150, 100), NONE, [rows, rows, sweeps]),
             ((192, 160, 128), NONE, [rows, sweeps, sweeps]), ((256, 256, 256), NONE, [sweeps] * 3),
             ((192, 160, 128), CELL, [rows] * 3), ((64, 64, 64), TILE, [sweeps] * 3),
             ((192, 160, 128), TUNED_CELL, [rows, sweeps, sweeps]), ((64, 64, 64), TUNED_TILE, [sweeps, rows, rows]),
             ((256, 256, 256), TUNED_CELL, [rows, sweeps, sweeps]), ((160, 150, 100), TUNED_CELL, [rows, rows, sweeps])]
    got = ask([f"kern 4 0 0 0 0 %d %d %d {k} 0 0" % g for g, k, _ in cases])
    for (g, k, want), r in zip(cases, got):
        assert r == want, (g, k)


def test_failed_tuner_leaves_nothing_selected(ask):
    """Without a device the tuner's events cannot be created: FD3D_EHIP, and the context's
    operations still pick their kernels."""
    import torch

    if torch.cuda.is_available():
        pytest.skip("needs a machine without a GPU")
    assert ask(["tuner 4 0 64 64 64"]) == [[-6, 1]]


def test_groups_use_the_tuned_sweep(ask):
    """Shots tuned to the cell variant keep the fastest sweep's tile (64 x 16 here) beside it; a
    group of them that exceeds the cache, and so runs sweeps, uses it, as one of shots tuned to
    that tile does; shots with the cell variant merely selected have no tile of their own."""
    big = (160, 150, 140)  # 154 MiB
    for kernel, tile in ((TUNED_CELL, (64, 16)), (TUNED_TILE, (64, 16)), (CELL, (64, 8))):
        assert groups(ask, (0, 0), 400, [(big, kernel), (big, kernel)]) == [(2, 0, *tile)], kernel
    assert groups(ask, (0, 0), 400, [(big, TUNED_CELL), (big, TUNED_TILE)]) == [(2, 0, 64, 16)]
    assert [g[1] for g in groups(ask, (0, 0), 160, [(big, TUNED_CELL)] * 2)] == [1, 1]


def test_fp64_rows_by_their_lanes(ask):
    """In FP64 every operation, and the shots of a launch together, run rows up to 400 thousand
    lanes, or 660 thousand with nine in ten filled (measured on both sides)."""
    cases = [((64, 64, 64), 0), ((48, 80, 64), 0), ((120, 64, 64), 0), ((128, 80, 64), 0), ((72, 56, 56), 1),
             ((72, 64, 64), 1), ((90, 60, 60), 1), ((128, 82, 64), 1), ((120, 112, 104), 1)]
    got = ask(["kern 8 0 0 0 0 %d %d %d -1 0 0" % g for g, _ in cases])
    for (g, want), r in zip(cases, got):
        assert r == [want] * 3, g
    for shots, want in ([(64, 64, 64)] * 2, 1), ([(40, 40, 40)] * 3, 1), ([(40, 40, 40)] * 6, 0):
        assert [g[1] for g in groups(ask, (0, 0), 0, [(s, NONE) for s in shots], ts=8)] == [want], shots


def test_long_sequences_are_not_captured(ask):
    """A batch's sequence becomes a graph up to 65536 launches, two per step and group: in
    lockstep by the steps alone, in groups by their number too."""
    shots = lambda n: " ".join("64 64 64 -1 0 0" for _ in range(n))
    cases = [(32768, 0, 24, 1), (32769, 0, 1, 0), (4096, 12, 8, 1), (4097, 12, 8, 0), (8000, 12, 16, 0), (8000, -1, 16, 1)]
    got = ask([f"graph 4 0 {nt} 0 {mib} {shots(n)}" for nt, mib, n, _ in cases])
    assert [r[0] for r in got] == [c[3] for c in cases]

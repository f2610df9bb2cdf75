"""Row kernels (the cell variant, and the default on grids that stay in the cache): the same
operations per sample as the tile sweeps, so every operation gives the same bits with either.
Sizes at the edges of a row block (64, 128, 256 columns), of its rows, of the slabs and strips
that are dealt to the XCDs (planes above 128 KiB are cut into strips), and smaller than all of
them.  The tile sweeps themselves are compared with the oracle elsewhere."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

H, DT, NT = 10.0, 5e-4, 9
SIZES = [(7, 6, 5), (63, 9, 17), (64, 16, 8), (65, 33, 9), (130, 21, 10), (257, 11, 7), (192, 190, 6), (300, 130, 12)]


def setup(shape, seed=11):
    nx, ny, nz = shape
    lam, mu, rho = W.layered_perturbed(shape, H, seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    mid = np.array(shape) / 2 - 0.4  # within a few cells of the source, which the waves reach
    rec = np.clip(mid + rng.uniform(-4, 4, (9, 3)), 0.6, np.array(shape) - 2.6)
    shot = dict(src_pos=(nx / 2 - 0.3, ny / 2 - 0.2, nz / 2 - 0.45), moment=W.random_mt(rng, 1e15), force=(2e9, -1e9, 3e9),
                wavelet=np.linspace(1.0, 2.0, NT), rec_pos=rec)
    return (lam, mu, rho), shot


def both(model, dtype, fn, **kw):
    """fn(sim) with the row kernels and with a tile sweep."""
    from paper_2112_15071_amd import Simulator

    out = []
    for kernel in (("cell", 4, 8, 64), ("tile", 8, 5, 64)):
        sim = Simulator(*model, H, DT, NT, dtype=dtype, sponge=3, **kw)
        sim.set_kernel(*kernel)
        out.append([t.clone() for t in fn(sim)])
        sim.close()
    return out


def same(out):
    for k, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a, b), f"output {k}: {int((a != b).sum())} values differ"
        assert bool(torch.isfinite(a).all()) and float(a.abs().max()) > 0.0, f"output {k} is zero or not finite"


@pytest.mark.parametrize("shape", SIZES)
@pytest.mark.parametrize("opts", [dict(), dict(free_surface=True), dict(vacuum_top=2), dict(layout="separate")],
                         ids=["damped", "free", "vacuum", "separate"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_forward(shape, opts, dtype):
    (lam, mu, rho), shot = setup(shape)
    same(both((lam, mu, rho), dtype, lambda s: (s.forward(**shot), s.state()), **opts))


@pytest.mark.parametrize("shape", SIZES[1:])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_gradient_and_born(shape, dtype):
    model, shot = setup(shape)

    def gradient(sim):
        g = [torch.zeros_like(sim.lam) for _ in range(3)]
        gws = sim.grad_workspace(4)
        obs = torch.zeros((len(shot["rec_pos"]), 3, NT), dtype=dtype, device="cuda")
        tr, J = sim.gradient(gws, obs, *g, **shot)
        return (tr, J, *g, sim.adjoint_state(gws))

    same(both(model, dtype, gradient))
    rng = np.random.Generator(np.random.PCG64(3))
    dm = [0.02 * m * rng.standard_normal(m.shape) for m in model]
    same(both(model, dtype, lambda s: s.born(*dm, **shot)))


@pytest.mark.parametrize("shape", [(40, 36, 20), (160, 150, 100), (300, 260, 80)])
def test_default_choice(shape):
    """With no kernel selected, small working sets run the rows and large ones the sweeps; the
    operations of one context may differ in that (160 x 150 x 100: the forward's arrays fit the
    cache, the adjoint's do not) and still give the selected kernels' bits."""
    from paper_2112_15071_amd import Simulator

    model, shot = setup(shape)
    sim = Simulator(*model, H, DT, NT, sponge=3)
    assert sim.kernel()["variant"] == ("cell" if np.prod(shape) < 3e6 else "tile")
    ref = Simulator(*model, H, DT, NT, sponge=3)
    ref.set_kernel("tile", 8, 16, 64)
    res = []
    for s in (sim, ref):
        g = [torch.zeros_like(s.lam) for _ in range(3)]
        obs = torch.zeros((len(shot["rec_pos"]), 3, NT), device="cuda")
        tr, J = s.gradient(s.grad_workspace(4), obs, *g, **shot)
        res.append([tr, J, *g, *s.born(*(0.01 * m for m in model), **shot)])
        s.close()
    same(res)


@pytest.mark.parametrize("select", [False, True])
def test_batch(select):
    """A batch of uneven shots with no kernel selected runs the rows in lockstep and in groups,
    eager and from a graph, forward and gradient, and equals the tile sweeps (select: the cell
    kernels chosen on every shot)."""
    from paper_2112_15071_amd import Simulator
    from paper_2112_15071_amd.batch import BatchSimulator

    shapes = [(40, 33, 21), (70, 20, 9), (192, 190, 6)]
    parts = [setup(s, seed=30 + k) for k, s in enumerate(shapes)]
    sims = [Simulator(*m, H, DT, NT, sponge=3) for m, _ in parts]
    shots = [sh for _, sh in parts]
    if select:
        for s in sims:
            s.set_kernel("cell", 4, 8, 64)
    obs = [torch.zeros((len(sh["rec_pos"]), 3, NT), device="cuda") for sh in shots]

    def gradient(batch):
        g = [[torch.zeros_like(s.lam) for s in sims] for _ in range(3)]
        tr, J = batch.gradient(shots, obs, *g, ckpt_every=4)
        return [*tr, J, *(x for q in g for x in q)]

    batch = BatchSimulator(sims)
    rows = [[t.clone() for t in batch.forward(shots, use_graph=graph)] for graph in (False, True, True)]
    batch.set_schedule(1 << 20)
    rows += [[t.clone() for t in batch.forward(shots, use_graph=False)]]
    batch.set_schedule(0)
    grad = gradient(batch)
    batch.close()
    batch = BatchSimulator(sims)
    batch.set_kernel(64, 8)
    ref = [t.clone() for t in batch.forward(shots, use_graph=False)]
    for r in rows:
        same([r, ref])
    same([grad, gradient(batch)])
    batch.close()
    for s in sims:
        s.close()


@pytest.mark.parametrize("tune", [False, True])
def test_batch_default_groups(tune):
    """Shots that exceed the cache together run in groups when no schedule is selected (one shot
    alone, two rows shots, one sweep of a large shot), untuned and tuned, and equal the lockstep."""
    from paper_2112_15071_amd import Simulator
    from paper_2112_15071_amd.batch import BatchSimulator

    shapes = [(256, 200, 110), (120, 110, 100), (128, 96, 80), (130, 128, 120)]  # 258, 60, 45, 92 MiB
    parts = [setup(s, seed=50 + k) for k, s in enumerate(shapes)]
    sims = [Simulator(*m, H, DT, NT, sponge=3) for m, _ in parts]
    shots = [sh for _, sh in parts]
    batch = BatchSimulator(sims)
    if tune:
        batch.autotune(1, cache=False)
    out = [[t.clone() for t in batch.forward(shots, use_graph=graph)] for graph in (False, True, True)]
    batch.close()
    batch = BatchSimulator(sims)
    batch.set_kernel(64, 8)
    batch.set_schedule(0)
    ref = [t.clone() for t in batch.forward(shots, use_graph=False)]
    for r in out:
        same([r, ref])
    batch.close()
    for s in sims:
        s.close()


@pytest.mark.parametrize("shape", [(4, 5, 70000), (70000, 4, 5), (5, 70000, 4)])
def test_thin_grids(shape):
    """Rows, planes and column blocks by the ten thousand: the longest axis decides which of a
    launch's dimensions grows (planes per slab, strips, blocks of a row)."""
    (lam, mu, rho), shot = setup((12, 11, 10))
    n = max(shape)
    model = [m.mean() * (1.0 + 0.1 * np.sin(np.arange(np.prod(shape)) / 3.0).reshape(shape[::-1])) for m in (lam, mu, rho)]
    pos = np.array([0.5 * k if k == n else 1.6 for k in shape])
    shot["src_pos"] = tuple(pos)
    shot["rec_pos"] = [pos + [2.2 if k == n else 0.2 for k in shape]]
    same(both(model, torch.float32, lambda s: (s.forward(**shot), s.state())))

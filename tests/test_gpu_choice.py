"""Which kernels a call runs (from a trace of its launches) after the tuners and the calls that
carry a kernel choice from one simulator to another.  All kernels give the same bits, so only the
launches can tell."""
from __future__ import annotations

import json
import re

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

H, DT, NT = 10.0, 5e-4, 3
SMALL = (40, 36, 32)      # every operation's arrays stay in the cache: rows
MIDDLE = (192, 160, 128)  # the forward's do (180 MiB), Born's (360) and the adjoint's (435) do not


def launched(fn) -> set:
    """Names of the library's kernels that fn launches."""
    from torch.profiler import ProfilerActivity, profile

    fn()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    names = {m.group(1) for e in p.key_averages() for m in [re.search(r"fd3d::(\w+)<", e.key)] if m}
    assert names, "no launch was recorded"
    return names


def simulator(shape, nt=NT, **kw):
    from paper_2112_15071_amd import Simulator

    nx, ny, nz = shape
    lam = torch.full((nz, ny, nx), 7.5e9, device="cuda")
    return Simulator(lam, lam, torch.full_like(lam, 2500.0), H, DT, nt, sponge=3, **kw)


def shot(shape, nt=NT):
    mid = np.array(shape) / 2 + 0.3
    return dict(src_pos=tuple(mid), moment=W.explosion(1e15), wavelet=np.ones(nt), rec_pos=[mid + 2, mid - 3])


def gradient(sim):
    obs = torch.zeros((2, 3, sim.nt), device="cuda")
    g = [torch.zeros_like(sim.lam) for _ in range(3)]
    gws = sim.grad_workspace(2)
    return lambda: sim.gradient(gws, obs, *g, **shot(sim.shape, sim.nt))


def born(sim):
    return lambda: sim.born(sim.lam, sim.lam, sim.rho, **shot(sim.shape, sim.nt))


def forward(sim):
    return lambda: sim.forward(**shot(sim.shape, sim.nt))


ROWS = dict(forward={"vel_row", "stress_row"}, gradient={"vel_row_io", "stress_row_io"}, born={"vel_row_io", "stress_row_io"})
SWEEPS = dict(forward={"vel_tile", "stress_tile"}, gradient={"vel_tile_adj", "stress_tile_adj"},
              born={"vel_tile_adj", "stress_tile_born"})


def runs(sim, what) -> str:
    names = launched(dict(forward=forward, gradient=gradient, born=born)[what](sim))
    rows, sweeps = ROWS[what] <= names, SWEEPS[what] <= names
    assert rows != sweeps, names
    return "rows" if rows else "sweeps"


@pytest.mark.parametrize("cached", [False, True])
def test_forward_tuner_leaves_the_other_operations_alone(cached, tmp_path, monkeypatch):
    """The forward of a tuned simulator runs the tuner's kernel; Born and the gradient, which it
    did not time, rows or sweeps by the size of their arrays, on the simulator that was tuned and
    (cached: the cell variant as the saved winner) on one that takes the saved result."""
    monkeypatch.setenv("FD3D_AUTOTUNE_CACHE", str(tmp_path / "tuned.json"))
    for shape, others in ((SMALL, "rows"), (MIDDLE, "sweeps")):
        sim = simulator(shape)
        sim.autotune(steps=1)
        if cached:
            sim.close()
            table = json.loads((tmp_path / "tuned.json").read_text())
            for e in table.values():
                e["variant"] = "cell"
            (tmp_path / "tuned.json").write_text(json.dumps(table))
            sim = simulator(shape)
            assert sim.autotune(steps=1)["cached"] and sim.kernel()["variant"] == "cell"
        variant = sim.kernel()["variant"]
        if variant != "fused":
            assert runs(sim, "forward") == {"cell": "rows", "tile": "sweeps"}[variant], shape
            assert runs(sim, "born") == others, shape
        assert runs(sim, "gradient") == others, shape
        sim.close()


def test_selected_kernel_runs_every_operation():
    sim = simulator(MIDDLE)
    for kernel, want in ((("cell", 4, 8, 64), "rows"), (("tile", 4, 32, 256), "sweeps")):
        sim.set_kernel(*kernel)
        assert [runs(sim, w) for w in ("forward", "born", "gradient")] == [want] * 3
    sim.close()


@pytest.mark.parametrize("state", ["default", "tuned", "selected"])
def test_copies_carry_the_choice(state):
    """Simulator.like, and the z chunk that the batched-gradient tuner sets, leave what was
    selected, tuned or open as it is (MIDDLE: the forward of an open choice runs rows, the other
    operations sweeps)."""
    from paper_2112_15071_amd.batch import BatchSimulator

    sim = simulator(MIDDLE)
    want = ["rows", "sweeps", "sweeps"]
    if state == "tuned":
        sim.set_tuned(dict(variant="cell", tile_x=256, tile_y=4, zchunk=32))
    elif state == "selected":
        sim.set_kernel("cell", 4, 32, 64)
        want = ["rows"] * 3
    BatchSimulator._set_zchunk([sim], 16)
    assert sim.kernel()["zchunk"] == 16
    copy = sim.like(NT + 1)
    assert copy.kernel() == sim.kernel()
    for s in (sim, copy):
        assert [runs(s, w) for w in ("forward", "born", "gradient")] == want
        s.close()


def test_copy_and_depth_are_checked():
    from paper_2112_15071_amd import _abi

    a, b, c = simulator(SMALL), simulator((41, 36, 32)), simulator(SMALL, dtype=torch.float64)
    for other in (b, c):
        with pytest.raises(_abi.FD3DError) as e:
            _abi.fd3d_copy_kernel(a.ctx, other.ctx)
        assert e.value.code == _abi.FD3D_EINVAL
    with pytest.raises(_abi.FD3DError):
        _abi.fd3d_set_zchunk(a.ctx, 3)
    _abi.fd3d_limit_window(a.ctx, 12 * 9 * 40 * 36 * 4)  # sweeps of 4 planes
    _abi.fd3d_set_zchunk(a.ctx, 4)
    with pytest.raises(_abi.FD3DError):
        _abi.fd3d_set_zchunk(a.ctx, 5)
    for s in (a, b, c):
        s.close()


@pytest.mark.parametrize("selected", ["background", "perturbation"])
def test_born_with_one_selected_context(selected):
    """A kernel selected on one of Born's two contexts runs both when the other has nothing
    selected (SMALL: an open choice is rows), with the bits of the open choice."""
    from paper_2112_15071_amd import _abi
    from paper_2112_15071_amd.simulator import make_source

    ref = simulator(SMALL)
    born(ref)()
    want = [ref.state(), ref._born_sim.state()]  # three steps reach few receivers: the whole states
    assert runs(ref, "born") == "rows" and all(float(x.abs().max()) > 0 for x in want)
    from paper_2112_15071_amd import Simulator

    a = simulator(SMALL)
    b = Simulator(a.lam, a.mu, a.rho, H, DT, NT, sponge=3, layout=a.layout())
    (a if selected == "background" else b).set_kernel("tile", 8, 32, 64)
    sh = shot(SMALL)
    rec = np.array(sh["rec_pos"], dtype=np.float64)
    w = torch.ones(NT, device="cuda")
    out = [torch.zeros((2, 3, NT), device="cuda") for _ in range(2)]
    src = make_source(sh["src_pos"], sh["moment"], (0.0,) * 3, w)

    def call():
        _abi.fd3d_born(a.ctx, b.ctx, src, a.lam.data_ptr(), a.lam.data_ptr(), a.rho.data_ptr(), 2, rec.ctypes.data,
                       out[0].data_ptr(), out[1].data_ptr(), torch.cuda.current_stream().cuda_stream)

    assert SWEEPS["born"] <= launched(call)
    assert torch.equal(a.state(), want[0]) and torch.equal(b.state(), want[1])
    for s in (ref, a, b):
        s.close()


def test_gradient_tuner_tries_the_rows_and_the_own_sweep():
    """The tuner's candidates hold the row kernels and the sweep that the grid would run untuned
    (60 x 50 x 45: no fixed candidate's), so that the fastest found is no slower than either."""
    shape = (60, 50, 45)
    sim = simulator(shape, nt=40)
    k = sim.kernel()
    own = f"tile,{k['tile_x']},{k['tile_y']},{k['zchunk']}"
    assert tuple(own.split(",")) not in [tuple(map(str, c)) for c in sim.GRADIENT_CANDIDATES]
    t = sim.autotune_gradient(shot(shape, 40))
    assert "cell,64,8,32" in t["tried"] and own in t["tried"]
    k = sim.kernel()
    assert f"{k['variant']},{k['tile_x']},{k['tile_y']}," in min(t["tried"], key=t["tried"].get) + ","
    assert runs(sim, "gradient") == {"cell": "rows", "tile": "sweeps"}[k["variant"]]
    t = sim.autotune_gradient(shot(shape, 40), candidates=[("tile", 64, 8, 32)])  # the caller's only
    assert list(t["tried"]) == ["tile,64,8,32"] and sim.kernel()["variant"] == "tile"
    sim.close()


def batch_of(n=2):
    from paper_2112_15071_amd.batch import BatchSimulator

    sims = [simulator(SMALL, nt=6) for _ in range(n)]
    return BatchSimulator(sims), sims, [shot(SMALL, 6)] * n


def batch_runs(batch, sims, shots, what) -> str:
    obs = [torch.zeros((2, 3, s.nt), device="cuda") for s in sims]
    g = [[torch.zeros_like(s.lam) for s in sims] for _ in range(3)]
    call = {"forward": lambda: batch.forward(shots, use_graph=False),
            "gradient": lambda: batch.gradient(shots, obs, *g, ckpt_every=3)}[what]
    names = launched(call)
    kinds = {k for k in ("row", "tile") if {f"vel_{k}_multi", f"stress_{k}_multi"} & names}
    assert len(kinds) == 1, names
    return {"row": "rows", "tile": "sweeps"}[kinds.pop()]


def test_batched_gradient_tuner_leaves_the_forward_alone():
    """Two small shots: forward and gradient run rows by default.  The gradient tuner tries that
    too, and what it sets counts for the gradient alone, until tiles are selected on the batch."""
    batch, sims, shots = batch_of()
    both = lambda: [batch_runs(batch, sims, shots, w) for w in ("forward", "gradient")]
    assert both() == ["rows", "rows"]
    zc = sims[0].kernel()["zchunk"]
    t = batch.autotune_gradient(shots, steps=6, ckpt_every=3)
    assert "0x0,4" in t["tried"] and len(t["tried"]) > 5
    assert both() == ["rows", "rows" if t["tile"] == [0, 0] else "sweeps"]
    assert t["zchunk"] == sims[0].kernel()["zchunk"] and (t["tile"] != [0, 0] or t["zchunk"] == zc)
    t = batch.autotune_gradient(shots, steps=6, ckpt_every=3, candidates=[(64, 8, 16)])
    assert t["tile"] == [64, 8] and t["zchunk"] == 16 == sims[1].kernel()["zchunk"]
    assert both() == ["rows", "sweeps"]
    t = batch.autotune_gradient(shots, steps=6, ckpt_every=3, candidates=[(0, 0, 4)])
    assert both() == ["rows", "rows"]
    batch.set_kernel(64, 8)
    assert both() == ["sweeps", "sweeps"]
    batch.close()
    for s in sims:
        s.close()


def test_batched_gradient_kernels_give_the_same_bits():
    """Every shape and depth (whole, ragged, deeper than the grid) of the gradient's sweeps, and
    the library's choice; unsupported shapes and depths are refused."""
    from paper_2112_15071_amd import _abi

    batch, sims, shots = batch_of()
    rng = np.random.default_rng(2)
    obs = [torch.as_tensor(rng.standard_normal((2, 3, 6)) * 1e-6, dtype=torch.float32, device="cuda") for _ in sims]
    ref = None
    for k in [(0, 0, 0), (64, 8, 0), (64, 16, 5), (128, 4, 64), (256, 4, 32)]:
        batch.set_gradient_kernel(*k)
        g = [[torch.zeros_like(s.lam) for s in sims] for _ in range(3)]
        tr, J = batch.gradient(shots, obs, *g, ckpt_every=4)
        out = [*tr, J, *(x for q in g for x in q)]
        ref = ref or out
        assert all(torch.equal(a, b) for a, b in zip(ref, out)), k
    assert all(float(x.abs().max()) > 0 for x in ref[-6:])
    for bad in [(64, 5, 8), (0, 8, 8), (64, 8, 3), (-1, -1, 0)]:
        with pytest.raises(_abi.FD3DError):
            batch.set_gradient_kernel(*bad)
    batch.close()
    for s in sims:
        s.close()


def test_saved_tuning_of_another_version_is_not_taken(tmp_path, monkeypatch):
    """A saved result counts for the library version that timed it: a table without the version
    in its keys, or of another one, is tuned anew and kept beside."""
    from paper_2112_15071_amd import _abi

    path = tmp_path / "tuned.json"
    monkeypatch.setenv("FD3D_AUTOTUNE_CACHE", str(path))
    sim = simulator(SMALL)
    assert not sim.autotune(steps=1)["cached"] and sim.autotune(steps=1)["cached"]
    (key, e), = json.loads(path.read_text()).items()
    assert key.endswith(_abi.fd3d_version())
    for old in (key[:-len(_abi.fd3d_version()) - 1], key + ".older"):
        path.write_text(json.dumps({old: e}))
        assert not sim.autotune(steps=1)["cached"]
        assert set(json.loads(path.read_text())) == {old, key}
    sim.close()

"""The kernels with a bounds test per load (vel_cell, stress_cell, their adjoint and the Born
source passes), which the cell variant runs where a few planes exceed the row kernels' buffer
window.  fd3d_limit_window brings them to small grids: every selection of the cell variant in
the tests called here gets a window of one byte first.  Tolerances are those of the other
kernels' tests."""
import numpy as np
import pytest
import torch

import test_gpu_born as born
import test_gpu_forward as forward
import test_gpu_gradient as gradient
import test_gpu_vacuum as vacuum
from gpu_cases import compare, gpu_run, oracle_run
from helpers import rel_l2
from test_gpu_gradient import case  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

CELL = ("cell", 4, 8, 64)


@pytest.fixture(autouse=True)
def bounds(monkeypatch):
    from paper_2112_15071_amd import Simulator, _abi

    plain = Simulator.set_kernel
    limited = []

    def set_kernel(self, variant="tile", *a, **kw):
        if variant == "cell":
            _abi.fd3d_limit_window(self.ctx, 1)
            with pytest.raises(_abi.FD3DError):  # no sweep fits
                plain(self, "tile", 4, 4, 64)
            limited.append(self)
        plain(self, variant, *a, **kw)

    monkeypatch.setattr(Simulator, "set_kernel", set_kernel)
    yield limited
    assert limited, "no context ran the kernels under test"


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("free_surface", [False, True])
@pytest.mark.parametrize("layout", ["rows", "separate"])
def test_forward(dtype, free_surface, layout):
    """Against the oracle, and bit for bit the tile sweep."""
    shot = forward.ragged_shot(free_surface, 77 + int(free_surface), True)
    got = gpu_run(shot, dtype, kernel=CELL, layout=layout)
    compare(got, oracle_run(shot), forward.TOL[dtype], f"bounds fs={free_surface} {layout}")
    ref = gpu_run(shot, dtype, kernel=("tile", 8, 5, 64), layout=layout)
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_vacuum(dtype):
    shot = vacuum.vacuum_shot(True, (10.0, 12.0, 8.0))
    got = gpu_run(shot, dtype, kernel=CELL, vacuum_top=vacuum.KS)
    compare(got, vacuum.run_oracle(shot), forward.TOL[dtype], "bounds vacuum")


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-4), (torch.float64, 1e-10)])
def test_gradient(case, dtype, tol):  # noqa: F811
    """The buoyancy gradient from each step's v^{n+1/2} and v^{n-1/2}; the row kernels' sum by
    parts rounds otherwise, so equal bits would mean that those ran."""
    from paper_2112_15071_amd import Simulator

    model, shots, d_obs, g_ref = case
    _, g = gradient.gpu_gradient(model, shots, d_obs, dtype, ckpt_every=7, kernel=CELL)
    for p in range(3):
        assert rel_l2(g[p], g_ref[p]) <= tol, (p, rel_l2(g[p], g_ref[p]))
    _, rows = gradient.gpu_gradient(model, shots, d_obs, dtype, ckpt_every=7)
    assert not np.array_equal(g[2], rows[2])


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-4), (torch.float64, 1e-10)])
def test_gradient_from_a_given_initial_state(dtype, tol):
    gradient.test_gradient_from_a_given_initial_state(CELL, dtype, tol)


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-4), (torch.float64, 1e-12)])
@pytest.mark.parametrize("kind", ["moment", "force"])
def test_born(dtype, tol, kind):
    born.test_born_matches_oracle(dtype, tol, kind, CELL, (10.0, 12.0, 8.0))


def test_largest_window():
    """The tile sweep whose windows are exactly 1 GiB against 64-bit addresses and bounds tests
    (the row kernels share the sweeps' window offsets)."""
    forward.test_largest_tile_window_equals_cell()

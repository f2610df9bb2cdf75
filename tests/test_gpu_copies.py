"""Copies and fills around the step loop: state access at row lengths and alignments that take
16-byte or single-sample accesses, a gradient workspace whose previous contents must not
matter, and the final reductions of the misfit and the model statistics."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as W
from helpers import active_mask

pytestmark = pytest.mark.gpu

H, DT = 10.0, 5e-4


def simulator(shape, nt, dtype, **kw):
    from paper_2112_15071_amd import Simulator

    return Simulator(*W.layered_perturbed(shape, H, 17), H, DT, nt, dtype=dtype, sponge=3, **kw)


@pytest.mark.parametrize("layout", ["rows", "separate"])
@pytest.mark.parametrize("nx,offset", [(64, 0), (64, 1), (62, 0), (61, 3), (4, 2)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_state_round_trip(nx, offset, layout, dtype):
    """set_state then get_state returns the samples with the pinned slots zeroed, from and to
    arrays that start `offset` samples past an aligned address."""
    from paper_2112_15071_amd import _abi

    shape = (nx, 9, 7)
    n = nx * 9 * 7
    sim = simulator(shape, 4, dtype, layout=layout)
    src = torch.randn(9, n + offset, dtype=dtype, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    dst = torch.full((9, n + offset), float("nan"), dtype=dtype, device="cuda")
    stream = int(torch.cuda.current_stream().cuda_stream)
    _abi.fd3d_set_state(sim.ctx, [src[f, offset:].data_ptr() for f in range(9)], stream)
    _abi.fd3d_get_state(sim.ctx, [dst[f, offset:].data_ptr() for f in range(9)], stream)
    torch.cuda.synchronize()
    for f in range(9):
        keep = torch.as_tensor(active_mask(f, shape), device="cuda").reshape(-1)
        assert torch.equal(dst[f, offset:], torch.where(keep, src[f, offset:], torch.zeros_like(src[f, offset:])))
        assert bool(torch.isnan(dst[f, :offset]).all())
    sim.close()


@pytest.mark.parametrize("kernel", [("cell", 4, 8, 64), ("tile", 8, 16, 64)])
@pytest.mark.parametrize("layout", ["rows", "separate"])
def test_gradient_workspace_contents(kernel, layout):
    """A workspace full of NaN gives the gradient that a zeroed one gives, at segment lengths
    that leave one, two and no free slots in the last group; the misfit is half the squared
    residual summed in 64 bits."""
    shape, nt = (40, 33, 18), 11
    nx, ny, nz = shape
    rng = np.random.Generator(np.random.PCG64(4))
    rec = np.array([nx / 2, ny / 2, nz / 2]) + rng.uniform(-4, 4, (7, 3))
    shot = dict(src_pos=(nx / 2, ny / 2, nz / 2), moment=W.random_mt(rng, 1e15), wavelet=np.linspace(1, 2, nt), rec_pos=rec)
    sim = simulator(shape, nt, torch.float32, layout=layout)
    sim.set_kernel(*kernel)
    obs = torch.zeros((7, 3, nt), device="cuda")
    for k in (4, 5, 6, 11):
        out = []
        for fill in (0, 255):  # 255: NaN in every sample
            gws = sim.grad_workspace(k)
            gws.fill_(fill)
            g = [torch.zeros_like(sim.lam) for _ in range(3)]
            tr, J = sim.gradient(gws, obs, *g, **shot)
            out.append([tr, J, *g])
        for a, b in zip(*out):
            assert torch.equal(a, b) and float(a.abs().max()) > 0.0
        ref = 0.5 * float((tr.double() ** 2).sum())
        assert abs(float(J) - ref) <= 4e-7 * ref  # the residual in FP32, then one rounding
    sim.close()


def test_model_statistics():
    """The statistics that create reads back, against torch on the same arrays."""
    sim = simulator((70, 33, 21), 4, torch.float64)
    vp = torch.sqrt((sim.lam + 2 * sim.mu) / sim.rho)
    vs = torch.sqrt(sim.mu / sim.rho)
    got = sim.info()
    for a, b in zip(got[:3], (vp.max(), vs.min(), sim.rho.min())):
        assert abs(a - float(b)) <= 1e-14 * float(b)
    sim.close()

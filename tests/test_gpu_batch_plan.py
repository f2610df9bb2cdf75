"""Batches in the launch configurations that a default or a selection chooses: groups of one and
of several shots with row kernels, sweeps beside them, and lockstep with the library's sweep."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import test_gpu_batch as batches
from test_gpu_choice import launched
from test_gpu_rows import DT, H, NT, setup

pytestmark = pytest.mark.gpu


def run_groups(shapes, budget, kinds):
    """Forward of the batch in groups (budget None: the library's), eager and replayed from a
    graph, against lockstep sweeps; kinds: which multi-shot kernels the groups launch."""
    from paper_2112_15071_amd import Simulator
    from paper_2112_15071_amd.batch import BatchSimulator

    parts = [setup(s, seed=70 + k) for k, s in enumerate(shapes)]
    sims = [Simulator(*m, H, DT, NT, sponge=3) for m, _ in parts]
    shots = [sh for _, sh in parts]
    batch = BatchSimulator(sims)
    if budget is not None:
        batch.set_schedule(budget)
    got = []
    for graph in (False, True, True):
        got.append([t.clone() for t in batch.forward(shots, use_graph=graph)] + [s.state() for s in sims])
    names = launched(lambda: batch.forward(shots, use_graph=False))
    assert {k for k in ("row", "tile") if f"stress_{k}_multi" in names} == set(kinds), names
    batch.close()
    batch = BatchSimulator(sims)
    batch.set_kernel(64, 8)
    ref = [t.clone() for t in batch.forward(shots, use_graph=False)] + [s.state() for s in sims]
    for out in got:
        for k, (a, b) in enumerate(zip(out, ref)):
            assert torch.equal(a, b), k
    assert all(float(t.abs().max()) > 0 for t in ref)
    batch.close()
    for s in sims:
        s.close()


def test_default_groups_of_one_and_of_several_shots():
    """72, 91, 151 and 258 MiB under the library's 230 MiB, out of order: two rows shots, one rows
    shot alone (third in the order) and one sweep of the large shot."""
    run_groups([(256, 200, 110), (120, 110, 119), (130, 128, 120), (160, 150, 137)], None, ["row", "tile"])


def test_rows_groups_of_several_shots_after_the_first():
    """12 to 16 MiB under 30 MiB: groups of two, two and one, all rows."""
    run_groups([(64, 64, n) for n in (84, 64, 70, 76, 80)], 30 << 20, ["row"])


@pytest.mark.parametrize("group_bytes", [0, 4 << 20])
def test_rows_with_many_receivers(group_bytes, monkeypatch):
    """700, 1, 350 and 45 receivers sampled by the first blocks of the row launches (3288 items in
    13 blocks, shot boundaries inside a block), against single-shot sweeps and the oracle."""
    from paper_2112_15071_amd.batch import BatchSimulator

    monkeypatch.setattr(BatchSimulator, "set_kernel", lambda self, *tile: None)  # nothing selected
    batches.test_many_receivers_batch_equals_single_shots(group_bytes)


def test_full_size_lockstep(monkeypatch):
    """The 24 shots at full size in lockstep, with the sweep that the library picks for all."""
    from paper_2112_15071_amd.batch import BatchSimulator

    init = BatchSimulator.__init__

    def lockstep(self, sims):
        init(self, sims)
        self.set_schedule(0)

    monkeypatch.setattr(BatchSimulator, "__init__", lockstep)
    batches.test_full_size_uneven_batch_truncated()


def test_long_sequence():
    """Two shots of 20000 steps in groups of one (80000 launches, more than are captured) give the
    lockstep batch's traces (40000 launches, a graph), asked for a graph twice each."""
    from paper_2112_15071_amd import Simulator
    from paper_2112_15071_amd.batch import BatchSimulator

    nt = 20000
    (model, sh) = setup((7, 6, 5))
    sh["wavelet"] = np.exp(-((np.arange(nt) - 30.0) / 9.0) ** 2)
    sims = [Simulator(*model, H, DT, nt, sponge=3) for _ in range(2)]
    out = []
    for budget in (1, 0):
        batch = BatchSimulator(sims)
        batch.set_schedule(budget)
        for _ in range(2):
            out.append([t.clone() for t in batch.forward([sh, sh], use_graph=True)])
        batch.close()
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], o))
    assert all(float(t.abs().max()) > 0 for t in out[0])
    for s in sims:
        s.close()

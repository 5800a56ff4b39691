"""Calls at the edges of what the on-chip preconditioner changed around itself: they do
what they did by sweep launches."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import grid_of, ragged_stack, rise_err, say, t64
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 3 + ["TIM", "TIM", "Cu", "Cu"]


@pytest.mark.parametrize("nx,ny,nz", [(16383, 1, 16), (16255, 2, 15), (13057, 3, 8)])
def test_long_thin_grids_solve_in_every_precision(nx, ny, nz):
    """Odd rows as long as the device has compute units: the smaller tiles that CG takes
    beside an on-chip preconditioner are four times as many here, and the outer residual
    keeps five sums for each."""
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=True)
    g, P = grid_of(st), t64(np.random.default_rng(nx).uniform(0.0, 1e-3, nx * ny * nz))
    ref = g.solve(P, precision="fp64")[0].cpu().numpy()
    for precision in ("mixed", "adaptive"):
        say(f"long thin {nx}x{ny}x{nz} {precision}")
        T, _ = g.solve(P, precision=precision)
        assert rise_err(T.cpu().numpy(), ref, st.t_amb) <= 1.01e-8
    g.close()


def test_without_memory_for_the_exchange(monkeypatch):
    """No room for the tiles' exchange (a limit of 0 MiB): solves, batches and
    applications run by sweep launches."""
    sts = [ragged_stack(130, 70, LAYERS[:9], mult=True), ragged_stack(64, 20, LAYERS[:3], mult=True, seed=5)]
    P = [t64(np.random.default_rng(q).uniform(0.0, 1e-3, st.n)) for q, st in enumerate(sts)]
    r = torch.as_tensor(np.random.default_rng(3).standard_normal(sts[0].n), dtype=torch.float32, device="cuda")

    def results():
        grids = [grid_of(st) for st in sts]
        b = grids[0].spectral_bounds()
        out = [grids[0].precond_apply(x, b["lmin"], b["lmax"], 12) for x in (r, r.double())]
        stats = []
        for precision in ("mixed", "adaptive", "fp64"):
            say(f"no memory for the exchange: {precision}")
            T, s = grids[0].solve(P[0], precision=precision)
            out.append(T)
            stats.append(s)
            if precision != "adaptive":
                Ts, ss = solve_batch(grids, P, precision=precision)
                out += Ts
                stats += ss
        for g in grids:
            g.close()
        return out, [s["alg_bytes"] / s["cg_iters"] for s in stats]

    monkeypatch.setenv("CUTH_GRAPH", "0")
    on_chip = results()[1]
    monkeypatch.setenv("CUTH_RESIDENT_MB", "0")
    got, launched = results()
    assert all(a > 2 * b for a, b in zip(launched, on_chip))
    monkeypatch.setenv("CUTH_RESIDENT", "0")
    want = results()[0]
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    for T, ref in zip(got[2:], want[2:]):   # (the tiles of the CG sums differ: bits may)
        assert rise_err(T.cpu().numpy(), ref.cpu().numpy(), sts[0].t_amb) <= 2.02e-8

"""Calls at the edges of what the on-chip preconditioner changed around itself: they do
what they did by sweep launches."""

from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import grid_of, ragged_stack, rise_err, say, t64

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

"""The on-chip Chebyshev preconditioner on 17 to 20 layers: tiles of 14 rows
(per-layer conductances, up to two x-edge cells a lane) and of 4 and 8."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import fp32_cheb_bar, grid_of, ragged_stack, rise_err, say, t32, t64
from oracle import assembly, krylov
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 4 + ["TIM", "TIM", "Cu", "Cu"]
# tiles of 4 and of 8 rows; of 14 with ragged columns and rows (257 x 460: 165 of
# them, 290 of 8 rows), and in slabs (the last)
SHAPES = [(1, 1, 18), (64, 4, 17), (65, 9, 20), (130, 131, 18), (257, 460, 19), (129, 1210, 17)]


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,nz", SHAPES[1:])   # (one column: too few modes for a Lanczos interval)
def test_preconditioner_matches_oracle(nx, ny, nz, per_cell):
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=per_cell, seed=nx + nz)
    A = assembly.assemble(st)
    g = grid_of(st)
    r = np.random.default_rng(nx * ny).standard_normal(st.n).astype(np.float32).astype(np.float64)
    v0 = np.random.default_rng(4).standard_normal(st.n)
    for jacobi in (False, True):
        name = "chebyshev_jacobi" if jacobi else "chebyshev"
        lo, hi = (krylov.jacobi_spectral_bounds if jacobi else krylov.spectral_bounds)(A, v0)
        for degree in (2, 3, 8, 67) if st.n < 200000 else (5, 30):
            say(f"tall {nx}x{ny}x{nz} {'cells' if per_cell else 'layers'} {name} k={degree}")
            if jacobi:
                ref = krylov.jacobi_chebyshev_precondition(A, r, lo, hi, degree)
            else:
                ref = krylov.chebyshev_precondition(lambda v: A @ v, r, lo, hi, degree)
            z = g.precond_apply(t32(r), lo, hi, degree, preconditioner=name)
            bar = fp32_cheb_bar(A, r, lo, hi, degree, ref, jacobi=jacobi)
            assert np.abs(z.cpu().numpy().astype(np.float64) - ref).max() <= bar
            assert torch.equal(z, g.precond_apply(t32(r), lo, hi, degree, preconditioner=name))
    g.close()


@pytest.mark.parametrize("spin", ["", "1"])
def test_solves_and_batches(monkeypatch, spin):
    """Against FP64 solves (bar: the documented 1e-8 of the largest rise, plus the
    FP64 reference's own 1e-10): alone, in a batch of such stacks only, and with
    thinner ones, whose tiles then have 8 rows too."""
    sts = [ragged_stack(nx, ny, LAYERS[:nz], mult=False, seed=q) for q, (nx, ny, nz) in enumerate(SHAPES)]
    sts.append(ragged_stack(70, 50, LAYERS[:9], mult=False, seed=9))
    grids = [grid_of(st) for st in sts]
    P = [np.random.default_rng(st.n).uniform(0.0, 1e-3, st.n) for st in sts]
    ref = [g.solve(t64(p), precision="fp64")[0].cpu().numpy() for g, p in zip(grids, P)]
    if spin:
        monkeypatch.setenv("CUTH_RESIDENT_SPIN", spin)
    for pc in ("chebyshev", "chebyshev_jacobi"):
        for n in (len(SHAPES), len(sts)):
            say(f"tall batch of {n} {pc} spin={spin}")
            T, _ = solve_batch(grids[:n], [t64(p) for p in P[:n]], precision="mixed", preconditioner=pc)
            for a, b, st in zip(T, ref, sts):
                assert rise_err(a.cpu().numpy(), b, st.t_amb) <= 1.01e-8
    for g, p, b, st in zip(grids, P, ref, sts):
        T, _ = g.solve(t64(p), precision="mixed")
        assert rise_err(T.cpu().numpy(), b, st.t_amb) <= 1.01e-8
        g.close()

"""The on-chip Chebyshev preconditioner on FP64 vectors: by itself against the
oracle, inside solves and batches, in slabs, and when its tiles give up."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import fp32_cheb_bar, grid_of, ragged_stack, rise_err, say, t64
from oracle import assembly, krylov
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 3 + ["TIM", "TIM", "Cu", "Cu"]
# the edges of its tiles (64 columns; 4 or 8 rows) and layer counts (8, 12, 16);
# the last two in slabs where the conductances are per cell
SHAPES = [(5, 3, 2), (64, 4, 8), (65, 5, 9), (63, 17, 12), (129, 33, 13), (128, 64, 16), (191, 259, 7),
          (513, 300, 3), (128, 1090, 9)]


def _power(st):
    return np.random.default_rng(st.n).uniform(0.0, 1e-3, st.n)


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,nz", SHAPES)
def test_preconditioner_matches_oracle(nx, ny, nz, per_cell):
    """Bar: the FP32 one (which the FP32 rounding of the oracle's own listing
    sets), scaled by the ratio of the unit roundoffs, 2^-53 / 2^-24, once for the
    kernel and once for the oracle, whose FP64 rounding is of the same size."""
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=per_cell, seed=nx + nz)
    A = assembly.assemble(st)
    g = grid_of(st)
    r = np.random.default_rng(nx * ny).standard_normal(st.n)
    v0 = np.random.default_rng(4).standard_normal(st.n)
    for jacobi in (False, True):
        name = "chebyshev_jacobi" if jacobi else "chebyshev"
        lo, hi = (krylov.jacobi_spectral_bounds if jacobi else krylov.spectral_bounds)(A, v0)
        for degree in (2, 3, 8, 67) if st.n < 200000 else (5, 30):
            say(f"on chip fp64 {nx}x{ny}x{nz} {'cells' if per_cell else 'layers'} {name} k={degree}")
            if jacobi:
                ref = krylov.jacobi_chebyshev_precondition(A, r, lo, hi, degree)
            else:
                ref = krylov.chebyshev_precondition(lambda v: A @ v, r, lo, hi, degree)
            z = g.precond_apply(t64(r), lo, hi, degree, preconditioner=name)
            bar = 2.0 * 2.0 ** -29 * fp32_cheb_bar(A, r, lo, hi, degree, ref, jacobi=jacobi)
            assert np.abs(z.cpu().numpy() - ref).max() <= bar
            y = torch.empty_like(z)
            assert torch.equal(z, g.precond_apply_noalloc(t64(r), y, lo, hi, degree, preconditioner=name))
    g.close()


@pytest.mark.parametrize("spin", ["", "1"])
@pytest.mark.parametrize("graph", ["0", "1"])
def test_solves_and_batches(monkeypatch, graph, spin):
    """Against the same solves by sweep launches.  Bar: both meet the relative
    residual of 1e-10 that FP64 solves stop at, whose rise errors the parity tests
    hold to 1e-10 each."""
    monkeypatch.setenv("CUTH_GRAPH", graph)
    sizes = [(70, 50, 3), (130, 33, 9), (192, 100, 13), (64, 64, 8)]
    sts = [ragged_stack(nx, ny, LAYERS[:nz], mult=q != 1, seed=q) for q, (nx, ny, nz) in enumerate(sizes)]
    grids = [grid_of(st) for st in sts]
    P = [_power(st) for st in sts]

    def all_of(pc):
        single = [g.solve(t64(p), precision="fp64", preconditioner=pc) for g, p in zip(grids, P)]
        T, s = solve_batch(grids, [t64(p) for p in P], precision="fp64", preconditioner=pc)
        return [x.cpu().numpy() for x, _ in single] + [x.cpu().numpy() for x in T], [x for _, x in single] + list(s)

    for pc in ("chebyshev", "chebyshev_jacobi"):
        monkeypatch.setenv("CUTH_RESIDENT", "0")
        ref, s0 = all_of(pc)
        monkeypatch.delenv("CUTH_RESIDENT")
        if spin:
            monkeypatch.setenv("CUTH_RESIDENT_SPIN", spin)
        for call in range(2):
            say(f"on chip fp64 solves {pc} graph={graph} spin={spin} call {call}")
            got, s1 = all_of(pc)
            for q, (a, b) in enumerate(zip(got, ref)):
                assert rise_err(a, b, sts[q % len(sts)].t_amb) <= 2e-10
                if not spin:   # the sweeps ran on chip
                    assert s1[q]["alg_bytes"] / s1[q]["cg_iters"] < s0[q]["alg_bytes"] / s0[q]["cg_iters"]
    for g in grids:
        g.close()

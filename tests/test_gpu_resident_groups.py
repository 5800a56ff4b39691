"""The on-chip Chebyshev preconditioner over several groups of tiles: grids of more
tiles than the device has compute units, which go through it in slabs of rows
with recomputed halos, and batches, where every problem is a group."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import fp32_cheb_bar, grid_of, ragged_stack, rise_err, say, t32, t64
from oracle import assembly, krylov
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 3 + ["TIM", "TIM", "Cu", "Cu"]
# (64 x 16 columns a tile, 256 tiles at once): one column of tiles; two, ragged in
# both directions; eight and nine with slabs of uneven last rows; all three layer classes
SLABS = [(1, 5000, 3), (65, 2100, 9), (129, 1500, 3), (512, 530, 2), (570, 460, 13)]


def _power(st):
    return np.random.default_rng(st.n).uniform(0.0, 1e-3, st.n)


def _per_iter(stats):
    return stats["alg_bytes"] / max(stats["cg_iters"], 1)


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,nz", SLABS)
def test_slabs_match_oracle(nx, ny, nz, per_cell):
    """One application against the oracle's polynomial.  A wrong halo shows as an
    error of z's own size in the rows next to a cut."""
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=per_cell, seed=nx + nz)
    A = assembly.assemble(st)
    g = grid_of(st)
    r = np.random.default_rng(nx * ny).standard_normal(st.n).astype(np.float32).astype(np.float64)
    v0 = np.random.default_rng(4).standard_normal(st.n)
    for jacobi in (False, True):
        name = "chebyshev_jacobi" if jacobi else "chebyshev"
        lo, hi = (krylov.jacobi_spectral_bounds if jacobi else krylov.spectral_bounds)(A, v0)
        for degree in (2, 7, 30):
            say(f"slabs {nx}x{ny}x{nz} {'cells' if per_cell else 'layers'} {name} k={degree}")
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
@pytest.mark.parametrize("nx,ny,nz", SLABS[1:3])
def test_solves_in_slabs(monkeypatch, nx, ny, nz, spin):
    """Solves against FP64 (bar: the documented 1e-8 of the largest rise, plus the
    FP64 reference's own 1e-10), also when tiles give up after one poll."""
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=True)
    g = grid_of(st)
    P = t64(_power(st))
    ref = g.solve(P, precision="fp64")[0].cpu().numpy()
    if spin:
        monkeypatch.setenv("CUTH_RESIDENT_SPIN", spin)
    for precision, pc in [("mixed", "chebyshev"), ("mixed16", "chebyshev"), ("adaptive", "chebyshev_jacobi")]:
        say(f"slabs {nx}x{ny}x{nz} {precision} {pc} spin={spin}")
        T, s = g.solve(P, precision=precision, preconditioner=pc)
        assert rise_err(T.cpu().numpy(), ref, st.t_amb) <= 1.01e-8
        if not spin:
            monkeypatch.setenv("CUTH_RESIDENT", "0")
            s0 = g.solve(P, precision=precision, preconditioner=pc)[1]
            monkeypatch.delenv("CUTH_RESIDENT")
            assert _per_iter(s) < _per_iter(s0)   # the sweeps ran on chip
    g.close()


@pytest.mark.parametrize("spin", ["", "1"])
@pytest.mark.parametrize("graph", ["0", "1"])
def test_batches_on_chip(monkeypatch, graph, spin):
    """Batches of per-layer and per-cell stacks of every layer class, one of them
    in slabs, over two calls, against FP64 solves; and when tiles give up."""
    monkeypatch.setenv("CUTH_GRAPH", graph)
    sizes = [(70, 50, 3), (64, 64, 8), (130, 33, 9), (5, 7, 12), (192, 200, 13), (65, 2100, 4)]
    sts = [ragged_stack(nx, ny, LAYERS[:nz], mult=q % 2 == 1, seed=q) for q, (nx, ny, nz) in enumerate(sizes)]
    grids = [grid_of(st) for st in sts]
    if spin:
        monkeypatch.setenv("CUTH_RESIDENT_SPIN", spin)
    for call in range(2):
        P = [np.stack([_power(st) * (1 + call), _power(st)[::-1] * 0.3]) for st in sts]
        for pc in ("chebyshev", "chebyshev_jacobi"):
            say(f"on-chip batch {pc} graph={graph} spin={spin} call {call}")
            T, s = solve_batch(grids, [t64(p.ravel()) for p in P], nrhs=2, precision="mixed", preconditioner=pc)
            for q, st in enumerate(sts):
                for m in range(2):
                    ref = grids[q].solve(t64(P[q][m].copy()), precision="fp64")[0].cpu().numpy()
                    got = T[q].view(2, -1)[m].cpu().numpy()
                    assert rise_err(got, ref, st.t_amb) <= 1.01e-8
    for g in grids:
        g.close()

"""The on-chip Chebyshev preconditioner (every sweep in one launch), by itself
and inside solves: grids at the edges of its tiles (64 columns; 4, 8 or 16 rows) and of
its layer counts (8, 12, 16), per-layer and per-cell conductivities, against the
oracle and FP64 solves, and the way back to sweep launches when its tiles wait in
vain for each other.

That it ran shows in a solve's algorithmic bytes (its sweeps read and write
their vectors once per application)."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as w
from gpu_helpers import fp32_cheb_bar, grid_of, ragged_stack, rise_err, say, t32, t64
from oracle import assembly, krylov

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 3 + ["TIM", "TIM", "Cu", "Cu"]
SHAPES = [(1, 1, 1), (5, 3, 2), (64, 4, 8), (65, 5, 9), (63, 17, 12), (129, 33, 13), (128, 64, 16),
          (191, 259, 7), (256, 256, 3), (257, 511, 5), (512, 512, 2)]


def _power(st):
    return np.random.default_rng(st.n).uniform(0.0, 1e-3, st.n)


def _per_iter(stats):
    return stats["alg_bytes"] / max(stats["cg_iters"], 1)


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,nz", SHAPES[1:])   # (one cell: its interval is a point)
def test_preconditioner_matches_oracle(nx, ny, nz, per_cell):
    """One application against the oracle's polynomial, at degrees that end on
    either of the kernel's two buffers and past its 64 constants at a time."""
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=per_cell, seed=nx + nz)
    A = assembly.assemble(st)
    g = grid_of(st)
    r = np.random.default_rng(nx * ny).standard_normal(st.n).astype(np.float32).astype(np.float64)
    v0 = np.random.default_rng(4).standard_normal(st.n)
    for jacobi in (False, True):
        name = "chebyshev_jacobi" if jacobi else "chebyshev"
        lo, hi = (krylov.jacobi_spectral_bounds if jacobi else krylov.spectral_bounds)(A, v0)
        for degree in (2, 3, 8, 67) if st.n < 200000 else (5,):
            say(f"on chip {nx}x{ny}x{nz} {'cells' if per_cell else 'layers'} {name} k={degree}")
            if jacobi:
                ref = krylov.jacobi_chebyshev_precondition(A, r, lo, hi, degree)
            else:
                ref = krylov.chebyshev_precondition(lambda v: A @ v, r, lo, hi, degree)
            z = g.precond_apply(t32(r), lo, hi, degree, preconditioner=name)
            bar = fp32_cheb_bar(A, r, lo, hi, degree, ref, jacobi=jacobi)
            assert np.abs(z.cpu().numpy().astype(np.float64) - ref).max() <= bar
            assert torch.equal(z, g.precond_apply(t32(r), lo, hi, degree, preconditioner=name))
    g.close()


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,nz", SHAPES)
def test_solves_on_chip(monkeypatch, nx, ny, nz, per_cell):
    """Mixed, mixed16, stage-switched and Jacobi-scaled solves against the FP64
    solve of the same system.  Bar: the mixed solves' documented 1e-8 of the
    largest rise, plus the FP64 reference's own 1e-10."""
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=per_cell, seed=nx + nz)
    g = grid_of(st)
    P = t64(_power(st))
    ref = g.solve(P, precision="fp64")[0].cpu().numpy()
    runs = [("mixed", "chebyshev", 30), ("mixed", "chebyshev_jacobi", 17), ("adaptive", "chebyshev", 8),
            ("mixed", "chebyshev", 2)]
    for precision, pc, degree in runs + ([("mixed16", "chebyshev", 7)] if per_cell else []):
        say(f"on chip {nx}x{ny}x{nz} {'cells' if per_cell else 'layers'} {precision} {pc} k={degree}")
        kw = dict(precision=precision, preconditioner=pc, cheb_degree=degree)
        T, s = g.solve(P, **kw)
        assert rise_err(T.cpu().numpy(), ref, st.t_amb) <= 1.01e-8
        monkeypatch.setenv("CUTH_RESIDENT", "0")
        s0 = g.solve(P, **kw)[1]
        monkeypatch.delenv("CUTH_RESIDENT")
        if degree > 2:
            assert _per_iter(s) < _per_iter(s0)   # the sweeps ran on chip
    g.close()


def test_repeat_solves_are_bitwise_equal():
    """Two solves by the same launches (the second knows where the first
    stopped) return the same bits."""
    st = ragged_stack(130, 70, LAYERS[:12], mult=True)
    g = grid_of(st)
    P = t64(_power(st))
    T = [g.solve(P, precision="mixed")[0] for _ in range(3)]
    assert bool((T[0] == T[1]).all()) and bool((T[1] == T[2]).all())
    g.close()


@pytest.mark.parametrize("precision,pc", [("mixed", "chebyshev"), ("mixed", "chebyshev_jacobi"),
                                          ("adaptive", "chebyshev")])
@pytest.mark.parametrize("graph", ["0", "1"])
def test_tiles_that_give_up(monkeypatch, precision, pc, graph):
    """A bound of one poll: tiles give up on a neighbour whose values are not
    there yet.  The solve goes on with sweep launches, reports no error and
    meets the same bar; after two such applications the handle keeps to sweep
    launches (their bytes show it)."""
    monkeypatch.setenv("CUTH_GRAPH", graph)
    st = ragged_stack(200, 100, LAYERS[:10], mult=True)
    g = grid_of(st)
    P = t64(_power(st))
    ref = g.solve(P, precision="fp64")[0].cpu().numpy()
    monkeypatch.setenv("CUTH_RESIDENT_SPIN", "1")
    for q in range(4):
        say(f"one poll {precision} {pc} graph={graph} solve {q}")
        T, s = g.solve(P, precision=precision, preconditioner=pc)
        assert rise_err(T.cpu().numpy(), ref, st.t_amb) <= 1.01e-8
    monkeypatch.setenv("CUTH_RESIDENT", "0")
    s0 = g.solve(P, precision=precision, preconditioner=pc)[1]
    assert _per_iter(s) == pytest.approx(_per_iter(s0), rel=0.2)
    g.close()


def test_transient_steps_on_chip():
    """Backward-Euler steps (capacity in every layer's sink) against FP64."""
    st = w.uniform_stack(150, 67, LAYERS[:11])
    g = grid_of(st)
    P = t64(_power(st))
    T = t64(np.full(st.n, st.t_amb))
    for step in range(3):
        say(f"on-chip transient step {step}")
        a, _ = g.transient_step(1e-4, P, T, precision="mixed")
        b, _ = g.transient_step(1e-4, P, T, precision="fp64")
        assert rise_err(a.cpu().numpy(), b.cpu().numpy(), st.t_amb) <= 1.01e-8
        T = b
    g.close()

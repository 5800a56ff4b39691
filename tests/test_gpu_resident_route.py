"""Which calls the on-chip preconditioner takes: where it is the shorter way, and with
CUTH_RESIDENT=1 wherever it fits.  A call that it does not take returns the bits of the
same call with CUTH_RESIDENT=0; one that it takes returns others and moves less."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import fp32_cheb_bar, grid_of, ragged_stack, rise_err, say, t32, t64
from oracle import assembly, krylov
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 4 + ["TIM", "TIM", "Cu", "Cu"]


def _power(n, q=0):
    return t64(np.random.default_rng(n + q).uniform(0.0, 1e-3, n))


# (stacks, layers of conductances per cell, precision, preconditioner, degree): measured
# on both sides in the rule's comment and around it
LAUNCHES = [([(1024, 1024, 1)], False, "mixed", "chebyshev", 30), ([(1024, 1024, 2)], True, "mixed16", "chebyshev", 30),
            ([(1023, 1023, 1)], True, "mixed", "chebyshev", 30), ([(1024, 1024, 2)], False, "adaptive", "chebyshev", 30),
            ([(512, 530, 2)], True, "mixed", "chebyshev_jacobi", 30), ([(512, 512, 16)], True, "mixed", "chebyshev", 2),
            ([(512, 512, 4)], False, "mixed", "chebyshev", 3), ([(512, 512, 2)], True, "fp64", "chebyshev", 30),
            ([(512, 512, 16)], True, "fp64", "chebyshev", 4), ([(256, 256, 1)] * 16, False, "mixed", "chebyshev", 30),
            ([(256, 256, 8)] * 16, False, "mixed", "chebyshev", 2), ([(128, 128, 2)] * 32, False, "fp64", "chebyshev", 30)]
ON_CHIP = [([(256, 256, 1)], False, "mixed", "chebyshev", 30), ([(1024, 1024, 6)], True, "mixed", "chebyshev", 30),
           ([(129, 1500, 3)], True, "mixed", "chebyshev", 30), ([(256, 256, 10)], False, "mixed", "chebyshev", 2),
           ([(512, 512, 8)], True, "mixed", "chebyshev", 3), ([(512, 512, 8)], True, "fp64", "chebyshev", 30),
           ([(128, 1090, 9)], True, "fp64", "chebyshev", 30), ([(256, 256, 4)] * 16, True, "mixed", "chebyshev", 30),
           ([(8, 8, 8)] * 400, False, "mixed", "chebyshev", 30)]


@pytest.mark.parametrize("sizes,cells,precision,pc,degree", LAUNCHES + ON_CHIP)
def test_the_shorter_way(monkeypatch, sizes, cells, precision, pc, degree):
    on_chip = (sizes, cells, precision, pc, degree) in ON_CHIP
    sts = [ragged_stack(nx, ny, LAYERS[:nz], mult=cells, seed=q) for q, (nx, ny, nz) in enumerate(sizes)]
    kw = dict(precision=precision, preconditioner=pc, cheb_degree=degree)

    def solve():
        # (new handles: one that has solved before checks at other iterations)
        grids = [grid_of(st) for st in sts]
        P = [_power(st.n, q) for q, st in enumerate(sts)]
        T = [grids[0].solve(P[0], **kw)[0]] if len(sts) == 1 else solve_batch(grids, P, **kw)[0]
        for g in grids:
            g.close()
        return T

    say(f"{len(sizes)} of {sizes[0]} {'cells' if cells else 'layers'} {precision} {pc} k={degree}")
    got = solve()
    monkeypatch.setenv("CUTH_RESIDENT", "0")
    want = solve()
    same = [torch.equal(a, b) for a, b in zip(got, want)]
    assert not any(same) if on_chip else all(same)


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,nz", [(512, 530, 2), (129, 2100, 1), (570, 460, 13)])
def test_forced_slabs_match_oracle(monkeypatch, nx, ny, nz, per_cell):
    """Slabs that only CUTH_RESIDENT=1 asks for, thin ones and short polynomials."""
    monkeypatch.setenv("CUTH_RESIDENT", "1")
    st = ragged_stack(nx, ny, LAYERS[:nz], mult=per_cell, seed=nx + nz)
    A = assembly.assemble(st)
    g = grid_of(st)
    r = np.random.default_rng(nx * ny).standard_normal(st.n).astype(np.float32).astype(np.float64)
    v0 = np.random.default_rng(4).standard_normal(st.n)
    for jacobi in (False, True):
        name = "chebyshev_jacobi" if jacobi else "chebyshev"
        lo, hi = (krylov.jacobi_spectral_bounds if jacobi else krylov.spectral_bounds)(A, v0)
        for degree in (2, 3, 7):
            say(f"forced slabs {nx}x{ny}x{nz} {'cells' if per_cell else 'layers'} {name} k={degree}")
            if jacobi:
                ref = krylov.jacobi_chebyshev_precondition(A, r, lo, hi, degree)
            else:
                ref = krylov.chebyshev_precondition(lambda v: A @ v, r, lo, hi, degree)
            z = g.precond_apply(t32(r), lo, hi, degree, preconditioner=name)
            bar = fp32_cheb_bar(A, r, lo, hi, degree, ref, jacobi=jacobi)
            assert np.abs(z.cpu().numpy().astype(np.float64) - ref).max() <= bar
            monkeypatch.setenv("CUTH_RESIDENT", "0")
            assert not torch.equal(z, g.precond_apply(t32(r), lo, hi, degree, preconditioner=name))
            monkeypatch.setenv("CUTH_RESIDENT", "1")
    g.close()


@pytest.mark.parametrize("precision,pc", [("mixed", "chebyshev"), ("mixed", "chebyshev_jacobi"), ("fp64", "chebyshev")])
def test_every_class_of_a_batch_runs_on_chip(monkeypatch, precision, pc):
    """Stacks of every layer class, ragged, in slabs (FP32) and of 17 to 20 layers (FP32):
    alone and together each moves less than by launches."""
    sizes = [(70, 50, 3), (64, 64, 8), (130, 33, 9), (5, 7, 12), (192, 200, 13), (257, 130, 16)]
    if precision == "mixed":
        sizes += [(65, 2100, 4), (65, 9, 20), (257, 460, 19)]
    sts = [ragged_stack(nx, ny, LAYERS[:nz], mult=False, seed=q) for q, (nx, ny, nz) in enumerate(sizes)]
    P = [_power(st.n) for st in sts]
    kw = dict(precision=precision, preconditioner=pc)

    def run():
        grids = [grid_of(st) for st in sts]
        T, stats = solve_batch(grids, P, **kw)
        single = [g.solve(p, **kw) for g, p in zip(grids, P)]
        for g in grids:
            g.close()
        return list(T) + [x for x, _ in single], [s["alg_bytes"] / s["cg_iters"] for s in stats + [s for _, s in single]]

    say(f"batch of {len(sizes)} classes {precision} {pc}")
    monkeypatch.setenv("CUTH_RESIDENT", "1")
    got, moved = run()
    monkeypatch.setenv("CUTH_RESIDENT", "0")
    want, moved0 = run()
    assert all(a < b / 2 for a, b in zip(moved, moved0))
    bar = 2.02e-8 if precision == "mixed" else 2e-10
    for q, (a, b) in enumerate(zip(got, want)):
        assert rise_err(a.cpu().numpy(), b.cpu().numpy(), sts[q % len(sts)].t_amb) <= bar

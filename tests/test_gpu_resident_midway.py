"""On-chip applications that give up in the middle of a solve: single solves go on from
their iterates, batches solve the problem again, entry points repeat the call."""

from __future__ import annotations

import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from gpu_helpers import grid_of, ragged_stack, rise_err, say, t64
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

LAYERS = ["Si", "Si", "BEOL", "bond"] * 3
BAR = {"mixed": 1.01e-8, "fp64": 2e-10, "adaptive": 1.01e-8}   # (the resident tests')


def _power(st):
    return np.random.default_rng(st.n).uniform(0.0, 1e-3, st.n)


@pytest.mark.parametrize("precision,pc", [("mixed", "chebyshev"), ("mixed", "chebyshev_jacobi"), ("adaptive", "chebyshev"),
                                          ("fp64", "chebyshev"), ("fp64", "chebyshev_jacobi")])
@pytest.mark.parametrize("m", [1, 2, 5])
def test_solve_goes_on(monkeypatch, precision, pc, m):
    """Application m gives up, so m updates of x, r and p have run.  FP64 solves, whose
    preconditioner differs between the two paths by FP64 rounding only, take the same
    number of iterations, one more or less."""
    monkeypatch.setenv("CUTH_GRAPH", "0")
    st = ragged_stack(200, 100, LAYERS[:10], mult=True)
    g, P = grid_of(st), t64(_power(st))
    ref = g.solve(P, precision="fp64")[0].cpu().numpy()
    _, sound = g.solve(P, precision=precision, preconditioner=pc)
    monkeypatch.setenv("CUTH_RESIDENT_SPIN", f"1@{m}")
    say(f"gives up at application {m}: {precision} {pc}")
    T, s = g.solve(P, precision=precision, preconditioner=pc)
    assert rise_err(T.cpu().numpy(), ref, st.t_amb) <= BAR[precision]
    if precision == "fp64":
        assert abs(s["cg_iters"] - sound["cg_iters"]) <= 1
    g.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_batch_problem_is_solved_again(monkeypatch, precision):
    """x and p hold several updates when the problem starts again."""
    monkeypatch.setenv("CUTH_GRAPH", "0")
    sts = [ragged_stack(nx, ny, LAYERS[:nz], mult=False, seed=q)
           for q, (nx, ny, nz) in enumerate([(130, 70, 3), (64, 8, 8), (200, 100, 9)])]
    grids = [grid_of(st) for st in sts]
    P = [_power(st) for st in sts]
    monkeypatch.setenv("CUTH_RESIDENT_SPIN", "1@3")
    say(f"batch gives up at application 3: {precision}")
    T, _ = solve_batch(grids, [t64(p) for p in P], precision=precision)
    monkeypatch.delenv("CUTH_RESIDENT_SPIN")
    for g, p, x, st in zip(grids, P, T, sts):
        ref = g.solve(t64(p), precision="fp64")[0].cpu().numpy()
        assert rise_err(x.cpu().numpy(), ref, st.t_amb) <= BAR[precision]
        g.close()


def test_give_up_at_the_iteration_limit():
    """The application after the last allowed update gives up: the inner solve's
    reduction of the residual is that of its last check, as by sweep launches."""
    code = (
        "import sys; sys.path.insert(0, 'tests')\n"
        "import numpy as np\n"
        "from gpu_helpers import grid_of, ragged_stack, t64\n"
        "st = ragged_stack(200, 100, ['Si', 'BEOL', 'bond', 'Cu'], mult=True)\n"
        "g = grid_of(st)\n"
        "P = t64(np.random.default_rng(1).uniform(0.0, 1e-3, st.n))\n"
        "try: g.solve(P, precision='mixed', max_inner=3)\n"
        "except Exception as e: assert 'limit' in str(e), e\n"
    )
    def last_reduction(**env):
        run = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, CUTH_LOG="1", CUTH_GRAPH="0", **env),
                             cwd=os.path.dirname(os.path.dirname(__file__)), stderr=subprocess.PIPE, timeout=100,
                             check=True)
        text = run.stderr.decode()
        assert ("gave up" in text) == ("CUTH_RESIDENT_SPIN" in env)
        cycle1 = next(line for line in text.splitlines() if " cycle 1 " in line)
        return float(cycle1.split("last reduction ")[1].split()[0])

    say("gives up at the iteration limit")
    # (by sweep launches throughout: three updates with a preconditioner that
    # differs in its FP32 rounding, far below a hundredth of the residual)
    want = last_reduction(CUTH_RESIDENT="0")
    assert want > 0.0 and last_reduction(CUTH_RESIDENT_SPIN="1@3") == pytest.approx(want, rel=1e-2)


@pytest.mark.parametrize("precision", ["mixed", "adaptive", "fp64"])
@pytest.mark.parametrize("m", [0, 4])
def test_bytes_are_those_of_the_launches_that_ran(monkeypatch, precision, m):
    """The solve's algorithmic bytes once application m has given up, against a solve
    by single sweep launches.  Per iteration and cycle they differ by the m + 1
    applications on chip (at most 5 of more than 20) and, FP32 aside, no more; what
    an iteration of the sound on-chip solve moves is below a third."""
    monkeypatch.setenv("CUTH_GRAPH", "0")
    st = ragged_stack(200, 100, LAYERS[:10], mult=True)
    g, P = grid_of(st), t64(_power(st))

    def per_iter():
        s = g.solve(P, precision=precision)[1]
        assert s["cg_iters"] > 20
        return s["alg_bytes"] / s["cg_iters"]

    sound = per_iter()
    monkeypatch.setenv("CUTH_RESIDENT_SPIN", f"1@{m}")
    say(f"bytes after giving up at application {m}: {precision}")
    gave_up = per_iter()
    monkeypatch.setenv("CUTH_FUSE", "0")
    sweeps = per_iter()
    assert sound < sweeps / 3
    assert gave_up == pytest.approx(sweeps, rel=0.05 + 5.0 * (m + 1) / 100)
    g.close()


@pytest.mark.parametrize("precision", ["mixed", "adaptive", "fp64"])
def test_a_handle_tries_again(monkeypatch, precision):
    """After two applications that gave up a handle keeps to sweep launches for 8 calls,
    then runs on chip again; if that gives up at once, for 16."""
    monkeypatch.setenv("CUTH_GRAPH", "0")
    st = ragged_stack(200, 100, LAYERS[:10], mult=True)
    g, P = grid_of(st), t64(_power(st))

    def on_chip():
        s = g.solve(P, precision=precision)[1]
        return s["alg_bytes"] / s["cg_iters"] < 1.1 * sound

    s = g.solve(P, precision=precision)[1]
    sound = s["alg_bytes"] / s["cg_iters"]
    for pause, gives_up in ((8, 2), (16, 1)):
        say(f"gives up {gives_up} times, then {pause} calls: {precision}")
        monkeypatch.setenv("CUTH_RESIDENT_SPIN", "1")
        for _ in range(gives_up):
            cycles = g.solve(P, precision=precision, max_outer=20)[1]["outer_cycles"]
            if cycles > 1:   # (one application gave up in each of two cycles)
                break
        monkeypatch.delenv("CUTH_RESIDENT_SPIN")
        assert not any(on_chip() for _ in range(pause))
        if pause == 16:
            assert on_chip() and on_chip()
    g.close()


@pytest.mark.parametrize("precision,dtype", [("mixed", "float32"), ("mixed16", "float32"), ("fp64", "float64")])
@pytest.mark.parametrize("pc", ["chebyshev", "chebyshev_jacobi"])
def test_entry_points_repeat_an_application(monkeypatch, precision, dtype, pc):
    """precond_apply and its allocation-free form, whose tiles give up: what they return
    by sweep launches, and on chip again after the pause."""
    st = ragged_stack(200, 100, LAYERS[:10], mult=True)
    r = torch.as_tensor(np.random.default_rng(3).standard_normal(st.n), dtype=getattr(torch, dtype), device="cuda")
    for alloc in (True, False):
        g = grid_of(st)
        b = g.spectral_bounds(preconditioner=pc)

        def apply():
            kw = dict(fp16_coef=precision == "mixed16", preconditioner=pc)
            if alloc:
                return g.precond_apply(r, b["lmin"], b["lmax"], 12, **kw)
            return g.precond_apply_noalloc(r, torch.full_like(r, float("nan")), b["lmin"], b["lmax"], 12, **kw)

        sound = apply()
        monkeypatch.setenv("CUTH_RESIDENT", "0")
        sweeps = apply()
        monkeypatch.delenv("CUTH_RESIDENT")
        assert not torch.equal(sound, sweeps)
        monkeypatch.setenv("CUTH_RESIDENT_SPIN", "1")
        say(f"application by itself gives up: {precision} {pc} {'' if alloc else 'no '}alloc")
        assert torch.equal(apply(), sweeps) and torch.equal(apply(), sweeps)
        monkeypatch.delenv("CUTH_RESIDENT_SPIN")
        assert all(torch.equal(apply(), sweeps) for _ in range(8))
        assert torch.equal(apply(), sound)
        g.close()

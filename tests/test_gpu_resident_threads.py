"""Solves of several threads at once on one device: the same bits as alone."""

from __future__ import annotations

import threading
import time

import numpy as np
import pytest
import torch

from gpu_helpers import dev, grid_of, ragged_stack, say, t64
from paper_2606_17850_amd import solve_batch

pytestmark = pytest.mark.gpu

# tiles that fit the device together, and two that need most or all of it
SIZES = [(64, 64, 8), (100, 40, 5), (384, 256, 9), (512, 512, 16)]
LAYERS = ["Si", "Si", "BEOL", "bond"] * 3 + ["TIM", "TIM", "Cu", "Cu"]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_results_do_not_depend_on_other_threads(precision):
    work = []
    for q, (nx, ny, nz) in enumerate(SIZES):
        st = ragged_stack(nx, ny, LAYERS[:nz], mult=q % 2 == 0, seed=q)
        with torch.cuda.stream(torch.cuda.Stream(dev())):
            g = grid_of(st)
        P = t64(np.random.default_rng(q).uniform(0.0, 1e-3, st.n))
        torch.cuda.synchronize()
        work.append((g, P, *g.solve(P, precision=precision)))
    wrong, start = [], threading.Barrier(len(work))

    def solve(q):
        g, P, T, s = work[q]
        start.wait(60)
        for turn in range(6 if q < 3 else 2):
            T1, s1 = g.solve(P, precision=precision)
            if not torch.equal(T, T1) or s1["cg_iters"] != s["cg_iters"] or s1["alg_bytes"] != s["alg_bytes"]:
                wrong.append((q, turn, s["cg_iters"], s1["cg_iters"]))

    say(f"{len(work)} threads, {precision}")
    threads = [threading.Thread(target=solve, args=(q,)) for q in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for g, *_ in work:
        g.close()


def test_a_small_solve_does_not_wait_for_a_long_one():
    """A batch that takes every compute unit for some 400 ms, and a solve of 3 ms that
    begins meanwhile: it is back before the batch is, and neither's bits change."""
    st, small = ragged_stack(512, 512, LAYERS, mult=True), ragged_stack(64, 64, LAYERS[:8], mult=False)
    with torch.cuda.stream(torch.cuda.Stream(dev())):
        g = grid_of(st)
    with torch.cuda.stream(torch.cuda.Stream(dev())):
        h = grid_of(small)
    rng = np.random.default_rng(2)
    P, Q = t64(rng.uniform(0.0, 1e-3, 4 * st.n)), t64(rng.uniform(0.0, 1e-3, small.n))
    torch.cuda.synchronize()
    long_one = lambda: solve_batch([g], [P], nrhs=4, precision="fp64")[0][0]
    want, want_small = long_one(), h.solve(Q)[0]
    t0 = time.perf_counter()
    long_one()
    alone = time.perf_counter() - t0
    h.solve(Q)
    got = []
    thread = threading.Thread(target=lambda: got.append(long_one()))
    say(f"a small solve beside one of {alone * 1e3:.0f} ms")
    thread.start()
    time.sleep(alone / 4)
    small_again = [h.solve(Q)[0] for _ in range(3)]
    running = thread.is_alive()
    thread.join()
    assert running
    assert torch.equal(got[0], want) and all(torch.equal(x, want_small) for x in small_again)
    g.close()
    h.close()

"""Solves of several threads at once on one device: the same bits as alone."""

from __future__ import annotations

import threading

import numpy as np
import pytest
import torch

from gpu_helpers import dev, grid_of, ragged_stack, say, t64

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

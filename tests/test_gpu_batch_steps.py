"""Batches whose members take different numbers of steps or converge at
different iterations (FP64 P3: the stage kernel deals its workgroups out to
the members that still run): every member equals its single solve, and the
members that are done leave the device to the others."""
from __future__ import annotations

import time

import numpy as np
import pytest

from paper_2106_02858_amd import inputs

pytestmark = pytest.mark.gpu


def _problems(lib, n, q, precision, omegas, seed=0):
    xyz, tet, tags = inputs.cube_mesh(n)
    s = lib.cmcg_space_create(lib.cmcg_mesh_create(xyz, tet, tags), q, precision)
    K, Np = len(tet), lib.cmcg_space_info(s)["Np"]
    rng = np.random.default_rng(seed)
    return K, Np, [lib.cmcg_problem_create(s, np.ones(K), np.ones(K), None, w, rng.standard_normal((K, Np, 3)))
                   for w in omegas]


def _fields(lib, r, K, Np):
    import torch
    f = [torch.zeros((K, 6, Np), dtype=torch.float64, device="cuda") for _ in range(3)]
    lib.cmcg_result_filtered_device(r, f[0], f[1])
    lib.cmcg_result_initial_device(r, f[2])
    return f


@pytest.mark.parametrize("n,omegas,opts", [
    (1, [9.0], dict(fixed_iters=2)),
    (2, [12.0, 3.0, 30.0, 12.0, 7.0], dict(fixed_iters=2)),          # unequal step counts
    (4, [12.0, 3.0, 30.0, 25.0], dict(fixed_iters=1)),               # more blocks than one per XCD
    (2, [8.0, 20.0, 40.0, 8.0, 60.0], dict(tol=0.3, max_iter=6)),    # converging one by one
    (1, [9.0 + 0.1 * b for b in range(100)], dict(fixed_iters=1)),   # more members than workgroups of a round
])
@pytest.mark.parametrize("use_graph", [1, 0])
def test_fp64_p3_members_equal_single_solves(lib, n, omegas, opts, use_graph):
    import torch
    print(f"batch steps n={n} B={len(omegas)} {opts} graph={use_graph}", flush=True)
    K, Np, probs = _problems(lib, n, 3, 0, omegas)
    res = lib.cmcg_solve_batch(probs, lib.cmcg_options_default(use_graph=use_graph, **opts))
    for p, r in zip(probs, res):
        one = lib.cmcg_solve(p, lib.cmcg_options_default(use_graph=0, **opts))
        assert lib.cmcg_result_stats(r)["iters"] == lib.cmcg_result_stats(one)["iters"]
        for x, y in zip(_fields(lib, r, K, Np), _fields(lib, one, K, Np)):
            assert torch.isfinite(x).all() and torch.equal(x, y)


def test_fp64_p3_long_member_has_the_device(lib):
    """15 members and one with six times their steps: no longer than the
    members together and the long one alone (a member's steps past the others'
    once ran on a sixteenth of the device: 1.34 s against 0.65)."""
    w = 6 * np.pi

    def seconds(omegas):
        K, Np, probs = _problems(lib, 12, 3, 0, omegas)
        o = lib.cmcg_options_default(fixed_iters=1)
        best = np.inf
        for _ in range(3):
            t0 = time.perf_counter()
            lib.cmcg_solve_batch(probs, o)
            best = min(best, time.perf_counter() - t0)
        return best

    print("batch with a long member", flush=True)
    both, short, long_ = seconds([w / 6] + [w] * 15), seconds([w] * 15), seconds([w / 6])
    print(f"  together {both:.3f} s, apart {short:.3f} + {long_:.3f} s")
    assert both < 1.25 * (short + long_)

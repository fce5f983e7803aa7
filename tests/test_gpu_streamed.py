"""Launches whose vectors exceed the Infinity Cache carry non-temporal hints
in the stage update; the hints change no value.

A batch whose members exceed the cache only together (the first one only
with the filter's accumulators) gives each member's single solve, which is
below the line, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2106_02858_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2106_02858_amd import cmcg
    return cmcg


# 622080 (q = 2) or 1244160 values a member, 18 B (FP32) or 32 B (FP64) each and 16 B of
# the filter, against 256 MB: the first passes it with the filter only (168 + 149 MB)
@pytest.mark.parametrize("q,precision,members", [(2, 1, 15), (2, 1, 24), (3, 1, 12), (2, 0, 13), (3, 0, 7)])
def test_streamed_batch_equals_single_solves(lib, q, precision, members):
    import torch
    print(f"streamed q={q} prec={precision} members={members}", flush=True)
    xyz, tet, tags = inputs.cube_mesh(12)
    K = len(tet)
    s = lib.cmcg_space_create(lib.cmcg_mesh_create(xyz, tet, tags), q, precision)
    Np = lib.cmcg_space_info(s)["Np"]
    rng = np.random.default_rng(3)
    j = np.zeros((K, Np, 3), dtype=complex)
    j[::17] = rng.standard_normal((len(j[::17]), Np, 3))
    probs = [lib.cmcg_problem_create(s, np.ones(K), np.ones(K), None, 7.0 + 0.1 * b, j) for b in range(members)]
    o = lib.cmcg_options_default(fixed_iters=1)  # the CFL step count

    def fields(r):
        f = [torch.zeros((K, 6, Np), dtype=torch.float64, device="cuda") for _ in range(3)]
        lib.cmcg_result_filtered_device(r, f[0], f[1])
        lib.cmcg_result_initial_device(r, f[2])
        return f

    batch = lib.cmcg_solve_batch(probs, o)
    for b in (0, members - 1):
        for x, y in zip(fields(batch[b]), fields(lib.cmcg_solve(probs[b], o))):
            assert torch.isfinite(x).all() and torch.equal(x, y)

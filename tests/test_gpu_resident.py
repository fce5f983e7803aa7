"""Periods run as one launch (meshes whose element blocks fit on the device at
once) against the same periods run by stage launches (use_graph = 0, itself
checked against the oracle elsewhere): the two do the same arithmetic, so
every comparison is bit for bit.

Covered: element counts around the block size, meshes numbered at random
(every face of a block then has its neighbour in another one, more exchanged
values than a block has threads), both time schemes, both directions, source
with boundary data and conductivity, the filter, and batches whose members do
not fit on the device together."""
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


def _strip(n):
    """n triangles in a zigzag strip (every second vertex on one side)."""
    i = np.arange(n + 2)
    xy = np.stack([i // 2 + 0.3 * (i % 2), (i % 2) * 1.0], axis=1) / 4.0
    tri = np.stack([i[:-2], i[1:-1], i[2:]], axis=1)
    tri[1::2] = tri[1::2][:, [1, 0, 2]]
    tags = np.full((n, 3), inputs.TAG_IMPEDANCE, dtype=np.int8)
    tags[::3] = inputs.TAG_PEC
    return xy, tri.astype(np.int64), tags


def _mesh2d(kind):
    if isinstance(kind, int):
        return _strip(kind)
    xy, tri, tags = inputs.cartesian_triangles(12, 9, side_tags=(1, 2, 1, 2))
    p = np.random.default_rng(8).permutation(len(tri))
    return xy, tri[p], tags[p]


def _problem(lib, dim, mesh, q, precision, seed, omega=9.0):
    """A problem with conductivity, current and boundary data on random coefficients."""
    rng = np.random.default_rng(seed)
    xyz, el, tags = mesh
    K = len(el)
    m = (lib.cmcg_mesh2d_create if dim == 2 else lib.cmcg_mesh_create)(xyz, el, tags)
    s = lib.cmcg_space_create(m, q, precision)
    return s, _member(lib, s, dim, K, q, rng, omega)


def _member(lib, s, dim, K, q, rng, omega):
    Np = lib.cmcg_space_info(s)["Np"]
    shape = (K, Np) if dim == 2 else (K, Np, 3)
    gshape = (K, 3, q + 1) if dim == 2 else (K, 4, (q + 1) * (q + 2) // 2, 3)
    j = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    j[rng.random(K) < 0.5] = 0.0
    return lib.cmcg_problem_create(s, rng.choice([1.0, 2.0, 4.0], K), rng.choice([1.0, 1.5], K),
                                   rng.uniform(0, 0.4, K), omega, j, 0.1 * rng.standard_normal(gshape))


def _periods(lib, p, K, comps, Np, q, use_graph):
    import torch
    U = torch.tensor(np.random.default_rng(2).standard_normal((K, comps, Np)), device="cuda")
    out = []
    for scheme in (2, 4):
        o = lib.cmcg_options_default(use_graph=use_graph, scheme=scheme)  # the CFL step count
        for direction, source, filt in ((1, False, False), (1, True, True), (-1, False, False), (1, True, False)):
            ut, fr, fi = (torch.zeros_like(U) for _ in range(3))
            lib.cmcg_debug_period(p, U, ut, direction, source, fr if filt else None, fi if filt else None, opts=o)
            out += [ut, fr, fi]
    return out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("q", [1, 2, 3])
@pytest.mark.parametrize("kind", [1, 20, 21, 22, 43, "shuffled"])
def test_period2d_equals_stage_launches(lib, kind, q, precision):
    import torch
    print(f"resident 2-D {kind} q={q} prec={precision}", flush=True)
    mesh = _mesh2d(kind)
    s, p = _problem(lib, 2, mesh, q, precision, seed=5)
    K, Np = len(mesh[1]), lib.cmcg_space_info(s)["Np"]
    a, b = (_periods(lib, p, K, 3, Np, q, g) for g in (1, 0))
    for x, y in zip(a, b):
        assert torch.isfinite(x).all() and torch.equal(x, y)


def _mesh3d(kind):
    """The first tets of a cube (the faces of the cut become walls), or all of them numbered at random."""
    xyz, tet, tags = inputs.cube_mesh(3)
    if kind == "shuffled":
        p = np.random.default_rng(8).permutation(len(tet))
        return xyz, tet[p], tags[p]
    return xyz, tet[:kind], np.where(tags[:kind] == 0, inputs.TAG_IMPEDANCE, tags[:kind]).astype(tags.dtype)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("q", [1, 2, 3])
@pytest.mark.parametrize("kind", [1, 9, 10, 11, 43, "shuffled"])
def test_period3d_equals_stage_launches(lib, kind, q, precision):
    import torch
    print(f"resident 3-D {kind} q={q} prec={precision}", flush=True)
    mesh = _mesh3d(kind)
    s, p = _problem(lib, 3, mesh, q, precision, seed=5)
    K, Np = len(mesh[1]), lib.cmcg_space_info(s)["Np"]
    a, b = (_periods(lib, p, K, 6, Np, q, g) for g in (1, 0))
    for x, y in zip(a, b):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("precision", [0, 1])
def test_batch2d_in_groups_equals_stage_launches(lib, precision):
    """30 members of 1200 triangles (58 blocks each) do not fit on the device
    together: the period runs in groups of members, each with its own step
    count."""
    import torch
    print(f"resident 2-D batch prec={precision}", flush=True)
    q = 3
    xy, tri, tags = inputs.cartesian_triangles(20, 15)
    m = lib.cmcg_mesh2d_create(xy, tri, tags)
    s = lib.cmcg_space_create(m, q, precision)
    K, Np = len(tri), lib.cmcg_space_info(s)["Np"]
    probs = [_member(lib, s, 2, K, q, np.random.default_rng(b), 20.0 + b) for b in range(30)]
    got = []
    for g in (1, 0):
        for r in lib.cmcg_solve_batch(probs, lib.cmcg_options_default(fixed_iters=2, use_graph=g)):
            f = [torch.zeros((K, 3, Np), dtype=torch.float64, device="cuda") for _ in range(3)]
            lib.cmcg_result_filtered_device(r, f[0], f[1])
            lib.cmcg_result_initial_device(r, f[2])
            got.append(f)
    for x, y in zip(got[:30], got[30:]):
        assert all(torch.isfinite(u).all() and torch.equal(u, v) for u, v in zip(x, y))

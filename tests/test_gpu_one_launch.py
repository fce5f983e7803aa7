"""Which periods run as one launch: the library's own count of them.  Results
do not tell (they equal those of stage launches, bit for bit; see
test_gpu_resident.py), so the tests here ask the counters."""
from __future__ import annotations

import threading
import time

import numpy as np
import pytest

from paper_2106_02858_amd import inputs
from tests.test_gpu_resident import _member, _mesh2d, _mesh3d, _periods, _problem

pytestmark = pytest.mark.gpu


def _period(lib, p, K, comps, Np, n=1, **kw):
    """n forward periods; how many of them (ran as one launch, were restarted)."""
    import torch
    U = torch.tensor(np.random.default_rng(3).standard_normal((K, comps, Np)), device="cuda")
    V = torch.zeros_like(U)
    a = lib.cmcg_debug_period_counts()
    for _ in range(n):
        lib.cmcg_debug_period(p, U, V, 1, True, opts=lib.cmcg_options_default(**kw))
    b = lib.cmcg_debug_period_counts()
    assert torch.isfinite(V).all()
    return tuple(y - x for x, y in zip(a, b))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dim,q", [(2, 1), (2, 2), (2, 3), (3, 2), (3, 3)])
@pytest.mark.parametrize("kind", [43, "shuffled"])
def test_small_meshes_run_as_one_launch(lib, kind, dim, q, precision):
    print(f"one launch dim={dim} q={q} prec={precision} {kind}", flush=True)
    mesh = (_mesh2d if dim == 2 else _mesh3d)(kind)
    s, p = _problem(lib, dim, mesh, q, precision, seed=4)
    K, Np, comps = len(mesh[1]), lib.cmcg_space_info(s)["Np"], 3 if dim == 2 else 6
    assert _period(lib, p, K, comps, Np, n=2) == (2, 0)
    assert _period(lib, p, K, comps, Np, scheme=4 if q == 1 else 2) == (1, 0)
    assert _period(lib, p, K, comps, Np, use_graph=0) == (0, 0)


@pytest.mark.parametrize("precision", [0, 1])
def test_batch2d_periods_run_as_one_launch(lib, precision):
    print(f"one launch 2-D batch prec={precision}", flush=True)
    xy, tri, tags = inputs.cartesian_triangles(12, 9)
    s = lib.cmcg_space_create(lib.cmcg_mesh2d_create(xy, tri, tags), 3, precision)
    probs = [_member(lib, s, 2, len(tri), 3, np.random.default_rng(b), 20.0 + b) for b in range(6)]
    a = lib.cmcg_debug_period_counts()
    res = lib.cmcg_solve_batch(probs, lib.cmcg_options_default(fixed_iters=2))
    b = lib.cmcg_debug_period_counts()
    periods = lib.cmcg_result_stats(res[0])["periods"]
    assert (b[0] - a[0], b[1] - a[1]) == (periods, 0)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("q", [1, 2, 3])
def test_default_stage_variant_put_back(lib, q, precision):
    """A variant set by hand keeps periods on its stage launches; the default
    put back, as read before, gives the one-launch periods back."""
    print(f"tune q={q} prec={precision}", flush=True)
    mesh = _mesh3d("shuffled")
    s, p = _problem(lib, 3, mesh, q, precision, seed=6)
    K, Np = len(mesh[1]), lib.cmcg_space_info(s)["Np"]
    saved = lib.cmcg_tune_get_stage(q, precision)
    try:
        lib.cmcg_tune_stage(q, precision, 1)
        assert _period(lib, p, K, 6, Np) == (0, 0)
    finally:
        lib.cmcg_tune_stage(q, precision, saved)
    assert _period(lib, p, K, 6, Np) == (1, 0)


def test_mesh_that_does_not_fit_is_not_restarted(lib):
    """24576 P1 FP64 tets do not fit on the device at once: their periods run
    by stage launches, each from the one start state written for it."""
    print("one launch: too large", flush=True)
    mesh = inputs.cube_mesh(16)
    s, p = _problem(lib, 3, mesh, 1, 0, seed=2)
    assert _period(lib, p, len(mesh[1]), 6, 4, n=3, steps=120) == (0, 0)


def test_batch_members_left_run_as_one_launch(lib):
    """24 members of 750 P1 FP64 tets (75 blocks each) do not fit together; the
    few that are still to converge do."""
    print("one launch: batch members left", flush=True)
    xyz, tet, tags = inputs.cube_mesh(5)
    s = lib.cmcg_space_create(lib.cmcg_mesh_create(xyz, tet, tags), 1, 0)
    probs = [_member(lib, s, 3, len(tet), 1, np.random.default_rng(b), 4.0 if b < 22 else 30.0) for b in range(24)]
    o = lib.cmcg_options_default(tol=0.2, max_iter=25)
    a = lib.cmcg_debug_period_counts()
    res = [lib.cmcg_result_stats(r) for r in lib.cmcg_solve_batch(probs, o)]
    b = lib.cmcg_debug_period_counts()
    alone = [lib.cmcg_result_stats(lib.cmcg_solve(q, lib.cmcg_options_default(tol=0.2, max_iter=25, use_graph=0)))
             for q in probs]
    assert [r["iters"] for r in res] == [r["iters"] for r in alone]
    assert [r["rel_res"] for r in res] == [r["rel_res"] for r in alone]
    iters = sorted(r["iters"] for r in res)
    assert iters[0] < iters[-1]  # the members do converge apart
    print(f"  iterations {iters}, one-launch periods {b[0] - a[0]}")
    # the members in the last iterations are few enough to fit (3 workgroups per compute unit, 80 slots each)
    few = sum(1 for i in range(iters[-1]) if sum(1 for r in res if r["iters"] > i) * 80 <= 512)
    assert b[0] - a[0] >= 2 * few > 0 and b[1] == a[1]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dim,q", [(2, 1), (2, 3), (3, 1), (3, 2), (3, 3)])
def test_period_that_gives_up_runs_by_stage_launches(lib, dim, q, precision):
    """A launch whose blocks are not all there gives up: its period starts
    again (state and filter) by stage launches, and neither this problem nor
    another of the device waits for such a launch again while the pause lasts."""
    import torch
    print(f"give up dim={dim} q={q} prec={precision}", flush=True)
    mesh = (_mesh2d if dim == 2 else _mesh3d)("shuffled")
    s, p = _problem(lib, dim, mesh, q, precision, seed=7)
    K, Np, comps = len(mesh[1]), lib.cmcg_space_info(s)["Np"], 3 if dim == 2 else 6
    other = _member(lib, s, dim, K, q, np.random.default_rng(1), 9.0)
    try:
        lib.cmcg_debug_period_stall(p, 1e-3)
        a = lib.cmcg_debug_period_counts()
        got = _periods(lib, p, K, comps, Np, q, 1)
        b = lib.cmcg_debug_period_counts()
        assert (b[0] - a[0], b[1] - a[1]) == (0, 1)
        assert _period(lib, other, K, comps, Np) == (0, 0)
    finally:
        lib.cmcg_debug_period_stall(p, 0)
    for x, y in zip(got, _periods(lib, p, K, comps, Np, q, 0)):
        assert torch.isfinite(x).all() and torch.equal(x, y)
    assert _period(lib, other, K, comps, Np) == (1, 0)
    assert _period(lib, p, K, comps, Np) == (1, 0)


def test_filtered_period_that_gives_up(lib):
    """The accumulators of a filtered period that gave up are begun again too."""
    import torch
    print("give up, filtered", flush=True)
    mesh = _mesh3d("shuffled")
    s, p = _problem(lib, 3, mesh, 2, 1, seed=7)
    U = torch.tensor(np.random.default_rng(3).standard_normal((len(mesh[1]), 6, 10)), device="cuda")
    out = []
    for stall, graph in ((1e-3, 1), (0, 0)):
        lib.cmcg_debug_period_stall(p, stall)
        V, F, G = (torch.zeros_like(U) for _ in range(3))
        a = lib.cmcg_debug_period_counts()
        lib.cmcg_debug_period(p, U, V, 1, True, F, G, opts=lib.cmcg_options_default(use_graph=graph))
        assert lib.cmcg_debug_period_counts()[1] - a[1] == graph
        out.append((V, F, G))
    assert all(torch.equal(x, y) and torch.isfinite(x).all() for x, y in zip(*out))


def test_batch_that_gives_up(lib):
    import torch
    print("give up, batch", flush=True)
    xy, tri, tags = inputs.cartesian_triangles(12, 9)
    K, q = len(tri), 3
    s = lib.cmcg_space_create(lib.cmcg_mesh2d_create(xy, tri, tags), q, 1)
    probs = [_member(lib, s, 2, K, q, np.random.default_rng(b), 20.0 + b) for b in range(6)]
    out = []
    for stall, graph in ((1e-3, 1), (0, 0)):
        lib.cmcg_debug_period_stall(probs[0], stall)
        a = lib.cmcg_debug_period_counts()
        res = lib.cmcg_solve_batch(probs, lib.cmcg_options_default(fixed_iters=2, use_graph=graph))
        b = lib.cmcg_debug_period_counts()
        assert (b[0] - a[0], b[1] - a[1]) == (0, graph)
        f = [[torch.zeros((K, 3, 10), dtype=torch.float64, device="cuda") for _ in range(2)] for _ in res]
        for r, (x, y) in zip(res, f):
            lib.cmcg_result_filtered_device(r, x, y)
        out.append([x for pair in f for x in pair])
    assert all(torch.equal(x, y) and torch.isfinite(x).all() for x, y in zip(*out))


def test_stall_arguments(lib):
    mesh = _mesh3d(43)  # five blocks: none can be left out of each range
    _, p = _problem(lib, 3, mesh, 1, 0, seed=1)
    for bad in (1e-3, -1.0, 3.0, float("nan")):
        with pytest.raises(lib.CmcgError) as err:
            lib.cmcg_debug_period_stall(p, bad)
        assert err.value.code == lib.CMCG_ERR_ARG


def _solves(lib, n, q, precision, count, fixed_iters, repeat, threads):
    """`count` problems solved `repeat` times each, on a host thread and stream
    each or one after the other: seconds, filtered fields, results' counts."""
    import torch
    xyz, tet, tags = inputs.cube_mesh(n)
    s = lib.cmcg_space_create(lib.cmcg_mesh_create(xyz, tet, tags), q, precision)
    K, Np = len(tet), lib.cmcg_space_info(s)["Np"]
    probs = [_member(lib, s, 3, K, q, np.random.default_rng(b), 9.0 + 0.5 * b) for b in range(count)]
    streams = [torch.cuda.Stream() for _ in probs]
    o = lib.cmcg_options_default(fixed_iters=fixed_iters)
    out, errors = [None] * count, []

    def work(i, times):
        try:
            for _ in range(times):
                r = lib.cmcg_solve(probs[i], o, stream=streams[i])
            f = [torch.zeros((K, 6, Np), dtype=torch.float64, device="cuda") for _ in range(2)]
            lib.cmcg_result_filtered_device(r, *f)
            out[i] = f
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(e)

    for i in range(count):
        work(i, 1)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    if threads:
        th = [threading.Thread(target=work, args=(i, repeat)) for i in range(count)]
        [t.start() for t in th]
        [t.join() for t in th]
    else:
        for i in range(count):
            work(i, repeat)
    torch.cuda.synchronize()
    seconds = time.perf_counter() - t0
    assert not errors, errors
    lib.cmcg_debug_period_stall(probs[0], 0)  # ends a pause, if the threads' first launches met
    return seconds, out


@pytest.mark.parametrize("n,q,precision,fits_together", [(8, 2, 1, True), (6, 1, 0, True), (12, 1, 1, False),
                                                         (8, 3, 1, False)])
def test_threads_share_the_device(lib, n, q, precision, fits_together):
    """Solves on four host threads give what they give one after the other, and
    small ones take less time together (one after another, each waiting for
    the others' whole periods, took as long: 0.97 of it; together 0.5)."""
    import torch
    print(f"threads n={n} q={q} prec={precision}", flush=True)
    ratios = []
    for _ in range(3):
        a, x = _solves(lib, n, q, precision, 4, 2, 4, threads=False)
        b, y = _solves(lib, n, q, precision, 4, 2, 4, threads=True)
        for u, v in zip(x, y):
            assert all(torch.isfinite(f).all() and torch.equal(f, g) for f, g in zip(u, v))
        ratios.append(b / a)
    print(f"  together / one after the other: {ratios}")
    if fits_together:
        assert min(ratios) < 0.8


def test_small_solve_beside_stage_launches(lib):
    """Beside a call that runs by stage launches a small solve does too (its
    workgroups would wait for room behind that call's launches)."""
    import torch
    print("small solve beside stage launches", flush=True)
    big = _problem(lib, 3, inputs.cube_mesh(16), 1, 0, seed=2)[1]
    mesh = _mesh3d("shuffled")
    small = _problem(lib, 3, mesh, 2, 1, seed=7)[1]
    ref = lib.cmcg_solve(small, lib.cmcg_options_default(fixed_iters=2, use_graph=0))
    o = lib.cmcg_options_default(fixed_iters=400)
    started, stop = threading.Event(), threading.Event()
    o.set_progress(lambda it, rel: started.set() or stop.is_set())
    stream = torch.cuda.Stream()
    t = threading.Thread(target=lambda: lib.cmcg_solve(big, o, stream=stream))
    t.start()
    try:
        assert started.wait(60)
        a = lib.cmcg_debug_period_counts()
        r = lib.cmcg_solve(small, lib.cmcg_options_default(fixed_iters=2))
        b = lib.cmcg_debug_period_counts()
        running = t.is_alive()
    finally:
        stop.set()
        t.join()
    assert running and a == b
    f = [torch.zeros((len(mesh[1]), 6, 10), dtype=torch.float64, device="cuda") for _ in range(4)]
    lib.cmcg_result_filtered_device(r, f[0], f[1])
    lib.cmcg_result_filtered_device(ref, f[2], f[3])
    assert torch.equal(f[0], f[2]) and torch.equal(f[1], f[3])
    lib.cmcg_debug_period_stall(small, 0)
    lib.cmcg_solve(small, lib.cmcg_options_default(fixed_iters=2))
    assert lib.cmcg_debug_period_counts()[0] > b[0]


@pytest.mark.parametrize("q,precision,n,B,groups", [
    (3, 1, 20, 30, 2), (3, 0, 20, 30, 3),   # 77 blocks a member; 1280 and 1024 fit
    (2, 0, 20, 20, 2), (1, 1, 20, 30, 2),
    (2, 0, 20, 30, 0), (1, 0, 20, 20, 0), (1, 1, 20, 60, 0),  # as many groups as lose to stage launches
])
def test_batch2d_groups(lib, q, precision, n, B, groups):
    """Batches of triangles run in equal groups of members while these win
    (groups = 0: they do not, the batch runs by stage launches)."""
    import torch
    print(f"groups q={q} prec={precision} B={B}", flush=True)
    xy, tri, tags = inputs.cartesian_triangles(n, n)
    K, Np = len(tri), (q + 1) * (q + 2) // 2
    s = lib.cmcg_space_create(lib.cmcg_mesh2d_create(xy, tri, tags), q, precision)
    probs = [_member(lib, s, 2, K, q, np.random.default_rng(b), 20.0 + b) for b in range(B)]
    out = []
    for g in (1, 0):
        a = lib.cmcg_debug_period_counts(launches=True)
        res = lib.cmcg_solve_batch(probs, lib.cmcg_options_default(fixed_iters=1, use_graph=g))
        b = lib.cmcg_debug_period_counts(launches=True)
        periods = lib.cmcg_result_stats(res[0])["periods"] if g and groups else 0
        assert [y - x for x, y in zip(a, b)] == [periods, 0, periods * groups]
        f = [[torch.zeros((K, 3, Np), dtype=torch.float64, device="cuda") for _ in range(2)] for _ in res]
        for r, (x, y) in zip(res, f):
            lib.cmcg_result_filtered_device(r, x, y)
        out.append([x for pair in f for x in pair])
    assert all(torch.isfinite(x).all() and torch.equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("n,one_launch", [(7, True), (8, True), (9, False)])
@pytest.mark.parametrize("q", [2, 3])
def test_fp64_block_limit(lib, q, n, one_launch):
    """FP64 P2 and P3 run as one launch up to 350 blocks (n = 8: 308, n = 9: 438)."""
    print(f"FP64 limit q={q} n={n}", flush=True)
    mesh = inputs.cube_mesh(n)
    s, p = _problem(lib, 3, mesh, q, 0, seed=3)
    got = _period(lib, p, len(mesh[1]), 6, lib.cmcg_space_info(s)["Np"])
    assert got == (int(one_launch), 0)


def test_footprint_counts_what_one_launch_periods_hold(lib):
    """A plain solve leaves exchange buffers and a step table with the problem;
    its footprint says so, and the engine, whose slots run none, gives them back."""
    print("footprint", flush=True)
    mesh = _mesh3d("shuffled")
    s, p = _problem(lib, 3, mesh, 2, 1, seed=8)
    K = len(mesh[1])
    before = lib.cmcg_problem_footprint(p)
    o = lib.cmcg_options_default(fixed_iters=1)
    lib.cmcg_solve(p, o)
    M = lib.cmcg_problem_steps(p, o)[0]
    held = lib.cmcg_problem_footprint(p) - before
    # two buffers of 8-byte pairs for the 6 x 6 values of every cut face, and 9 scalars per stage
    assert 2 * 8 * 36 * 2 * K < held - (M + 1) * 4 * 9 * 8 <= 2 * 8 * 36 * 4 * K + 64
    e = lib.cmcg_engine_create(before, 2)
    slot = lib.cmcg_engine_admit(e, p, o)
    assert slot is not None and lib.cmcg_engine_info(e)["used"] == before
    assert lib.cmcg_problem_footprint(p) == before
    while lib.cmcg_engine_poll(e, slot) == 1:
        lib.cmcg_engine_step(e)
    lib.cmcg_engine_collect(e, slot, p)
    assert _period(lib, p, K, 6, 10) == (1, 0)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("q", [1, 2, 3])
def test_autotuner_times_every_kernel_once(lib, q, precision):
    """Variants that stand for one kernel get one time; the choice is the lowest
    of the fastest kernel's."""
    print(f"autotune q={q} prec={precision}", flush=True)
    mesh = _mesh3d("shuffled")
    _, p = _problem(lib, 3, mesh, q, precision, seed=9)
    saved = lib.cmcg_tune_get_stage(q, precision)
    try:
        v, us = lib.cmcg_autotune_stage(p)
    finally:
        lib.cmcg_tune_stage(q, precision, saved)
    us = list(us)
    assert us[0] > 0 and us[1] > 0
    rest = [x for i, x in enumerate(us) if i > 1 and not (q == 2 and i in (6, 7))]
    assert len(set(rest)) == 1 and (rest[0] > 0) == (q > 1)
    assert us[v] == min(x for x in us if x > 0) and v <= 2


def test_engine_slots_leave_the_device_when_done(lib):
    """While a slot runs, plain solves beside it run by stage launches; when it
    has finished, failed or been cancelled -- collected or not -- they do not."""
    print("engine slots", flush=True)
    mesh = _mesh3d("shuffled")
    s, p = _problem(lib, 3, mesh, 2, 1, seed=8)
    K = len(mesh[1])
    rng = np.random.default_rng(3)
    slots = [_member(lib, s, 3, K, 2, rng, 9.0) for _ in range(3)]
    e = lib.cmcg_engine_create(1 << 30, 4)

    def run(slot):
        while lib.cmcg_engine_poll(e, slot) == 1:
            lib.cmcg_engine_step(e)

    a = lib.cmcg_engine_admit(e, slots[0], lib.cmcg_options_default(fixed_iters=2))
    assert _period(lib, p, K, 6, 10) == (0, 0)
    run(a)
    assert lib.cmcg_engine_poll(e, a) == 2 and _period(lib, p, K, 6, 10) == (1, 0)
    b = lib.cmcg_engine_admit(e, slots[1], lib.cmcg_options_default(fixed_iters=2, steps=3))  # far too few steps
    run(b)
    assert lib.cmcg_engine_poll(e, b) == 3 and _period(lib, p, K, 6, 10) == (1, 0)
    c = lib.cmcg_engine_admit(e, slots[2], lib.cmcg_options_default(fixed_iters=50))
    assert _period(lib, p, K, 6, 10) == (0, 0)
    lib.cmcg_engine_cancel(e, c)
    assert _period(lib, p, K, 6, 10) == (1, 0)

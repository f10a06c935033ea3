"""Narrow lattices (the column kernel: several steps per launch): parity with
the oracle at the edges of its tiles and any split of a run into calls."""
import math

import numpy as np
import pytest

import lbm_inputs as W
import oracle as O
from tests.test_parity_gpu import P, _f0, _oracle_params  # noqa: F401

pytestmark = pytest.mark.gpu

# rows of a workgroup are 8 and up: one tile, a full one, one row over, several
SIZES = [(3, 3), (4, 8), (4, 9), (5, 37), (7, 64), (16, 29), (15, 130)]


@pytest.mark.parametrize("geom,far,wall,sigma,coll", [
    (W.PLATE, W.FAR_WALL, "bb", 1.0, "regularized"),
    (W.PLATE, W.FAR_EQ, "maxwell", 0.35, "regularized"),
    (W.PLATE, W.FAR_WALL, "ds", 1.0, "bgk"),
    (W.PERIODIC, W.FAR_EQ, "bb", 1.0, "bgk"),
])
@pytest.mark.parametrize("Q", [9, 37])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_column_kernel(P, nx, ny, Q, geom, far, wall, sigma, coll):  # noqa: F811
    """Fields and forces after 71 steps in calls of 1, 2, 13, 32 and 23 against
    the long-double oracle (FP64: 71 steps of a few roundings, 1e-12), and the
    same bits from one call per step; FP32 within 2e-5."""
    calls = [1, 2, 13, 32, 23]
    n = sum(calls)
    print(f"case {nx}x{ny} Q{Q} {geom} {far} {wall} {coll}", flush=True)
    v, w, th = P.lattice(Q)
    for storage in ("f64", "f32dev"):
        s = W.Solve(Q=Q, geometry=geom, far=far, nx=nx, ny=ny, tau=0.9, omega=2 * math.pi / 40,
                    nsteps=n, window_first=5, window_count=n - 9, storage=storage,
                    collision=coll, wall=wall, accommodation=sigma)
        f0 = _f0(s, w, seed=11, amp=1e-3)
        out = []
        for split in (calls, [1] * n):
            with P.Solver(P.params_from_solve(s)) as sv:
                sv.set_populations(f0)
                for k in split:
                    sv.step(k)
                out.append((*sv.force_history(), sv.get_deviations(), sv.lockin()[0]))
        assert all(np.array_equal(a, b) for a, b in zip(*out))
        ox, oy, of = O.run(_oracle_params(s), n, f0=f0, want_state=True, variant="ld")
        rest = w[:, None, None] * s.rho0
        tol = 1e-12 if storage == "f64" else 2e-5
        fx, fy, f, _ = out[0]
        assert np.max(np.abs(f - (of - rest))) <= tol * np.max(np.abs(of - rest)) + \
            2 * np.spacing(np.max(w))
        if geom == W.PLATE:
            scale = max(np.max(np.abs(ox)), np.max(np.abs(oy)))
            assert np.max(np.abs(fx - ox)) <= tol * scale
            assert np.max(np.abs(fy - oy)) <= tol * scale


# lattices so long that a workgroup's rows fill the LDS planes, some tiles'
# regions just reaching a wall
FULL = [(37, 16, 2309), (37, 16, 2310), (37, 8, 3339), (37, 7, 2307), (9, 16, 2309)]


@pytest.mark.parametrize("far,wall,sigma", [(W.FAR_WALL, "bb", 1.0), (W.FAR_EQ, "bb", 1.0),
                                            (W.FAR_WALL, "ds", 1.0), (W.FAR_EQ, "maxwell", 0.35)])
@pytest.mark.parametrize("Q,nx,ny", FULL)
def test_full_planes(P, Q, nx, ny, far, wall, sigma):  # noqa: F811
    """14 steps of full planes in one call, and the same bits from one step per
    call; FP64 against the long-double oracle within 1e-12."""
    n = 14
    print(f"case {nx}x{ny} Q{Q} {far} {wall}", flush=True)
    v, w, th = P.lattice(Q)
    for storage in ("f64", "f32dev"):
        s = W.Solve(Q=Q, geometry=W.PLATE, far=far, nx=nx, ny=ny, tau=0.9,
                    omega=2 * math.pi / 40, nsteps=n, window_first=2, window_count=n - 4,
                    storage=storage, wall=wall, accommodation=sigma)
        f0 = _f0(s, w, seed=13, amp=1e-3)
        out = []
        for split in ([n], [1] * n):
            with P.Solver(P.params_from_solve(s)) as sv:
                sv.set_populations(f0)
                for k in split:
                    sv.step(k)
                out.append((*sv.force_history(), sv.get_deviations(), sv.lockin()[0]))
        assert all(np.array_equal(a, b) for a, b in zip(*out))
        if storage == "f64":
            ox, oy, of = O.run(_oracle_params(s), n, f0=f0, want_state=True, variant="ld")
            dev = of - w[:, None, None] * s.rho0
            assert np.max(np.abs(out[0][2] - dev)) <= \
                1e-12 * np.max(np.abs(dev)) + 2 * np.spacing(np.max(w))
            scale = max(np.max(np.abs(ox)), np.max(np.abs(oy)))
            assert np.max(np.abs(out[0][0] - ox)) <= 1e-12 * scale
            assert np.max(np.abs(out[0][1] - oy)) <= 1e-12 * scale


@pytest.mark.parametrize("nx,lengths", [(8, [3101] * 8), (16, [700, 1311, 902]),
                                        (4, [5832, 6795, 1186, 6816, 4385])])
def test_batch_of_long_plates(P, nx, lengths):  # noqa: F811
    """Plates whose total length makes the workgroups of their launch take more
    rows than each plate's own: the bits of every plate alone."""
    import torch
    n = 21
    solves = [W.Solve(Q=37, geometry=W.PLATE, far=(W.FAR_WALL, W.FAR_EQ)[i % 2], nx=nx, ny=ny,
                      tau=0.8, omega=2 * math.pi / 40, nsteps=n, window_first=0, window_count=n)
              for i, ny in enumerate(lengths)]
    alone = []
    for s in solves:
        with P.Solver(P.params_from_solve(s)) as sv:
            for _ in range(n):
                sv.step(1)
            alone.append((*sv.force_history(), sv.get_deviations()))
    stream = torch.cuda.Stream()
    members = [P.Solver(P.params_from_solve(s), stream=stream) for s in solves]
    with P.Batch(stream) as batch:
        for m in members:
            batch.add(m)
        batch.step(n)
        for m, a in zip(members, alone):
            got = (*m.force_history(), m.get_deviations())
            assert all(np.array_equal(x, y) for x, y in zip(got, a))
    for m in members:
        m.close()


@pytest.mark.parametrize("geom,far,wall,sigma,coll", [
    (W.PLATE, W.FAR_WALL, "bb", 1.0, "regularized"),
    (W.PLATE, W.FAR_EQ, "bb", 1.0, "bgk"),
    (W.PLATE, W.FAR_EQ, "maxwell", 0.35, "regularized"),
    (W.PLATE, W.FAR_WALL, "ds", 1.0, "bgk"),
    (W.PERIODIC, W.FAR_EQ, "bb", 1.0, "regularized"),
    (W.PERIODIC, W.FAR_EQ, "bb", 1.0, "bgk"),
])
@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("Q,nx,lengths", [(37, 16, [3301, 3300, 3, 3299, 3310, 3400]),
                                          (37, 3, [77000] * 3),
                                          (9, 16, [7300] * 8 + [4])])
def test_single_steps(P, Q, nx, lengths, storage, geom, far, wall, sigma, coll):  # noqa: F811
    """Batches so long that calls of one step go straight through memory: the
    fields, forces and lock-in sums of each lattice alone in one call (several
    steps per launch in LDS), bit for bit."""
    import torch
    n = 5
    print(f"case {nx} Q{Q} {storage} {geom} {far} {wall} {coll}", flush=True)
    v, w, th = P.lattice(Q)
    rng = np.random.default_rng(21)
    kinds = [rng.standard_normal((Q, 1, nx)) * 1e-3 * np.asarray(w)[:, None, None]
             for _ in range(2)]
    solves, fields, alone = [], [], []
    for i, ny in enumerate(lengths):
        s = W.Solve(Q=Q, geometry=geom, far=far, nx=nx, ny=ny, tau=0.9, omega=2 * math.pi / 40,
                    nsteps=n, window_first=1, window_count=n - 1, storage=storage,
                    collision=coll, wall=wall, accommodation=sigma)
        # different in every row
        f = kinds[i % 2] * np.cos(0.37 * np.arange(ny) + i)[None, :, None]
        with P.Solver(P.params_from_solve(s)) as sv:
            sv.set_deviations(f)
            sv.step(n)
            alone.append((*sv.force_history(), sv.lockin()[0], sv.get_deviations()))
        solves.append(s)
        fields.append(f)
    stream = torch.cuda.Stream()
    members = [P.Solver(P.params_from_solve(s), stream=stream) for s in solves]
    with P.Batch(stream) as batch:
        for m, f in zip(members, fields):
            batch.add(m)
            m.set_deviations(f)
        for k in (1, 2, 1, 1):
            batch.step(k)
        for m, a in zip(members, alone):
            got = (*m.force_history(), m.lockin()[0], m.get_deviations())
            assert all(np.array_equal(x, y) for x, y in zip(got, a))
    for m in members:
        m.close()


@pytest.mark.parametrize("nx,ny", [(16, 6250), (16, 6251), (14, 7142), (14, 7143), (13, 7700)])
def test_wide_line(P, nx, ny):  # noqa: F811
    """Lengths on both sides of the line where D2Q37 lattices of 14 to 16 columns
    leave the column kernel: 5 FP64 steps against the long-double oracle."""
    n = 5
    s = W.Solve(Q=37, geometry=W.PLATE, far=W.FAR_WALL, nx=nx, ny=ny, tau=0.9, storage="f64",
                omega=2 * math.pi / 40, nsteps=n, window_first=0, window_count=n)
    v, w, th = P.lattice(37)
    f0 = _f0(s, w, seed=17, amp=1e-3)
    with P.Solver(P.params_from_solve(s)) as sv:
        sv.set_populations(f0)
        sv.step(n)
        fx, fy = sv.force_history()
        dev = sv.get_deviations()
    ox, oy, of = O.run(_oracle_params(s), n, f0=f0, want_state=True, variant="ld")
    want = of - w[:, None, None] * s.rho0
    assert np.max(np.abs(dev - want)) <= 1e-12 * np.max(np.abs(want)) + 2 * np.spacing(np.max(w))
    scale = max(np.max(np.abs(ox)), np.max(np.abs(oy)))
    assert np.max(np.abs(fx - ox)) <= 1e-12 * scale and np.max(np.abs(fy - oy)) <= 1e-12 * scale


@pytest.mark.parametrize("capacity", [1, 2, 5])
@pytest.mark.parametrize("Q", [9, 37])
def test_short_force_ring(P, Q, capacity):  # noqa: F811
    """A force ring shorter than the steps of one launch holds the newest
    samples after every call."""
    n = 97
    s = W.Solve(Q=Q, geometry=W.PLATE, far=W.FAR_EQ, nx=4, ny=40, tau=0.9,
                omega=2 * math.pi / 40, nsteps=n, window_first=0, window_count=n)
    with P.Solver(P.params_from_solve(s)) as sv:
        sv.step(n)
        fx, fy = sv.force_history()
    with P.Solver(P.params_from_solve(s, history_capacity=capacity)) as sv:
        for k in (31, 3, 2, 61):
            sv.step(k)
            at, m = sv.steps_done, min(capacity, sv.steps_done)
            gx, gy = sv.force_history(at - m, m)
            assert np.array_equal(gx, fx[at - m:at]) and np.array_equal(gy, fy[at - m:at])


@pytest.mark.parametrize("own_stream", [True, False])
@pytest.mark.parametrize("graphs", [32, 0])
def test_columns_beside_tiles(P, own_stream, graphs):  # noqa: F811
    """Narrow plates in a batch with a box and a population member (their
    launches run beside the others'): reads between calls, members that leave
    and a member that ends early see the same bits as each solve alone."""
    import torch
    n = 150
    kw = dict(Q=37, tau=0.9, omega=2 * math.pi / 40, window_first=5)
    solves = [
        W.Solve(geometry=W.PLATE, far=W.FAR_WALL, nx=4, ny=700, nsteps=n, window_count=n - 9, **kw),
        W.Solve(geometry=W.BOX, far=W.FAR_EQ, nx=90, ny=75, box=(40, 30, 9, 11), nsteps=n,
                window_count=n - 9, **kw),
        W.Solve(geometry=W.PLATE, far=W.FAR_EQ, nx=7, ny=64, nsteps=n - 40, window_count=n - 60,
                wall="ds", **kw),
        W.Solve(geometry=W.PLATE, far=W.FAR_EQ, nx=40, ny=64, nsteps=n, window_count=n - 9, **kw),
    ]
    alone = []
    for s in solves:
        with P.Solver(P.params_from_solve(s)) as sv:
            sv.step(s.nsteps)
            alone.append((*sv.force_history(), sv.get_deviations(), sv.lockin()[0]))
    stream = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
    members = [P.Solver(P.params_from_solve(s), stream=stream) for s in solves]
    with P.Batch(stream) as batch:
        batch.set_graphs(graphs)
        for m in members:
            batch.add(m)
        for k in (1, 64, 33):
            batch.step(k)
            for m, a in zip(members, alone):
                fx, fy = m.force_history(m.steps_done - 1, 1)
                assert (fx[0], fy[0]) == (a[0][m.steps_done - 1], a[1][m.steps_done - 1])
        batch.remove(members[1])
        members[1].step(n - 98)
        batch.step(n - 98)
        for m, a in zip(members, alone):
            got = (*m.force_history(), m.get_deviations(), m.lockin()[0])
            assert all(np.array_equal(x, y) for x, y in zip(got, a))
    for m in members:
        m.close()

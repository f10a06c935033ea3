"""GPU parity at the edges of the wall code: bodies of the least accepted
thickness, bodies across tile borders, plates thinner than two wall bands."""
import math

import numpy as np
import pytest

import lbm_inputs as W
import oracle as O
from tests.test_parity_gpu import P, _f0, _gpu, _oracle_params  # noqa: F401

pytestmark = pytest.mark.gpu

EDGE = {
    # name: (Q, geometry, far, nx, ny, box)
    "q37_thin_box": (37, W.BOX, W.FAR_EQ, 70, 40, (30, 19, 3, 3)),
    "q37_box_on_borders": (37, W.BOX, W.FAR_EQ, 140, 40, (61, 10, 6, 17)),
    "q37_box_least_margin": (37, W.BOX, W.FAR_EQ, 70, 21, (3, 3, 64, 15)),
    "q9_thin_box": (9, W.BOX, W.FAR_EQ, 70, 20, (63, 11, 1, 2)),
    "q37_plate_thin": (37, W.PLATE, W.FAR_WALL, 65, 4, (0, 0, 0, 0)),
    "q37_plate_five": (37, W.PLATE, W.FAR_WALL, 128, 5, (0, 0, 0, 0)),
    "q9_plate_thin": (9, W.PLATE, W.FAR_WALL, 64, 3, (0, 0, 0, 0)),
}


@pytest.mark.parametrize("wall,sigma", [("bb", 1.0), ("ds", 1.0), ("maxwell", 0.3)])
@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("name", list(EDGE))
def test_wall_edges(P, name, storage, wall, sigma):  # noqa: F811
    """Fields after 12 steps and every force against the long-double oracle
    (FP64: 1e-12; FP32: 12 steps of a few roundings each, 2e-5)."""
    Q, geom, far, nx, ny, box = EDGE[name]
    n = 12
    s = W.Solve(Q=Q, geometry=geom, far=far, nx=nx, ny=ny, tau=1.1, omega=2 * math.pi / 32,
                box=box, nsteps=n, window_first=0, window_count=n, storage=storage, wall=wall,
                accommodation=sigma)
    print(f"case {name} {storage} {wall} {sigma}", flush=True)
    v, w, th = P.lattice(Q)
    f0 = _f0(s, w, seed=77, amp=1e-3)
    fx, fy, z, f = _gpu(P, s, f0, state=True, repr_=2)
    ox, oy, of = O.run(_oracle_params(s), n, f0=f0, want_state=True, variant="ld")
    rest = w[:, None, None] * s.rho0
    mask = np.ones((ny, nx))
    x0, y0, lx, ly = s.box
    mask[y0:y0 + ly, x0:x0 + lx] = 0
    scale = np.max(np.abs((of - rest) * mask))
    tol = 1e-12 if storage == "f64" else 2e-5
    assert np.max(np.abs((f - of) * mask)) <= tol * scale + 2 * np.spacing(np.max(w))
    fscale = max(np.max(np.abs(ox)), np.max(np.abs(oy)))
    assert np.max(np.abs(fx - ox)) <= tol * fscale
    assert np.max(np.abs(fy - oy)) <= tol * fscale


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("wall", ["bb", "ds"])
def test_launch_size_does_not_change_bits(P, storage, wall):  # noqa: F811
    """A small box alone (one row per wavefront), with each explicit tile, and
    beside a member large enough for the launch to take more rows: the same
    forces and fields bit for bit."""
    import torch
    n = 40
    small = W.Solve(Q=37, geometry=W.BOX, far=W.FAR_EQ, nx=90, ny=75, tau=0.8,
                    omega=2 * math.pi / 40, box=(40, 30, 9, 11), nsteps=n, window_first=0,
                    window_count=n, storage=storage, wall=wall)
    large = W.Solve(Q=37, geometry=W.PLATE, far=W.FAR_EQ, nx=1000, ny=800, tau=0.7,
                    omega=2 * math.pi / 40, nsteps=n, window_first=0, window_count=n,
                    storage=storage)
    out = []
    for tile in (0, 1, 2, 3):
        with P.Solver(P.params_from_solve(small, tile=tile)) as sv:
            sv.step(n)
            out.append((*sv.force_history(), sv.get_deviations()))
    stream = torch.cuda.Stream()
    with P.Solver(P.params_from_solve(small), stream=stream) as a, \
            P.Solver(P.params_from_solve(large, loads=False), stream=stream) as b, \
            P.Batch(stream) as batch:
        batch.add(a)
        batch.add(b)
        batch.step(33)
        batch.step(n - 33)
        out.append((*a.force_history(), a.get_deviations()))
    for o in out[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(o, out[0]))


@pytest.mark.parametrize("nx", [64, 102, 103, 128, 161])
@pytest.mark.parametrize("geom,wall", [(W.BOX, "bb"), (W.PLATE, "ds"), (W.PERIODIC, "bb")])
def test_population_rows(P, nx, geom, wall):  # noqa: F811
    """Populations at widths on both sides of the line where the kernel's tiles
    cover rows padded to whole wavefronts: 12 FP64 steps against the long-double
    oracle within 1e-12, the same bits with every tile."""
    n, ny = 12, 29
    s = W.Solve(Q=37, geometry=geom, far=W.FAR_WALL if geom == W.PLATE else W.FAR_EQ, nx=nx,
                ny=ny, tau=0.9, omega=2 * math.pi / 32,
                box=(25, 9, 12, 8) if geom == W.BOX else (0, 0, 0, 0), nsteps=n,
                window_first=0, window_count=n, storage="f64", collision="bgk", wall=wall)
    v, w, th = P.lattice(37)
    f0 = _f0(s, w, seed=5, amp=1e-3)
    fx, fy, z, f = _gpu(P, s, f0, state=True, repr_=1)
    ox, oy, of = O.run(_oracle_params(s), n, f0=f0, want_state=True, variant="ld")
    x0, y0, lx, ly = s.box
    mask = np.ones((ny, nx))
    mask[y0:y0 + ly, x0:x0 + lx] = 0
    rest = w[:, None, None]
    assert np.max(np.abs((f - of) * mask)) <= \
        1e-12 * np.max(np.abs((of - rest) * mask)) + 2 * np.spacing(np.max(w))
    assert np.max(np.abs(fx - ox)) <= 1e-12 * max(np.max(np.abs(ox)), np.max(np.abs(oy)), 1e-3)
    for tile in (2, 4):
        gx, gy, _, g = _gpu(P, s, f0, state=True, repr_=1, tile=tile)
        assert np.array_equal(g, f) and np.array_equal(gx, fx) and np.array_equal(gy, fy)

"""FP32 states: what a diffuse or Maxwell wall sends back is formed in FP64 (the
emission, the specular share and their mixing) and rounded once."""
import math

import numpy as np
import pytest

import lbm_inputs as W
from tests.test_parity_gpu import P  # noqa: F401

pytestmark = pytest.mark.gpu
SIGMA = 0.37


def _emission(U, rho0, cm, w, vx, th, Mr, Z1, Z2, L1):
    """Deviation of the diffuse arrivals from a column with constants Mr .. L1."""
    e = vx * U / th + U * U * (vx * vx / (2 * th * th) - 1 / (2 * th))
    z = Mr + Z1 * U + Z2 * U * U
    return w * (rho0 * (Mr * e + L1 * U * (1 + e) - Z1 * U - Z2 * U * U) + cm * (1 + e)) / z


@pytest.mark.parametrize("wall", ["ds", "maxwell"])
@pytest.mark.parametrize("Q", [9, 37])
def test_narrow_plate(P, Q, wall):  # noqa: F811
    """One step without relaxation (tau infinite, plain BGK) is the streaming
    alone, so the populations of the wall rows are the arrivals: each within
    half a unit of the last FP32 place of its FP64 value."""
    sigma = SIGMA if wall == "maxwell" else 1.0
    v, w, th = P.lattice(Q)
    v = np.asarray(v)
    index = {tuple(p): q for q, p in enumerate(v.tolist())}
    nx, ny = 5, 8
    s = W.Solve(Q=Q, geometry=W.PLATE, far=W.FAR_WALL, nx=nx, ny=ny, tau=math.inf,
                omega=math.pi, u0=0.05, nsteps=1, window_first=0, window_count=0,
                storage="f32dev", collision="bgk", wall=wall, accommodation=sigma)
    rng = np.random.default_rng(3)
    f = (rng.uniform(-1e-2, 1e-2, (Q, ny, nx)) * w[:, None, None]).astype(np.float32)
    f = f.astype(np.float64)
    with P.Solver(P.params_from_solve(s)) as sv:
        sv.set_deviations(f)
        sv.step(1)
        out = sv.get_deviations()
    U = s.u0 * math.sin(s.omega * 0.5)
    up = v[:, 1] > 0
    flux, vx = (v[:, 1] * w)[up], v[up, 0]
    A1, A2 = flux.sum(), (flux * (vx ** 2 / (2 * th * th) - 1 / (2 * th))).sum()
    cm = sum(f[q, r] for q in range(Q) for r in range(max(0, -v[q, 1])))
    n = 0
    for q in range(Q):
        vx, vy = v[q]
        for y in range(max(0, vy)):
            exact = sigma * _emission(U, s.rho0, cm, w[q], vx, th, A1, 0.0, A2, 0.0)
            if sigma != 1.0:
                spec = f[index[(vx, -vy)], vy - 1 - y]
                exact = exact + (1 - sigma) * np.roll(spec, vx)
            ulp = np.spacing(np.abs(exact).astype(np.float32)).astype(np.float64)
            assert np.all(np.abs(out[q, y] - exact) <= 0.5 * ulp * (1 + 1e-6) + 1e-18)
            n += nx
    assert n > 0


def _face_sums(v, w, n, sg, ax, lo, hi):
    """Velocities of normal speed n towards the fluid and their tangential part,
    those with a source behind the wall."""
    for q, (vx, vy) in enumerate(v.tolist()):
        vn, t = (vx, vy) if ax else (vy, vx)
        if vn == sg * n and -lo <= t <= hi:
            yield w[q], vx, vy


@pytest.mark.parametrize("wall", ["ds", "maxwell"])
@pytest.mark.parametrize("Q", [9, 37])
@pytest.mark.parametrize("geom", [W.PLATE, W.BOX])
def test_coefficients(P, geom, Q, wall):  # noqa: F811
    """First step from rest of a coefficient state.  The cells R - 1 cells from a face
    get one set of arrivals (normal speed R) and nothing from the stream: their
    mass and momentum sums, rounded to FP32 once, then the FP32 scaling to
    the coefficients j / theta, to the last FP32 bit."""
    sigma = SIGMA if wall == "maxwell" else 1.0
    v, w, th = P.lattice(Q)
    v = np.asarray(v)
    R = int(v.max())
    nx, ny, box = (70, 12, (0, 0, 0, 0)) if geom == W.PLATE else (80, 50, (30, 20, 12, 9))
    x0, y0, lx, ly = box
    x1, y1 = x0 + lx, y0 + ly
    f32 = np.float32
    ith = f32(1.0 / th)
    checked = 0
    for k in range(24):
        s = W.Solve(Q=Q, geometry=geom, far=W.FAR_WALL if geom == W.PLATE else W.FAR_EQ, nx=nx,
                    ny=ny, tau=1.3, omega=math.pi, u0=1e-3 * 1.37 ** k / 10, box=box, nsteps=1,
                    window_first=0, window_count=0, storage="f32dev", wall=wall,
                    accommodation=sigma)
        with P.Solver(P.params_from_solve(s, representation=2)) as sv:
            sv.step(1)
            dev = sv.get_deviations()
        U = s.u0 * math.sin(s.omega * 0.5)
        ladd = 2 * s.rho0 / th * U
        # coefficients (by)(bx) back from the populations of speed 1
        def coef(axis):
            a = [q for q, p in enumerate(v.tolist()) if p == ([1, 0] if axis == 0 else [0, 1])][0]
            b = [q for q, p in enumerate(v.tolist()) if p == ([-1, 0] if axis == 0 else [0, -1])][0]
            return ((dev[a] - dev[b]) / (2 * w[a])).astype(f32)
        bx, by = coef(0), coef(1)
        if geom == W.PLATE:
            cells = [(0, x, R - 1, False, 1, R, R) for x in (0, 1, 33, nx - 1)]
        else:
            cells = [(0, x, y0 - R, False, -1, min(R, x1 - x - 1), min(R, x - x0))
                     for x in range(x0 + R, x1 - R)]
            cells += [(1, x, y1 + R - 1, False, 1, min(R, x1 - x - 1), min(R, x - x0))
                      for x in range(x0 + R, x1 - R)]
            cells += [(2, x0 - R, y, True, -1, min(R, y1 - y - 1), min(R, y - y0))
                      for y in range(y0 + R, y1 - R)]
            cells += [(3, x1 + R - 1, y, True, 1, min(R, y1 - y - 1), min(R, y - y0))
                      for y in range(y0 + R, y1 - R)]
        for face, x, y, ax, sg, lo, hi in cells:
            # the column's constants over all its links
            Mr = Z1 = Z2 = L1 = 0.0
            for n in range(1, R + 1):
                for wq, vx, vy in _face_sums(v, w, n, sg, ax, lo, hi):
                    Mr += n * wq
                    if geom == W.BOX:
                        Z1 += n * wq * vx / th
                        L1 += n * 2 * wq * vx / th
                    Z2 += n * wq * (vx * vx / (2 * th * th) - 1 / (2 * th))
            jn = jt = m0 = size = 0.0
            for wq, vx, vy in _face_sums(v, w, R, sg, ax, lo, hi):
                arr = sigma * _emission(U, s.rho0, 0.0, wq, vx, th, Mr, Z1, Z2, L1)
                if ax:
                    arr += (1 - sigma) * wq * vx * ladd
                m0 += arr
                size += abs(arr)
                jt += arr * (vy if ax else vx)
            jn = f32(sg * R) * f32(m0)
            want_n, want_t = f32(jn * ith), f32(f32(jt) * ith)
            got_n, got_t = (bx[y, x], by[y, x]) if ax else (by[y, x], bx[y, x])
            # (a sum that cancels is the rounding error of its FP64 terms)
            eps = 16 * np.spacing(size) * R / th
            assert abs(float(got_n) - float(want_n)) <= eps, (k, face, x, y, got_n, want_n)
            assert abs(float(got_t) - float(want_t)) <= eps, (k, face, x, y, got_t, want_t)
            checked += 1
    assert checked >= 24 * 4

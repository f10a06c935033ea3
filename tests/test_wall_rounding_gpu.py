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

"""lbm_create_static at its limit: what one row per wavefront adds to the work
list of a small lattice does not count."""
import dataclasses
import math

import numpy as np
import pytest

import lbm_inputs as W
from tests.test_parity_gpu import P  # noqa: F401

pytestmark = pytest.mark.gpu


def _box(n):
    return W.Solve(Q=37, geometry=W.BOX, far=W.FAR_EQ, nx=640, ny=520, tau=0.9,
                   omega=2 * math.pi / 64, box=(300, 250, 20, 12), nsteps=n, window_first=0,
                   window_count=64)


def _at(P, need):  # noqa: F811
    """The box with as many steps (drive and history) as need `need` bytes."""
    lo, hi = 64, 1 << 22
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if P.required_bytes(P.params_from_solve(_box(mid))) <= need else (lo, mid)
    return _box(lo)


def test_static_limit_ignores_finer_tiles(P):  # noqa: F811
    limit = P.lbm.STATIC_SCRATCH_BYTES
    s = _at(P, limit + 4096)
    assert limit < P.required_bytes(P.params_from_solve(s)) <= limit + 4096
    out = []
    for memory in ("torch", "static"):
        with P.Solver(P.params_from_solve(s), memory=memory) as sv:
            sv.step(24)
            sv.synchronize()
            out.append((*sv.force_history(0, 24), sv.get_deviations()))
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    over = _at(P, limit + 65536)
    with pytest.raises(P.LbmError) as e:
        P.Solver(P.params_from_solve(dataclasses.replace(over)), memory="static")
    assert e.value.code == P.lbm.ESCRATCH

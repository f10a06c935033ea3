"""Performance cases of the oscillating-body lattice-BGK solver.

A case is one chunk of work as a program of this framework does it: a solver
(or a batch of solvers) that lives on the GPU is advanced by a number of
steps, and the force on the body is read back, with the impedance where the
chunk is a whole drive period.  A run that has used up its drive table (one
period) is started again by lbm_seek to step 0: the drive goes on in phase and
the lock-in sums start anew, as a program that watches Z settle does.

The force of an FP32 state is kept as float32 (the state's precision), that
of an FP64 state as float64.  `exact` advances the same inputs in FP64 with
plain torch.
"""
import dataclasses
import math

import numpy as np
import torch

import lbm_inputs as W
from paper_0904_4504_amd import lbm as L


def listed():
    return [
        # a program that follows the force step by step: the smallest call,
        # one step and its force, on a small ragged box that starts from a
        # loaded perturbation
        _case("monitor_step", kind="box", nx=96, ny=77, lx=10, ly=9, steps=1, period=256,
              noise=1e-4),
        # the Stokes-layer check: D2Q9 FP64, Stokes depth 16, a narrow plate
        # started from seeded noise of 1e-9, its fields read at the end
        _case("stokes_plate", kind="plate", Q=9, storage="f64", nx=4, ny=256, steps=1024,
              period=8192, tw_lo=2.3e-4, tw_hi=2.4e-4, noise=1e-9, fields=True),
        # the plate sweep of the damping curve: five 4 x 2048 plates in one
        # batch, one drive period and the impedances
        _case("plate_sweep", kind="plate", nx=4, ny=2048, count=5, steps=1024, period=1024),
        # the same plate in FP64 with diffuse scattering, alone (parity runs)
        _case("plate_f64_diffuse", kind="plate", storage="f64", nx=4, ny=1531, wall="ds",
              far="eq", steps=512, period=1024),
        # plates wide enough for the coefficient state, Maxwell walls, a
        # stationary far wall
        _case("wide_plates", kind="plate", nx=64, ny=2048, count=4, wall="maxwell", sigma=0.6,
              steps=256, period=1024),
        # the diffuse beam section in a small domain, one period, Z and the
        # fields at its end
        _case("wall_box", kind="box", nx=256, ny=256, lx=32, ly=16, wall="ds", steps=1024,
              period=1024, fields=True),
        # the beam box: three tau*omega of a 32 x 16 section in 1024^2
        _case("beam_box", kind="box", nx=1024, ny=1024, lx=32, ly=16, count=3, steps=512,
              period=1024, tw_lo=0.1, tw_hi=10.0),
        # FP64 section of ragged size, alone
        _case("box_f64", kind="box", storage="f64", nx=515, ny=389, lx=33, ly=12, steps=128,
              period=1024),
        # a serving chunk: resident requests, one box to four plates
        _case("serving_mix", kind="mix", nx=1024, ny=1024, lx=32, ly=16, count=2, plates=8,
              ny_lo=1024, ny_hi=8192, order=5, steps=256, period=1024, tw_lo=0.1, tw_hi=10.0),
        # the batched sweep: 256 uneven solves (256 .. 2048 cells per side),
        # 13 GB of state streaming from HBM
        _case("batch_sweep", kind="sweep", count=256, order=4, steps=64, period=1024),
        # plain BGK for checks: the populations themselves are the state
        _case("bgk_box", kind="box", nx=641, ny=1000, lx=21, ly=40, collision="bgk", steps=64,
              period=1024),
        # a run from given fields: load deviations, a few steps, read fields
        _case("fields_io", kind="box", nx=205, ny=150, lx=16, ly=24, steps=16, period=1024,
              noise=1e-4, reload=True, fields=True),
    ]


def _case(name, **kw):
    c = dict(kind="box", Q=37, storage="f32dev", collision="regularized", wall="bb", sigma=1.0,
             far="", nx=0, ny=0, lx=0, ly=0, count=1, plates=0, ny_lo=0, ny_hi=0, order=0,
             steps=1, period=1024, tw_lo=1e-2, tw_hi=1e2, noise=0.0, reload=False,
             fields=False)
    c.update(kw)
    if not c["far"]:
        c["far"] = "wall" if c["kind"] == "plate" else "eq"
    if name:
        c["name"] = name
    return c


def draw(rng):
    """One more case: a kind of work, sizes log-uniform over its range."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    pick = rng.choice(["plate", "plate", "wide", "box", "box", "mix", "sweep", "bgk", "fields"])
    wall, sigma = rng.choice([("bb", 1.0), ("bb", 1.0), ("ds", 1.0),
                              ("maxwell", round(rng.uniform(0.0, 1.0), 3))])
    f64 = rng.random() < 0.25
    storage = "f64" if f64 else "f32dev"
    Q = rng.choice([37, 37, 37, 9])
    if pick == "plate":
        return _case("", kind="plate", Q=Q, storage=storage, wall=wall, sigma=sigma,
                     far=rng.choice(["wall", "eq"]), nx=rng.choice([3, 4, 4, 5, 8]),
                     ny=size(100, 8192), count=rng.randint(1, 8), steps=size(100, 1024))
    if pick == "wide":
        return _case("", kind="plate", storage=storage, wall=wall, sigma=sigma,
                     far=rng.choice(["wall", "eq"]), nx=size(64, 600), ny=size(128, 2048),
                     count=rng.randint(1, 3), steps=size(16, 256))
    if pick == "box":
        small = rng.random() < 0.4
        steps = size(1, 256) if small else size(16, 256)
        return _case("", kind="box", Q=Q, storage=storage, wall=wall, sigma=sigma,
                     nx=size(80, 320 if small else 1280), ny=size(80, 320 if small else 1280),
                     lx=rng.randint(8, 64), ly=rng.randint(8, 64), count=rng.randint(1, 3),
                     steps=steps, noise=1e-4 if steps < 8 else 0.0)
    if pick == "mix":
        n = size(256, 1024)
        return _case("", kind="mix", nx=n, ny=n, lx=rng.randint(8, 64), ly=rng.randint(8, 64),
                     count=rng.randint(1, 3), plates=rng.randint(2, 12), ny_lo=1024, ny_hi=8192,
                     order=rng.randint(0, 10 ** 6), steps=size(32, 256))
    if pick == "sweep":
        return _case("", kind="sweep", count=size(4, 64), order=rng.randint(0, 10 ** 6),
                     steps=size(16, 64))
    if pick == "bgk":
        return _case("", kind="box", Q=Q, storage=storage, collision="bgk", nx=size(100, 900),
                     ny=size(100, 900), lx=rng.randint(8, 64), ly=rng.randint(8, 64),
                     steps=size(16, 64))
    return _case("", kind="box", Q=Q, storage=storage, nx=size(80, 400), ny=size(80, 400),
                 lx=rng.randint(8, 32), ly=rng.randint(8, 32), steps=size(2, 32), noise=1e-4,
                 reload=True, fields=True)


# ------------------------------------------------------------------ inputs


def _solves(case, seed):
    """The solves of a case, tau*omega drawn log-uniformly from the seed."""
    rng = np.random.default_rng([int(seed), 2009])
    c = case
    # the drive table is one period, a whole number of passes
    period = c["steps"] * max(1, c["period"] // c["steps"])
    omega = 2 * math.pi / period

    def plate(nx, ny, far, **kw):
        return W.Solve(Q=c["Q"], geometry=W.PLATE, far=far, nx=nx, ny=ny, tau=1.0, omega=omega,
                       storage=c["storage"], collision=c["collision"], **kw)

    def box(nx, ny, lx, ly, **kw):
        return W.Solve(Q=c["Q"], geometry=W.BOX, far=W.FAR_EQ, nx=nx, ny=ny, tau=1.0, omega=omega,
                       box=((nx - lx) // 2, (ny - ly) // 2, lx, ly), storage=c["storage"],
                       collision=c["collision"], **kw)

    walls = dict(wall=c["wall"], accommodation=c["sigma"])
    if c["kind"] == "plate":
        out = [plate(c["nx"], c["ny"], c["far"], **walls) for _ in range(c["count"])]
    elif c["kind"] == "box":
        out = [box(c["nx"], c["ny"], c["lx"], c["ly"], **walls) for _ in range(c["count"])]
    elif c["kind"] == "mix":
        sizes = np.random.default_rng(c["order"])
        out = [box(c["nx"], c["ny"], c["lx"], c["ly"]) for _ in range(c["count"])]
        out += [plate(4, int(sizes.integers(c["ny_lo"], c["ny_hi"] + 1)), W.FAR_WALL)
                for _ in range(c["plates"])]
    else:
        out = W.batch_sweep(count=c["count"], seed=c["order"], period=period)
    tws = np.exp(rng.uniform(math.log(c["tw_lo"]), math.log(c["tw_hi"]), len(out)))
    return [dataclasses.replace(s, tau=float(W.tau_lb(tw, omega)), tau_omega=float(tw),
                                nsteps=period, window_first=0, window_count=period,
                                noise=c["noise"], seed=int(seed) * 1000 + i)
            for i, (s, tw) in enumerate(zip(out, tws))]


def prepare(case, seed):
    solves = _solves(case, seed)
    stream = torch.cuda.Stream()
    loads = case["noise"] > 0
    fields = [W.initial_noise(s) for s in solves] if loads else None
    solvers = [L.Solver(L.params_from_solve(s, loads=loads), stream=stream) for s in solves]
    if loads:
        for sv, f in zip(solvers, fields):
            sv.set_deviations(f)
    batch = None
    if len(solvers) > 1:
        batch = L.Batch(stream)
        for sv in solvers:
            batch.add(sv)
    return {"case": case, "solves": solves, "solvers": solvers, "batch": batch,
            "fields": fields}


def run(state):
    case, solvers, batch = state["case"], state["solvers"], state["batch"]
    n = case["steps"]
    for i, sv in enumerate(solvers):
        if case["reload"]:
            sv.set_deviations(state["fields"][i])
        if case["reload"] or sv.steps_done + n > state["solves"][i].nsteps:
            sv.seek(0)
    if batch is not None:
        batch.step(n)
    else:
        solvers[0].step(n)
    real = np.float64 if case["storage"] == "f64" else np.float32
    out = {"plate_fx": [], "plate_fy": [], "box_f": [], "Z": []}
    for s, sv in zip(state["solves"], solvers):
        fx, fy = sv.force_history(sv.steps_done - n, n)
        if s.geometry == W.PLATE:
            out["plate_fx"].append(fx)
            out["plate_fy"].append(fy)
        else:
            out["box_f"].append(np.stack([fx, fy]))
        if n == s.nsteps:
            z = sv.impedance()
            out["Z"].append([z["R"], z["X"]])
    out = {k: np.stack(v).astype(real) for k, v in out.items() if v}
    if case["fields"]:
        out["fields"] = np.stack([sv.get_deviations() for sv in solvers]).astype(real)
    return out


def work(case):
    """Bytes: the state read once and written once -- by every step where it
    exceeds the chip's caches (256 MB), once per pass where it does not -- in
    its smallest form (six Hermite coefficients per cell after a regularized
    collision, else Q populations).  Flops: eight per velocity and update."""
    solves = _solves(case, 0)
    es = 8 if case["storage"] == "f64" else 4
    cells = sum(s.fluid_cells for s in solves)
    values = 6 if case["collision"] == "regularized" else case["Q"]
    sweeps = case["steps"] if cells * values * es * 2 > 256e6 else 1
    nbytes = 2 * cells * values * es * sweeps + 16 * case["steps"] * len(solves)
    if case["fields"]:
        nbytes += 8 * case["Q"] * sum(s.nx * s.ny for s in solves) * (2 if case["reload"] else 1)
    return {"bytes": nbytes, "flops": 8 * case["Q"] * cells * case["steps"]}


# ------------------------------------------------------- the same in 64 bits

# Gauss-Hermite velocity sets: orbit representatives, weights, theta (D2Q37:
# the table of the paper's appendix)
_SETS = {
    9: ([(0, 0), (1, 0), (1, 1)], [4 / 9, 1 / 9, 1 / 36], 1 / 3),
    37: ([(0, 0), (1, 0), (1, 1), (2, 0), (2, 2), (3, 0), (1, 2), (1, 3)],
         [0.233150669132352000, 0.107306091542219000, 0.057667859888794800,
          0.014208216158450700, 0.001011937592673570, 0.000245301027757717,
          0.005353049000513770, 0.000283414252994198], 0.69795332201968309),
}


def _lattice(Q):
    v, w = [], []
    orbits, weights, theta = _SETS[Q]
    for (a, b), wt in zip(orbits, weights):
        pts = {(s * p, t * q) for p, q in ((a, b), (b, a)) for s in (1, -1) for t in (1, -1)}
        for p in sorted(pts, key=lambda u: math.atan2(u[1], u[0]) % (2 * math.pi)):
            v.append(p)
            w.append(wt)
    return np.array(v), np.array(w), theta


def _links(s, v, R):
    """Wall links of a solve: arrival (direction, cell), bounce-back partner,
    specular source (flat indices into [Q][ny][nx]), column (-1: bounce-back),
    whether the face is normal to the motion, whether the wall moves."""
    index = {tuple(p): q for q, p in enumerate(v.tolist())}
    nx, ny = s.nx, s.ny
    diffuse = s.wall != "bb"
    rows = []

    def flat(q, y, x):
        return (q * ny + y) * nx + x

    if s.geometry == W.PLATE:
        x = np.arange(nx)
        for q, (vx, vy) in enumerate(v.tolist()):
            o, r = index[(-vx, -vy)], index[(vx, -vy)]
            for y in range(min(max(vy, 0), ny)):
                py = vy - 1 - y
                rows.append((q, flat(q, y, x), flat(o, py, x), flat(r, py, (x - vx) % nx),
                             x if diffuse else x * 0 - 1, x * 0, x * 0 + 1))
            if s.far == W.FAR_WALL:
                for y in range(max(0, ny + vy), ny):
                    py = 2 * ny - 1 - (y - vy)
                    rows.append((q, flat(q, y, x), flat(o, py, x), flat(o, py, x), x * 0 - 1,
                                 x * 0, x * 0))
    else:
        x0, y0, lx, ly = s.box
        x1, y1 = x0 + lx, y0 + ly
        gy, gx = np.mgrid[y0 - R:y1 + R, x0 - R:x1 + R]
        gy, gx = gy.ravel(), gx.ravel()
        inx, iny = (gx >= x0) & (gx < x1), (gy >= y0) & (gy < y1)
        for q, (vx, vy) in enumerate(v.tolist()):
            sx, sy = gx - vx, gy - vy
            hit = ~(inx & iny) & (sx >= x0) & (sx < x1) & (sy >= y0) & (sy < y1)
            x, y, sx, sy, ix, iy = (a[hit] for a in (gx, gy, sx, sy, inx, iny))
            px = np.where(x < x0, 2 * x0 - 1 - sx, np.where(x >= x1, 2 * x1 - 1 - sx, x))
            py = np.where(y < y0, 2 * y0 - 1 - sy, np.where(y >= y1, 2 * y1 - 1 - sy, y))
            o, ry, rx = index[(-vx, -vy)], index[(vx, -vy)], index[(-vx, vy)]
            col = np.where(ix, (x - x0) + np.where(y < y0, 0, lx),
                           np.where(iy, 2 * lx + (y - y0) + np.where(x < x0, 0, ly), -1))
            spec = np.where(ix, flat(ry, py, sx), np.where(iy, flat(rx, sy, px), 0))
            one = np.ones_like(x)
            rows.append((q, flat(q, y, x), flat(o, py, px), spec, col if diffuse else -one,
                         (iy & ~ix) * one, one))
    q = np.concatenate([np.full(len(r[1]), r[0]) for r in rows])
    return (q,) + tuple(np.concatenate([r[k] for r in rows]) for k in range(1, 7))


def _advance(s, f, n, dev):
    """n FP64 steps from rest or from the deviations f: forces [2][n] and the
    final deviations [Q][ny][nx]."""
    v, w, th = _lattice(s.Q)
    R = int(np.abs(v).max())
    Q, ny, nx = s.Q, s.ny, s.nx
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=dev)  # noqa: E731
    f = torch.zeros(Q, ny, nx, dtype=torch.float64, device=dev) if f is None else t(f).clone()
    lq, dst, part, spec, col, normal, moving = _links(s, v, R)
    lw, lvx, lvy = w[lq], v[lq, 0].astype(float), v[lq, 1].astype(float)
    ncol = int(col.max()) + 1 if len(col) else 0
    on = col >= 0
    e1, e2 = lvx / th, lvx ** 2 / (2 * th * th) - 1 / (2 * th)
    sums = [np.bincount(col[on], k[on], minlength=max(ncol, 1))
            for k in (lw, lw * e1, lw * e2, 2 * lw * e1)]
    static = -2 * s.rho0 * np.array([(lw * lvx * moving).sum(), (lw * lvy * moving).sum()])
    dst, part, spec, con = t(dst), t(part), t(spec), t(on)
    ccol, lwt, vxt, vyt = t(np.maximum(col, 0)), t(lw), t(lvx), t(lvy)
    e1, e2, movt, nort = t(e1), t(e2), t(moving.astype(float)), t(normal.astype(float))
    mr, z1, z2, l1 = (t(a)[ccol] for a in sums)
    ladd = 2 * s.rho0 / th
    sigma = s.accommodation if s.wall == "maxwell" else 1.0
    vx, vy = t(v[:, 0].astype(float)), t(v[:, 1].astype(float))
    basis = torch.stack([vx * 0 + 1, vx, vy, vx * vx, vx * vy, vy * vy])
    post = (basis * t(w)).t().contiguous()
    fluid = torch.ones(ny, nx, dtype=torch.float64, device=dev)
    if s.geometry == W.BOX:
        x0, y0, lx, ly = s.box
        fluid[y0:y0 + ly, x0:x0 + lx] = 0
    f *= fluid
    om = 1.0 / s.tau
    pad = torch.zeros(Q, ny + 2 * R, nx + 2 * R, dtype=torch.float64, device=dev)
    adv = torch.empty_like(f)
    force = torch.zeros(n, 2, dtype=torch.float64, device=dev)
    for k in range(n):
        U = s.u0 * math.sin(s.omega * (k + 0.5))
        pad[:, R:R + ny, R:R + nx] = f
        if s.geometry == W.PLATE:
            pad[:, :, :R] = pad[:, :, nx:nx + R].clone()
            pad[:, :, R + nx:] = pad[:, :, R:2 * R].clone()
        for q, (a, b) in enumerate(v.tolist()):
            adv[q] = pad[q, R - b:R - b + ny, R - a:R - a + nx]
        if len(lq):
            p = f.view(-1)[part]
            arr = p + lwt * vxt * movt * (ladd * U)
            if ncol:
                cm = torch.zeros(ncol, dtype=torch.float64, device=dev)
                cm.index_add_(0, ccol[con], p[con])
                cm = cm[ccol]
                e = e1 * U + e2 * U * U
                em = lwt * (s.rho0 * (mr * e + l1 * U * (1 + e) - z1 * U - z2 * U * U)
                            + cm * (1 + e)) / (mr + z1 * U + z2 * U * U)
                sp = f.view(-1)[spec] + lwt * vxt * nort * (ladd * U)
                arr = torch.where(con, sigma * em + (1 - sigma) * sp, arr)
            adv.view(-1)[dst] = arr
            both = (p + arr) * movt
            force[k, 0] = static[0] - (vxt * both).sum()
            force[k, 1] = static[1] - (vyt * both).sum()
        m = basis @ adv.view(Q, -1)
        rho = s.rho0 + m[0]
        ex, exy, ey = m[1] * m[1] / rho, m[1] * m[2] / rho, m[2] * m[2] / rho
        if s.collision == "bgk":
            bx, bxy, by = ex, exy, ey
        else:
            axx, ayy = m[3] - m[0] * th, m[5] - m[0] * th
            bx, bxy, by = axx - om * (axx - ex), m[4] - om * (m[4] - exy), ayy - om * (ayy - ey)
        c = torch.stack([m[0] - (bx + by) / (2 * th), m[1] / th, m[2] / th,
                         bx / (2 * th * th), bxy / (th * th), by / (2 * th * th)])
        g = (post @ c).view(Q, ny, nx)
        f = (adv + om * (g - adv) if s.collision == "bgk" else g) * fluid
    return force.t().cpu().numpy(), f


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    n = case["steps"]
    out = {"plate_fx": [], "plate_fy": [], "box_f": [], "Z": []}
    fields = []
    for s in _solves(case, seed):
        f0 = W.initial_noise(s) if case["noise"] > 0 else None
        force, f = _advance(s, f0, n, dev)
        if s.geometry == W.PLATE:
            out["plate_fx"].append(force[0])
            out["plate_fy"].append(force[1])
        else:
            out["box_f"].append(force)
        if n == s.nsteps:
            arg = s.omega * (np.arange(n) + 0.5)
            A = np.stack([np.sin(arg), np.cos(arg), np.ones(n)], 1)
            a, b, _ = np.linalg.lstsq(A, force[0], rcond=None)[0]
            out["Z"].append([-a / s.u0, -b / s.u0])
        if case["fields"]:
            fields.append(f.cpu().numpy())
        del f
    out = {k: np.stack(v) for k, v in out.items() if v}
    if case["fields"]:
        out["fields"] = np.stack(fields)
    return out

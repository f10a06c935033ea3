// Several steps of narrow lattices in one launch (population state).
//
// A plate of a few columns (nx <= kColumnMaxNx, periodic in x) has too few
// cells for a step to be anything but latency: a launch of the population
// kernel and one for the force per step took 6-17 us for 1 k to 40 k cells
// (D2Q9 FP64 4 x 256: 6.5 us, five D2Q37 FP32 4 x 2048: 10.3 us, D2Q37 FP64
// 4 x 1531 with a diffuse wall: 16.6 us), nearly all of it launch, cold
// caches and dependent round trips.  Here one workgroup owns `rows` lattice
// rows, loads them with a halo of R rows per step and side into LDS, and takes
// `nsub` steps there: step s updates the rows that later steps still need, so
// the halo shrinks by R rows a step and the owned rows are exact.  The halo is
// work done twice, on compute units that would idle otherwise.  Per step now
// 0.76, 2.6 and 2.2 us.
//
// One thread per cell: it pulls the Q populations of its cell from LDS,
// collides, and writes them back between two barriers.  The sums and the
// output polynomial are formed per set of mirrored velocities (+-a, +-b), 230
// instead of 400 operations per D2Q37 cell.  What bounds a step is the vector
// issue and the LDS traffic of a compute unit (2 Q values per cell), with the
// launch's 4 us spread over nsub steps; two threads per cell, on two halves of
// the velocity set that a rotation maps onto each other, took as long (2.08
// against 2.27 us per step without walls, 3.4 against 2.8 with).
//
// Walls: the populations that cross a wall are written a second time, into
// the row behind the wall that their arrival pulls from (bounce-back with the
// moving-wall term of the next step, or the specular image of the Maxwell
// wall; zero for the rest-equilibrium far field), so the pull is one rule for
// every cell.  Rows past the region's ends are left out (row_behind_moving).  At
// a diffuse or Maxwell wall the arrivals of the wall rows mix it with the
// emission, in FP64.
// A cell's arithmetic does not depend on the split into workgroups or
// launches, so any sequence of calls gives the same bits.
//
// The workgroup that holds the moving wall (tile 0) has the wall force's
// populations in LDS at every step: its last wavefront, which owns no cell,
// sums the momentum exchange in FP64 in a fixed order and accumulates the
// lock-in sums, beside the other wavefronts' update.
//
// State buffers: step n reads buf[n & 1].  nsub is odd, so a launch writes the
// other buffer than the one that its neighbours' halos are read from, and the
// rule holds after it.  The step counter is read by every workgroup and
// advanced by a launch of its own after the last of a call (advance_kernel);
// `dn` counts the steps of the launches in between.
#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "lattice.hpp"
#include "solver.hpp"
#include "walls.hpp"

namespace lbm {

namespace {

// The crossing populations of one wall column, in a fixed order: population q
// (v_y < 0) at row r < -v_y; its reflection leaves along -v_q.
template <class L>
struct CrossTable {
  static constexpr int count() {
    int n = 0;
    for (int q = 0; q < L::Q; ++q) n += L::vy[q] < 0 ? -L::vy[q] : 0;
    return n;
  }
  static constexpr int N = count();
  int8_t q[N], r[N], vx[N], vy[N];  // vx, vy: the reflected direction
  constexpr CrossTable() : q(), r(), vx(), vy() {
    int n = 0;
    for (int i = 0; i < L::Q; ++i)
      for (int k = 0; k < -L::vy[i]; ++k) {
        q[n] = (int8_t)i;
        r[n] = (int8_t)k;
        vx[n] = (int8_t)-L::vx[i];
        vy[n] = (int8_t)-L::vy[i];
        ++n;
      }
  }
};
template <class L>
__device__ constexpr CrossTable<L> kCross{};

// Calls axis(a, i, along_y) for the velocities +-a along each axis and
// four(a, b) for the mirrored sets (+-a, +-b).
template <class L, class A, class F>
__device__ __forceinline__ void for_sets(A&& axis, F&& four) {
  static_for<1, L::R + 1>([&](auto ac) __attribute__((always_inline)) {
    constexpr int a = decltype(ac)::value;
    if constexpr (find_velocity<L>(a, 0) >= 0) {
      axis(ac, std::false_type{});
      axis(ac, std::true_type{});
    }
    static_for<1, L::R + 1>([&](auto bc) __attribute__((always_inline)) {
      if constexpr (find_velocity<L>(a, decltype(bc)::value) >= 0) four(ac, bc);
    });
  });
}

// Moments (delta rho, jx, jy, Pxx, Pxy, Pyy) of the populations f.
template <class L, typename S>
__device__ __forceinline__ void moments_of(const S (&f)[L::Q], S (&m)[6]) {
  m[0] = f[0];
  m[1] = m[2] = m[3] = m[4] = m[5] = S(0);
  for_sets<L>(
      [&](auto ac, auto along_y) __attribute__((always_inline)) {
        constexpr int a = decltype(ac)::value;
        constexpr bool y = decltype(along_y)::value;
        constexpr int p = find_velocity<L>(y ? 0 : a, y ? a : 0), n = opposite<L>(p);
        const S s = f[p] + f[n];
        m[0] += s;
        m[y ? 2 : 1] += S(a) * (f[p] - f[n]);
        m[y ? 5 : 3] += S(a * a) * s;
      },
      [&](auto ac, auto bc) __attribute__((always_inline)) {
        constexpr int a = decltype(ac)::value, b = decltype(bc)::value;
        constexpr int pp = find_velocity<L>(a, b), pn = find_velocity<L>(a, -b);
        constexpr int nn = opposite<L>(pp), np = opposite<L>(pn);
        const S s1 = f[pp] + f[nn], d1 = f[pp] - f[nn];  // along (a, b)
        const S s2 = f[pn] + f[np], d2 = f[pn] - f[np];  // along (a, -b)
        const S s = s1 + s2;
        m[0] += s;
        m[1] += S(a) * (d1 + d2);
        m[2] += S(b) * (d1 - d2);
        m[3] += S(a * a) * s;
        m[4] += S(a * b) * (s1 - s2);
        m[5] += S(b * b) * s;
      });
}

// out(q, p) for every velocity: p = a0 + v.b + cxx vx^2 + cxy vx vy + cyy vy^2.
template <class L, typename S, class F>
__device__ __forceinline__ void expand(S a0, S bx, S by, S cxx, S cxy, S cyy, F&& out) {
  out(std::integral_constant<int, 0>{}, a0);
  for_sets<L>(
      [&](auto ac, auto along_y) __attribute__((always_inline)) {
        constexpr int a = decltype(ac)::value;
        constexpr bool y = decltype(along_y)::value;
        constexpr int p = find_velocity<L>(y ? 0 : a, y ? a : 0);
        const S e = a0 + S(a * a) * (y ? cyy : cxx), o = S(a) * (y ? by : bx);
        out(std::integral_constant<int, p>{}, e + o);
        out(std::integral_constant<int, opposite<L>(p)>{}, e - o);
      },
      [&](auto ac, auto bc) __attribute__((always_inline)) {
        constexpr int a = decltype(ac)::value, b = decltype(bc)::value;
        constexpr int pp = find_velocity<L>(a, b), pn = find_velocity<L>(a, -b);
        const S e = a0 + S(a * a) * cxx + S(b * b) * cyy;
        const S e1 = e + S(a * b) * cxy, e2 = e - S(a * b) * cxy;
        const S o1 = S(a) * bx + S(b) * by, o2 = S(a) * bx - S(b) * by;
        out(std::integral_constant<int, pp>{}, e1 + o1);
        out(std::integral_constant<int, opposite<L>(pp)>{}, e1 - o1);
        out(std::integral_constant<int, pn>{}, e2 + o2);
        out(std::integral_constant<int, opposite<L>(pn)>{}, e2 - o2);
      });
}

// A solve's constants of the update and of its moving wall.
template <typename S>
struct StepConst {
  double rho0d, ladd_scale, sigma, ds0, ds1, inv_thd;
  S rho0, th, inv_th, h2, om;
  __device__ __forceinline__ StepConst(const SolveDesc& d, const KernelLattice& lat)
      : rho0d(d.rho0),
        ladd_scale(d.ladd_scale),
        sigma(d.sigma),
        ds0(d.ds[0]),
        ds1(d.ds[1]),
        inv_thd(1.0 / lat.theta),
        rho0((S)d.rho0),
        th((S)lat.theta),
        inv_th((S)(1.0 / lat.theta)),
        h2((S)(0.5 / (lat.theta * lat.theta))),
        om((S)d.inv_tau) {}
};

// The arrivals of a row y < R from a diffuse or Maxwell wall: the emission
// w (ea + eb (e1 vx + e2 vx^2)) of the cell's column (see ds_arrival; cm: the
// deviation of the mass crossing the wall in it), mixed in FP64 with the
// specular image that f holds, rounded once.
template <class L, typename S>
__device__ __forceinline__ void emission_arrivals(S (&f)[L::Q], const StepConst<S>& c,
                                                  const KernelLattice& lat, int y, double U,
                                                  double cm) {
  const double emit = c.sigma / (c.ds0 + U * U * c.ds1);
  const double e0 = 0.5 * U * U * c.inv_thd, e1 = U * c.inv_thd, e2 = e0 * c.inv_thd;
  const double eb = (c.rho0d * c.ds0 + cm) * emit;
  const double ea = (cm - c.rho0d * (U * U * c.ds1)) * emit - eb * e0;
  // (a share of zero leaves the emission as it is)
  const double ws = 1.0 - c.sigma;
  static_for<0, L::Q>([&](auto qc) __attribute__((always_inline)) {
    constexpr int q = decltype(qc)::value;
    constexpr int vx = L::vx[q], vy = L::vy[q];
    if constexpr (vy > 0) {
      const double e = lat.w[L::orbit[q]] * (ea + eb * (vx * (e1 + vx * e2)));
      f[q] = y < vy ? (S)__builtin_fma(ws, (double)f[q], e) : f[q];
    }
  });
}

// The collision of the pulled populations f; returns the density.
template <class L, typename S, bool BGK>
__device__ __forceinline__ S collide(S (&f)[L::Q], const StepConst<S>& c,
                                     const KernelLattice& lat) {
  S m[6];
  moments_of<L>(f, m);
  const S drho = m[0], jx = m[1], jy = m[2];
  const S rho = c.rho0 + drho;
  const S inv_rho = S(1) / rho;
  const S uxx = jx * jx * inv_rho, uxy = jx * jy * inv_rho, uyy = jy * jy * inv_rho;
  S bxx = uxx, bxy = uxy, byy = uyy;
  if constexpr (!BGK) {
    const S axx = m[3] - drho * c.th, ayy = m[5] - drho * c.th, axy = m[4];
    bxx = axx - c.om * (axx - uxx);
    bxy = axy - c.om * (axy - uxy);
    byy = ayy - c.om * (ayy - uyy);
  }
  expand<L>(drho - (bxx + byy) * (S(0.5) * c.inv_th), jx * c.inv_th, jy * c.inv_th, bxx * c.h2,
            bxy * (S(2) * c.h2), byy * c.h2, [&](auto qc, S p) __attribute__((always_inline)) {
              constexpr int q = decltype(qc)::value;
              const S g = (S)lat.w[L::orbit[q]] * p;
              f[q] = BGK ? f[q] + c.om * (g - f[q]) : g;
            });
  return rho;
}

// Force of a step by one wavefront: the momentum exchange of the moving wall's
// links (value(i): the crossing population of link i, vel(i, k): its reflected
// velocity) in a fixed order, complete in lane 63; and its share of the lock-in
// sums.
struct WallForce {
  double mwx, mwy, fs0, fs1, kl0, kl1;
  WallEmission emission;
  bool diffuse;
  __device__ __forceinline__ WallForce(const SolveDesc& d, bool diffuse_wall)
      : mwx(diffuse_wall ? d.sigma : 2.0),
        mwy(diffuse_wall ? 2.0 - d.sigma : 2.0),
        fs0(d.fstatic[0]),
        fs1(d.fstatic[1]),
        kl0(d.kladd[0]),
        kl1(d.kladd[1]),
        emission(wall_emission(d)),
        diffuse(diffuse_wall) {}
  template <class V, class W>
  __device__ __forceinline__ void sum(int lane, int nlinks, V&& value, W&& vel, double& fx,
                                      double& fy, double& fm) const {
    fx = fy = fm = 0.0;
    for (int i = lane; i < nlinks; i += 64) {
      const double v = value(i);
      fx -= mwx * vel(i, 0) * v;
      fy -= mwy * vel(i, 1) * v;
      fm += v;
    }
    fx = wave_sum_63(fx);
    fy = wave_sum_63(fy);
    if (diffuse) fm = wave_sum_63(fm);
  }
  // lane 63
  __device__ __forceinline__ void finish(const Drive& dr, bool in_window, double& fx, double& fy,
                                         double fm, double (&lk)[6]) const {
    fx += fs0 + kl0 * dr.u;
    fy += fs1 + kl1 * dr.u;
    if (diffuse) add_emission_force(emission, dr.u, fm, &fx, &fy);
    if (in_window) {
      lk[0] += fx * dr.s;
      lk[1] += fx * dr.c;
      lk[2] += fx;
      lk[3] += fy * dr.s;
      lk[4] += fy * dr.c;
      lk[5] += fy;
    }
  }
};

}  // namespace

// LDS: the populations as Q planes of a compile-time size, column x of a plane
// contiguous in y with R nsub rows before and after the owned ones (behind a
// wall: the rows that its arrivals pull from), so that the pull of velocity
// (vx, vy) is one read at a constant offset from the base of column x - vx.
template <class L, typename S, bool BGK, bool DSW>
__global__ __launch_bounds__(kColumnThreads) void column_kernel(
    const SolveDesc* __restrict__ descs, const WorkItem* __restrict__ work, KernelLattice lat,
    int rows, int nsub, int dn) {
  constexpr int Q = L::Q, R = L::R;
  constexpr int cap = kColumnCells;
  __shared__ Drive drive[kColumnMaxSub];
  __shared__ S pop[Q * cap];
  __shared__ double hist[2 * kColumnMaxSub];  // the steps' forces
  // wall links: LDS index of the crossing population, reflected velocity
  __shared__ int link_at[CrossTable<L>::N * kColumnMaxNx];
  __shared__ int8_t link_v[CrossTable<L>::N * kColumnMaxNx][2];
  // diffuse wall: deviation of the mass crossing it, per row and column
  __shared__ double cross[DSW ? R * kColumnMaxNx : 1];
  // a launch over one solve needs no work list
  const WorkItem wi = work ? work[blockIdx.x] : WorkItem{0, (int32_t)blockIdx.x};
  const SolveDesc& d = descs[wi.solve];
  const int64_t n0 = d.state->step + dn;
  const S* __restrict__ fin = static_cast<const S*>(d.buf[n0 & 1]);
  S* __restrict__ fout = static_cast<S*>(d.buf[(n0 + nsub) & 1]);
  const int nx = d.nx, ny = d.ny, tid = (int)threadIdx.x;
  const int64_t qs = d.qs;
  const bool yper = d.geom == GEOM_PERIODIC;
  const int y0 = wi.tile * rows, y1 = y0 + rows < ny ? y0 + rows : ny;  // owned rows
  const int ylo = y0 - R * nsub, region = rows + 2 * R * nsub;          // LDS rows
  const int ys = column_stride(region, nx, sizeof(S));
  // threads in lattice order: the rows that a step still needs are whole
  // wavefronts but for two, the others skip it
  const int row = tid / nx, x = tid - row * nx, y = ylo + row;
  const int own = x * ys + row;
  const bool mine = row < region && (yper || (y >= 0 && y < ny));
  // the descriptor's values, read once: the loop below touches LDS only, so
  // that its barriers wait for no global access
  const StepConst<S> c(d, lat);
  const bool far_eq = d.far == FAR_EQ, diffuse = DSW && d.wall == WALL_DS;
  const WallForce wall(d, diffuse);
  const int64_t win0 = d.lockin_first - n0, win1 = win0 + d.lockin_count;

  for (int i = tid; i < 3 * nsub; i += (int)blockDim.x)
    reinterpret_cast<double*>(drive)[i] = reinterpret_cast<const double*>(d.drive + n0)[i];
  S f[Q];
  if (mine) {
    int gy = y;
    if (yper) gy = ((y % ny) + ny) % ny;
    const S* src = fin + gy * nx + x;
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      f[q] = src[q * qs];
    });
  }
  // bases of the columns x - vx, by vx + R.  Every row of the region reads
  // inside the planes (the first plane's velocity is at rest); a lane without
  // a cell reads somewhere in them.
  int base[2 * R + 1];
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) {
    int sx = x - (k - R);
    sx += sx < 0 ? nx : 0;
    sx -= sx >= nx ? nx : 0;
    base[k] = mine ? sx * ys + row : R;
  }
  // rows whose populations cross a wall, and the element of the column of
  // offset 0 that their reflections go to, relative to the column's base
  const bool low = mine && !yper && y < R, high = mine && !yper && y >= ny - R;
  const int behind_low = low ? row_behind_moving(row, y, region) : -1;
  const int behind_high = high ? row_behind_far(row, ny - 1 - y, region) : -1;
  const int to_low = behind_low - row, to_high = behind_high - row;
  // write the cell's populations, and those that cross a wall to where their
  // arrivals in the step with wall velocity U pull from
  auto put = [&](double U) __attribute__((always_inline)) {
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      pop[own + q * cap] = f[q];
    });
    if (low) {
      if (diffuse) {
        // specular images: reflected in y only, in the same column
        double cm = 0.0;
        static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value, to = reflect_y<L>(q);
          if constexpr (L::vy[q] < 0)
            if (y < -L::vy[q]) {
              cm += (double)f[q];
              if (behind_low >= 0) pop[own + to_low + to * cap] = f[q];
            }
        });
        cross[y * kColumnMaxNx + x] = cm;
      } else if (behind_low >= 0) {
        const double ladd = c.ladd_scale * U;
        static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;  // the arrival
          constexpr int vx = L::vx[q], vy = L::vy[q], o = opposite<L>(q);
          if constexpr (vy > 0)
            if (y < vy)
              pop[base[R + vx] + to_low + q * cap] =
                  f[o] + (S)(lat.w[L::orbit[q]] * vx * ladd);
        });
      }
    }
    if (behind_high >= 0 && !far_eq) {
      const int k = ny - 1 - y;
      static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        constexpr int vx = L::vx[q], vy = L::vy[q], o = opposite<L>(q);
        if constexpr (vy < 0)
          if (k < -vy) pop[base[R + vx] + to_high + q * cap] = f[o];
      });
    }
  };
  if (behind_high >= 0 && far_eq) {
    const int k = ny - 1 - y;
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      constexpr int vx = L::vx[q], vy = L::vy[q];
      if constexpr (vy < 0)
        if (k < -vy) pop[base[R + vx] + to_high + q * cap] = S(0);
    });
  }
  if (mine) put(d.drive[n0].u);
  // force wavefront of the tile at the moving wall: the last one, without cells
  const int lane = tid & 63;
  const bool force = wi.tile == 0 && tid >= (int)blockDim.x - 64;
  const int nlinks = yper ? 0 : CrossTable<L>::N * nx;
  double lk[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (force) {
    for (int i = lane; i < nlinks; i += 64) {
      const int k = i / nx, lx = i - k * nx;
      link_at[i] = kCross<L>.q[k] * cap + lx * ys + kCross<L>.r[k] - ylo;
      link_v[i][0] = kCross<L>.vx[k];
      link_v[i][1] = kCross<L>.vy[k];
    }
    if (lane == 63)
      for (int k = 0; k < 6; ++k) lk[k] = d.state->lockin[k];
  }
  bool bad = false;
  __syncthreads();

#pragma unroll 1
  for (int s = 0; s < nsub; ++s) {
    const int more = R * (nsub - 1 - s);
    const bool active = mine && y >= y0 - more && y < y1 + more;
    if (force) {
      double fx, fy, fm;
      wall.sum(
          lane, nlinks, [&](int i) { return (double)pop[link_at[i]]; },
          [&](int i, int k) { return link_v[i][k]; }, fx, fy, fm);
      if (lane == 63) {
        wall.finish(drive[s], s >= win0 && s < win1, fx, fy, fm, lk);
        hist[2 * s] = fx;
        hist[2 * s + 1] = fy;
      }
    }
    if (__any(active)) {
      static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        f[q] = pop[base[R + L::vx[q]] + (q * cap - L::vy[q])];
      });
      if (DSW && diffuse && low) {
        double cm = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) cm += cross[r * kColumnMaxNx + x];
        emission_arrivals<L>(f, c, lat, y, drive[s].u, cm);
      }
      const S rho = collide<L, S, BGK>(f, c, lat);
      bad |= active && !(rho > S(0) && rho < S(INFINITY));
    }
    if (s + 1 < nsub) {
      __syncthreads();
      if (active) put(drive[s + 1].u);
      __syncthreads();
    } else if (active) {
      S* dst = fout + y * nx + x;
      static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        dst[q * qs] = f[q];
      });
    }
  }
  if (force) {
    // the forces of the steps, written by lane 63 above; of a ring shorter than
    // the launch the last hist_cap only, so that each slot is written once
    const int64_t cap_h = d.hist_cap;
    const int s0 = nsub > cap_h ? nsub - (int)cap_h : 0;
    for (int i = 2 * s0 + lane; i < 2 * nsub; i += 64)
      d.hist[2 * ((n0 + (i >> 1)) % cap_h) + (i & 1)] = hist[i];
    if (lane == 63)
      for (int k = 0; k < 6; ++k) d.state->lockin[k] = lk[k];
  }
  if (bad) d.state->unstable = 1;
}

// One step of the same lattices, straight from and to the state buffers: the
// same arithmetic on the same values as a step of column_kernel, so the same
// bits, and the choice is free per launch.  One thread per cell of 256
// consecutive ones, and a workgroup for the force (kForceTile).  For calls of
// one step and the odd steps of others where a launch of column_kernel takes
// many rounds of workgroups (column_single): its LDS leaves one or two
// workgroups per compute unit, and loading, update and storing of a workgroup
// follow one another.  Bound by memory: 31 plates of 16 x 2048 D2Q37, us per step,
// FP32 69 (column_kernel 77 at 3 steps per launch, 93 at one), FP64 122 (121, 163):
// 4.4 and 4.9 TB/s.
template <class L, typename S, bool BGK, bool DSW>
__global__ __launch_bounds__(kBlock) void column_single_kernel(
    const SolveDesc* __restrict__ descs, const WorkItem* __restrict__ work, KernelLattice lat,
    int dn, int streaming) {
  constexpr int Q = L::Q, R = L::R;
  // a launch over one solve needs no work list
  const WorkItem wi =
      work ? work[blockIdx.x]
           : WorkItem{0, blockIdx.x ? (int32_t)blockIdx.x - 1 : kForceTile};
  const SolveDesc& d = descs[wi.solve];
  const int64_t n = d.state->step + dn;
  const S* __restrict__ fin = static_cast<const S*>(d.buf[n & 1]);
  S* __restrict__ fout = static_cast<S*>(d.buf[(n & 1) ^ 1]);
  const int nx = d.nx, ny = d.ny, tid = (int)threadIdx.x;
  const int64_t qs = d.qs;
  const bool yper = d.geom == GEOM_PERIODIC;
  const bool far_eq = d.far == FAR_EQ, diffuse = DSW && d.wall == WALL_DS;
  if (wi.tile == kForceTile) {
    if (tid >= 64) return;
    const WallForce wall(d, diffuse);
    double lk[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    Drive dr{};
    if (tid == 63) {
      dr = d.drive[n];
      for (int k = 0; k < 6; ++k) lk[k] = d.state->lockin[k];
    }
    double fx, fy, fm;
    wall.sum(
        tid, yper ? 0 : CrossTable<L>::N * nx,
        [&](int i) {
          const int k = i / nx;
          return (double)fin[kCross<L>.q[k] * qs + kCross<L>.r[k] * nx + (i - k * nx)];
        },
        [&](int i, int k) { return k ? kCross<L>.vy[i / nx] : kCross<L>.vx[i / nx]; }, fx, fy, fm);
    if (tid == 63) {
      wall.finish(dr, n >= d.lockin_first && n < d.lockin_first + d.lockin_count, fx, fy, fm, lk);
      const int64_t h = n % d.hist_cap;
      d.hist[2 * h] = fx;
      d.hist[2 * h + 1] = fy;
      for (int k = 0; k < 6; ++k) d.state->lockin[k] = lk[k];
    }
    return;
  }
  const StepConst<S> c(d, lat);
  const int at = wi.tile * kBlock + tid, cy = at / nx;
  const bool active = cy < ny;
  if (!__any(active)) return;
  // (lanes past the last cell read as cell 0 does, inside the buffer: rows before
  // a plane are the plane before's)
  const int y = active ? cy : 0, x = active ? at - cy * nx : 0;
  // the columns x - vx and the rows y - vy (those behind a wall are not read)
  int col[2 * R + 1], row[2 * R + 1];
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) {
    int sx = x - (k - R), sy = y - (k - R);
    sx += sx < 0 ? nx : 0;
    sx -= sx >= nx ? nx : 0;
    if (yper) {
      sy += sy < 0 ? ny : 0;
      sy -= sy >= ny ? ny : 0;
    }
    col[k] = sx;
    row[k] = sy * nx;
  }
  const bool low = active && !yper && y < R, high = active && !yper && y >= ny - R;
  S f[Q];
  if (!__any(low || high)) {
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      f[q] = fin[q * qs + (row[R + L::vy[q]] + col[R + L::vx[q]])];
    });
  } else {
    const double U = d.drive[n].u, ladd = c.ladd_scale * U;
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      constexpr int vx = L::vx[q], vy = L::vy[q], o = opposite<L>(q);
      int64_t src = q * qs + (row[R + vy] + col[R + vx]);
      bool moving = false, zero = false;
      if constexpr (vy > 0) {
        // from the moving wall: the reflection (bounce-back with the moving-wall
        // term, or the specular image)
        moving = low && y < vy;
        const int at_wall = (vy - 1 - y) * nx;
        if (diffuse)
          src = moving ? reflect_y<L>(q) * qs + (at_wall + col[R + vx]) : src;
        else
          src = moving ? o * qs + (at_wall + x) : src;
      }
      if constexpr (vy < 0) {
        // from the stationary far wall, or the rest-equilibrium far field
        const bool far = high && ny - 1 - y < -vy;
        src = far ? o * qs + ((2 * ny - 1 - (y - vy)) * nx + x) : src;
        zero = far && far_eq;
      }
      f[q] = fin[src];
      if constexpr (vy > 0)
        if (moving && !diffuse) f[q] = f[q] + (S)(lat.w[L::orbit[q]] * vx * ladd);
      if constexpr (vy < 0) f[q] = zero ? S(0) : f[q];
    });
    if (DSW && diffuse && low) {
      double cm = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        double cr = 0.0;
        static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          if constexpr (L::vy[q] < 0)
            if (r < -L::vy[q]) cr += (double)fin[q * qs + (r * nx + x)];
        });
        cm += cr;
      }
      emission_arrivals<L>(f, c, lat, y, U, cm);
    }
  }
  const S rho = collide<L, S, BGK>(f, c, lat);
  if (!active) return;
  if (!(rho > S(0) && rho < S(INFINITY))) d.state->unstable = 1;
  S* const dst = fout + at;
  if (streaming)
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      __builtin_nontemporal_store(f[q], &dst[q * qs]);
    });
  else
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      // (empty, but keeps the compiler from merging the two forms)
      asm volatile("" ::: "memory");
      dst[q * qs] = f[q];
    });
}

// Advance the step counters of solves stepped by column_kernel.
__global__ __launch_bounds__(64) void advance_kernel(const SolveDesc* __restrict__ descs,
                                                     const int32_t* __restrict__ solves,
                                                     int count, int nsteps) {
  const int i = (int)(blockIdx.x * 64 + threadIdx.x);
  if (i < count) descs[solves[i]].state->step += nsteps;
}

template <class L, typename S>
static hipError_t launch_column_l(bool bgk, bool ds, const ColumnShape& sh,
                                  const SolveDesc* descs, const WorkItem* work, int nwork,
                                  const KernelLattice& lat, int dn, hipStream_t stream,
                                  const KernelEvents& ev) {
  const dim3 grid(nwork), block(sh.threads);
  auto go = [&](auto kernel) {
    if (ev.start)
      hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, ev.start, ev.stop, 0u, descs,
                            work, lat, sh.rows, sh.nsub, dn);
    else
      hipLaunchKernelGGL(kernel, grid, block, 0, stream, descs, work, lat, sh.rows, sh.nsub,
                         dn);
    return hipGetLastError();
  };
  if (bgk) return ds ? go(column_kernel<L, S, true, true>) : go(column_kernel<L, S, true, false>);
  return ds ? go(column_kernel<L, S, false, true>) : go(column_kernel<L, S, false, false>);
}

hipError_t launch_column(int Q, bool f64, bool bgk, bool ds, const ColumnShape& sh,
                         const SolveDesc* descs, const WorkItem* work, int nwork,
                         const KernelLattice& lat, int dn, hipStream_t stream, KernelEvents ev) {
  if (nwork <= 0) return hipSuccess;
  // odd step counts only (the state buffers alternate), within the LDS planes
  if (sh.nsub < 1 || sh.nsub > kColumnMaxSub || sh.nsub % 2 == 0 || sh.rows < 1 ||
      sh.threads > kColumnThreads)
    return hipErrorInvalidValue;
  if (Q == 9)
    return f64 ? launch_column_l<D2Q9, double>(bgk, ds, sh, descs, work, nwork, lat, dn, stream, ev)
               : launch_column_l<D2Q9, float>(bgk, ds, sh, descs, work, nwork, lat, dn, stream, ev);
  return f64 ? launch_column_l<D2Q37, double>(bgk, ds, sh, descs, work, nwork, lat, dn, stream, ev)
             : launch_column_l<D2Q37, float>(bgk, ds, sh, descs, work, nwork, lat, dn, stream, ev);
}

template <class L, typename S>
static hipError_t launch_single_l(bool bgk, bool ds, const SolveDesc* descs, const WorkItem* work,
                                  int nwork, const KernelLattice& lat, int dn, bool streaming,
                                  hipStream_t stream, const KernelEvents& ev) {
  auto go = [&](auto kernel) {
    launch_kernel(kernel, dim3(nwork), dim3(kBlock), stream, ev, descs, work, lat, dn,
                  (int)streaming);
    return hipGetLastError();
  };
  if (bgk)
    return ds ? go(column_single_kernel<L, S, true, true>)
              : go(column_single_kernel<L, S, true, false>);
  return ds ? go(column_single_kernel<L, S, false, true>)
            : go(column_single_kernel<L, S, false, false>);
}

hipError_t launch_column_single(int Q, bool f64, bool bgk, bool ds, const SolveDesc* descs,
                                const WorkItem* work, int nwork, const KernelLattice& lat, int dn,
                                bool streaming, hipStream_t stream, KernelEvents ev) {
  if (nwork <= 0) return hipSuccess;
  if (Q == 9)
    return f64 ? launch_single_l<D2Q9, double>(bgk, ds, descs, work, nwork, lat, dn, streaming,
                                               stream, ev)
               : launch_single_l<D2Q9, float>(bgk, ds, descs, work, nwork, lat, dn, streaming,
                                              stream, ev);
  return f64 ? launch_single_l<D2Q37, double>(bgk, ds, descs, work, nwork, lat, dn, streaming,
                                              stream, ev)
             : launch_single_l<D2Q37, float>(bgk, ds, descs, work, nwork, lat, dn, streaming,
                                             stream, ev);
}

hipError_t launch_advance(const SolveDesc* descs, const int32_t* solves, int count, int nsteps,
                          hipStream_t stream) {
  if (count <= 0 || nsteps <= 0) return hipSuccess;
  hipLaunchKernelGGL(advance_kernel, dim3((count + 63) / 64), dim3(64), 0, stream, descs, solves,
                     count, nsteps);
  return hipGetLastError();
}

}  // namespace lbm

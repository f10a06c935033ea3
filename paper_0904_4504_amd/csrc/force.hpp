// Wall force of a step, computed by a workgroup of the step's own launch.
#pragma once

#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "solver.hpp"
#include "walls.hpp"

namespace lbm {

constexpr int kForceLinks = 3;  // links of a thread in flight (box_wall_force)

struct ForceLds {
  double emit[kMaxWallCols];  // box_wall_force: diffuse emission by column
  double red[3][kBlock / 64];
};

// Diffuse emission of a face column: the arrival on its link of weight w and
// velocity vx is w ((B + rho0) e + B) with e = vx e1 + vx^2 e2 - e0 (what
// ds_box_arrival forms per link), B from the deviation m of the mass crossing
// the wall in the column.
struct Emission {
  double e0, e1, e2;
  __device__ __forceinline__ Emission(double U, double theta) {
    e1 = U / theta;
    e0 = 0.5 * U * e1;
    e2 = 0.5 * e1 * e1;
  }
};
__device__ __forceinline__ double column_emission(const WallCol& col, double rho0, double U,
                                                  double m) {
  const double Zu = U * (col.Z1 + col.Z2 * U);
  return (rho0 * (col.L1 * U - Zu) + m) / (col.Mr + Zu);
}

// A link of a diffuse or Maxwell box between its loads and its use: its
// bounce-back partner, its specular source, weight, velocity, column.
struct BoxLink {
  double fp, sp, w, vx, vy;
  int32_t col;
};

// Links i, i + kBlock, .. (those past the end: weight zero at the last link).
template <typename S>
__device__ __forceinline__ void load_links(const SolveDesc& d, const S* __restrict__ f, int i,
                                           bool specular, BoxLink (&b)[kForceLinks]) {
  int64_t partner[kForceLinks], spec[kForceLinks];
#pragma unroll
  for (int u = 0; u < kForceLinks; ++u) {
    const int k = i + u * kBlock;
    const WallLink& l = d.wlinks[k < d.nwlinks ? k : d.nwlinks - 1];
    b[u].w = k < d.nwlinks ? l.w : 0.0;
    b[u].vx = k < d.nwlinks ? l.vx : 0.0;
    b[u].vy = k < d.nwlinks ? l.vy : 0.0;
    b[u].col = l.col;
    partner[u] = l.off_partner;
    spec[u] = l.col < 0 ? l.off_partner : l.off_spec;  // (corner links have none)
  }
#pragma unroll
  for (int u = 0; u < kForceLinks; ++u) {
    b[u].fp = (double)f[partner[u]];
    b[u].sp = specular ? (double)f[spec[u]] : 0.0;
  }
}

// Force sums of a population state's box with diffuse or Maxwell faces: every
// link's arrival as the step forms it -- the column's diffuse emission from
// the column's crossing mass (first pass), mixed with the specular image;
// corner links bounce back -- and the momentum exchange -v_l (f_partner +
// f_arrival); the moving-wall terms are in kladd.
template <typename S>
__device__ __forceinline__ void box_link_force(const SolveDesc& d, int64_t n, ForceLds& lds,
                                               int first, int stride, double& fx, double& fy) {
  const S* __restrict__ f = static_cast<const S*>(n & 1 ? d.buf[1] : d.buf[0]);
  const int nlinks = d.nwlinks;
  const double U = d.drive[n].u, rho0 = d.rho0, sigma = d.sigma;
  const bool specular = sigma != 1.0;
  // a thread's first links are under way during the first pass
  BoxLink b[kForceLinks];
  int i = first;
  if (i < nlinks) load_links(d, f, i, specular, b);
  for (int c = first; c < d.nwcols; c += stride) {
    const WallCol& col = d.wcols[c];
    double m = 0.0;
#pragma unroll 4
    for (int k = 0; k < col.count; ++k) m += (double)f[d.wlinks[col.first + k].off_partner];
    lds.emit[c] = column_emission(col, rho0, U, m);
  }
  __syncthreads();
  const Emission em(U, d.theta);
  while (i < nlinks) {
#pragma unroll
    for (int u = 0; u < kForceLinks; ++u) {
      const BoxLink& l = b[u];
      double a = l.fp;
      if (l.col >= 0) {
        const double B = lds.emit[l.col], e = l.vx * (em.e1 + l.vx * em.e2) - em.e0;
        a = l.w * ((B + rho0) * e + B);
        if (specular) a = sigma * a + (1.0 - sigma) * l.sp;
      }
      fx -= l.vx * (l.fp + a);
      fy -= l.vy * (l.fp + a);
    }
    i += kForceLinks * kBlock;
    if (i < nlinks) load_links(d, f, i, specular, b);
  }
}

// Wall force of step n by momentum exchange (Sec. 2 force F_f; eq. BB): every
// bounce-back link carries -v_i (f_opp(x_p) + f_i^adv(x)) = -v_i (2 f_opp(x_p)
// + 2 w_i rho0 (v_i.U_w)/theta) (+ the rest state), so F_n = F_static + K_ladd
// U_w(n) + sum over links of the reflected populations of step n's input
// state, read here from the step's input buffer (untouched by the step) and
// summed in a fixed order in FP64.  At a diffuse wall (eq. DS) f_i^adv is the
// wall's emission, which depends on the same input state only through the
// crossing mass of each column.  Then append F_n to the history ring and
// accumulate the lock-in sums when n lies in the window.
//
// The force reads nothing that the step writes, so one workgroup per solve
// (the first work items of a launch, tile kForceTile) does it beside the
// update.  As a launch of its own after every step it added 4.5 us (bounce-
// back) to 10 us (diffuse box) and a dependency between launches to each step:
// a 256 x 256 FP32 box took 21 us per step instead of 14.6 (both at K = 3), a
// 641 x 1000 box of populations 58.8 instead of 50.6.  The step counter, which
// every workgroup reads, is advanced by a launch of its own after the last step
// of a call or graph (advance_kernel); a launch is told how many steps lie in
// between.
// coeffs: the input state is H2 coefficients, else populations.
//
// Bound by the chain of dependent loads per thread.  The force of a
// coefficient state is therefore a sum over the wall's mirror cells with
// weights made at creation (a 32 x 16 body: 330 cells, two per thread) and,
// at diffuse faces, over the columns' emission (96 columns).  Summed over the
// 2500 links of that body, five to ten pairs of dependent loads per thread and
// a division each, the force set the time of a step of a 256 x 256 diffuse
// box: 10.0 us (two links of a thread in flight: 9.8), against 8.4.
template <typename S, bool DSW>
__device__ __forceinline__ void wall_force(const SolveDesc& d, bool coeffs, int64_t n,
                                           ForceLds& lds) {
  SolveState* st = d.state;
  const int tid = (int)threadIdx.x;
  // the first kBlock threads work, whatever the workgroup of the kernel
  const int stride = tid < kBlock ? kBlock : 0x40000000, first = tid < kBlock ? tid : 0x40000000;
  // the epilogue's loads (drive entry, lock-in sums), issued before the
  // force sums so that their latency overlaps them
  const bool in_window = n >= d.lockin_first && n < d.lockin_first + d.lockin_count;
  Drive dr{};
  double lk[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (tid == 0) {
    dr = d.drive[n];
    if (in_window)
      for (int k = 0; k < 6; ++k) lk[k] = st->lockin[k];
  }
  double fx = 0.0, fy = 0.0, fm = 0.0;
  if (DSW && !coeffs && d.nwlinks > 0) {
    box_link_force<S>(d, n, lds, first, stride, fx, fy);
  } else if (coeffs) {
    const S* __restrict__ c = static_cast<const S*>(d.mbuf[n & 1]);
    if (DSW && d.nwcols > 0) {
      // box with diffuse or Maxwell faces: what its columns emit, from the
      // crossing mass (linear in the column's cells) and the column's sums
      // over its links; all that is linear in the coefficients is in fcells
      const double U = d.drive[n].u, rho0 = d.rho0;
      const Emission em(U, d.theta);
      for (int k = first; k < d.nwcols; k += stride) {
        const WallCol& col = d.wcols[k];
        double m = 0.0;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int j = 0; j < 6; ++j) m += col.mc[r][j] * (double)c[j * d.mks + col.cell[r]];
        const double B = column_emission(col, rho0, U, m);
        fx -= d.sigma * ((B + rho0) * (em.e1 * col.ex[1] + em.e2 * col.ex[2] - em.e0 * col.ex[0]) +
                         B * col.ex[0]);
        fy -= d.sigma * ((B + rho0) * (em.e1 * col.ey[1] + em.e2 * col.ey[2] - em.e0 * col.ey[0]) +
                         B * col.ey[0]);
      }
    }
    const int64_t ks = d.mks;
    for (int i = first; i < d.nfcells; i += stride) {
      const ForceCell& cell = d.fcells[i];
      const CellWeights& fc = d.cweights[cell.pat];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const double v = (double)c[k * ks + cell.off];
        fx += fc.wx[k] * v;
        fy += fc.wy[k] * v;
        fm += fc.wm[k] * v;
      }
    }
  } else {
    const S* __restrict__ f = static_cast<const S*>(n & 1 ? d.buf[1] : d.buf[0]);
#pragma unroll 4
    for (int i = first; i < d.nlinks; i += stride) {
      const ForceLink& link = d.links[i];
      const LinkWeights& l = d.lweights[link.pat];
      const double v = (double)f[link.off];
      fx += l.wx * v;
      fy += l.wy * v;
      fm += l.wm * v;
    }
  }
  fx = wave_sum_63(fx);
  fy = wave_sum_63(fy);
  fm = wave_sum_63(fm);
  const int wave = tid >> 6;
  if ((tid & 63) == 63 && tid < kBlock) {
    lds.red[0][wave] = fx;
    lds.red[1][wave] = fy;
    lds.red[2][wave] = fm;
  }
  __syncthreads();
  if (tid == 0) {
    double sx = 0.0, sy = 0.0, sm = 0.0;
#pragma unroll
    for (int k = 0; k < kBlock / 64; ++k) {
      sx += lds.red[0][k];
      sy += lds.red[1][k];
      sm += lds.red[2][k];
    }
    fx = d.fstatic[0] + d.kladd[0] * dr.u + sx;
    fy = d.fstatic[1] + d.kladd[1] * dr.u + sy;
    if (d.wall == WALL_DS && d.geom == GEOM_PLATE)
      add_emission_force(wall_emission(d), dr.u, sm, &fx, &fy);
    const int64_t h = n % d.hist_cap;
    d.hist[2 * h] = fx;
    d.hist[2 * h + 1] = fy;
    if (in_window) {
      st->lockin[0] = lk[0] + fx * dr.s;
      st->lockin[1] = lk[1] + fx * dr.c;
      st->lockin[2] = lk[2] + fx;
      st->lockin[3] = lk[3] + fy * dr.s;
      st->lockin[4] = lk[4] + fy * dr.c;
      st->lockin[5] = lk[5] + fy;
    }
  }
}


}  // namespace lbm

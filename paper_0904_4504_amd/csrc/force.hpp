// Wall force of a step, computed by a workgroup of the step's own launch.
#pragma once

#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "solver.hpp"
#include "walls.hpp"

namespace lbm {

struct ForceLds {
  double cmass[kMaxWallCols];
  double red[3][kBlock / 64];
};

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
// 641 x 1000 box of populations 58.8 instead of 50.6.  The step counter, which every workgroup reads, is advanced by a
// launch of its own after the last step of a call or graph (advance_kernel);
// a launch is told how many steps lie in between.
// coeffs: the input state is H2 coefficients, else populations.
template <typename S>
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
  if (!coeffs && d.nwlinks > 0) {
    // box with diffuse or Maxwell faces: every link's arrival as the step
    // kernel formed it -- the column's diffuse emission from the column's
    // crossing mass (first pass), mixed with the specular image; corner links
    // bounce back -- and the momentum exchange -v_l (f_partner + f_arrival)
    const S* __restrict__ f = static_cast<const S*>(n & 1 ? d.buf[1] : d.buf[0]);
    for (int c = first; c < d.nwcols; c += stride) {
      const WallCol col = d.wcols[c];
      double m = 0.0;
      for (int k = 0; k < col.count; ++k) m += (double)f[d.wlinks[col.first + k].off_partner];
      lds.cmass[c] = m;
    }
    __syncthreads();
    const double U = d.drive[n].u;
    const double ladd = d.ladd_scale * U;
    for (int i = first; i < d.nwlinks; i += stride) {
      const WallLink l = d.wlinks[i];
      const double fp = (double)f[l.off_partner];
      double a;
      if (l.col < 0) {
        a = fp + l.w * l.vx * ladd;
      } else {
        a = ds_box_arrival(d.wcols[l.col], d.rho0, U, lds.cmass[l.col], l.w, l.vx, d.theta);
        if (d.sigma != 1.0) {
          const double sp = (double)f[l.off_spec] + (l.normal ? l.w * l.vx * ladd : 0.0);
          a = d.sigma * a + (1.0 - d.sigma) * sp;
        }
      }
      fx -= l.vx * (fp + a);
      fy -= l.vy * (fp + a);
    }
  } else if (coeffs && d.nwlinks > 0) {
    // the same two passes on the H2 coefficients of the input state: a
    // population of velocity v at cell o is w_v (a0 + vx bx + vy by + vx^2 cxx
    // + vx vy cxy + vy^2 cyy)(o)
    const S* __restrict__ c = static_cast<const S*>(d.mbuf[n & 1]);
    const int64_t ks = d.mks;
    auto pop = [&](int64_t o, double w, double vx, double vy) {
      return w * ((double)c[o] + vx * (double)c[ks + o] + vy * (double)c[2 * ks + o] +
                  vx * vx * (double)c[3 * ks + o] + vx * vy * (double)c[4 * ks + o] +
                  vy * vy * (double)c[5 * ks + o]);
    };
    for (int k = first; k < d.nwcols; k += stride) {
      const WallCol& col = d.wcols[k];
      double m = 0.0;
      for (int r = 0; r < 3; ++r)
        for (int j = 0; j < 6; ++j) m += col.mc[r][j] * (double)c[j * ks + col.cell[r]];
      lds.cmass[k] = m;
    }
    __syncthreads();
    const double U = d.drive[n].u;
    const double ladd = d.ladd_scale * U;
    for (int i = first; i < d.nwlinks; i += stride) {
      const WallLink l = d.wlinks[i];
      const double fp = pop(l.cell_partner, l.w, -l.vx, -l.vy);
      double a;
      if (l.col < 0) {
        a = fp + l.w * l.vx * ladd;
      } else {
        a = ds_box_arrival(d.wcols[l.col], d.rho0, U, lds.cmass[l.col], l.w, l.vx, d.theta);
        if (d.sigma != 1.0) {
          const double sp = l.normal ? pop(l.cell_spec, l.w, -l.vx, l.vy) + l.w * l.vx * ladd
                                     : pop(l.cell_spec, l.w, l.vx, -l.vy);
          a = d.sigma * a + (1.0 - d.sigma) * sp;
        }
      }
      fx -= l.vx * (fp + a);
      fy -= l.vy * (fp + a);
    }
  } else if (coeffs) {
    const S* __restrict__ c = static_cast<const S*>(d.mbuf[n & 1]);
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
    if (d.wall == WALL_DS && d.geom == GEOM_PLATE) add_emission_force(wall_emission(d), dr.u, sm, &fx, &fy);
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

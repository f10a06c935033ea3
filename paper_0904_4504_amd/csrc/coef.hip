// Regularized lattice-BGK step on H2-coefficient storage.
//
// The regularized collision (Sec. 5, eqs. regularization and fne) leaves
// every post-collision distribution in the span of the Hermite polynomials up
// to second order: with deviations from the rest state,
//   delta f_i(x) = w_i [ a0 + vx bx + vy by + vx^2 cxx + vx vy cxy + vy^2 cyy ](x).
// Six coefficients per cell describe the state exactly, so a step reads and
// writes 6 values per cell instead of Q and Q.
//
// A workgroup of four wavefronts updates a tile of 64 columns x 4 RB rows: it
// stages the coefficients of the tile and an R-cell halo in LDS, then the
// lane of column x in wavefront w computes the RB cells (x, w RB + k).  The
// pulled populations f_v(x) = delta f_v(x - v) (eq. advection) of those RB
// cells come from the union of their stencils; the lane reads each cell of
// the union from LDS once and adds its populations to every output cell that
// pulls from it.  For a source cell at column offset dx (so vx = -dx) the
// populations differ only through vy: f = g + vy^2 cyy + vy h with
// g = a0 + vx bx + vx^2 cxx and h = by + vx cxy.  Per output cell and source
// row the sums of w f, w vx f, w vx^2 f are gathered first and then scattered
// into the six moments (rho, j, Pi), which the collision turns into the six
// new coefficients.
//
// Walls (Sec. 4, eq. BB): cells inside the body and outside the domain are
// staged as zeros (the rest-equilibrium far field; the plate's wall
// half-spaces), so a population crossing the moving wall, the body or the
// stationary far wall arrives as zero; the lane of a cell within R of a wall
// then adds the moments of the bounce-back values f_opp(x_p) + 2 w_i rho0
// (v_i.U_w)/theta (moving wall only), x_p the half-way mirror cell of the link
// (the rules of the population kernel), read from the step's input state; at a
// plate or a box face with the diffuse or the Maxwell wall those of the
// diffuse emission (eq. DS) of the link's wall column, mixed with the specular
// image for the Maxwell wall.  The force's workgroup sums the momentum exchange from the same
// input state.
#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "force.hpp"
#include "lattice.hpp"
#include "solver.hpp"
#include "walls.hpp"

// No implicit contraction in this file: every fused multiply-add is written as
// one, so that a cell's bits do not depend on the unrolled copy, the tile
// shape or the segment length that computes it, and the host may choose those
// per launch.
#pragma clang fp contract(off)

namespace lbm {

// Constants of a launch in the storage precision: the orbit weights, their
// products with |vx| and vx^2 (the factors of the x-weighted sums; for
// |vx| = 1 the weight itself is used) and the theta factors of the
// coefficients.  Passed by value, so they sit in scalar registers.
template <typename S>
struct CoefConst {
  S w[8];
  S wx[8][4];   // w_o |vx|
  S wxx[8][4];  // w_o vx^2
  S theta;
  S inv_theta;        // 1 / theta
  S half_inv_theta;   // 1 / (2 theta)
  S inv_theta2;       // 1 / theta^2
  S half_inv_theta2;  // 1 / (2 theta^2)
};

template <typename S>
CoefConst<S> coef_const(const KernelLattice& lat) {
  CoefConst<S> c{};
  for (int o = 0; o < 8; ++o) {
    c.w[o] = (S)lat.w[o];
    for (int a = 0; a < 4; ++a) {
      c.wx[o][a] = (S)(lat.w[o] * a);
      c.wxx[o][a] = (S)(lat.w[o] * a * a);
    }
  }
  c.theta = (S)lat.theta;
  c.inv_theta = (S)(1.0 / lat.theta);
  c.half_inv_theta = (S)(0.5 / lat.theta);
  c.inv_theta2 = (S)(1.0 / (lat.theta * lat.theta));
  c.half_inv_theta2 = (S)(0.5 / (lat.theta * lat.theta));
  return c;
}

namespace {

template <typename S>
__device__ __forceinline__ S fmadd(S a, S b, S c) {
  if constexpr (sizeof(S) == 4)
    return __builtin_fmaf(a, b, c);
  else
    return __builtin_fma(a, b, c);
}

// Pointers into device global memory (loads and stores then address the
// global segment directly, with a scalar base and a 32-bit lane offset).
template <typename T>
using gptr = __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ gptr<T> as_global(T* p) {
  return (gptr<T>)p;
}

// A wave-uniform pointer held in scalar registers, so that every load or
// store through it is a scalar base plus a 32-bit per-lane byte offset.
template <typename T>
__device__ __forceinline__ gptr<T> scalar_ptr(gptr<T> p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (gptr<T>)(((uint64_t)hi << 32) | lo);
}

// Address of the element at byte offset `off` of plane `p`.
template <typename T>
__device__ __forceinline__ gptr<T> at(gptr<T> p, uint32_t off) {
  return (gptr<T>)((__attribute__((address_space(1))) char*)p + off);
}

// Two coefficients of a cell: (a0, bx), (by, cxx) or (cxy, cyy).
template <typename S>
using Pair = S __attribute__((ext_vector_type(2)));

template <typename T>
using lptr = __attribute__((address_space(3))) T*;

// The same LDS address, opaque to the compiler: reads relative to it use
// their small constant offsets directly instead of a new base register each.
template <typename T>
__device__ __forceinline__ lptr<const T> opaque(lptr<const T> p) {
  uint32_t a = (uint32_t)(uintptr_t)p;
  asm volatile("" : "+v"(a));
  return (lptr<const T>)(uintptr_t)a;
}

// Six running moment sums of one output row: delta rho, jx, jy, Pxx, Pxy, Pyy.
template <typename S>
struct Mom {
  S v[6];
};


// Empty instruction that takes the six sums as inputs and outputs and
// clobbers memory: the sums of one source row are complete here and the LDS
// reads of the next row are not hoisted above it, so the compiler keeps one
// source row in registers at a time.
template <typename S>
__device__ __forceinline__ void row_fence(Mom<S>& m) {
  asm volatile("" : "+v"(m.v[0]), "+v"(m.v[1]), "+v"(m.v[2]), "+v"(m.v[3]), "+v"(m.v[4]),
                    "+v"(m.v[5])::"memory");
}

// True if a source cell at column offset -vx and row offset iy (relative to
// the first of RB output rows) feeds any of those rows.
template <class L, int RB>
constexpr bool source_used(int vx, int iy) {
  for (int k = 0; k < RB; ++k) {
    const int vy = k - iy;
    if (vy >= -L::R && vy <= L::R && find_velocity<L>(vx, vy) >= 0) return true;
  }
  return false;
}

// Wall constants of a tile, in LDS, so that the lanes of a wavefront can look
// up different ones.  w: the weights by |vx| and |vy| (zero where the lattice
// has no such velocity).  s[n - 1][lo][hi][b]: the sum of w t^b over the
// velocities of normal speed n and tangential speed -lo <= t <= hi, b = 0..4;
// wd, sd: the same in FP64, for the diffuse wall.
template <typename S, bool DSW>
struct WallTable {
  S w[4][4];
  S s[3][4][4][5];
  double wd[DSW ? 4 : 1][4];
  double sd[DSW ? 3 : 1][4][4][5];
};

// Entries of thread i < 48: selected from the kernel's arguments, without a
// load (a table of orbits looked up in memory put two dependent cache misses
// in front of the staging loads).
template <class L, typename S, bool DSW>
__device__ __forceinline__ void fill_wall_table(WallTable<S, DSW>& tab, const KernelLattice& lat,
                                                int i) {
  constexpr int R = L::R;
  const int n = (i >> 4) + 1, lo = i >> 2 & 3, hi = i & 3;
  double w = 0, wn[4] = {0, 0, 0, 0};
  static_for<0, R + 1>([&](auto ac) __attribute__((always_inline)) {
    static_for<0, R + 1>([&](auto bc) __attribute__((always_inline)) {
      constexpr int a = decltype(ac)::value, b = decltype(bc)::value;
      constexpr int q = find_velocity<L>(a, b);
      if constexpr (q >= 0) {
        const double v = lat.w[L::orbit[q]];
        w = i == 4 * a + b ? v : w;
        if constexpr (a > 0) wn[b] = n == a ? v : wn[b];
      }
    });
  });
  if (i < 16) {
    tab.w[i >> 2][i & 3] = (S)w;
    if constexpr (DSW) tab.wd[i >> 2][i & 3] = w;
  }
  double m[5] = {wn[0], 0, 0, 0, 0};
#pragma unroll
  for (int t = 1; t <= R; ++t) {
    const double u = t <= hi ? wn[t] : 0.0, v = t <= lo ? wn[t] : 0.0;
    const double e = u + v, o = u - v, tt = t * t;
    m[0] += e;
    m[1] = fmadd((double)t, o, m[1]);
    m[2] = fmadd(tt, e, m[2]);
    m[3] = fmadd(t * tt, o, m[3]);
    m[4] = fmadd(tt * tt, e, m[4]);
  }
#pragma unroll
  for (int b = 0; b < 5; ++b) tab.s[n - 1][lo][hi][b] = (S)m[b];
  if constexpr (DSW)
#pragma unroll
    for (int b = 0; b < 5; ++b) tab.sd[n - 1][lo][hi][b] = m[b];
}

// Moments of the arrivals from the walls at fluid cell (x, y): each link
// population arrived as zero from the stream.  A wall or box face with normal
// axis n is a set of links per distance: at the k-th cell from the face
// (k = 0..R-1), the arrivals with normal speed |v_n| = k + 1 + r come from the
// one mirror cell r cells from the face (0 <= r < R - k), whatever their
// tangential velocity t.  So the links of a cell are summed per mirror cell:
// every arrival is w (G + t H + t^2 K) with G, H, K from the mirror cell's
// coefficients (bounce-back, f_opp(x_p) + the moving-wall term) or from the
// wall's emission (diffuse), and its moments need only S_b = sum w t^b,
// b = 0..4, over the tangential velocities whose source lies behind the wall
// (all of them, except near a box corner).  Cells outside the body on both
// axes have corner links, one mirror cell each (always bounce-back).
//
// The loops over mirror cells are kept rolled.  A tile with wall cells runs
// this code once per launch from a cold instruction cache: as one branch per
// velocity, unrolled for every row of a lane (20 to 150 KB of code), it took
// 25 us (bounce-back) and 36-45 us (diffuse) of a launch however small the
// lattice; per mirror cell (14 KB of code) a launch over a 256 x 256 box takes
// 14.3 and 23.3 us, over a 256 x 256 plate 9.9 and 15.0 us, without walls
// 7.8 us.
//
// What is left is a serial chain on the few wavefronts with wall cells, so it
// is kept short: the S_b come from a table by n and the range of t, filled by
// 48 threads while the staging loads are under way (summed by each lane from
// the weights they were seven look-ups and five chains of seven additions per
// mirror cell and as many again in FP64 for the crossing mass), the reads of
// a mirror cell, or of two specular sources, are in flight together, and
// the column constants arrive behind the crossing mass.  The corner links of
// a cell are one unrolled pass of selects (in a loop over pairs of speeds, up
// to nine round trips to LDS, they were the longest chain of a bounce-back
// box).  One row per wavefront, box of 256 x 256, bounce-back / diffuse /
// Maxwell, us per step: FP32 8.8 -> 6.7 / 12.5 -> 8.2 / - -> 12.6, FP64 9.9 ->
// 7.7 / - -> 9.0 / - -> 12.4 (5.0 and 6.2 without walls).  The specular share
// is the rest of the Maxwell wall: its 21 sources unrolled over t; rolled
// over t, the two signs together, 15.3.
//
// What a diffuse or Maxwell wall sends back is FP64 whatever the storage,
// emission, specular share and mixing, and a mirror cell's sums are rounded
// to S once (FP32 with sums and share in FP32: diffuse 8.1, Maxwell 11.6 us;
// registers and wavefronts per SIMD are the same).
//
// Every cell read here (mirror cells, the specular sources and the crossing
// rows of the diffuse wall) lies within R - 1 cells of (x, y) along each axis
// (specular: R tangentially, inside the halo), so inside the staged tile: the
// reads come from LDS (C, staged region starting at cell (ox, oy), rows of HW
// cells), not from global memory.
template <class L, typename S, bool DSW>
__device__ __forceinline__ Mom<S> wall_moments(const SolveDesc& d, const Pair<S>* C, int HW,
                                               int ox, int oy, int x, int y, S ladd, double U,
                                               const WallTable<S, DSW>& tab, double theta) {
  constexpr int R = L::R;
  const lptr<const Pair<S>> T = (lptr<const Pair<S>>)C;
  // (values: the fences below would have them loaded again)
  const int bx0 = d.bx0, bx1 = d.bx1, by0 = d.by0, by1 = d.by1, nyl = d.ny;
  const bool two_walls = d.geom == GEOM_PLATE && d.far == FAR_WALL, ds_wall = d.wall == WALL_DS;
  const double sigma = d.sigma, rho0 = d.rho0;
  Mom<S> m{{S(0), S(0), S(0), S(0), S(0), S(0)}};
  struct WallEmit {
    double Mr, Z1, Z2, L1;  // of a WallCol, or of a plate (ds)
  };
  // coefficients of cell (cx, cy) by normal axis: a0, b_t, b_n, c_tt, c_nt, c_nn
  struct Cell {
    S a0, bt, bn, ctt, cnt, cnn;
  };
  auto cell = [&](int cx, int cy, bool nx_axis) __attribute__((always_inline)) -> Cell {
    const int i = 3 * (cy - oy) * HW + (cx - ox);
    const Pair<S> p0 = T[i], p1 = T[i + HW], p2 = T[i + 2 * HW];
    // (selects per field: a choice of whole cells becomes a branch, and with it
    // a wait for every cell by itself)
    const S bt = nx_axis ? p1.x : p0.y, bn = nx_axis ? p0.y : p1.x;
    const S ctt = nx_axis ? p2.y : p1.y, cnn = nx_axis ? p1.y : p2.y;
    return Cell{p0.x, bt, bn, ctt, p2.x, cnn};
  };
  const bool is_box = d.geom == GEOM_BOX;
  const bool inx = !is_box || (x >= bx0 && x < bx1);
  const bool iny = is_box && y >= by0 && y < by1;
  // moments along the normal and the tangential axis
  Mom<S> a{{S(0), S(0), S(0), S(0), S(0), S(0)}};  // drho, j_t, j_n, P_tt, P_nt, P_nn
  auto add = [&](S t0, S t1, S t2, S vn) __attribute__((always_inline)) {
    a.v[0] += t0;
    a.v[1] += t1;
    a.v[2] = fmadd(vn, t0, a.v[2]);
    a.v[3] += t2;
    a.v[4] = fmadd(vn, t1, a.v[4]);
    a.v[5] = fmadd(vn * vn, t0, a.v[5]);
  };
  const bool ax = iny;  // normal along x: the faces left and right of the body
  if (inx || iny) {
    // a plate's cell may be in reach of both its walls
    const int npass = two_walls ? 2 : 1;
#pragma unroll 1
    for (int pass = 0; pass < npass; ++pass) {
      // first fluid cell along the normal, and the sign of the arrivals' v_n
      int w0, sg;
      if (!is_box) {
        w0 = pass ? nyl - 1 : 0;
        sg = pass ? -1 : 1;
      } else if (ax) {
        w0 = x < bx0 ? bx0 - 1 : bx1;
        sg = x < bx0 ? -1 : 1;
      } else {
        w0 = y < by0 ? by0 - 1 : by1;
        sg = y < by0 ? -1 : 1;
      }
      const int k = sg * ((ax ? x : y) - w0);
      if (k >= R) continue;
      // tangential velocities t with a source behind the wall: -lo <= t <= hi
      int lo = R, hi = R;
      if (is_box) {
        lo = min(R, (ax ? by1 - y : bx1 - x) - 1);
        hi = min(R, ax ? y - by0 : x - bx0);
      }
      const S lad = pass ? S(0) : ladd;
      const bool diffuse = DSW && ds_wall && pass == 0;
      // diffuse emission w (ea + eb (e1 v_x + e2 v_x^2)) of the cell's column
      double ea = 0, eb = 0, e1 = 0, e2 = 0;
      if (diffuse) {
        WallEmit em{d.ds[0], 0, d.ds[1], 0};
        if (is_box) {
          const int face = ax ? (sg < 0 ? 2 : 3) : (sg < 0 ? 0 : 1);
          const WallCol& wc = d.wcols[box_column(d, face, x, y)];
          em = {wc.Mr, wc.Z1, wc.Z2, wc.L1};
        }
        // deviation of the mass crossing the wall in this column: the
        // bounce-back partners of all its links (while em arrives)
        double cm = 0;
        const double sgn = sg;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int pc = w0 + sg * r;
          const Cell c = cell(ax ? pc : x, ax ? y : pc, ax);
          const double a0 = c.a0, bn = sgn * (double)c.bn, cnn = c.cnn, bt = c.bt, ctt = c.ctt;
          const double cnt = sgn * (double)c.cnt;
#pragma unroll
          for (int n = r + 1; n <= R; ++n) {
            const double* const sd = tab.sd[DSW ? n - 1 : 0][lo][hi];
            cm = fmadd(sd[0], fmadd((double)n, fmadd((double)n, cnn, -bn), a0), cm);
            cm = fmadd(sd[1], fmadd((double)n, cnt, -bt), cm);
            cm = fmadd(sd[2], ctt, cm);
          }
          asm volatile("" : "+v"(cm)::"memory");  // the reads of one cell in flight
        }
        // mass emitted per unit density: Mr + Zu
        const double Zu = fmadd(em.Z2, U, em.Z1) * U, Lu = em.L1 * U;
        const double it = 1.0 / theta, sz = sigma / (em.Mr + Zu), e0 = -0.5 * U * U * it;
        e1 = U * it;
        e2 = 0.5 * e1 * e1;
        eb = sz * fmadd(rho0, em.Mr + Lu, cm);
        ea = fmadd(eb, e0, sz * fmadd(rho0, Lu - Zu, cm));
      }
#pragma unroll 1
      for (int r = 0; r < R - k; ++r) {
        const int n = k + 1 + r;
        const S vn = (S)(sg * n);
        const int pc = w0 + sg * r;
        if (diffuse) {
          // in FP64, the emission and its mixing with the specular image, and
          // rounded once
          const double vd = sg * n;
          double f0 = 0, f1 = 0, f2 = 0;
          if (DSW && sigma != 1.0) {
            // Maxwell wall: the specular share, the population of (t, -v_n) that
            // crossed the wall from the mirror cell's neighbour t cells back
            // (plus the moving-wall term on the faces normal to the motion)
            const double ws = 1.0 - sigma, ladn = ax ? d.ladd_scale * U : 0.0;
            const double* const wt = tab.wd[DSW ? n : 0];
            auto source = [&](int t) __attribute__((always_inline)) {
              return cell(ax ? pc : x - t, ax ? y - t : pc, ax);
            };
            Cell next = source(-R);
#pragma unroll
            for (int t = -R; t <= R; ++t) {
              // the reads of the next source in flight, not of all
              const Cell c = next;
              if (t < R) next = source(t + 1);
              const double ts = t, bn = (double)c.bn - ladn;
              const double g =
                  fmadd(ts, fmadd(ts, (double)c.ctt, fmadd(-vd, (double)c.cnt, (double)c.bt)),
                        fmadd(vd, fmadd(vd, (double)c.cnn, -bn), (double)c.a0));
              const double f = t >= -lo && t <= hi ? wt[t < 0 ? -t : t] * g : 0.0;
              f0 += f;
              f1 = fmadd(ts, f, f1);
              f2 = fmadd(ts * ts, f, f2);
              asm volatile("" : "+v"(f0), "+v"(f1), "+v"(f2)::"memory");
            }
            f0 *= ws;
            f1 *= ws;
            f2 *= ws;
          }
          const double* const sd = tab.sd[DSW ? n - 1 : 0][lo][hi];
          const double s0 = sd[0], s1 = sd[1], s2 = sd[2], s3 = sd[3], s4 = sd[4];
          const double G = ax ? fmadd(eb, vd * fmadd(vd, e2, e1), ea) : ea;
          const double H = ax ? 0.0 : eb * e1, K = ax ? 0.0 : eb * e2;
          f0 = fmadd(s0, G, fmadd(s1, H, fmadd(s2, K, f0)));
          f1 = fmadd(s1, G, fmadd(s2, H, fmadd(s3, K, f1)));
          f2 = fmadd(s2, G, fmadd(s3, H, fmadd(s4, K, f2)));
          add((S)f0, (S)f1, (S)f2, vn);
        } else {
          const S* const st = tab.s[n - 1][lo][hi];
          const S s0 = st[0], s1 = st[1], s2 = st[2], s3 = st[3], s4 = st[4];
          Cell c = cell(ax ? pc : x, ax ? y : pc, ax);
          // the moving-wall term acts like a shift of bx by its amplitude
          c.bn -= ax ? lad : S(0);
          c.bt -= ax ? S(0) : lad;
          const S G = fmadd(vn, fmadd(vn, c.cnn, -c.bn), c.a0);
          const S H = fmadd(vn, c.cnt, -c.bt), K = c.ctt;
          add(fmadd(s0, G, fmadd(s1, H, s2 * K)), fmadd(s1, G, fmadd(s2, H, s3 * K)),
              fmadd(s2, G, fmadd(s3, H, s4 * K)), vn);
        }
      }
    }
  } else {
    // corner links: |v_x| >= i and |v_y| >= j, one mirror cell each
    const bool lo_x = x < bx0, lo_y = y < by0;
    const int i = lo_x ? bx0 - x : x - bx1 + 1, j = lo_y ? by0 - y : y - by1 + 1;
    const int wx = lo_x ? bx0 - 1 : bx1, wy = lo_y ? by0 - 1 : by1;
    const int sx = lo_x ? -1 : 1, sy = lo_y ? -1 : 1;
    static_for<1, R + 1>([&](auto bc) __attribute__((always_inline)) {
      static_for<1, R + 1>([&](auto ac) __attribute__((always_inline)) {
        constexpr int va = decltype(ac)::value, vb = decltype(bc)::value;
        if constexpr (find_velocity<L>(va, vb) >= 0) {
          const bool on = va >= i && vb >= j;
          Cell c = cell(on ? wx + sx * (va - i) : x, on ? wy + sy * (vb - j) : y, false);
          c.bt -= ladd;
          const S vx = (S)(sx * va), vy = (S)(sy * vb);
          const S g = tab.w[va][vb] *
                      fmadd(vx, fmadd(vx, c.ctt, fmadd(vy, c.cnt, -c.bt)),
                            fmadd(vy, fmadd(vy, c.cnn, -c.bn), c.a0));
          const S f = on ? g : S(0);
          add(f, vx * f, vx * vx * f, vy);
        }
      });
      // the reads of one row of velocities in flight
      row_fence(a);
    });
  }
  m.v[0] = a.v[0];
  m.v[1] = ax ? a.v[2] : a.v[1];
  m.v[2] = ax ? a.v[1] : a.v[2];
  m.v[3] = ax ? a.v[5] : a.v[3];
  m.v[4] = a.v[4];
  m.v[5] = ax ? a.v[3] : a.v[5];
  return m;
}

}  // namespace

// Tile shape of variant RB (RB cells per thread, four wavefronts).
template <class L, int RB>
struct CoefTile {
  static constexpr int R = L::R;
  static constexpr int NT = 64 * kCoefWaves;  // threads
  static constexpr int TH = kCoefWaves * RB;  // tile rows
  static constexpr int HW = kCoefTileW + 2 * R, HH = TH + 2 * R, NC = HW * HH;
  // staging: the 64 core cells of staged row r (columns R .. R + 63) are
  // loaded by wavefront r mod 4, one cell per lane; the 2R halo cells of
  // every staged row by the first NHALO threads
  static constexpr int NCR = (HH + kCoefWaves - 1) / kCoefWaves;  // core rows per wave
  static constexpr int NHALO = 2 * R * HH;
  static constexpr int NHIT = (NHALO + NT - 1) / NT;  // halo cells per thread
};

// A thread's share of a staged tile between its loads and its LDS writes.
template <class L, typename S, int RB>
struct StageRegs {
  S core[CoefTile<L, RB>::NCR][6];
  S halo[CoefTile<L, RB>::NHIT][6];
};

namespace {

// Raw buffer resource over `bytes` bytes at p (a wave-uniform address):
// loads at offsets past the end return zero.  Word 3 = 0x00020000 sets the
// 32-bit data format (bits 15-18 = 4) with no swizzle or index stride, the
// untyped-access setting of the gfx9 family.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void* p, uint32_t bytes) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, (int)bytes,
                                           0x00020000);
}

template <typename S>
__device__ __forceinline__ S buf_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(S) == 4)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  else
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

// Store bypassing the caches' retention (the nontemporal policy bit): a
// separate instruction form from a plain store, which the compiler cannot
// merge with one.
template <typename S>
__device__ __forceinline__ void buf_store_nt(__amdgpu_buffer_rsrc_t r, uint32_t off, S v) {
  if constexpr (sizeof(S) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 2);
  else
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(__attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t, v),
        r, off, 0, 2);
}

// Extent of one coefficient plane's buffer resource: from its first element
// to the last element of its last row.  Element (k, y, x) sits at
// k*ks + y*ys + x: six whole planes (ks >= ny*ys) or, row-interleaved, the
// six rows of a lattice row side by side (ks = row pitch, ys = 6 ks); either
// way plane 5's resource ends inside the buffer.  The library keeps the
// extent below 2 GiB.
template <typename S>
__device__ __forceinline__ uint32_t plane_bytes(int ny, int64_t ys, int64_t ks) {
  return (uint32_t)(((int64_t)(ny - 1) * ys + (ks < ys ? ks : ys)) * (int64_t)sizeof(S));
}

// An offset past the end of every plane's resource (all below 2 GiB).
constexpr uint32_t kNoCell = 0x80000000u;

// Population that output row k pulls from the source cell at column offset
// dx and row offset iy (both relative to the lane's column and the wave's
// first output row), or -1.
template <class L>
constexpr int pull_q(int dx, int iy, int k) {
  const int vy = k - iy;
  if (vy < -L::R || vy > L::R) return -1;
  return find_velocity<L>(-dx, vy);
}

// First column offset of source row iy that feeds output row k (with
// vx != 0 if nz), or R + 1.
template <class L>
constexpr int first_dx(int iy, int k, bool nz) {
  for (int dx = -L::R; dx <= L::R; ++dx)
    if (pull_q<L>(dx, iy, k) >= 0 && (!nz || dx != 0)) return dx;
  return L::R + 1;
}

}  // namespace

// Read of memory that no thread writes during the launch, through the
// constant address space: a scalar load (no wait on vector memory) for a
// wave-uniform address.
template <typename T>
__device__ __forceinline__ T kread(const T* p) {
  return *(const __attribute__((address_space(4))) T*)p;
}

__device__ __forceinline__ WorkItem kread_item(const WorkItem* p) {
  return WorkItem{kread(&p->solve), kread(&p->tile)};
}

// Step index and state buffers of a solve for this launch.
template <typename S>
struct TileCtx {
  const S* min;  // input coefficients
  S* mout;       // output coefficients
  int64_t n;     // step index
};

template <typename S>
__device__ __forceinline__ TileCtx<S> tile_ctx(const SolveDesc& d, int dn) {
  const int64_t n = kread(&d.state->step) + dn;
  void* const b0 = kread(&d.mbuf[0]);
  void* const b1 = kread(&d.mbuf[1]);
  return {static_cast<const S*>(n & 1 ? b1 : b0), static_cast<S*>(n & 1 ? b0 : b1), n};
}

// Load a tile's staged region (the tile and its R-cell halo) into registers:
// body and outside cells as zeros, periodic images where the geometry wraps.
// Each core load of a wavefront covers 64 consecutive cells of one row of one
// coefficient, starting at a multiple of 64 cells: a tile's loads touch whole
// aligned segments, and only the 2R halo cells per row come in separately
// (a 70-cell row loaded lane by lane straddles rows at unaligned starts:
// 11 % slower on the memory side of a state streaming from HBM).
template <class L, typename S, int RB>
__device__ __forceinline__ void stage_load(const SolveDesc& d, const TileCtx<S>& t, int tile,
                                           StageRegs<L, S, RB>& g, int tid) {
  using T = CoefTile<L, RB>;
  constexpr int R = T::R, HH = T::HH;
  constexpr uint32_t es = sizeof(S);
  const S* min = t.min;
  const int nx = d.nx, ny = d.ny;
  const int64_t ks = d.mks;
  const int ys = (int)d.mys;
  const uint32_t bytes = plane_bytes<S>(ny, ys, ks);
  __amdgpu_buffer_rsrc_t rs[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) rs[k] = plane_rsrc(min + k * ks, bytes);
  const int x0 = (tile % d.tiles_x) * kCoefTileW;
  const int y0 = (tile / d.tiles_x) * T::TH;
  const int lane = tid & 63, wv = tid >> 6;
  const bool xper = d.geom != GEOM_BOX, yper = d.geom == GEOM_PERIODIC;
  const bool is_box = d.geom == GEOM_BOX;
  const int bx0 = d.bx0, bx1 = d.bx1, by0 = d.by0, by1 = d.by1;
  // byte offsets first, then the loads (one code path, so the wait before
  // each use covers exactly the loads it needs)
  uint32_t oc[T::NCR], oh[T::NHIT];
  // a staged region inside the lattice, clear of the body: every cell is
  // read as is
  const bool inside = x0 >= R && x0 + kCoefTileW + R <= nx && y0 >= R && y0 + T::TH + R <= ny &&
                      !(is_box && x0 - R < bx1 && x0 + kCoefTileW + R > bx0 && y0 - R < by1 &&
                        y0 + T::TH + R > by0);
  if (inside) {
    uint32_t o = (uint32_t)((y0 - R + wv) * ys + x0 + lane) * es;
    const uint32_t step = (uint32_t)(kCoefWaves * ys) * es;
#pragma unroll
    for (int m = 0; m < T::NCR; ++m) {
      // rows past the region (wave-uniform) read nothing and are not written
      oc[m] = wv + kCoefWaves * m < HH ? o : kNoCell;
      o += step;
    }
#pragma unroll
    for (int it = 0; it < T::NHIT; ++it) {
      const int i = tid + it * T::NT, j = i % (2 * R), hy = i / (2 * R);
      const int hx = j < R ? j : kCoefTileW + j;
      oh[it] = i < T::NHALO ? (uint32_t)((y0 - R + hy) * ys + x0 - R + hx) * es : kNoCell;
    }
  } else {
    // lattices narrower than the staged tile wrap more than once
    const bool narrow = nx < T::HW || (yper && ny < HH);
    auto offset = [&](int hx, int hy) -> uint32_t {
      int gx = x0 - R + hx, gy = y0 - R + hy;
      if (xper) {
        gx += gx < 0 ? nx : 0;
        gx -= gx >= nx ? nx : 0;
      }
      if (yper) {
        gy += gy < 0 ? ny : 0;
        gy -= gy >= ny ? ny : 0;
      }
      if (__builtin_expect(narrow, 0)) {
        if (xper) gx = (((x0 - R + hx) % nx) + nx) % nx;
        if (yper) gy = (((y0 - R + hy) % ny) + ny) % ny;
      }
      const bool solid = is_box && gx >= bx0 && gx < bx1 && gy >= by0 && gy < by1;
      const bool load = gx >= 0 && gx < nx && gy >= 0 && gy < ny && !solid;
      // cells without data read past the end of the plane: zeros
      return load ? (uint32_t)(gy * ys + gx) * es : kNoCell;
    };
#pragma unroll
    for (int m = 0; m < T::NCR; ++m) {
      const int hy = wv + kCoefWaves * m;
      oc[m] = hy < HH ? offset(R + lane, hy) : kNoCell;
    }
#pragma unroll
    for (int it = 0; it < T::NHIT; ++it) {
      const int i = tid + it * T::NT, j = i % (2 * R), hy = i / (2 * R);
      oh[it] = i < T::NHALO ? offset(j < R ? j : kCoefTileW + j, hy) : kNoCell;
    }
  }
#pragma unroll
  for (int m = 0; m < T::NCR; ++m)
#pragma unroll
    for (int k = 0; k < 6; ++k) g.core[m][k] = buf_load<S>(rs[k], oc[m]);
#pragma unroll
  for (int it = 0; it < T::NHIT; ++it)
#pragma unroll
    for (int k = 0; k < 6; ++k) g.halo[it][k] = buf_load<S>(rs[k], oh[it]);
}

// The cells of a solve that may have a wall link: rows and columns within R of
// the body or of a plate's walls (uniform values).
template <class L>
struct WallBand {
  int x0 = 0, x1 = 0, y0 = 0, y1 = 0, far0;
  __device__ __forceinline__ explicit WallBand(const SolveDesc& d) {
    far0 = 0x7fffffff;
    if (d.geom == GEOM_BOX) {
      x0 = d.bx0 - L::R;
      x1 = d.bx1 + L::R;
      y0 = d.by0 - L::R;
      y1 = d.by1 + L::R;
    } else if (d.geom == GEOM_PLATE) {
      x1 = d.nx;
      y1 = L::R;  // moving wall below row 0
      if (d.far == FAR_WALL) far0 = d.ny - L::R;
    }
  }
  // some cell of the 64 columns from cx and the `rows` rows from cy
  __device__ __forceinline__ bool meets(int cx, int cy, int rows) const {
    return (cx < x1 && cx + kCoefTileW > x0 && cy < y1 && cy + rows > y0) || cy + rows > far0;
  }
  __device__ __forceinline__ bool has(int x, int y) const {
    return (x >= x0 && x < x1 && y >= y0 && y < y1) || y >= far0;
  }
};

// Moments, wall arrivals and collision of the RB cells of this
// thread, from the staged tile in LDS (staged row r holds the pairs
// (a0, bx), (by, cxx), (cxy, cyy) of its HW cells as three runs of HW): the
// new coefficients of the cells in the lattice and the fluid go to res.  U:
// the wall drive U_w of the step.
template <class L, typename S, int RB, bool DSW>
__device__ __forceinline__ void compute_tile(const SolveDesc& d, const TileCtx<S>& t, int tile,
                                             const Pair<S>* C, const WallTable<S, DSW>& tab,
                                             const KernelLattice& lat, const CoefConst<S>& cc,
                                             int tid, S (&res)[RB][6], uint32_t& valid,
                                             double U) {
  using T = CoefTile<L, RB>;
  constexpr int R = T::R, HW = T::HW;
  const int nx = d.nx, ny = d.ny;
  const int x0 = (tile % d.tiles_x) * kCoefTileW;
  const int y0 = (tile / d.tiles_x) * T::TH;
  const bool is_box = d.geom == GEOM_BOX;
  const int bx0 = d.bx0, bx1 = d.bx1, by0 = d.by0, by1 = d.by1;

  const int lane = tid & 63, wave = tid >> 6;
  const int x = x0 + lane, yb = y0 + wave * RB;

  Mom<S> acc[RB];
#pragma unroll
  for (int k = 0; k < RB; ++k)
#pragma unroll
    for (int j = 0; j < 6; ++j) acc[k].v[j] = S(0);

  static_for<0, RB + 2 * R>([&](auto ic) __attribute__((always_inline)) {
    constexpr int iy = decltype(ic)::value - R;
    // staged row of source row iy, from the cell at column offset -R
    const lptr<const Pair<S>> row =
        opaque((lptr<const Pair<S>>)(C + (wave * RB + R + iy) * 3 * HW + lane));
    // per output row k (pulling along vy = k - iy): sums of w f, w vx f, w vx^2 f
    S t0[RB], t1[RB], t2[RB];
#pragma unroll
    for (int k = 0; k < RB; ++k) t0[k] = t1[k] = t2[k] = S(0);
    static_for<0, 2 * R + 1>([&](auto dxc) __attribute__((always_inline)) {
      constexpr int dx = decltype(dxc)::value - R;
      constexpr int vx = -dx;  // the source x - v sits at x + dx
      if constexpr (source_used<L, RB>(vx, iy)) {
        const Pair<S> p0 = row[dx + R], p1 = row[HW + dx + R], p2 = row[2 * HW + dx + R];
        // populations of the source cell along vx: f = g + vy^2 cyy + vy h
        S g = p0.x, h = p1.x;
        if constexpr (vx != 0) {
          g = fmadd(S(vx * vx), p1.y, fmadd(S(vx), p0.y, g));
          h = fmadd(S(vx), p2.x, h);
        }
        const S cyy = p2.y;
        static_for<0, RB>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          constexpr int vy = k - iy;
          constexpr int q = pull_q<L>(dx, iy, k);
          if constexpr (q >= 0) {
            constexpr int o = L::orbit[q];
            S f = g;
            if constexpr (vy != 0) f = fmadd(S(vy), h, fmadd(S(vy * vy), cyy, g));
            const S w = cc.w[o];
            if constexpr (dx == first_dx<L>(iy, k, false))
              t0[k] = w * f;
            else
              t0[k] = fmadd(w, f, t0[k]);
            if constexpr (vx != 0) {
              constexpr int a = vx < 0 ? -vx : vx;
              const S wa = a == 1 ? w : cc.wx[o][a];
              const S wb = a == 1 ? w : cc.wxx[o][a];
              const S wsx = vx < 0 ? -wa : wa;
              if constexpr (dx == first_dx<L>(iy, k, true)) {
                t1[k] = wsx * f;
                t2[k] = wb * f;
              } else {
                t1[k] = fmadd(wsx, f, t1[k]);
                t2[k] = fmadd(wb, f, t2[k]);
              }
            }
          }
        });
      }
    });
    static_for<0, RB>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      constexpr int vy = k - iy;
      if constexpr (vy >= -R && vy <= R) {
        Mom<S>& m = acc[k];
        if constexpr (iy == k - R) {
          // first source row of output row k
          m.v[0] = t0[k];
          m.v[1] = t1[k];
          m.v[3] = t2[k];
          m.v[2] = S(vy) * t0[k];
          m.v[4] = S(vy) * t1[k];
          m.v[5] = S(vy * vy) * t0[k];
        } else {
          m.v[0] += t0[k];
          m.v[1] += t1[k];
          m.v[3] += t2[k];
          if constexpr (vy != 0) {
            m.v[2] = fmadd(S(vy), t0[k], m.v[2]);
            m.v[4] = fmadd(S(vy), t1[k], m.v[4]);
            m.v[5] = fmadd(S(vy * vy), t0[k], m.v[5]);
          }
        }
      }
    });
#pragma unroll
    for (int k = 0; k < RB; ++k) row_fence(acc[k]);
  });

  // wall arrivals of the cells within R of a wall (uniform per wavefront: the
  // band of rows and columns whose cells may have a link)
  const WallBand<L> band(d);
  if (band.meets(x0, yb, RB)) {
#pragma unroll 1
    for (int k = 0; k < RB; ++k) {
      const int y = yb + k;
      const bool in = y < ny && x < nx && !(is_box && y >= by0 && y < by1 && x >= bx0 && x < bx1);
      if (!(in && band.has(x, y))) continue;
      const Mom<S> m = wall_moments<L, S, DSW>(d, C, HW, x0 - R, y0 - R, x, y,
                                               (S)(d.ladd_scale * U), U, tab, lat.theta);
#pragma unroll
      for (int kk = 0; kk < RB; ++kk)
#pragma unroll
        for (int j = 0; j < 6; ++j) acc[kk].v[j] += k == kk ? m.v[j] : S(0);
    }
  }

  const S th = cc.theta;
  const S inv_th = cc.inv_theta;
  const S h2 = cc.half_inv_theta2;
  const S om = (S)d.inv_tau;
  const S rho0 = (S)d.rho0;
  // Every lane runs the collision of all its rows: cells outside the lattice
  // or inside the body see only staged zeros and finite sums, and their
  // results are dropped by the store (bit k of `valid`), so no lane leaves
  // the straight-line code.
  bool bad = false;
  // (a compile-time loop: unrolled whatever the size of the wall code)
  static_for<0, RB>([&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const Mom<S>& m = acc[k];
    const int y = yb + k;
    const bool in = y < ny && x < nx && !(is_box && y >= by0 && y < by1 && x >= bx0 && x < bx1);
    valid |= in ? 1u << k : 0u;
    const S drho = m.v[0], jx = m.v[1], jy = m.v[2];
    const S rho = rho0 + drho;
    S inv_rho;
    if constexpr (sizeof(S) == 4)
      inv_rho = __builtin_amdgcn_rcpf(rho);  // 1 ulp; the FP32 form's error is dominated by storage
    else
      inv_rho = S(1) / rho;
    bad |= in && !(rho > S(0) && rho < S(INFINITY));
    const S ux = jx * inv_rho, uy = jy * inv_rho;
    const S axx = fmadd(-drho, th, m.v[3]), ayy = fmadd(-drho, th, m.v[5]), axy = m.v[4];
    const S bxx = fmadd(-om, fmadd(-jx, ux, axx), axx);
    const S bxy = fmadd(-om, fmadd(-jx, uy, axy), axy);
    const S byy = fmadd(-om, fmadd(-jy, uy, ayy), ayy);
    res[k][0] = fmadd(-(bxx + byy), cc.half_inv_theta, drho);
    res[k][1] = jx * inv_th;
    res[k][2] = jy * inv_th;
    res[k][3] = bxx * h2;
    res[k][4] = bxy * cc.inv_theta2;
    res[k][5] = byy * h2;
  });
  if (bad) d.state->unstable = 1;
}

// Store the new coefficients of this thread's cells (those in the lattice
// and the fluid: bit k of `valid` for row k).
template <class L, typename S, int RB>
__device__ __forceinline__ void store_tile(const SolveDesc& d, const TileCtx<S>& t, int tile,
                                           int tid, const S (&res)[RB][6], uint32_t valid,
                                           bool streaming) {
  using T = CoefTile<L, RB>;
  const gptr<S> mout = as_global(t.mout);
  const int64_t ks = d.mks;
  const int ys = (int)d.mys;
  gptr<S> pout[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) pout[k] = scalar_ptr(mout + k * ks);
  // the same planes as buffer resources, for the nontemporal stores
  const uint32_t bytes = plane_bytes<S>(d.ny, ys, ks);
  __amdgpu_buffer_rsrc_t ro[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) ro[k] = plane_rsrc(t.mout + k * ks, bytes);
  const int x = (tile % d.tiles_x) * kCoefTileW + (tid & 63);
  const int yb = (tile / d.tiles_x) * T::TH + (tid >> 6) * RB;
#pragma unroll
  for (int k = 0; k < RB; ++k) {
    if (!(valid & (1u << k))) continue;
    const int y = yb + k;
    const uint32_t o = (uint32_t)(y * ys + x) * (uint32_t)sizeof(S);
    // a state that stays in the last-level cache between steps is stored
    // through it (the next step reads it back from there: 36.7 against
    // 43.3 us per beam-box launch); a state streaming from HBM bypasses it
    // (2.84 against 3.03 ms per launch of the 256-solve batch)
    if (streaming) {
#pragma unroll
      for (int j = 0; j < 6; ++j) buf_store_nt(ro[j], o, res[k][j]);
    } else {
#pragma unroll
      for (int j = 0; j < 6; ++j) *at(pout[j], o) = res[k][j];
    }
  }
}

// Write a loaded tile (stage_load) to LDS.
template <class L, typename S, int RB>
__device__ __forceinline__ void stage_store(Pair<S>* C, const StageRegs<L, S, RB>& g, int tid) {
  using T = CoefTile<L, RB>;
  constexpr int R = T::R, HW = T::HW;
  const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int m = 0; m < T::NCR; ++m) {
    const int hy = wv + kCoefWaves * m;
    if (hy < T::HH)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        C[(hy * 3 + j) * HW + R + lane] = Pair<S>{g.core[m][2 * j], g.core[m][2 * j + 1]};
  }
#pragma unroll
  for (int it = 0; it < T::NHIT; ++it) {
    const int i = tid + it * T::NT, jj = i % (2 * R), hy = i / (2 * R);
    const int hx = jj < R ? jj : kCoefTileW + jj;
    if (i < T::NHALO)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        C[(hy * 3 + j) * HW + hx] = Pair<S>{g.halo[it][2 * j], g.halo[it][2 * j + 1]};
  }
}

// LDS of a workgroup: a staged tile, or the force's sums.
template <class L, typename S, int RB, bool DSW>
union CoefLds {
  struct {
    // staged row r, pair j, column c at C[(3 r + j) HW + c]: the reads of a
    // pair are 64-bit (128-bit) loads at consecutive lanes
    Pair<S> C[CoefTile<L, RB>::HH * 3 * CoefTile<L, RB>::HW];
    WallTable<S, DSW> tab;
  } tile;
  ForceLds force;
};

// Update of one tile by a workgroup.
template <class L, typename S, int RB, bool DSW>
__device__ __forceinline__ void tile_update(const SolveDesc& d, const TileCtx<S>& ctx, int tile,
                                            const KernelLattice& lat, const CoefConst<S>& cc,
                                            int tid, bool streaming,
                                            CoefLds<L, S, RB, DSW>& lds) {
  using T = CoefTile<L, RB>;
  Pair<S>* const C = lds.tile.C;
  WallTable<S, DSW>& tab = lds.tile.tab;
  // wall drive of the step (for the links): a new table entry every step, so
  // a cache miss; a vector load issued before the staging loads hides it
  // behind them (a scalar load would share its counter with the LDS reads)
  uint32_t nv = drive_index(ctx.n);
  asm volatile("" : "+v"(nv));
  const double U = as_global(d.drive)[nv].u;
  {
    // all loads of a thread are issued before the first LDS store, so the
    // block waits for one memory round trip, not one per staged cell
    StageRegs<L, S, RB> g;
    stage_load<L, S, RB>(d, ctx, tile, g, tid);
    if (tid < 48 &&
        WallBand<L>(d).meets((tile % d.tiles_x) * kCoefTileW, (tile / d.tiles_x) * T::TH, T::TH))
      fill_wall_table<L>(tab, lat, tid);
    stage_store<L, S, RB>(C, g, tid);
  }
  __syncthreads();
  S res[RB][6];
  uint32_t valid = 0;
  compute_tile<L, S, RB, DSW>(d, ctx, tile, C, tab, lat, cc, tid, res, valid, U);
  store_tile<L, S, RB>(d, ctx, tile, tid, res, valid, streaming);
}

// DSW: with the diffuse-scattering wall (a separate instantiation, so that
// the bounce-back kernel carries none of its code).  One workgroup per work
// item.
template <class L, typename S, int RB, bool DSW>
__global__ __launch_bounds__(64 * kCoefWaves) void coef_kernel(const SolveDesc* __restrict__ descs,
                                                   const WorkItem* __restrict__ work,
                                                   KernelLattice lat, CoefConst<S> cc,
                                                   int streaming, int dn) {
  __shared__ CoefLds<L, S, RB, DSW> lds;
  const WorkItem wi = kread_item(&work[blockIdx.x]);
  if (wi.tile == kNoTile) return;
  const SolveDesc& d = descs[wi.solve];
  const TileCtx<S> ctx = tile_ctx<S>(d, dn);
  if (wi.tile == kForceTile) {
    wall_force<S, DSW>(d, true, ctx.n, lds.force);
    return;
  }
  tile_update<L, S, RB, DSW>(d, ctx, wi.tile, lat, cc, (int)threadIdx.x, streaming != 0, lds);
}

template <class L, typename S, int RB>
static hipError_t launch_rb(bool ds, bool streaming, const SolveDesc* descs, const WorkItem* work,
                            int nwork, const KernelLattice& lat, int dn, hipStream_t stream,
                            const KernelEvents& ev) {
  const CoefConst<S> cc = coef_const<S>(lat);
  const dim3 grid(nwork), block(64 * kCoefWaves);
  const int st = streaming ? 1 : 0;
  if (ds)
    launch_kernel(coef_kernel<L, S, RB, true>, grid, block, stream, ev, descs, work, lat, cc, st,
                  dn);
  else
    launch_kernel(coef_kernel<L, S, RB, false>, grid, block, stream, ev, descs, work, lat, cc, st,
                  dn);
  return hipGetLastError();
}

template <class L, typename S>
static hipError_t launch_coef_t(int k, bool ds, bool streaming, const SolveDesc* descs,
                                const WorkItem* work, int nwork, const KernelLattice& lat, int dn,
                                hipStream_t stream, const KernelEvents& ev) {
  switch (k) {
    case 1:
      return launch_rb<L, S, 1>(ds, streaming, descs, work, nwork, lat, dn, stream, ev);
    case 2:
      return launch_rb<L, S, 2>(ds, streaming, descs, work, nwork, lat, dn, stream, ev);
    case 3:
      return launch_rb<L, S, 3>(ds, streaming, descs, work, nwork, lat, dn, stream, ev);
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_coef(int Q, bool f64, int k, bool ds, bool streaming, const SolveDesc* descs,
                       const WorkItem* work, int nwork, const KernelLattice& lat, int dn,
                       hipStream_t stream, KernelEvents ev) {
  if (nwork <= 0) return hipSuccess;
  if (Q == 9)
    return f64 ? launch_coef_t<D2Q9, double>(k, ds, streaming, descs, work, nwork, lat, dn, stream,
                                             ev)
               : launch_coef_t<D2Q9, float>(k, ds, streaming, descs, work, nwork, lat, dn, stream,
                                            ev);
  return f64 ? launch_coef_t<D2Q37, double>(k, ds, streaming, descs, work, nwork, lat, dn, stream, ev)
             : launch_coef_t<D2Q37, float>(k, ds, streaming, descs, work, nwork, lat, dn, stream, ev);
}

}  // namespace lbm

// C ABI of the solver: validation, device memory layout, lifecycle, the
// per-step launch sequence, and host-side read-out (force history, lock-in
// fit, populations).  See include/lbm.h for the contract of each call.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <thread>
#include <unordered_map>
#include <vector>

#include "internal.hpp"

using namespace lbm;

namespace lbm {

// Workgroups of a launch are dealt to the 8 XCDs in turn (workgroup b runs on
// XCD b % 8), and each XCD has its own L2.  Tiles of one lattice row share the
// cache lines at their ends (the pulls are shifted by up to 3 cells), so the
// rows ("super-rows" of `span` tiles, about one lattice row) are dealt to the
// XCDs in turn: workgroups 8k..8k+7 take tile j of 8 consecutive rows.  All
// XCDs then work on one compact band of rows at a time (good HBM page
// locality) while every row stays within one L2.  Positions without a tile
// are no-op items (tile -1), which also keeps the next solve aligned.
void order_tiles(std::vector<WorkItem>* out, int32_t solve, int32_t ntiles, int32_t span) {
  while (out->size() % 8) out->push_back(WorkItem{solve, -1});
  span = std::max<int32_t>(1, span);
  const int32_t nrows = (ntiles + span - 1) / span;
  for (int32_t g = 0; g < nrows; g += 8)
    for (int32_t k = 0; k < span; ++k)
      for (int32_t i = 0; i < 8; ++i) {
        const int32_t row = g + i, t = row * span + k;
        out->push_back(WorkItem{solve, row < nrows && t < ntiles ? t : -1});
      }
}

// Small launches take one row per wavefront: few workgroups per compute unit,
// so a step is the chain of one wavefront, which K rows make K times as long
// (a 256 x 256 box, K = 1, 2, 3: FP32 6.9, 9.1, 10.8 us per step, FP64 7.9,
// 10.4, 12.8).  Large ones share the halo and the source cells among more rows.
// The lines: FP32 640 x 640 10.6, 10.7, 12.3, 768 x 768 13.0, 11.8, 12.4,
// 848 x 848 16.0, 14.9, 13.7, 1024 x 1024 20.3, 17.7, 17.9, 1400 x 1400 32.5,
// 26.6, 25.7; FP64 512 x 512 12.5, 12.3, 13.5, 640 x 640 17.4, 17.2, 17.6,
// 768 x 768 21.8, 20.1, 21.0, 1400 x 1400 54.3, 46.3, 48.6 (K = 3 leaves two
// workgroups per compute unit by LDS).  States that stream from HBM: FP32
// 3000 x 3000 133, 102, 91, 4096 x 4096 254, 180, 158; FP64 1800 x 1800 94, 80, 86,
// 3000 x 3000 243, 205, 230, 4096 x 4096 439, 362, 398 (the larger halo of K = 2
// costs less than the third workgroup brings).  The lines are D2Q37's; D2Q9 differs
// by less than 4 % but for FP32 near 640 x 640 (7.9, 7.1, 7.3).  The cells are those
// of whole tile columns (coef_cells), since a wavefront with idle lanes takes as
// long as a full one: D2Q37 FP32 12 x 39318 42.4, 32.2, 27.4, 20 x 12000 16.6, 13.9,
// 11.9, 70 x 9000 21.3, 17.5, 16.8.  A cell's bits do not depend on K.
int coef_k_for(uint32_t tile, bool f64, int64_t cells) {
  if (tile) return (int)tile;
  if (f64) return cells <= 400000 ? 1 : 2;
  return cells <= 420000 ? 1 : cells <= 650000 ? 2 : kCoefKDefault;
}

int64_t coef_cells(const lbm_params* p) {
  return (int64_t)(p->nx + kCoefTileW - 1) / kCoefTileW * kCoefTileW * p->ny;
}

CoefGrid coef_grid(const lbm_params* p, int K) {
  const int th = coef_tile_rows(K);
  CoefGrid g;
  g.tiles_x = (p->nx + kCoefTileW - 1) / kCoefTileW;
  g.ntiles = g.tiles_x * ((p->ny + th - 1) / th);
  return g;
}

// Coefficient-kernel tiles (of K cells per thread) that hold a cell
// with a wall link: the band of R cells around the body, the plate's wall rows
// (the same band the kernel tests per wavefront).
std::vector<char> coef_wall_tiles(const lbm_params* p, int K, int R) {
  const CoefGrid grid = coef_grid(p, K);
  std::vector<char> wall((size_t)grid.ntiles, 0);
  int wx0 = 0, wx1 = p->nx, wy0 = 0, wy1 = 0;
  bool far_band = false;
  if (p->geometry == LBM_GEOM_BOX) {
    wx0 = p->box_x0 - R;
    wx1 = p->box_x0 + p->box_lx + R;
    wy0 = p->box_y0 - R;
    wy1 = p->box_y0 + p->box_ly + R;
  } else if (p->geometry == LBM_GEOM_PLATE) {
    wy1 = R;
    far_band = p->far == LBM_FAR_WALL;
  }
  const int th = coef_tile_rows(K);
  for (int32_t t = 0; t < grid.ntiles; ++t) {
    const int x0 = (t % grid.tiles_x) * kCoefTileW, y0 = (t / grid.tiles_x) * th;
    wall[t] = (x0 < wx1 && x0 + kCoefTileW > wx0 && y0 < wy1 && y0 + th > wy0) ||
              (far_band && y0 + th > p->ny - R);
  }
  return wall;
}

void order_coef_tiles(std::vector<WorkItem>* front, std::vector<WorkItem>* rest, int32_t solve,
                      const std::vector<char>& wall, int32_t ntiles, int32_t span, bool banded) {
  for (int32_t t = 0; t < ntiles; ++t)
    if (wall[t]) front->push_back(WorkItem{solve, t});
  const size_t from = rest->size();
  if (banded)
    order_tiles_banded(rest, solve, ntiles, span);
  else
    order_tiles(rest, solve, ntiles, span);
  for (size_t i = from; i < rest->size(); ++i) {
    WorkItem& w = (*rest)[i];
    if (w.tile >= 0 && wall[w.tile]) w.tile = -1;
  }
}

void join_front(std::vector<WorkItem>* front, const std::vector<WorkItem>& rest) {
  while (front->size() % 8) front->push_back(WorkItem{0, -1});
  front->insert(front->end(), rest.begin(), rest.end());
}

void order_tiles_banded(std::vector<WorkItem>* out, int32_t solve, int32_t ntiles,
                        int32_t span) {
  while (out->size() % 8) out->push_back(WorkItem{solve, -1});
  span = std::max<int32_t>(1, span);
  const int32_t nrows = (ntiles + span - 1) / span;
  const int32_t band = (nrows + 7) / 8, per = band * span;
  for (int32_t j = 0; j < per; ++j)
    for (int32_t x = 0; x < 8; ++x) {
      const int32_t row = x * band + j / span, t = row * span + j % span;
      out->push_back(WorkItem{solve, row < nrows && t < ntiles ? t : -1});
    }
}

ColumnShape column_shape(int Q, int nx, int rows, int nsub) {
  const int R = Q == 9 ? D2Q9::R : D2Q37::R;
  const int cells = (rows + 2 * R * nsub) * nx;
  ColumnShape sh;
  sh.rows = rows;
  sh.nsub = nsub;
  sh.threads = (cells + 63) / 64 * 64 + 64;  // the last wavefront for the force
  return sh;
}

// Lanes per LDS bank, on average over the parts of a wavefront that are served
// together, when it reads one element per cell of rows of nx columns.
static double bank_load(int nx, int ys, int es) {
  const int part = es == 8 ? 16 : 32;  // lanes served together, and banks
  int sum = 0;
  for (int l0 = 0; l0 < 64; l0 += part) {
    int hits[32] = {}, most = 0;
    for (int l = l0; l < l0 + part; ++l)
      most = std::max(most, ++hits[(l % nx * ys + l / nx) % part]);
    sum += most;
  }
  return (double)sum / (64 / part);
}

// A step's share of a launch (about 4 us) falls as 1/T, the halo it updates
// grows as R (T - 1) / 2 rows per side.
// While the workgroups all run at once (one per compute unit, two of D2Q9's FP32
// ones): the fewest rows for that, 8 at least (below, the halo is most of the
// work), and the most steps that fit, up to 11 (D2Q37; 4 x 2048 FP32, us per step
// in calls of 1024: 1.89 at 5, 1.62 at 9, 1.56 at 11, 1.67 at 13) or 27 (D2Q9;
// 4 x 256, FP32 / FP64: 0.77 / 0.82 at 15, 0.70 / 0.75 at 23, 0.69 / 0.76 at 27,
// 0.78 / 0.87 at 31).
// Longer lattices and batches, or widths that leave one step only: what costs
// least, in updates of a row: the rounds of workgroups (two of D2Q9 at once) times
// what one does per step -- the loads and stores of its region (a row 3 or 5
// updates, FP32 or FP64; fitted) once in T steps, the updates, a tenth more for
// every further lane per bank, and the barriers, 100 cells' updates -- and the
// launch, 1300 (D2Q9) or 500 cells' updates.
// D2Q37 FP32, us per step, against the most steps that leave 8 rows of a full
// plane: 7 x 16384 6.0 and 21.8 (64 rows per column, a row's lanes all on one
// bank), 8 x 16384 6.9 and 10.0, 61 plates of 8 x 2048 62 and 83 (FP64 98 and 119).
ColumnPlan column_plan(int Q, bool f64, int nx, const std::vector<int>& ny) {
  const int R = Q == 9 ? D2Q9::R : D2Q37::R;
  const int most = Q == 9 ? kColumnMaxSub : 11, fit = kColumnCells / nx, es = f64 ? 8 : 4;
  auto groups = [&](int rows) {
    int64_t g = 0;
    for (int n : ny) g += (n + rows - 1) / rows;
    return g;
  };
  auto banks = [&](int region) { return bank_load(nx, column_stride(region, nx, es), es); };
  ColumnPlan plan;
  plan.rows = 8;
  const int abreast = Q == 9 ? 512 : 256;
  while (plan.rows < fit && groups(plan.rows) > (f64 ? 256 : abreast)) ++plan.rows;
  plan.max_sub = most;
  while (plan.max_sub > 1) {
    const int region = plan.rows + 2 * R * plan.max_sub;
    if (region <= fit && banks(region) <= 4) {
      plan.groups = groups(plan.rows);
      return plan;
    }
    plan.max_sub -= 2;
  }
  double load[kColumnCells + 1], least = INFINITY;  // by region
  for (int region = 1; region <= fit; ++region) load[region] = banks(region);
  for (int rows = 4; rows + 2 * R <= fit; ++rows) {
    double rounds = (double)groups(rows) / abreast;
    rounds = rounds < 4 ? std::ceil(rounds) : rounds + 0.5;
    for (int t = 1; t <= most && rows + 2 * R * t <= fit; t += 2) {
      const int region = rows + 2 * R * t;
      if (load[region] > 4) continue;
      const double work = (f64 ? 5.0 : 3.0) * region / t +
                          (rows + R * (t - 1)) * (0.9 + 0.1 * load[region]) + 100.0 / nx;
      const double cost = rounds * work + (Q == 9 ? 1300.0 : 500.0) / (nx * t);
      if (cost < least) {
        least = cost;
        plan.rows = rows;
        plan.max_sub = t;
      }
    }
  }
  plan.groups = groups(plan.rows);
  // about as much halo as rows: steps one by one (column_single_kernel) are faster
  // (31 plates of 16 x 2048 FP32 69 us per step against 77, 12 x 16384 alone 14.4 against 12.1)
  if (Q == 37 && !f64 && nx >= 14 && plan.groups > 1500) plan.max_sub = 1;
  return plan;
}

// A launch of one step: column_kernel where a few rounds of workgroups do,
// column_single_kernel above (us per call of one step, column / single).  D2Q37
// bounce-back: FP32 4 x 10448 (255 workgroups) 7.8 / 9.2, 8 x 13217 (509) 14 / 13,
// 16 x 6000 (750) 17 / 11, 61 of 8 x 2048 (3294) 96 / 72; FP64 8 x 4000 (250) 9.9 / 11,
// 61 of 8 x 2048 172 / 128.  With a diffuse wall the single kernel's wall cells are
// a chain of 15 us more: FP32 two of 12 x 8000 (1000) 24 / 29, 8 x 40000 (1177)
// 29 / 29; FP64, one workgroup per compute unit, 16 x 6000 (750) 23 / 29, two of
// 12 x 8000 38 / 33, 8 x 40000 46 / 34.  D2Q9 has no such chain: 4 x 2048 6.0 / 5.6,
// six of 16 x 4096 16 / 10, FP64 20 / 14.
bool column_single(int Q, bool f64, const ColumnPlan& plan, bool ds) {
  if (Q == 9 || plan.max_sub == 1) return true;
  return plan.groups > (!ds ? 400 : f64 ? 900 : 1600);
}

std::vector<int> odd_pieces(int64_t n, int max_sub) {
  std::vector<int> out;
  if (n <= 0) return out;
  int64_t m = (n + max_sub - 1) / max_sub;
  m += (m ^ n) & 1;  // as many odd numbers as n is odd or even
  int64_t base = n / m;
  base -= base % 2 == 0;
  int64_t twos = (n - m * base) / 2;
  for (int64_t i = 0; i < m; ++i) out.push_back((int)(base + (i < twos ? 2 : 0)));
  return out;
}

// Work-list length order_tiles (and order_tiles_banded) produces for one
// solve starting aligned.
int64_t ordered_length(int64_t ntiles, int64_t span) {
  span = std::max<int64_t>(1, span);
  const int64_t nrows = (ntiles + span - 1) / span;
  return (nrows + 7) / 8 * 8 * span;
}

}  // namespace lbm

namespace {

template <class L>
void fill_lattice(HostLattice* h) {
  h->Q = L::Q;
  h->R = L::R;
  for (int i = 0; i < L::Q; ++i) {
    h->vx.push_back(L::vx[i]);
    h->vy.push_back(L::vy[i]);
    h->orbit.push_back(L::orbit[i]);
    h->opp.push_back(opposite<L>(i));
  }
}

bool host_lattice(int Q, HostLattice* h) {
  if (Q == 9) fill_lattice<D2Q9>(h);
  else if (Q == 37) fill_lattice<D2Q37>(h);
  else return false;
  return lattice_weights(Q, &h->lw);
}

// One coefficient plane must stay addressable with 32-bit byte offsets.
bool coefficient_plane_fits(const lbm_params* p) {
  const uint64_t es = p->storage == LBM_STORE_F64 ? 8 : 4;
  return (uint64_t)p->ny * align_up((uint64_t)p->nx, kCoefTileW) * es < ((uint64_t)1 << 31);
}

// Device state kept as the six H2 coefficients (else the Q populations).
bool uses_coefficients(const lbm_params* p) {
  if (p->representation == LBM_REPR_COEFFICIENTS ||
      p->representation == LBM_REPR_COEFFICIENTS_NOLOAD)
    return true;
  return p->representation == LBM_REPR_AUTO && p->collision == LBM_COLL_REGULARIZED &&
         p->nx >= kCoefTileW && coefficient_plane_fits(p);
}

// Stepped by the column kernel: plates and periodic lattices of a few columns
// kept as populations (see column.hip).  14 to 16 columns of D2Q37 leave room for
// 3 steps per launch and about as much halo as rows, so long ones go to the
// population kernel (16 columns, us per step, column / population kernel: 4096
// rows FP32 6.2 / 7.5, FP64 9.6 / 10.9, 8192 rows 11.8 / 9.1, 19.2 / 14.4).  The choice
// is by the lattice alone, since its bits follow from it; batches of many short ones
// are column_plan's.
bool uses_columns(const lbm_params* p) {
  if (uses_coefficients(p) || p->geometry == LBM_GEOM_BOX || p->nx > kColumnMaxNx) return false;
  return p->lattice == 9 || p->nx < 14 || (int64_t)p->nx * p->ny <= kColumnWideCells;
}

int validate(const lbm_params* p, HostLattice* lat) {
  if (!p) return LBM_EINVAL;
  if (p->abi_version != LBM_ABI_VERSION) return LBM_EABI;
  if (!host_lattice((int)p->lattice, lat)) return LBM_EINVAL;
  if (p->storage != LBM_STORE_F64 && p->storage != LBM_STORE_F32_DEV) return LBM_EINVAL;
  if (p->collision != LBM_COLL_REGULARIZED && p->collision != LBM_COLL_BGK) return LBM_EINVAL;
  if (p->wall != LBM_WALL_BB && p->wall != LBM_WALL_DS && p->wall != LBM_WALL_MAXWELL)
    return LBM_EINVAL;
  if (p->wall != LBM_WALL_BB && p->geometry == LBM_GEOM_PERIODIC) return LBM_EINVAL;
  if (p->wall == LBM_WALL_MAXWELL && !(p->accommodation >= 0.0 && p->accommodation <= 1.0))
    return LBM_EINVAL;
  if (p->far != LBM_FAR_WALL && p->far != LBM_FAR_EQ) return LBM_EINVAL;
  if (p->representation > LBM_REPR_COEFFICIENTS_NOLOAD) return LBM_EINVAL;
  const bool coef_asked = p->representation == LBM_REPR_COEFFICIENTS ||
                          p->representation == LBM_REPR_COEFFICIENTS_NOLOAD;
  if (coef_asked && p->collision != LBM_COLL_REGULARIZED) return LBM_EINVAL;
  // a box with diffuse or Maxwell faces: at most kMaxWallCols face columns
  if (p->wall != LBM_WALL_BB && p->geometry == LBM_GEOM_BOX &&
      2 * ((int64_t)p->box_lx + p->box_ly) > kMaxWallCols)
    return LBM_EINVAL;
  const int R = lat->R;
  if (p->nx < std::max(3, R) || p->ny < std::max(3, R)) return LBM_EINVAL;
  if ((int64_t)p->nx * p->ny > (int64_t)1 << 30) return LBM_EINVAL;
  if (coef_asked && !coefficient_plane_fits(p)) return LBM_EINVAL;
  // tile: cells per thread of the population kernel, or tile variant of the
  // coefficient kernel
  if (uses_coefficients(p)) {
    if (p->tile > (uint32_t)kCoefKMax) return LBM_EINVAL;
  } else if (p->tile != 0 && p->tile != 1 && p->tile != 2 && p->tile != 4) {
    return LBM_EINVAL;
  }
  if (!(p->tau > 0.5)) return LBM_EINVAL;  // rejects NaN too; +inf allowed
  if (!std::isfinite(p->omega) || !std::isfinite(p->u0)) return LBM_EINVAL;
  if (!(p->rho0 > 0) || !std::isfinite(p->rho0)) return LBM_EINVAL;
  if (p->max_steps < 1 || p->max_steps > ((int64_t)1 << 32)) return LBM_EINVAL;
  if (p->lockin_first < 0 || p->lockin_count < 0 ||
      p->lockin_first + p->lockin_count > p->max_steps)
    return LBM_EINVAL;
  if (p->history_capacity < 0 || p->history_capacity > p->max_steps) return LBM_EINVAL;
  switch (p->geometry) {
    case LBM_GEOM_PLATE:
    case LBM_GEOM_PERIODIC:
      break;
    case LBM_GEOM_BOX:
      if (p->far != LBM_FAR_EQ) return LBM_EINVAL;
      if (p->box_lx < R || p->box_ly < R || p->box_x0 < R || p->box_y0 < R) return LBM_EINVAL;
      if ((int64_t)p->box_x0 + p->box_lx + R > p->nx ||
          (int64_t)p->box_y0 + p->box_ly + R > p->ny)
        return LBM_EINVAL;
      break;
    default:
      return LBM_EINVAL;
  }
  return LBM_OK;
}

bool in_body(const lbm_params* p, int x, int y) {
  return p->geometry == LBM_GEOM_BOX && x >= p->box_x0 && x < p->box_x0 + p->box_lx &&
         y >= p->box_y0 && y < p->box_y0 + p->box_ly;
}

// True if a population arriving at fluid cell (x, y) along q comes from the
// moving wall or body (a bounce-back link that carries force).
bool is_link(const lbm_params* p, const HostLattice& L, int x, int y, int q) {
  const int sx = x - L.vx[q], sy = y - L.vy[q];
  if (p->geometry == LBM_GEOM_PLATE) return sy < 0;
  if (p->geometry == LBM_GEOM_BOX) return in_body(p, sx, sy);
  return false;
}

// Mirror cell of the bounce-back link arriving at fluid cell (x, y) along q
// (half-way walls; the same rules as the kernels).
void mirror_of(const lbm_params* p, const HostLattice& L, int x, int y, int q, int* px, int* py) {
  const int sx = x - L.vx[q], sy = y - L.vy[q];
  if (p->geometry == LBM_GEOM_PLATE) {
    *px = x;
    *py = -1 - sy;
    return;
  }
  const int x0 = p->box_x0, x1 = p->box_x0 + p->box_lx;
  const int y0 = p->box_y0, y1 = p->box_y0 + p->box_ly;
  *px = x < x0 ? 2 * x0 - 1 - sx : (x >= x1 ? 2 * x1 - 1 - sx : x);
  *py = y < y0 ? 2 * y0 - 1 - sy : (y >= y1 ? 2 * y1 - 1 - sy : y);
}

// Momentum-exchange tables of the wall force.  Each bounce-back link (fluid
// arrival x along v_i, mirror cell x_p) contributes
//   -v_i (f_opp(x_p) + f_i^adv(x)) = -v_i (2 w_i rho0 + 2 df_opp(x_p) + 2 w_i rho0 (v_i.U_w)/theta)
// with df the stored deviation.  The rest part and the moving-wall part are
// geometry constants (fstatic, kladd times U_w), summed here in long double;
// the deviation part becomes the link list (population state) or, per mirror
// cell, two 6-vectors acting on the cell's H2 coefficients (coefficient state:
// df_opp(x_p) = w_i (a0 - vx bx - vy by + vx^2 cxx + vx vy cxy + vy^2 cyy)).
// At a diffuse wall (eq. DS) the arrival f_i^adv is the wall's emission: the
// tables then carry -v_i df_opp(x_p) and the crossing mass df_opp(x_p), and
// the emission's share follows from the lattice sums in `ds` (wall_force).
struct ForceTables {
  std::vector<ForceLink> links;
  std::vector<ForceCell> cells;
  std::vector<LinkWeights> lweights;
  std::vector<CellWeights> cweights;
  double fstatic[2] = {0, 0}, kladd[2] = {0, 0};
  double ds[6] = {0, 0, 0, 0, 0, 0};
  // box with diffuse or Maxwell faces
  std::vector<WallCol> wcols;
  std::vector<WallLink> wlinks;
};

bool diffuse_box(const lbm_params* p) {
  return p->geometry == LBM_GEOM_BOX && p->wall != LBM_WALL_BB;
}

// The mirror cells of a coefficient state with their force weights; cells with
// equal weights (compared bit for bit) share a pattern.
struct CellTable {
  const Layout& lay;
  ForceTables* t;
  int x0 = 0, y0 = 0, w = 0;    // the cells within R of the moving wall
  std::vector<int32_t> index;   // of those cells: position in t->cells, or -1
  std::vector<CellWeights> cw;  // the weights of t->cells

  CellTable(const lbm_params* p, int R, const Layout& layout, ForceTables* tables)
      : lay(layout), t(tables), w(p->nx) {
    int h = R;
    if (p->geometry == LBM_GEOM_BOX) {
      x0 = p->box_x0 - R;
      y0 = p->box_y0 - R;
      w = p->box_lx + 2 * R;
      h = p->box_ly + 2 * R;
    }
    if (lay.mom && p->geometry != LBM_GEOM_PERIODIC) index.assign((size_t)w * h, -1);
  }
  CellWeights& at(int px, int py) {
    int32_t& pos = index[(size_t)(py - y0) * w + (px - x0)];
    if (pos >= 0) return cw[(size_t)pos];
    ForceCell fc{};
    fc.off = (int64_t)py * lay.mpitch + px;
    pos = (int32_t)t->cells.size();
    t->cells.push_back(fc);
    cw.push_back(CellWeights{});
    return cw.back();
  }
  void assign_patterns() {
    std::unordered_map<std::string, int32_t> pats;
    for (size_t i = 0; i < t->cells.size(); ++i)
      t->cells[i].pat = pattern(pats, t->cweights, cw[i]);
  }
  template <class P, class V, class W>
  static int32_t pattern(P& pats, V& table, const W& wts) {
    const std::string key(reinterpret_cast<const char*>(&wts), sizeof(wts));
    auto it = pats.find(key);
    if (it != pats.end()) return it->second;
    const int32_t k = (int32_t)table.size();
    table.push_back(wts);
    pats.emplace(key, k);
    return k;
  }
};

// Tables of a box with diffuse or Maxwell faces: its links face column by
// face column (faces below, above the body by arrival x, left, right of it
// by arrival y; in a column by arrival cell and direction), then the corner
// links; per column the lattice sums of its links (long double).  The force
// is -sum v_l (f_partner + f_arrival) over every link: the rest-state parts
// give fstatic, the moving-wall terms of the corner links and of the specular
// share at the x faces give kladd.  The rest is formed per link (population
// state); of a coefficient state all but the columns' emission is linear in
// the cells' coefficients and becomes weights per cell, as for bounce-back.
void build_wall_tables(const lbm_params* p, const HostLattice& L, const Layout& lay,
                       ForceTables* t) {
  const int R = L.R;
  const int x0 = p->box_x0, x1 = p->box_x0 + p->box_lx;
  const int y0 = p->box_y0, y1 = p->box_y0 + p->box_ly;
  const long double th = L.lw.theta_ld;
  auto find = [&](int vx, int vy) {
    for (int j = 0; j < L.Q; ++j)
      if (L.vx[j] == vx && L.vy[j] == vy) return j;
    return -1;
  };
  auto face_of = [&](int x, int y) {
    const bool inx = x >= x0 && x < x1, iny = y >= y0 && y < y1;
    if (inx && !iny) return y < y0 ? 0 : 1;
    if (iny && !inx) return x < x0 ? 2 : 3;
    return -1;
  };
  const long double spec =
      1.0L - (p->wall == LBM_WALL_MAXWELL ? (long double)p->accommodation : 1.0L);
  long double sx = 0, sy = 0, kx = 0, ky = 0;
  CellTable cells(p, L.R, lay, t);
  // -scale v_l times the population of velocity (ux, uy) and weight w at a cell
  auto add_pop = [&](int cx, int cy, long double scale, long double w, int vx, int vy, int ux,
                     int uy) {
    CellWeights& fc = cells.at(cx, cy);
    const double sw = (double)(-scale * w);
    const int g[6] = {1, ux, uy, ux * ux, ux * uy, uy * uy};
    for (int k = 0; k < 6; ++k) {
      fc.wx[k] += sw * (vx * g[k]);
      fc.wy[k] += sw * (vy * g[k]);
    }
  };
  // crossing-mass weights of the current column over its cells' coefficients
  long double mc[3][6];
  // the links of a fluid cell, in direction order
  auto add_cell = [&](int x, int y, int col) {
    for (int q = 0; q < L.Q; ++q) {
      const int vx = L.vx[q], vy = L.vy[q];
      const int sxs = x - vx, sys = y - vy;
      if (!in_body(p, sxs, sys)) continue;
      int px, py;
      mirror_of(p, L, x, y, q, &px, &py);
      const long double w = L.lw.w_orbit_ld[L.orbit[q]];
      WallLink l{};
      l.off_partner = L.opp[q] * lay.qs + py * lay.ys + px;
      l.col = col;
      l.w = (double)w;
      l.vx = vx;
      l.vy = vy;
      const int face = face_of(x, y);
      // where and with which velocity the specular source crossed
      const bool xface = face >= 2;
      const int ux = xface ? -vx : vx, uy = xface ? vy : -vy;
      const int cx = xface ? px : sxs, cy = xface ? sys : py;
      if (face >= 0) l.off_spec = find(ux, uy) * lay.qs + cy * lay.ys + cx;
      // a corner link's arrival is its partner again
      if (lay.mom) add_pop(px, py, face < 0 ? 2.0L : 1.0L, w, vx, vy, -vx, -vy);
      if (lay.mom && face >= 0 && spec != 0) add_pop(cx, cy, spec, w, vx, vy, ux, uy);
      if (face < 0 || xface) {
        const long double share = face < 0 ? 1.0L : spec;
        kx -= share * vx * w * 2.0L * p->rho0 * vx / th;
        ky -= share * vy * w * 2.0L * p->rho0 * vx / th;
      }
      if (col >= 0) {
        // the partner's distance from the face (it lies in the link's column)
        const int k = face == 0 ? y0 - py : face == 1 ? py - (y1 - 1) : face == 2 ? x0 - px
                                                                                  : px - (x1 - 1);
        const long double g[6] = {1, -(long double)vx, -(long double)vy,
                                  (long double)vx * vx, (long double)vx * vy,
                                  (long double)vy * vy};
        for (int j = 0; j < 6; ++j) mc[k - 1][j] += w * g[j];
      }
      sx -= 2.0L * w * p->rho0 * vx;
      sy -= 2.0L * w * p->rho0 * vy;
      t->wlinks.push_back(l);
    }
  };
  // columns: cells of a face column from the face outwards
  const int ncol = 2 * (p->box_lx + p->box_ly);
  t->wcols.assign((size_t)ncol, WallCol{});
  for (int c = 0; c < ncol; ++c) {
    int face, at;
    if (c < p->box_lx) { face = 0; at = x0 + c; }
    else if (c < 2 * p->box_lx) { face = 1; at = x0 + c - p->box_lx; }
    else if (c < 2 * p->box_lx + p->box_ly) { face = 2; at = y0 + c - 2 * p->box_lx; }
    else { face = 3; at = y0 + c - 2 * p->box_lx - p->box_ly; }
    WallCol& wc = t->wcols[(size_t)c];
    wc.first = (int32_t)t->wlinks.size();
    for (auto& row : mc)
      for (auto& v : row) v = 0;
    for (int k = 1; k <= R; ++k) {
      const int x = face <= 1 ? at : (face == 2 ? x0 - k : x1 - 1 + k);
      const int y = face >= 2 ? at : (face == 0 ? y0 - k : y1 - 1 + k);
      wc.cell[k - 1] = (int64_t)y * lay.mpitch + x;
      add_cell(x, y, c);
    }
    for (int k = 0; k < 3; ++k)
      for (int j = 0; j < 6; ++j) wc.mc[k][j] = (double)mc[k][j];
    wc.count = (int32_t)t->wlinks.size() - wc.first;
    long double mr = 0, z1 = 0, z2 = 0, l1 = 0;
    long double ex[3] = {0, 0, 0}, ey[3] = {0, 0, 0};
    for (int i = wc.first; i < wc.first + wc.count; ++i) {
      const WallLink& l = t->wlinks[(size_t)i];
      const long double w = L.lw.w_orbit_ld[L.orbit[find((int)l.vx, (int)l.vy)]];
      const long double vx = l.vx;
      mr += w;
      z1 += w * vx / th;
      z2 += w * (vx * vx / (2 * th * th) - 1 / (2 * th));
      l1 += 2 * w * vx / th;
      for (int k = 0; k < 3; ++k) {
        const long double pw = k == 0 ? w : k == 1 ? w * vx : w * vx * vx;
        ex[k] += pw * vx;
        ey[k] += pw * (long double)l.vy;
      }
    }
    for (int k = 0; k < 3; ++k) {
      wc.ex[k] = (double)ex[k];
      wc.ey[k] = (double)ey[k];
    }
    wc.Mr = (double)mr;
    wc.Z1 = (double)z1;
    wc.Z2 = (double)z2;
    wc.L1 = (double)l1;
  }
  // corner links: cells outside the body's range on both axes, within R
  for (int y = y0 - R; y < y1 + R; ++y)
    for (int x = x0 - R; x < x1 + R; ++x)
      if (!in_body(p, x, y) && face_of(x, y) < 0) add_cell(x, y, -1);
  cells.assign_patterns();
  t->fstatic[0] = (double)sx;
  t->fstatic[1] = (double)sy;
  t->kladd[0] = (double)kx;
  t->kladd[1] = (double)ky;
}

void build_force_tables(const lbm_params* p, const HostLattice& L, const Layout& lay,
                        ForceTables* t) {
  if (diffuse_box(p)) {
    build_wall_tables(p, L, lay, t);
    return;
  }
  long double sx = 0, sy = 0, kx = 0, ky = 0;
  // diffuse or Maxwell wall: a share sigma of every arrival is the diffuse
  // emission, the rest the specular image of a crossing population (the
  // same v_x): shear sees sigma of the reflected deviations, the normal
  // force 2 - sigma of them
  const bool diffuse = p->wall == LBM_WALL_DS || p->wall == LBM_WALL_MAXWELL;
  const long double sigma = p->wall == LBM_WALL_MAXWELL ? (long double)p->accommodation : 1.0L;
  const long double mwx = diffuse ? sigma : 2.0L, mwy = diffuse ? 2.0L - sigma : 2.0L;
  CellTable cells(p, L.R, lay, t);
  std::unordered_map<std::string, int32_t> lpat;
  int x0 = 0, x1 = 0, y0 = 0, y1 = 0;
  if (p->geometry == LBM_GEOM_PLATE) {
    x0 = 0; x1 = p->nx; y0 = 0; y1 = std::min(L.R, p->ny);
  } else if (p->geometry == LBM_GEOM_BOX) {
    x0 = p->box_x0 - L.R; x1 = p->box_x0 + p->box_lx + L.R;
    y0 = p->box_y0 - L.R; y1 = p->box_y0 + p->box_ly + L.R;
  }
  for (int y = y0; y < y1; ++y)
    for (int x = x0; x < x1; ++x) {
      if (in_body(p, x, y)) continue;
      for (int q = 0; q < L.Q; ++q) {
        if (!is_link(p, L, x, y, q)) continue;
        const long double w = L.lw.w_orbit_ld[L.orbit[q]];
        const int vx = L.vx[q], vy = L.vy[q];
        sx -= vx * 2.0L * w * p->rho0;
        sy -= vy * 2.0L * w * p->rho0;
        if (!diffuse) {
          kx -= vx * 2.0L * w * p->rho0 * vx / L.lw.theta_ld;
          ky -= vy * 2.0L * w * p->rho0 * vx / L.lw.theta_ld;
        }
        int px, py;
        mirror_of(p, L, x, y, q, &px, &py);
        const LinkWeights lwt{(double)(-mwx * vx), (double)(-mwy * vy), diffuse ? 1.0 : 0.0,
                              0.0};
        t->links.push_back(ForceLink{L.opp[q] * lay.qs + py * lay.ys + px,
                                     CellTable::pattern(lpat, t->lweights, lwt), 0});
        if (lay.mom) {
          CellWeights& fc = cells.at(px, py);
          // basis of the opposite direction -v at the mirror cell
          const long double g[6] = {1, -(long double)vx, -(long double)vy,
                                    (long double)vx * vx, (long double)vx * vy,
                                    (long double)vy * vy};
          for (int k = 0; k < 6; ++k) {
            fc.wx[k] += (double)(-mwx * vx * w * g[k]);
            fc.wy[k] += (double)(-mwy * vy * w * g[k]);
            if (diffuse) fc.wm[k] += (double)(w * g[k]);
          }
        }
      }
    }
  cells.assign_patterns();
  t->fstatic[0] = (double)sx;
  t->fstatic[1] = (double)sy;
  t->kladd[0] = (double)kx;
  t->kladd[1] = (double)ky;
  if (diffuse) {
    // lattice sums over the directions the wall emits (v_y > 0)
    const long double th = L.lw.theta_ld;
    long double a1 = 0, a2 = 0, bx = 0, by0 = 0, by2 = 0;
    for (int q = 0; q < L.Q; ++q) {
      if (L.vy[q] <= 0) continue;
      const long double w = L.lw.w_orbit_ld[L.orbit[q]];
      const long double vx = L.vx[q], vy = L.vy[q];
      const long double e2 = vx * vx / (2 * th * th) - 1 / (2 * th);
      a1 += vy * w;
      a2 += vy * w * e2;
      bx += vy * vx * vx * w / th;
      by0 += vy * vy * w;
      by2 += vy * vy * w * e2;
    }
    t->ds[0] = (double)a1;
    t->ds[1] = (double)a2;
    t->ds[2] = (double)bx;
    t->ds[3] = (double)by0;
    t->ds[4] = (double)by2;
    t->ds[5] = (double)((long double)p->nx * p->rho0);
  }
}

// The layout, and the force tables whose sizes it holds.
void make_layout(const lbm_params* p, const HostLattice& L, Layout* lay, ForceTables* tables) {
  const uint64_t es = p->storage == LBM_STORE_F64 ? 8 : 4;
  if (p->nx >= 64) {
    // row-interleaved: the Q rows of lattice row y are contiguous, so the Q
    // streams of a workgroup touch a few contiguous rows of Q*pitch elements
    lay->pitch = (int64_t)align_up(p->nx, 64);
    lay->qs = lay->pitch;
    lay->ys = (int64_t)L.Q * lay->pitch;
    lay->buf_elems = lay->ys * p->ny;
  } else {
    // narrow lattices: whole-lattice planes (a wavefront covers several rows
    // of one plane contiguously); planes start 256 elements past a
    // 256-element boundary apart to spread them over HBM channels
    lay->pitch = p->nx;
    lay->qs = (int64_t)align_up((uint64_t)p->ny * lay->pitch, 256) + 256;
    lay->ys = lay->pitch;
    lay->buf_elems = lay->qs * L.Q;
  }
  lay->mom = uses_coefficients(p);
  lay->column = uses_columns(p);
  lay->loadable = !(lay->mom && p->representation == LBM_REPR_COEFFICIENTS_NOLOAD);
  if (lay->mom) {
    lay->coef_k = p->tile ? (int32_t)p->tile : kCoefKDefault;
    lay->launch_k = coef_k_for(p->tile, es == 8, coef_cells(p));
    // element (k, y, x) of a buffer at k*mks + y*mpitch + x.  Row-interleaved
    // where the whole buffer stays addressable with 32-bit byte offsets: the
    // six coefficient rows of lattice row y side by side, so the staged rows
    // and the stores of a tile fall in one contiguous span (2 % faster on a
    // state streaming from HBM than six whole planes).  Larger lattices keep
    // six planes, each under 2 GiB, spaced 256 elements past a 256-element
    // boundary.
    const int64_t pitch = (int64_t)align_up(p->nx, 64);
    if ((uint64_t)p->ny * 6 * (uint64_t)pitch * es < ((uint64_t)1 << 31)) {
      lay->mpitch = 6 * pitch;
      lay->mks = pitch;
      lay->mbuf_bytes = ((uint64_t)align_up((uint64_t)p->ny * lay->mpitch, 256) + 256) * es;
    } else {
      lay->mpitch = pitch;
      lay->mks = (int64_t)align_up((uint64_t)p->ny * pitch, 256) + 256;
      lay->mbuf_bytes = 6 * (uint64_t)lay->mks * es;
    }
  }
  // the coefficient solver's population kernel (first step after a load)
  // runs with one cell per thread
  lay->cpt = lay->mom ? 1 : (p->tile ? (int32_t)p->tile : 1);
  lay->cells_per_tile = kBlock * lay->cpt;
  // rows padded to the pitch, so that every wavefront covers an aligned segment
  // of one row (641 x 1000 BGK FP32: 40.3 us per step against 49.2 with 256
  // consecutive cells per workgroup, both with nontemporal stores), unless a
  // fifth or more of the lanes would idle
  lay->mw = lay->pitch * 4 <= (int64_t)p->nx * 5 ? (int32_t)lay->pitch : p->nx;
  const int64_t mapped = (int64_t)lay->mw * p->ny;
  lay->ntiles = (int32_t)((mapped + lay->cells_per_tile - 1) / lay->cells_per_tile);
  lay->hist_cap = p->history_capacity ? p->history_capacity : p->max_steps;
  uint64_t o = 0;
  auto take = [&](uint64_t bytes) {
    uint64_t at = o;
    o = align_up(o + std::max<uint64_t>(bytes, 1), kAlign);
    return at;
  };
  lay->off_desc = take(sizeof(SolveDesc));
  lay->off_state = take(sizeof(SolveState));
  // the force's item and padding, then the XCD-aware order, which pads each
  // group of 8 rows to full length
  // (none for the column kernel, which needs no list and sums the force itself)
  lay->nwork = lay->column ? 0
                           : 8 + (int32_t)ordered_length(
                                     lay->ntiles, (lay->mw + lay->cells_per_tile - 1) /
                                                      lay->cells_per_tile);
  lay->off_work = take(sizeof(WorkItem) * (uint64_t)lay->nwork);
  if (lay->mom) {
    int64_t nfront = 1;  // the force's item and the wall tiles
    for (char w : coef_wall_tiles(p, lay->launch_k, L.R)) nfront += w;
    const CoefGrid g = coef_grid(p, lay->launch_k);
    lay->mnwork = (int32_t)((nfront + 7) / 8 * 8 + ordered_length(g.ntiles, g.tiles_x));
    lay->off_mwork = take(sizeof(WorkItem) * (uint64_t)lay->mnwork);
  }
  lay->off_solves = take(sizeof(int32_t));
  ForceTables& ft = *tables;
  build_force_tables(p, L, *lay, &ft);
  if (lay->column) {
    lay->unused_bytes = (int64_t)(sizeof(ForceLink) * ft.links.size() +
                                  sizeof(LinkWeights) * ft.lweights.size());
    ft.links.clear();
    ft.lweights.clear();
  }
  lay->nlinks = (int32_t)ft.links.size();
  lay->nfcells = (int32_t)ft.cells.size();
  lay->off_links = take(sizeof(ForceLink) * ft.links.size());
  lay->off_fcells = take(sizeof(ForceCell) * ft.cells.size());
  lay->nlweights = (int32_t)ft.lweights.size();
  lay->ncweights = (int32_t)ft.cweights.size();
  lay->off_lweights = take(sizeof(LinkWeights) * ft.lweights.size());
  lay->off_cweights = take(sizeof(CellWeights) * ft.cweights.size());
  lay->nwcols = (int32_t)ft.wcols.size();
  lay->nwlinks = (int32_t)ft.wlinks.size();
  lay->off_wcols = take(sizeof(WallCol) * ft.wcols.size());
  lay->off_wlinks = take(sizeof(WallLink) * ft.wlinks.size());
  lay->off_drive = take(sizeof(Drive) * (uint64_t)p->max_steps);
  lay->off_hist = take(sizeof(double) * 2 * (uint64_t)lay->hist_cap);
  // a coefficient solver that cannot load populations has no population buffer
  lay->buf_bytes = lay->loadable ? (uint64_t)lay->buf_elems * es : 0;
  o = align_up(o, 4096);
  lay->off_buf[0] = lay->loadable ? take(lay->buf_bytes) : 0;
  if (lay->mom) {
    // one population buffer (a loaded state, read by the next step; none
    // without loads) and two coefficient buffers
    lay->off_buf[1] = lay->off_buf[0];
    o = align_up(o, 4096);
    lay->off_mbuf[0] = take(lay->mbuf_bytes);
    o = align_up(o, 4096);
    lay->off_mbuf[1] = take(lay->mbuf_bytes);
  } else {
    o = align_up(o, 4096);
    lay->off_buf[1] = take(lay->buf_bytes);
  }
  lay->total = o;
}


}  // namespace

namespace {

int init_solver(lbm_solver* s, const ForceTables& ft) {
  const lbm_params* p = &s->p;
  const Layout& lay = s->lay;
  char* b = s->base;

  SolveDesc& d = s->desc;
  std::memset(&d, 0, sizeof(d));
  if (lay.loadable) {
    s->bufs[0] = d.buf[0] = b + lay.off_buf[0];
    s->bufs[1] = d.buf[1] = b + lay.off_buf[1];
  }
  d.drive = reinterpret_cast<const Drive*>(b + lay.off_drive);
  d.hist = reinterpret_cast<double*>(b + lay.off_hist);
  d.state = reinterpret_cast<SolveState*>(b + lay.off_state);
  d.links = reinterpret_cast<const ForceLink*>(b + lay.off_links);
  d.fcells = reinterpret_cast<const ForceCell*>(b + lay.off_fcells);
  d.lweights = reinterpret_cast<const LinkWeights*>(b + lay.off_lweights);
  d.cweights = reinterpret_cast<const CellWeights*>(b + lay.off_cweights);
  d.nlinks = lay.nlinks;
  if (lay.nwlinks > 0) {
    d.wcols = reinterpret_cast<const WallCol*>(b + lay.off_wcols);
    d.wlinks = reinterpret_cast<const WallLink*>(b + lay.off_wlinks);
    d.nwcols = lay.nwcols;
    d.nwlinks = lay.nwlinks;
  }
  d.theta = s->lat.lw.theta;
  d.nfcells = lay.nfcells;
  d.qs = lay.qs;
  d.ys = lay.ys;
  d.max_steps = p->max_steps;
  d.hist_cap = lay.hist_cap;
  d.lockin_first = p->lockin_first;
  d.lockin_count = p->lockin_count;
  d.nx = p->nx;
  d.ny = p->ny;
  d.mw = lay.mw;
  d.geom = (int32_t)p->geometry;
  d.far = (int32_t)p->far;
  if (p->geometry == LBM_GEOM_BOX) {
    d.bx0 = p->box_x0;
    d.by0 = p->box_y0;
    d.bx1 = p->box_x0 + p->box_lx;
    d.by1 = p->box_y0 + p->box_ly;
  }
  d.inv_tau = std::isinf(p->tau) ? 0.0 : 1.0 / p->tau;
  d.rho0 = p->rho0;
  d.ladd_scale = 2.0 * p->rho0 / s->lat.lw.theta;
  d.fstatic[0] = ft.fstatic[0];
  d.fstatic[1] = ft.fstatic[1];
  d.kladd[0] = ft.kladd[0];
  d.kladd[1] = ft.kladd[1];
  d.wall = p->wall == LBM_WALL_BB ? WALL_BB : WALL_DS;
  d.sigma = p->wall == LBM_WALL_MAXWELL ? p->accommodation : 1.0;
  for (int k = 0; k < 6; ++k) d.ds[k] = ft.ds[k];
  if (lay.mom) {
    d.mbuf[0] = b + lay.off_mbuf[0];
    d.mbuf[1] = b + lay.off_mbuf[1];
    d.mks = lay.mks;
    d.mys = lay.mpitch;
    d.tiles_x = coef_grid(p, lay.launch_k).tiles_x;
  }

  for (int k = 0; k < 8; ++k) s->klat.w[k] = s->lat.lw.w_orbit[k];
  s->klat.theta = s->lat.lw.theta;

  std::vector<WorkItem> work, mwork, rest;
  if (lay.nwork > 0) {
    work.push_back(WorkItem{0, kForceTile});
    order_tiles(&rest, 0, lay.ntiles, (lay.mw + lay.cells_per_tile - 1) / lay.cells_per_tile);
    join_front(&work, rest);
  }
  if (lay.mom) {
    const CoefGrid g = coef_grid(p, lay.launch_k);
    mwork.push_back(WorkItem{0, kForceTile});
    rest.clear();
    order_coef_tiles(&mwork, &rest, 0, coef_wall_tiles(p, lay.launch_k, s->lat.R), g.ntiles,
                     g.tiles_x, 2 * lay.mbuf_bytes <= kCachedStateBytes);
    join_front(&mwork, rest);
    if ((int32_t)mwork.size() != lay.mnwork) return LBM_EINVAL;
  }
  std::vector<Drive> drive((size_t)p->max_steps);
  for (int64_t n = 0; n < p->max_steps; ++n) {
    const double arg = p->omega * ((double)n + 0.5);
    drive[n].u = p->u0 * std::sin(arg);
    drive[n].s = std::sin(arg);
    drive[n].c = std::cos(arg);
  }
  const int32_t solve0 = 0;
  s->d_desc = reinterpret_cast<SolveDesc*>(b + lay.off_desc);
  s->d_work = reinterpret_cast<WorkItem*>(b + lay.off_work);
  s->d_solves = reinterpret_cast<int32_t*>(b + lay.off_solves);
  s->d_mwork = lay.mom ? reinterpret_cast<WorkItem*>(b + lay.off_mwork) : nullptr;

  hipStream_t st = s->stream;
  int rc;
  if ((rc = hip_rc(hipMemcpyAsync(s->d_desc, &d, sizeof(d), hipMemcpyHostToDevice, st)))) return rc;
  if (!work.empty() &&
      (rc = hip_rc(hipMemcpyAsync(s->d_work, work.data(), sizeof(WorkItem) * work.size(),
                                  hipMemcpyHostToDevice, st))))
    return rc;
  if ((rc = hip_rc(hipMemcpyAsync(s->d_solves, &solve0, sizeof(solve0), hipMemcpyHostToDevice,
                                  st))))
    return rc;
  if (!ft.links.empty() &&
      (rc = hip_rc(hipMemcpyAsync(b + lay.off_links, ft.links.data(),
                                  sizeof(ForceLink) * ft.links.size(), hipMemcpyHostToDevice, st))))
    return rc;
  if (!ft.cells.empty() &&
      (rc = hip_rc(hipMemcpyAsync(b + lay.off_fcells, ft.cells.data(),
                                  sizeof(ForceCell) * ft.cells.size(), hipMemcpyHostToDevice, st))))
    return rc;
  if (!ft.lweights.empty() &&
      (rc = hip_rc(hipMemcpyAsync(b + lay.off_lweights, ft.lweights.data(),
                                  sizeof(LinkWeights) * ft.lweights.size(), hipMemcpyHostToDevice,
                                  st))))
    return rc;
  if (!ft.cweights.empty() &&
      (rc = hip_rc(hipMemcpyAsync(b + lay.off_cweights, ft.cweights.data(),
                                  sizeof(CellWeights) * ft.cweights.size(), hipMemcpyHostToDevice,
                                  st))))
    return rc;
  if (!ft.wcols.empty() &&
      (rc = hip_rc(hipMemcpyAsync(b + lay.off_wcols, ft.wcols.data(),
                                  sizeof(WallCol) * ft.wcols.size(), hipMemcpyHostToDevice, st))))
    return rc;
  if (!ft.wlinks.empty() &&
      (rc = hip_rc(hipMemcpyAsync(b + lay.off_wlinks, ft.wlinks.data(),
                                  sizeof(WallLink) * ft.wlinks.size(), hipMemcpyHostToDevice,
                                  st))))
    return rc;
  if ((rc = hip_rc(hipMemcpyAsync(b + lay.off_drive, drive.data(), sizeof(Drive) * drive.size(),
                                  hipMemcpyHostToDevice, st))))
    return rc;
  if (lay.mom) {
    if ((rc = hip_rc(hipMemcpyAsync(s->d_mwork, mwork.data(), sizeof(WorkItem) * mwork.size(),
                                    hipMemcpyHostToDevice, st))))
      return rc;

    if ((rc = hip_rc(hipMemsetAsync(b + lay.off_mbuf[0], 0, lay.mbuf_bytes, st)))) return rc;
    if ((rc = hip_rc(hipMemsetAsync(b + lay.off_mbuf[1], 0, lay.mbuf_bytes, st)))) return rc;
  }
  // rest state (zero deviations), zero counters, sums and history
  if ((rc = hip_rc(hipMemsetAsync(b + lay.off_state, 0, sizeof(SolveState), st)))) return rc;

  if ((rc = hip_rc(hipMemsetAsync(b + lay.off_hist, 0, sizeof(double) * 2 * lay.hist_cap, st))))
    return rc;
  if (lay.loadable && (rc = hip_rc(hipMemsetAsync(b + lay.off_buf[0], 0, lay.buf_bytes, st))))
    return rc;
  if (!lay.mom && (rc = hip_rc(hipMemsetAsync(b + lay.off_buf[1], 0, lay.buf_bytes, st))))
    return rc;
  return hip_rc(hipStreamSynchronize(st));
}

}  // namespace

int lbm::create_solver(const lbm_params* p, void* stream, void* dev_buf, uint64_t bytes,
                       bool graphs, lbm_solver** out) {
  if (!out) return LBM_EINVAL;
  *out = nullptr;
  lbm_solver* s = new (std::nothrow) lbm_solver();
  if (!s) return LBM_ENOMEM;
  int rc = validate(p, &s->lat);
  if (rc) {
    delete s;
    return rc;
  }
  s->p = *p;
  ForceTables tables;
  make_layout(p, s->lat, &s->lay, &tables);
  s->stream = static_cast<hipStream_t>(stream);
  if (hipGetDevice(&s->device) != hipSuccess) {
    delete s;
    return LBM_EHIP;
  }
  if (dev_buf) {
    if (bytes < s->lay.total || (reinterpret_cast<uintptr_t>(dev_buf) % kAlign) != 0) {
      delete s;
      return bytes < s->lay.total ? LBM_ENOMEM : LBM_EINVAL;
    }
    s->base = static_cast<char*>(dev_buf);
  } else {
    void* ptr = nullptr;
    if (hipMalloc(&ptr, s->lay.total) != hipSuccess) {
      (void)hipGetLastError();
      delete s;
      return LBM_ENOMEM;
    }
    s->base = static_cast<char*>(ptr);
    s->owned = true;
  }
  s->graphs_ok = graphs;
  if (s->lay.column)
    s->column = column_plan((int)p->lattice, p->storage == LBM_STORE_F64, p->nx, {p->ny});
  rc = init_solver(s, tables);
  if (rc) {
    if (s->owned) (void)hipFree(s->base);
    delete s;
    return rc;
  }
  readout_users(1);
  *out = s;
  return LBM_OK;
}

// One step of a single solver: the population kernel, the population kernel
// writing coefficients (first step after populations were loaded into a
// coefficient solver), or the coefficient kernel.
namespace {

// Enqueue one step's launch, dn steps after the last advance of the counter.
int launch_one_step(lbm_solver* s, int dn) {
  const bool f64 = s->p.storage == LBM_STORE_F64;
  const bool bgk = s->p.collision == LBM_COLL_BGK;
  const int Q = (int)s->p.lattice;
  const bool ds = s->p.wall != LBM_WALL_BB;
  hipError_t e;
  if (!s->lay.mom) {
    e = launch_step(Q, f64, bgk, ds, s->lay.cpt, false, s->d_desc, s->d_work, s->lay.nwork,
                    s->klat, dn, 2 * s->lay.buf_bytes > kCachedPopBytes, s->stream);
  } else if (s->pop_pending) {
    e = launch_step(Q, f64, false, ds, 1, true, s->d_desc, s->d_work, s->lay.nwork, s->klat, dn,
                    false, s->stream);
    if (e == hipSuccess) s->pop_pending = false;
  } else {
    e = launch_coef(Q, f64, s->lay.launch_k, ds, 2 * s->lay.mbuf_bytes > kCachedStateBytes,
                    s->d_desc, s->d_mwork, s->lay.mnwork, s->klat, dn, s->stream);
  }
  return e == hipSuccess ? LBM_OK : LBM_EHIP;
}

// Enqueue the launches of n steps; *done: how many were (less than n after a
// failure), the device's counter advanced by as many.
int launch_steps(lbm_solver* s, int64_t n, int64_t* done) {
  const bool f64 = s->p.storage == LBM_STORE_F64;
  const int Q = (int)s->p.lattice, rows = s->column.rows;
  *done = 0;
  while (*done < n) {
    // one advance of the step counter for all the launches of a block
    const int block = (int)std::min<int64_t>(n - *done, kStepBlock);
    int rc = LBM_OK, k = 0;
    if (!s->lay.column)
      for (; k < block && !(rc = launch_one_step(s, k)); ++k) {
      }
    else
      for (int nsub : odd_pieces(block, s->column.max_sub)) {
        const bool bgk = s->p.collision == LBM_COLL_BGK, ds = s->p.wall != LBM_WALL_BB;
        const hipError_t e =
            nsub == 1 && column_single(Q, f64, s->column, ds)
                ? launch_column_single(Q, f64, bgk, ds, s->d_desc, nullptr,
                                       column_single_items(s->p.nx, s->p.ny), s->klat, k,
                                       2 * s->lay.buf_bytes > kCachedPopBytes, s->stream)
                : launch_column(Q, f64, bgk, ds, column_shape(Q, s->p.nx, rows, nsub), s->d_desc,
                                nullptr, (s->p.ny + rows - 1) / rows, s->klat, k, s->stream);
        if (e != hipSuccess) {
          rc = LBM_EHIP;
          break;
        }
        k += nsub;
      }
    if (launch_advance(s->d_desc, s->d_solves, 1, k, s->stream) != hipSuccess) return LBM_EHIP;
    *done += k;
    if (rc) return rc;
  }
  return LBM_OK;
}

// Capture kGraphSteps steps of a solver whose state is in its steady
// representation (no pending population load).
bool capture_steps(lbm_solver* s) {
  if (s->stream == nullptr || s->pop_pending) return false;  // the null stream cannot be captured
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(s->stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  int64_t done;
  const bool ok = launch_steps(s, kGraphSteps, &done) == LBM_OK;
  if (hipStreamEndCapture(s->stream, &g) != hipSuccess || !ok) {
    (void)hipGetLastError();
    if (g) (void)hipGraphDestroy(g);
    return false;
  }
  hipGraphExec_t ex = nullptr;
  const bool inst = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) == hipSuccess;
  (void)hipGraphDestroy(g);
  if (!inst) {
    (void)hipGetLastError();
    return false;
  }
  s->graph = ex;
  return true;
}

}  // namespace

int step_one(lbm_solver* s) {
  int64_t done;
  const int rc = launch_steps(s, 1, &done);
  s->steps += done;
  return rc;
}

namespace {

// fn(y0, y1) over the rows [0, ny), by up to 8 threads where the `row` values
// per row make that worth their start.
template <class F>
void host_rows(int ny, size_t row, F&& fn) {
  const size_t most = std::min<size_t>(8, std::max(1u, std::thread::hardware_concurrency()));
  const int n = (int)std::min<size_t>({most, (size_t)ny, 1 + row * ny / (1 << 18)});
  std::vector<std::thread> team;
  int y = 0;
  try {
    team.reserve((size_t)n);
    for (int i = 0; i + 1 < n; ++i) {
      const int y1 = (int)((int64_t)ny * (i + 1) / n);
      team.emplace_back([&fn, y, y1] { fn(y, y1); });
      y = y1;
    }
  } catch (...) {
    // fewer threads than wanted: the rest of the rows here
  }
  fn(y, ny);
  for (std::thread& t : team) t.join();
}

// Wait for the solver's work and read its flag, and the lock-in sums and
// `count` force samples from step `first` into `force` (pairs) if wanted.
int sync_and_check(lbm_solver* s, double lockin[6] = nullptr, int64_t first = 0,
                   int64_t count = 0, double* force = nullptr) {
  int32_t flag = 0;
  const int small = (int)std::min<int64_t>(count, kReadoutSamples);
  int rc = read_out(s->d_desc, s->device, s->stream, first, small, &flag, lockin, force);
  int64_t done = small;
  if (rc == LBM_ENOMEM) {
    // no pinned memory: a wait and copies
    SolveState st;
    if (hipStreamSynchronize(s->stream) != hipSuccess ||
        hipMemcpy(&st, s->desc.state, sizeof(st), hipMemcpyDeviceToHost) != hipSuccess)
      return LBM_EHIP;
    flag = st.unstable;
    if (lockin) std::memcpy(lockin, st.lockin, sizeof(st.lockin));
    done = 0;
    rc = LBM_OK;
  }
  if (rc) return rc;
  const int64_t cap = s->lay.hist_cap;
  while (done < count) {
    const int64_t h = (first + done) % cap;
    const int64_t run = std::min(count - done, cap - h);
    if (hipMemcpy(force + 2 * done, s->desc.hist + 2 * h, sizeof(double) * 2 * run,
                  hipMemcpyDeviceToHost) != hipSuccess)
      return LBM_EHIP;
    done += run;
  }
  if (flag) s->sticky_unstable = true;
  return s->sticky_unstable ? LBM_EUNSTABLE : LBM_OK;
}

}  // namespace

namespace lbm {

int required_bytes(const lbm_params* p, uint64_t* bytes, int64_t* beyond) {
  if (!bytes) return LBM_EINVAL;
  HostLattice lat;
  int rc = validate(p, &lat);
  if (rc) return rc;
  Layout lay;
  ForceTables tables;
  make_layout(p, lat, &lay, &tables);
  *bytes = lay.total;
  if (!beyond) return LBM_OK;
  // the same lists over plain cells and with the default K, wall tiles aside
  const int64_t cells = (int64_t)p->nx * p->ny, per = lay.cells_per_tile;
  int64_t items = lay.nwork - ordered_length((cells + per - 1) / per, (p->nx + per - 1) / per);
  if (lay.mom) {
    const CoefGrid g = coef_grid(p, lay.coef_k);
    items += lay.mnwork - ordered_length(g.ntiles, g.tiles_x);
  }
  const int64_t force_cells =
      diffuse_box(p) && lay.mom
          ? (int64_t)sizeof(ForceCell) * lay.nfcells + (int64_t)sizeof(CellWeights) * lay.ncweights
          : 0;
  // (a kAlign for the rounding of each)
  *beyond = items * (int64_t)sizeof(WorkItem) + force_cells - lay.unused_bytes +
            4 * (int64_t)kAlign;
  return LBM_OK;
}

}  // namespace lbm

extern "C" {

int lbm_params_init(lbm_params* p) {
  if (!p) return LBM_EINVAL;
  std::memset(p, 0, sizeof(*p));
  p->abi_version = LBM_ABI_VERSION;
  p->lattice = LBM_D2Q37;
  p->storage = LBM_STORE_F32_DEV;
  p->collision = LBM_COLL_REGULARIZED;
  p->wall = LBM_WALL_BB;
  p->accommodation = 1.0;
  p->geometry = LBM_GEOM_PLATE;
  p->far = LBM_FAR_WALL;
  p->rho0 = 1.0;
  return LBM_OK;
}

int lbm_lattice(int Q, int32_t* vx, int32_t* vy, double* w, double* theta) {
  HostLattice h;
  if (!host_lattice(Q, &h)) return LBM_EINVAL;
  for (int i = 0; i < Q; ++i) {
    if (vx) vx[i] = h.vx[i];
    if (vy) vy[i] = h.vy[i];
    if (w) w[i] = h.lw.w_orbit[h.orbit[i]];
  }
  if (theta) *theta = h.lw.theta;
  return LBM_OK;
}

int lbm_required_bytes(const lbm_params* p, uint64_t* bytes) {
  return lbm::required_bytes(p, bytes, nullptr);
}

int lbm_create(const lbm_params* p, void* hip_stream, lbm_solver** out) {
  return create_solver(p, hip_stream, nullptr, 0, true, out);
}

int lbm_create_in(const lbm_params* p, void* hip_stream, void* dev_buf, uint64_t bytes,
                  lbm_solver** out) {
  if (!dev_buf) return LBM_EINVAL;
  return create_solver(p, hip_stream, dev_buf, bytes, true, out);
}

int lbm_step(lbm_solver* s, int64_t nsteps) {
  if (!s || nsteps < 0) return LBM_EINVAL;
  if (s->steps + nsteps > s->p.max_steps) return LBM_ERANGE;
  int64_t k = 0;
  // a coefficient solver whose state was loaded as populations converts it
  // in its first step (another kernel than the steady one)
  if (s->pop_pending && k < nsteps) {
    int rc = step_one(s);
    if (rc) return rc;
    ++k;
  }
  // steady chunks replay one captured graph
  // (not of the column kernel: its launches of several steps keep the device
  // busy without, and one advance of the counter serves them all)
  if (nsteps - k >= kGraphSteps && s->graphs_ok && !s->lay.column && !s->graph &&
      !capture_steps(s))
    s->graphs_ok = false;
  for (; s->graph && k + kGraphSteps <= nsteps; k += kGraphSteps) {
    if (hipGraphLaunch(s->graph, s->stream) != hipSuccess) return LBM_EHIP;
    s->steps += kGraphSteps;
  }
  if (k < nsteps) {
    int64_t done;
    const int rc = launch_steps(s, nsteps - k, &done);
    s->steps += done;
    return rc;
  }
  return LBM_OK;
}

int lbm_synchronize(lbm_solver* s) {
  if (!s) return LBM_EINVAL;
  return sync_and_check(s);
}

int lbm_representation(const lbm_solver* s, int* repr) {
  if (!s || !repr) return LBM_EINVAL;
  *repr = s->lay.mom ? LBM_REPR_COEFFICIENTS : LBM_REPR_POPULATIONS;
  return LBM_OK;
}

int lbm_steps_done(const lbm_solver* s, int64_t* n) {
  if (!s || !n) return LBM_EINVAL;
  *n = s->steps;
  return LBM_OK;
}

int lbm_force_history(lbm_solver* s, int64_t first, int64_t count, double* fx, double* fy) {
  if (!s || first < 0 || count < 0) return LBM_EINVAL;
  const int64_t cap = s->lay.hist_cap;
  if (first + count > s->steps || first < std::max(s->hist_from, s->steps - std::min(s->steps, cap)))
    return LBM_ERANGE;
  std::vector<double> tmp((size_t)count * 2);
  const int rc = sync_and_check(s, nullptr, first, count, tmp.data());
  if (rc && rc != LBM_EUNSTABLE) return rc;
  for (int64_t i = 0; i < count; ++i) {
    if (fx) fx[i] = tmp[2 * i];
    if (fy) fy[i] = tmp[2 * i + 1];
  }
  return rc;
}

int lbm_lockin(lbm_solver* s, double sums[6], int64_t* nsamples) {
  if (!s || !sums) return LBM_EINVAL;
  const int rc = sync_and_check(s, sums);
  if (rc && rc != LBM_EUNSTABLE) return rc;
  if (nsamples)
    *nsamples = std::max<int64_t>(
        0, std::min(s->steps, s->p.lockin_first + s->p.lockin_count) - s->p.lockin_first);
  return rc;
}

int lbm_impedance(lbm_solver* s, double out[5]) {
  if (!s || !out) return LBM_EINVAL;
  double sums[6];
  int64_t ns = 0;
  int rc = lbm_lockin(s, sums, &ns);
  if (rc && rc != LBM_EUNSTABLE) return rc;
  if (ns < 3) return LBM_ERANGE;
  // normal equations of F ~ a sin + b cos + c with the drive table's basis
  long double G[3][4] = {{0}};
  for (int64_t n = s->p.lockin_first; n < s->p.lockin_first + ns; ++n) {
    const double arg = s->p.omega * ((double)n + 0.5);
    const long double b[3] = {std::sin(arg), std::cos(arg), 1.0L};
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) G[r][c] += b[r] * b[c];
  }
  G[0][3] = sums[0];
  G[1][3] = sums[1];
  G[2][3] = sums[2];
  for (int c = 0; c < 3; ++c) {
    int piv = c;
    for (int r = c + 1; r < 3; ++r)
      if (std::fabs(G[r][c]) > std::fabs(G[piv][c])) piv = r;
    if (G[piv][c] == 0) return LBM_ERANGE;
    for (int k = 0; k < 4; ++k) std::swap(G[c][k], G[piv][k]);
    for (int r = 0; r < 3; ++r) {
      if (r == c) continue;
      const long double m = G[r][c] / G[c][c];
      for (int k = c; k < 4; ++k) G[r][k] -= m * G[c][k];
    }
  }
  const long double a = G[0][3] / G[0][0], b = G[1][3] / G[1][1], c = G[2][3] / G[2][2];
  out[0] = (double)a;
  out[1] = (double)b;
  out[2] = (double)c;
  out[3] = (double)(-a / s->p.u0);
  out[4] = (double)(-b / s->p.u0);
  return rc;
}

namespace {

// Copy the current state out as FP64 [q][y][x] populations; with_rest adds
// w_i rho0.  A coefficient state is expanded to populations
// w_i (a0 + vx bx + vy by + vx^2 cxx + vx vy cxy + vy^2 cyy).
int copy_out(lbm_solver* s, double* host, uint64_t n, bool with_rest) {
  if (!s || !host) return LBM_EINVAL;
  const lbm_params& p = s->p;
  const HostLattice& L = s->lat;
  const int Q = L.Q;
  if (n != (uint64_t)Q * p.ny * p.nx) return LBM_EINVAL;
  if (hipStreamSynchronize(s->stream) != hipSuccess) return LBM_EHIP;
  const bool f64 = p.storage == LBM_STORE_F64;
  const bool coeffs = s->lay.mom && !s->pop_pending;
  const uint64_t bytes = coeffs ? s->lay.mbuf_bytes : s->lay.buf_bytes;
  const void* src = coeffs ? s->desc.mbuf[s->steps & 1] : s->bufs[s->steps & 1];
  std::unique_ptr<char[]> stage(new (std::nothrow) char[bytes]);
  if (!stage) return LBM_ENOMEM;
  if (hipMemcpy(stage.get(), src, bytes, hipMemcpyDeviceToHost) != hipSuccess) return LBM_EHIP;
  auto rows = [&](const auto* buf, int y0, int y1) {
    for (int y = y0; y < y1; ++y)
      for (int q = 0; q < Q; ++q) {
        const double w = L.lw.w_orbit[L.orbit[q]];
        const double wr = with_rest ? w * p.rho0 : 0.0;
        double* out = host + ((size_t)q * p.ny + y) * p.nx;
        if (coeffs) {
          const double vx = L.vx[q], vy = L.vy[q];
          const double xx = vx * vx, xy = vx * vy, yy = vy * vy;
          const int64_t ks = s->lay.mks;
          const auto* c = buf + y * s->lay.mpitch;
          for (int x = 0; x < p.nx; ++x)
            out[x] = wr + w * ((double)c[x] + vx * (double)c[ks + x] + vy * (double)c[2 * ks + x] +
                               xx * (double)c[3 * ks + x] + xy * (double)c[4 * ks + x] +
                               yy * (double)c[5 * ks + x]);
        } else {
          const auto* f = buf + q * s->lay.qs + y * s->lay.ys;
          for (int x = 0; x < p.nx; ++x) out[x] = wr + (double)f[x];
        }
        if (in_body(&p, p.box_x0, y)) std::fill_n(out + p.box_x0, p.box_lx, 0.0);
      }
  };
  host_rows(p.ny, (size_t)Q * p.nx, [&](int y0, int y1) {
    if (f64) rows(reinterpret_cast<const double*>(stage.get()), y0, y1);
    else rows(reinterpret_cast<const float*>(stage.get()), y0, y1);
  });
  return LBM_OK;
}

// Copy FP64 [q][y][x] into the current population buffer; with_rest
// subtracts w_i rho0.  A coefficient solver reads it in its next step.
int copy_in(lbm_solver* s, const double* host, uint64_t n, bool with_rest) {
  if (!s || !host) return LBM_EINVAL;
  const lbm_params& p = s->p;
  const int Q = s->lat.Q;
  if (n != (uint64_t)Q * p.ny * p.nx) return LBM_EINVAL;
  if (!s->lay.loadable) return LBM_EINVAL;  // no population buffer to load into
  if (hipStreamSynchronize(s->stream) != hipSuccess) return LBM_EHIP;
  const bool f64 = p.storage == LBM_STORE_F64;
  std::unique_ptr<char[]> stage(new (std::nothrow) char[s->lay.buf_bytes]);
  if (!stage) return LBM_ENOMEM;
  // elements after a row of a population: the row's padding, or the gap
  // between two planes (zeros)
  const int64_t qs = s->lay.qs, ys = s->lay.ys;
  auto rows = [&](auto* buf, int y0, int y1) {
    for (int y = y0; y < y1; ++y)
      for (int q = 0; q < Q; ++q) {
        const double wr = with_rest ? s->lat.lw.w_orbit[s->lat.orbit[q]] * p.rho0 : 0.0;
        const double* in = host + ((size_t)q * p.ny + y) * p.nx;
        auto* out = buf + q * qs + y * ys;
        for (int x = 0; x < p.nx; ++x) out[x] = in[x] - wr;
        if (in_body(&p, p.box_x0, y)) std::fill_n(out + p.box_x0, p.box_lx, 0);
        const int64_t gap = ys > qs ? s->lay.pitch - p.nx : y + 1 == p.ny ? qs - p.ny * ys : 0;
        std::fill_n(out + p.nx, gap, 0);
      }
  };
  host_rows(p.ny, (size_t)Q * p.nx, [&](int y0, int y1) {
    if (f64) rows(reinterpret_cast<double*>(stage.get()), y0, y1);
    else rows(reinterpret_cast<float*>(stage.get()), y0, y1);
  });
  if (hipMemcpy(s->bufs[s->steps & 1], stage.get(), s->lay.buf_bytes,
                hipMemcpyHostToDevice) != hipSuccess)
    return LBM_EHIP;
  if (s->lay.mom) s->pop_pending = true;
  return LBM_OK;
}

// Raw state blob: header, then the current buffer.
struct StateHeader {
  uint32_t magic, lattice, storage, coeffs;
  int32_t nx, ny;
  uint64_t bytes;
};
constexpr uint32_t kStateMagic = 0x4c424d32;  // "LBM2": row-interleaved coefficient buffers

uint64_t state_payload(const lbm_solver* s) {
  return (s->lay.mom && !s->pop_pending) ? s->lay.mbuf_bytes : s->lay.buf_bytes;
}

}  // namespace

int lbm_get_populations(lbm_solver* s, double* host, uint64_t n) {
  return copy_out(s, host, n, true);
}

int lbm_set_populations(lbm_solver* s, const double* host, uint64_t n) {
  return copy_in(s, host, n, true);
}

int lbm_get_deviations(lbm_solver* s, double* host, uint64_t n) {
  return copy_out(s, host, n, false);
}

int lbm_set_deviations(lbm_solver* s, const double* host, uint64_t n) {
  return copy_in(s, host, n, false);
}

int lbm_seek(lbm_solver* s, int64_t step, const double lockin_sums[6]) {
  if (!s || step < 0 || step >= s->p.max_steps) return LBM_EINVAL;
  if (hipStreamSynchronize(s->stream) != hipSuccess) return LBM_EHIP;
  if ((step & 1) != (s->steps & 1)) {
    // the current state moves to the buffer that step n reads
    void* const* bufs = s->lay.mom && !s->pop_pending ? s->desc.mbuf : s->bufs;
    if (bufs[step & 1] != bufs[s->steps & 1] &&
        hipMemcpy(bufs[step & 1], bufs[s->steps & 1], state_payload(s),
                  hipMemcpyDeviceToDevice) != hipSuccess)
      return LBM_EHIP;
  }
  SolveState st{};
  st.step = step;
  for (int k = 0; k < 6; ++k) st.lockin[k] = lockin_sums ? lockin_sums[k] : 0.0;
  if (hipMemcpy(s->desc.state, &st, sizeof(st), hipMemcpyHostToDevice) != hipSuccess)
    return LBM_EHIP;
  s->steps = step;
  s->hist_from = step;
  s->sticky_unstable = false;
  return LBM_OK;
}

int lbm_state_size(const lbm_solver* s, uint64_t* bytes) {
  if (!s || !bytes) return LBM_EINVAL;
  *bytes = sizeof(StateHeader) + state_payload(s);
  return LBM_OK;
}

int lbm_get_state(lbm_solver* s, void* host, uint64_t bytes) {
  if (!s || !host) return LBM_EINVAL;
  const uint64_t payload = state_payload(s);
  if (bytes != sizeof(StateHeader) + payload) return LBM_EINVAL;
  if (hipStreamSynchronize(s->stream) != hipSuccess) return LBM_EHIP;
  const bool coeffs = s->lay.mom && !s->pop_pending;
  StateHeader h{kStateMagic, s->p.lattice, s->p.storage, coeffs ? 1u : 0u, s->p.nx, s->p.ny,
                payload};
  std::memcpy(host, &h, sizeof(h));
  const void* src = coeffs ? s->desc.mbuf[s->steps & 1] : s->bufs[s->steps & 1];
  if (hipMemcpy(static_cast<char*>(host) + sizeof(h), src, payload, hipMemcpyDeviceToHost) !=
      hipSuccess)
    return LBM_EHIP;
  return LBM_OK;
}

int lbm_set_state(lbm_solver* s, const void* host, uint64_t bytes) {
  if (!s || !host || bytes < sizeof(StateHeader)) return LBM_EINVAL;
  StateHeader h;
  std::memcpy(&h, host, sizeof(h));
  if (h.magic != kStateMagic || h.lattice != s->p.lattice || h.storage != s->p.storage ||
      h.nx != s->p.nx || h.ny != s->p.ny || (h.coeffs && !s->lay.mom) ||
      (!h.coeffs && !s->lay.loadable))
    return LBM_EINVAL;
  const uint64_t payload = h.coeffs ? s->lay.mbuf_bytes : s->lay.buf_bytes;
  if (h.bytes != payload || bytes != sizeof(h) + payload) return LBM_EINVAL;
  if (hipStreamSynchronize(s->stream) != hipSuccess) return LBM_EHIP;
  void* dst = h.coeffs ? s->desc.mbuf[s->steps & 1] : s->bufs[s->steps & 1];
  if (hipMemcpy(dst, static_cast<const char*>(host) + sizeof(h), payload,
                hipMemcpyHostToDevice) != hipSuccess)
    return LBM_EHIP;
  if (s->lay.mom) s->pop_pending = !h.coeffs;
  return LBM_OK;
}

int lbm_destroy(lbm_solver* s) {
  if (!s) return LBM_OK;
  int rc = hipStreamSynchronize(s->stream) == hipSuccess ? LBM_OK : LBM_EHIP;
  if (s->graph) (void)hipGraphExecDestroy(s->graph);
  if (s->owned && hipFree(s->base) != hipSuccess) rc = LBM_EHIP;
  if (s->in_scratch) release_scratch(s->device);
  readout_users(-1);
  delete s;
  return rc;
}

const char* lbm_strerror(int code) {
  switch (code) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument";
    case LBM_ENOMEM: return "out of memory or buffer too small";
    case LBM_EHIP: return "HIP runtime error";
    case LBM_ERANGE: return "out of range";
    case LBM_EUNSTABLE: return "unstable: non-positive or non-finite density";
    case LBM_EABI: return "ABI version mismatch";
    case LBM_ESCRATCH:
      return "static scratch buffer too small for these parameters, or in use by a live solver";
    default: return "unknown error";
  }
}

}  // extern "C"

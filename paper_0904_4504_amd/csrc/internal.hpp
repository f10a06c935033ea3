// Host-side internals shared by the C ABI translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "lattice.hpp"
#include "lbm.h"
#include "solver.hpp"

namespace lbm {

// dn (here and below): steps enqueued since the last advance of the step
// counters.  ds: some solve of the launch has a diffuse-scattering wall.
hipError_t launch_step(int Q, bool f64, bool bgk, bool ds, int cpt, bool outm,
                       const SolveDesc* descs, const WorkItem* work, int nwork,
                       const KernelLattice& lat, int dn, bool streaming, hipStream_t stream,
                       KernelEvents ev = {});
// ds: some solve of the launch has a diffuse-scattering wall.  streaming:
// the launch's state exceeds what stays in the last-level cache between
// steps (its new coefficients then go out with nontemporal stores).
hipError_t launch_coef(int Q, bool f64, int k, bool ds, bool streaming, const SolveDesc* descs,
                       const WorkItem* work, int nwork, const KernelLattice& lat, int dn,
                       hipStream_t stream, KernelEvents ev = {});
// nsub steps of narrow lattices.
// work: (solve, tile of `rows` rows) items, or null for nwork tiles of solve 0.
hipError_t launch_column(int Q, bool f64, bool bgk, bool ds, const ColumnShape& shape,
                         const SolveDesc* descs, const WorkItem* work, int nwork,
                         const KernelLattice& lat, int dn, hipStream_t stream,
                         KernelEvents ev = {});
// One step of narrow lattices.
// work: (solve, tile of kBlock cells or kForceTile) items, or null for solve 0
// (nwork: its tiles and one).
hipError_t launch_column_single(int Q, bool f64, bool bgk, bool ds, const SolveDesc* descs,
                                const WorkItem* work, int nwork, const KernelLattice& lat, int dn,
                                bool streaming, hipStream_t stream, KernelEvents ev = {});
// Advance the step counters of the listed solves.
hipError_t launch_advance(const SolveDesc* descs, const int32_t* solves, int count, int nsteps,
                          hipStream_t stream);

// What a read-out brings to the host, in pinned memory.
constexpr int kReadoutSamples = 4096;
struct Readout {
  int32_t unstable, pad;
  double lockin[6];
  double force[kReadoutSamples][2];
};
// A pinned buffer (null: not to be had), and its return once nothing writes it.
Readout* take_readout();
void give_readout(Readout* r);
// Solvers created (1) and destroyed (-1): idle buffers are freed with the last.
void readout_users(int change);
// Wait for the stream and read a solver's flag, lock-in sums and `count` force
// samples from step `first` (null: not wanted).  LBM_ENOMEM: no pinned memory
// (nothing was enqueued or waited for).
int read_out(const SolveDesc* desc, int device, hipStream_t stream, int64_t first, int count,
             int32_t* unstable, double lockin[6], double* force);

constexpr uint64_t kAlign = 256;

inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

inline int hip_rc(hipError_t e) { return e == hipSuccess ? LBM_OK : LBM_EHIP; }

// Velocity set of a lattice id, host copies.
struct HostLattice {
  int Q = 0, R = 0;
  std::vector<int> vx, vy, orbit, opp;
  LatticeWeights lw{};
};

// Where every region lives inside the one device allocation.
struct Layout {
  bool column = false;  // stepped by the column kernel
  int64_t pitch = 0, qs = 0, ys = 0, buf_elems = 0;
  int32_t ntiles = 0, cells_per_tile = kBlock, cpt = 1;
  int32_t mw = 0;  // population kernel: cells per row of its tiles
  int32_t nlinks = 0, nfcells = 0, nwcols = 0, nwlinks = 0, nlweights = 0, ncweights = 0;
  uint64_t off_links = 0, off_fcells = 0, off_wcols = 0, off_wlinks = 0;
  uint64_t off_lweights = 0, off_cweights = 0;
  int64_t unused_bytes = 0;  // force links left out (column kernel)
  // coefficient representation (mom): six coefficient planes, updated in
  // tiles of kCoefTileW columns x coef_tile_rows(K) rows
  bool mom = false;
  bool loadable = true;  // has the population buffer a populations load needs
  int32_t coef_k = 0;  // tile asked for (0: the default's rank among batch members)
  int32_t launch_k = 0;  // K of a launch over this solve alone
  int64_t mpitch = 0, mks = 0;  // coefficient buffers: row and plane strides (elements)
  uint64_t mbuf_bytes = 0, off_mwork = 0, off_mbuf[2] = {0, 0};
  int32_t nwork = 0, mnwork = 0;  // population-kernel and coefficient-kernel work items
  int64_t hist_cap = 0;
  uint64_t off_desc = 0, off_state = 0, off_work = 0, off_solves = 0, off_drive = 0,
           off_hist = 0, off_buf[2] = {0, 0};
  uint64_t buf_bytes = 0, total = 0;
};

// Append the tiles of one solve to a launch work list in XCD-aware order
// (rows of `span` tiles dealt to the 8 XCDs in turn).
void order_tiles(std::vector<WorkItem>* out, int32_t solve, int32_t ntiles, int32_t span);
// The same tiles with each XCD taking one contiguous band of tile rows (the
// halo rows shared by vertically adjacent tiles stay in that XCD's L2);
// the same length as order_tiles.
void order_tiles_banded(std::vector<WorkItem>* out, int32_t solve, int32_t ntiles,
                        int32_t span);
// Cells per thread of the coefficient kernel for a launch over `cells` cells
// (coef_cells of each lattice): the tile asked for, or (0) by the launch's size.
int coef_k_for(uint32_t tile, bool f64, int64_t cells);
// The cells of a lattice, its width rounded up to whole tiles.
int64_t coef_cells(const lbm_params* p);
// Tiles of a solve for K cells per thread, and the mask of those with a wall link.
struct CoefGrid {
  int32_t tiles_x = 0, ntiles = 0;
};
CoefGrid coef_grid(const lbm_params* p, int K);
std::vector<char> coef_wall_tiles(const lbm_params* p, int K, int R);
// The tiles of one coefficient solve: its wall tiles to `front` (they are the
// slowest of a launch, so they start first), the rest to `rest` in the order
// of order_tiles_banded (banded) or order_tiles with the wall tiles made
// no-ops (keeping the XCD structure).
void order_coef_tiles(std::vector<WorkItem>* front, std::vector<WorkItem>* rest, int32_t solve,
                      const std::vector<char>& wall, int32_t ntiles, int32_t span, bool banded);
// Coefficient launches whose two state buffers together take at most this
// many bytes stay in the 256 MB last-level cache between steps: their tiles
// go in bands (reuse of the halo rows within an XCD's L2) and their stores
// are plain, so the next step reads the state from the cache.  Larger ones
// stream from HBM: the row-interleaved order (adjacent rows in flight on all
// XCDs at once) and nontemporal stores.
constexpr uint64_t kCachedStateBytes = (uint64_t)192 << 20;
// The same line for the stores of the population kernel (two populations
// buffers of all the launch's members; stores plain against nontemporal: 209 MB
// 32.2 against 40.3 us per step, 310 MB 57.1 against 57.3, 931 MB 167 against
// 160).
constexpr uint64_t kCachedPopBytes = (uint64_t)256 << 20;
// Most steps between two advances of the step counters.
constexpr int kStepBlock = 1024;
// Split of column-kernel launches: rows per workgroup and the most steps per
// launch, for lattices of ny rows each and at most nx columns.
struct ColumnPlan {
  int rows = 0, max_sub = 1;
  int64_t groups = 0;  // workgroups
};
// Whether launches of one step go to column_single_kernel.
bool column_single(int Q, bool f64, const ColumnPlan& plan, bool ds);
// Work items of a narrow lattice in a single-step launch: the force and the tiles.
inline int column_single_items(int nx, int ny) {
  return 1 + (int)(((int64_t)nx * ny + kBlock - 1) / kBlock);
}
ColumnPlan column_plan(int Q, bool f64, int nx, const std::vector<int>& ny);
ColumnShape column_shape(int Q, int nx, int rows, int nsub);
// n as a sum of odd numbers of at most max_sub (odd): the steps per launch of
// a call of n steps.
std::vector<int> odd_pieces(int64_t n, int max_sub);
// front, padded with no-ops to a multiple of 8 items, then rest.
void join_front(std::vector<WorkItem>* front, const std::vector<WorkItem>& rest);

}  // namespace lbm

struct lbm_solver;
// One step of a single solver (population, population-to-coefficient or
// coefficient kernel), its counter advanced; defined in api.cpp.
int step_one(lbm_solver* s);
// Steps of a single solver captured into one graph.
constexpr int kGraphSteps = 32;

struct lbm_solver {
  // solver state; host fields mirror the device counters after a sync
  lbm_params p{};
  lbm::HostLattice lat;
  lbm::Layout lay;
  lbm::KernelLattice klat{};
  lbm::ColumnPlan column;     // of lattices stepped by the column kernel
  hipStream_t stream = nullptr;
  char* base = nullptr;       // device allocation (owned or caller's)
  void* bufs[2] = {nullptr, nullptr};  // population buffers; bufs[steps & 1] is current
  bool owned = false;
  int device = 0;
  int64_t steps = 0;          // steps enqueued
  bool pop_pending = false;   // coefficient solver whose current state is populations
  lbm::WorkItem* d_mwork = nullptr;   // coefficient kernel: tiles in XCD-aware order
  lbm::SolveDesc desc{};      // host copy (device pointers)
  lbm::SolveDesc* d_desc = nullptr;
  lbm::WorkItem* d_work = nullptr;
  int32_t* d_solves = nullptr;
  bool sticky_unstable = false;
  int64_t hist_from = 0;      // first step whose force is in the ring
  // graph of kGraphSteps steps (captured on first use; the launches read the
  // step index from the device, so one graph serves every later chunk)
  hipGraphExec_t graph = nullptr;
  bool graphs_ok = true;
  // device memory is the library's static scratch array of `device`
  // (lbm_create_static), released by lbm_destroy
  bool in_scratch = false;
};

namespace lbm {
// lbm_required_bytes; beyond (if asked for): how much more (or less) that is
// than the state, every force table by links and the work lists of the default
// tiles, which the static scratch limit counts.
int required_bytes(const lbm_params* p, uint64_t* bytes, int64_t* beyond);
// Create a solver in caller-owned device memory (dev_buf, bytes) or, with
// dev_buf null, in memory the library allocates.  graphs: lbm_step may
// capture and replay HIP graphs (off: every step launches directly).
int create_solver(const lbm_params* p, void* stream, void* dev_buf, uint64_t bytes, bool graphs,
                  lbm_solver** out);
// Mark the static scratch array of `device` free again (lbm_destroy of a
// solver created by lbm_create_static).
void release_scratch(int device);
}  // namespace lbm


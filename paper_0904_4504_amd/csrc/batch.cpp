// Batched execution: many solvers (uneven lattices, same velocity set,
// storage and collision) advanced by one launch per step and kind of member
// over the tiles of all of them, each launch with a workgroup per member for
// its wall force.  Members join and leave between steps
// (continuous batching); a member stops when it reaches its max_steps.
// Steady-state chunks are replayed from a captured HIP graph.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>
#include <vector>

#include "internal.hpp"

using namespace lbm;

namespace {
// kinds of launch of a batch (even: bounce-back, odd: diffuse or Maxwell wall)
constexpr int kPop = 0, kTiles = 2, kColumns = 4, kGroups = 6;
// Least steps of a call for which column launches go beside the others: the
// events between two streams and the second advance of the counters cost a
// call about 25 us of waiting (a 512 x 512 box with four 4 x 2048 plates, us per
// call, beside / one after the other: 1 step 43 / 19, 2 42 / 35, 3 57 / 41,
// 4 53 / 57, 8 94 / 97; 1024 x 1024 with eight plates: 3 65 / 66, 4 82 / 89).
// Beside members of fewer cells than kBesideCells there is less to gain (a
// 20 x 300 plate with four of 4 x 2048, D2Q9 FP32: 5 steps 51 / 29, 8 68 / 46).
// The runtime deals a process's streams to its hardware queues (4 by default).  If
// both streams fall to one queue, the launches take turns and the call lasts as
// long as one after the other (two 1024 x 1024 boxes with eight plates, 256 steps: 8.8
// ms instead of 7.4).
constexpr int kBesideSteps = 4, kBesideStepsSmall = 12;
constexpr int64_t kBesideCells = 200000;
}  // namespace

struct lbm_batch {
  hipStream_t stream = nullptr;
  std::vector<lbm_solver*> members;
  int Q = 0;
  uint32_t storage = 0, collision = 0;
  int cpt = 1;
  bool have_pop = false;  // some member keeps populations (sets cpt)
  int coef_k = 0;         // their tile as asked for, and the K of their launch
  int launch_k = 0;
  bool have_mom = false;  // some member keeps coefficients (sets coef_k)
  // current launch set (members that still have steps to run)
  std::vector<lbm_solver*> active;
  bool dirty = true;
  // work items in consecutive groups, one launch each: population kernel
  // (bounce-back wall, diffuse wall), coefficient kernel, column
  // kernel (the same); every member runs the kernel it runs alone
  int ngroup[kGroups] = {};
  // items of single-step launches of column-kernel members, behind the groups
  int nsingle[kGroups] = {};
  int first[kGroups + 1] = {};  // the groups' ranges in the solve list
  ColumnPlan column;      // of the column-kernel members
  int column_nx = 0;      // their widest lattice
  int ncolumn = 0;        // how many
  int64_t tile_cells = 0; // cells of the others
  // where other members step too, the column launches go on a stream of their
  // own between these events on the batch's stream
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  // coefficient groups whose state streams from HBM (nontemporal stores)
  bool streaming[kGroups] = {};
  SolveDesc* d_descs = nullptr;
  WorkItem* d_work = nullptr;   // population-kernel items, then coefficient-kernel items
  int32_t* d_solves = nullptr;
  size_t cap_descs = 0, cap_work = 0, cap_solves = 0;
  // graph of `graph_steps` steps for the current launch set
  hipGraphExec_t graph = nullptr;
  int graph_steps = 0;
  int graph_chunk = 32;
  bool graphs_enabled = true;
  // per-launch timing of the fused step kernel
  bool timing = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  double kernel_ms = 0;
  int64_t launches = 0;
};

namespace {

void drop_graph(lbm_batch* b) {
  if (b->graph) (void)hipGraphExecDestroy(b->graph);
  b->graph = nullptr;
  b->graph_steps = 0;
}

template <class T>
int grow(T** ptr, size_t* cap, size_t need) {
  if (need <= *cap) return LBM_OK;
  size_t n = std::max(need, *cap * 2);
  if (*ptr) (void)hipFree(*ptr);
  *ptr = nullptr;
  *cap = 0;
  if (hipMalloc(reinterpret_cast<void**>(ptr), n * sizeof(T)) != hipSuccess) {
    (void)hipGetLastError();
    return LBM_ENOMEM;
  }
  *cap = n;
  return LBM_OK;
}

// The stream and events of column launches beside others; false: not to be had
// (the launches then go one after the other).
bool side_stream(lbm_batch* b) {
  if (b->join) return true;
  if (!b->side && hipStreamCreateWithFlags(&b->side, hipStreamNonBlocking) != hipSuccess)
    b->side = nullptr;
  if (b->side && !b->fork &&
      hipEventCreateWithFlags(&b->fork, hipEventDisableTiming) != hipSuccess)
    b->fork = nullptr;
  if (b->fork && hipEventCreateWithFlags(&b->join, hipEventDisableTiming) != hipSuccess)
    b->join = nullptr;
  if (!b->join) (void)hipGetLastError();
  return b->join != nullptr;
}

// The kind of launch that steps a member.
int kind(const lbm_solver* s) {
  const Layout& lay = s->lay;
  return (lay.mom ? kTiles : lay.column ? kColumns : kPop) + (s->p.wall != LBM_WALL_BB);
}

// Rebuild the device launch set from the given members.
int refresh(lbm_batch* b, const std::vector<lbm_solver*>& act) {
  if (!b->dirty && act == b->active) return LBM_OK;
  drop_graph(b);
  b->active = act;
  b->dirty = true;  // until the device has the whole set
  std::vector<SolveDesc> descs;
  // first every member's force item and (coefficient groups) its wall tiles,
  // the slowest tiles of the launch, then the rest
  std::vector<WorkItem> group[kGroups], front[kGroups], single[kGroups], work;
  std::vector<int32_t> solves;
  std::vector<int> column_ny;
  b->column_nx = 0;
  b->tile_cells = 0;
  for (lbm_solver* s : act)
    if (s->lay.column) {
      b->column_nx = std::max(b->column_nx, s->p.nx);
      column_ny.push_back(s->p.ny);
    } else {
      b->tile_cells += (int64_t)s->p.nx * s->p.ny;
    }
  if (b->column_nx)
    b->column = column_plan(b->Q, b->storage == LBM_STORE_F64, b->column_nx, column_ny);
  uint64_t state[kGroups] = {};  // state bytes per group
  uint32_t tile = 0;  // as a member asks (0: none does)
  int64_t cells = 0;
  for (const lbm_solver* s : act)
    if (!s->lay.mom) {
      state[kind(s)] += 2 * s->lay.buf_bytes;
    } else {
      state[kind(s)] += 2 * s->lay.mbuf_bytes;
      tile = std::max(tile, s->p.tile);
      cells += coef_cells(&s->p);
    }
  b->launch_k = cells ? coef_k_for(tile, b->storage == LBM_STORE_F64, cells) : 0;
  for (size_t i = 0; i < act.size(); ++i) {
    descs.push_back(act[i]->desc);
    const Layout& lay = act[i]->lay;
    const int k = kind(act[i]);
    if (!lay.column) front[k].push_back(WorkItem{(int32_t)i, kForceTile});
    if (lay.column) {
      const int tiles = (act[i]->p.ny + b->column.rows - 1) / b->column.rows;
      for (int t = 0; t < tiles; ++t) group[k].push_back(WorkItem{(int32_t)i, t});
      const int items = column_single_items(act[i]->p.nx, act[i]->p.ny);
      front[k].push_back(WorkItem{(int32_t)i, kForceTile});
      for (int t = 0; t + 1 < items; ++t) single[k].push_back(WorkItem{(int32_t)i, t});
    } else if (lay.mom) {
      const CoefGrid g = coef_grid(&act[i]->p, b->launch_k);
      order_coef_tiles(&front[k], &group[k], (int32_t)i,
                       coef_wall_tiles(&act[i]->p, b->launch_k, act[i]->lat.R), g.ntiles,
                       g.tiles_x, state[k] <= kCachedStateBytes);
    } else {
      order_tiles(&group[k], (int32_t)i, lay.ntiles,
                  (lay.mw + lay.cells_per_tile - 1) / lay.cells_per_tile);
    }
  }
  b->ncolumn = (int)column_ny.size();
  for (int k = 0; k < kGroups; ++k) {
    for (size_t i = 0; i < act.size(); ++i)
      if (kind(act[i]) == k) solves.push_back((int32_t)i);
    b->first[k + 1] = (int)solves.size();
    if (k >= kColumns) {
      single[k].insert(single[k].begin(), front[k].begin(), front[k].end());
      b->nsingle[k] = (int)single[k].size();
    } else if (!front[k].empty()) {
      join_front(&front[k], group[k]);
      group[k].swap(front[k]);
    }
    b->ngroup[k] = (int)group[k].size();
    b->streaming[k] =
        state[k] > (k < kTiles || k >= kColumns ? kCachedPopBytes : kCachedStateBytes);
    work.insert(work.end(), group[k].begin(), group[k].end());
  }
  for (int k = kColumns; k < kGroups; ++k)
    work.insert(work.end(), single[k].begin(), single[k].end());
  if (act.empty()) {
    b->dirty = false;
    return LBM_OK;
  }
  if (b->ncolumn && b->ncolumn < (int)act.size()) (void)side_stream(b);
  if (hipStreamSynchronize(b->stream) != hipSuccess) return LBM_EHIP;
  int rc;
  if ((rc = grow(&b->d_descs, &b->cap_descs, descs.size()))) return rc;
  if ((rc = grow(&b->d_work, &b->cap_work, work.size()))) return rc;
  if ((rc = grow(&b->d_solves, &b->cap_solves, solves.size()))) return rc;
  if (hipMemcpy(b->d_descs, descs.data(), sizeof(SolveDesc) * descs.size(),
                hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(b->d_work, work.data(), sizeof(WorkItem) * work.size(),
                hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(b->d_solves, solves.data(), sizeof(int32_t) * solves.size(),
                hipMemcpyHostToDevice) != hipSuccess)
    return LBM_EHIP;
  b->dirty = false;
  return LBM_OK;
}

hipEvent_t next_event(lbm_batch* b) {
  if (b->ev_used == b->ev_pool.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    b->ev_pool.push_back(e);
  }
  return b->ev_pool[b->ev_used++];
}

// Sum the durations of the recorded step-kernel launches (waits).
int collect_timing(lbm_batch* b) {
  if (b->ev_used == 0) return LBM_OK;
  if (hipStreamSynchronize(b->stream) != hipSuccess) return LBM_EHIP;
  for (size_t i = 0; i + 1 < b->ev_used; i += 2) {
    float ms = 0;
    if (hipEventElapsedTime(&ms, b->ev_pool[i], b->ev_pool[i + 1]) != hipSuccess) return LBM_EHIP;
    b->kernel_ms += ms;
    ++b->launches;
  }
  b->ev_used = 0;
  return LBM_OK;
}

// Steps of each kind of member enqueued since its counters were advanced, and in
// all (counters advanced).
struct Enqueued {
  int since[kGroups] = {};
  int64_t done[kGroups] = {};
};

// Advance the counters of the kinds [k0, k1) by the steps enqueued for each (the
// same for all of them unless a launch failed).
int advance(lbm_batch* b, int k0, int k1, Enqueued* q, hipStream_t stream) {
  int rc = LBM_OK;
  for (int k = k0, e; k < k1; k = e) {
    for (e = k + 1; e < k1 && q->since[e] == q->since[k]; ++e) {
    }
    if (launch_advance(b->d_descs, b->d_solves + b->first[k], b->first[e] - b->first[k],
                       q->since[k], stream) != hipSuccess)
      rc = LBM_EHIP;
    else
      for (int i = k; i < e; ++i) q->done[i] += q->since[i];
    for (int i = k; i < e; ++i) q->since[i] = 0;
  }
  return rc;
}

// The launches of column-kernel members, nsub steps each.
hipError_t launch_columns(lbm_batch* b, int nsub, Enqueued* q, hipStream_t stream,
                          KernelEvents ev) {
  const bool f64 = b->storage == LBM_STORE_F64, bgk = b->collision == LBM_COLL_BGK;
  const KernelLattice& lat = b->active[0]->klat;
  const WorkItem *work = b->d_work, *single = b->d_work;
  for (int k = 0; k < kGroups; ++k) (k < kColumns ? work : single) += b->ngroup[k];
  single += work - b->d_work;
  for (int k = kColumns; k < kGroups; ++k) {
    const int n = b->ngroup[k], dn = q->since[k];
    const bool ds = k & 1;
    hipError_t e = hipSuccess;
    if (nsub == 1 && n > 0 && column_single(b->Q, f64, b->column, ds))
      e = launch_column_single(b->Q, f64, bgk, ds, b->d_descs, single, b->nsingle[k], lat, dn,
                               b->streaming[k], stream, ev);
    else if (n > 0)
      e = launch_column(b->Q, f64, bgk, ds,
                        column_shape(b->Q, b->column_nx, b->column.rows, nsub), b->d_descs, work,
                        n, lat, dn, stream, ev);
    if (e != hipSuccess) return e;
    q->since[k] += nsub;
    work += n;
    single += b->nsingle[k];
  }
  return hipSuccess;
}

// The population- and coefficient-kernel launches of one step.
hipError_t launch_tiles(lbm_batch* b, Enqueued* q, KernelEvents ev) {
  const bool f64 = b->storage == LBM_STORE_F64, bgk = b->collision == LBM_COLL_BGK;
  const KernelLattice& lat = b->active[0]->klat;
  const WorkItem* work = b->d_work;
  for (int k = 0; k < kColumns; ++k) {
    const int n = b->ngroup[k], dn = q->since[k];
    const bool ds = k & 1;
    const hipError_t e =
        n == 0       ? hipSuccess
        : k < kTiles ? launch_step(b->Q, f64, bgk, ds, b->cpt, false, b->d_descs, work, n, lat, dn,
                                   b->streaming[k], b->stream, ev)
                     : launch_coef(b->Q, f64, b->launch_k, ds, b->streaming[k], b->d_descs, work, n,
                                   lat, dn, b->stream, ev);
    if (e != hipSuccess) return e;
    ++q->since[k];
    work += n;
  }
  return hipSuccess;
}

// One step of every member, its step-kernel launches timed.
int launch_timed(lbm_batch* b, Enqueued* q) {
  int nlaunch = 0;
  for (int k = 0; k < kGroups; ++k) nlaunch += b->ngroup[k] > 0;
  if (b->ev_used + 2 > 4096) {
    int rc = collect_timing(b);
    if (rc) return rc;
  }
  hipEvent_t e0 = next_event(b), e1 = next_event(b);
  if (!e0 || !e1) return LBM_EHIP;
  // a single launch records its own start and end; several: events around them
  const KernelEvents own = nlaunch == 1 ? KernelEvents{e0, e1} : KernelEvents{};
  if (nlaunch > 1 && hipEventRecord(e0, b->stream) != hipSuccess) return LBM_EHIP;
  int rc = LBM_OK;
  if (launch_columns(b, 1, q, b->stream, own) != hipSuccess ||
      launch_tiles(b, q, own) != hipSuccess)
    rc = LBM_EHIP;
  if (nlaunch > 1 && hipEventRecord(e1, b->stream) != hipSuccess) rc = LBM_EHIP;
  if (rc) b->ev_used -= 2;  // not both recorded: not a measured step
  if (advance(b, 0, kGroups, q, b->stream)) rc = LBM_EHIP;
  return rc;
}

// n steps of the column-kernel members, several per launch.
int launch_column_steps(lbm_batch* b, int64_t n, Enqueued* q, hipStream_t stream) {
  for (int64_t left = b->ncolumn ? n : 0; left > 0;) {
    const int block = (int)std::min<int64_t>(left, kStepBlock);
    int rc = LBM_OK;
    for (int nsub : odd_pieces(block, b->column.max_sub))
      if (!rc && launch_columns(b, nsub, q, stream, KernelEvents{}) != hipSuccess) rc = LBM_EHIP;
    if (advance(b, kColumns, kGroups, q, stream)) rc = LBM_EHIP;
    if (rc) return rc;
    left -= block;
  }
  return LBM_OK;
}

// Makes the batch's stream wait for the side stream's launches, at the latest
// when it goes out of scope.
struct Joined {
  lbm_batch* b;
  int wait() {
    lbm_batch* const w = b;
    b = nullptr;
    return !w || hipStreamWaitEvent(w->stream, w->join, 0) == hipSuccess ? LBM_OK : LBM_EHIP;
  }
  ~Joined() { (void)wait(); }
};

// n steps of the other members, step by step.
int launch_tile_steps(lbm_batch* b, int64_t n, Enqueued* q) {
  for (int64_t left = (int)b->active.size() > b->ncolumn ? n : 0; left > 0;) {
    const int block = (int)std::min<int64_t>(left, kStepBlock);
    int rc = LBM_OK;
    for (int k = 0; k < block && !rc; ++k)
      if (launch_tiles(b, q, KernelEvents{}) != hipSuccess) rc = LBM_EHIP;
    if (advance(b, 0, kColumns, q, b->stream)) rc = LBM_EHIP;
    if (rc) return rc;
    left -= block;
  }
  return LBM_OK;
}

// Capture graph_chunk steps of the members stepped by tiles into a graph.
bool capture(lbm_batch* b) {
  if (b->stream == nullptr) return false;  // the null stream cannot be captured
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  Enqueued q;
  const bool ok = launch_tile_steps(b, b->graph_chunk, &q) == LBM_OK;
  if (hipStreamEndCapture(b->stream, &g) != hipSuccess || !ok) {
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
  b->graph = ex;
  b->graph_steps = b->graph_chunk;
  return true;
}

// chunk steps of the launch set.
int step_chunk(lbm_batch* b, int64_t chunk, Enqueued* q) {
  int rc = LBM_OK;
  if (b->timing) {
    for (int64_t k = 0; k < chunk && !rc; ++k) rc = launch_timed(b, q);
    return rc;
  }
  // members do not interact: the column-kernel ones take the whole chunk,
  // several steps per launch, the others step by step, in graphs where the
  // chunk allows.  Both at once, on two streams: the column launches are
  // chains of a few hundred workgroups that leave most of the GPU idle (two
  // 1024 x 1024 boxes with eight plates: 28.9 us per step, one after the
  // other 35.1)
  const bool tiles = (int)b->active.size() > b->ncolumn;
  const bool beside = tiles && b->ncolumn && b->join;
  if (beside && chunk < (b->tile_cells < kBesideCells ? kBesideStepsSmall : kBesideSteps)) {
    for (int nsub : odd_pieces(chunk, b->column.max_sub))
      if (!rc && launch_columns(b, nsub, q, b->stream, KernelEvents{}) != hipSuccess)
        rc = LBM_EHIP;
    for (int64_t k = 0; k < chunk && !rc; ++k)
      if (launch_tiles(b, q, KernelEvents{}) != hipSuccess) rc = LBM_EHIP;
    return advance(b, 0, kGroups, q, b->stream) ? LBM_EHIP : rc;
  }
  if (beside && (hipEventRecord(b->fork, b->stream) != hipSuccess ||
                 hipStreamWaitEvent(b->side, b->fork, 0) != hipSuccess))
    return LBM_EHIP;
  rc = launch_column_steps(b, chunk, q, beside ? b->side : b->stream);
  // (also after a failed launch: nothing is left running beside the stream)
  if (beside && hipEventRecord(b->join, b->side) != hipSuccess) rc = LBM_EHIP;
  Joined joined{beside ? b : nullptr};
  if (rc) return rc;
  int64_t k = 0;
  if (tiles && b->graphs_enabled && chunk >= b->graph_chunk) {
    if (!b->graph && !capture(b)) b->graphs_enabled = false;
    for (; b->graph && k + b->graph_steps <= chunk; k += b->graph_steps) {
      if (hipGraphLaunch(b->graph, b->stream) != hipSuccess) return LBM_EHIP;
      for (int i = 0; i < kColumns; ++i) q->done[i] += b->graph_steps;
    }
  }
  if ((rc = launch_tile_steps(b, chunk - k, q))) return rc;
  return joined.wait();
}

}  // namespace

extern "C" {

int lbm_batch_create(void* hip_stream, lbm_batch** out) {
  if (!out) return LBM_EINVAL;
  lbm_batch* b = new (std::nothrow) lbm_batch();
  if (!b) return LBM_ENOMEM;
  b->stream = static_cast<hipStream_t>(hip_stream);
  *out = b;
  return LBM_OK;
}

int lbm_batch_add(lbm_batch* b, lbm_solver* s) {
  if (!b || !s) return LBM_EINVAL;
  if (s->stream != b->stream) return LBM_EINVAL;
  if (std::find(b->members.begin(), b->members.end(), s) != b->members.end()) return LBM_EINVAL;
  if (b->members.empty()) {
    b->Q = (int)s->p.lattice;
    b->storage = s->p.storage;
    b->collision = s->p.collision;
  } else if ((int)s->p.lattice != b->Q || s->p.storage != b->storage ||
             s->p.collision != b->collision) {
    return LBM_EINVAL;
  }
  // members kept as populations share one population-kernel launch, members
  // kept as coefficients one coefficient-kernel launch
  if (!s->lay.mom) {
    if (b->have_pop && s->lay.cpt != b->cpt) return LBM_EINVAL;
    b->have_pop = true;
    b->cpt = s->lay.cpt;
  } else {
    if (b->have_mom && s->lay.coef_k != b->coef_k) return LBM_EINVAL;
    b->have_mom = true;
    b->coef_k = s->lay.coef_k;
  }
  b->members.push_back(s);
  b->dirty = true;
  return LBM_OK;
}

int lbm_batch_remove(lbm_batch* b, lbm_solver* s) {
  if (!b || !s) return LBM_EINVAL;
  auto it = std::find(b->members.begin(), b->members.end(), s);
  if (it == b->members.end()) return LBM_EINVAL;
  if (hipStreamSynchronize(b->stream) != hipSuccess) return LBM_EHIP;
  b->members.erase(it);
  b->dirty = true;
  if (b->members.empty()) {
    b->Q = 0;
    b->have_pop = false;
    b->have_mom = false;
  }
  return LBM_OK;
}

int lbm_batch_size(const lbm_batch* b, int* members, int* active) {
  if (!b) return LBM_EINVAL;
  if (members) *members = (int)b->members.size();
  if (active) {
    int n = 0;
    for (lbm_solver* s : b->members) n += s->steps < s->p.max_steps;
    *active = n;
  }
  return LBM_OK;
}

int lbm_batch_step(lbm_batch* b, int64_t nsteps) {
  if (!b || nsteps < 0) return LBM_EINVAL;
  // steps each member still takes in this call
  std::vector<int64_t> left(b->members.size());
  for (size_t i = 0; i < b->members.size(); ++i) {
    lbm_solver* s = b->members[i];
    left[i] = std::min(nsteps, s->p.max_steps - s->steps);
    // a coefficient member whose state was just loaded as populations takes
    // that step alone (population kernel writing coefficients)
    if (s->pop_pending && left[i] > 0) {
      int rc = step_one(s);
      if (rc) return rc;
      --left[i];
    }
  }
  for (;;) {
    std::vector<lbm_solver*> act;
    int64_t chunk = 0;
    for (size_t i = 0; i < b->members.size(); ++i)
      if (left[i] > 0) {
        act.push_back(b->members[i]);
        chunk = chunk ? std::min(chunk, left[i]) : left[i];
      }
    if (act.empty()) break;
    int rc = refresh(b, act);
    if (rc) return rc;
    Enqueued q;
    rc = step_chunk(b, chunk, &q);
    // what was launched counts, also when a launch failed
    for (size_t i = 0; i < b->members.size(); ++i)
      if (left[i] > 0) {
        b->members[i]->steps += q.done[kind(b->members[i])];
        left[i] -= chunk;
      }
    if (rc) return rc;
  }
  return LBM_OK;
}

int lbm_batch_synchronize(lbm_batch* b) {
  if (!b) return LBM_EINVAL;
  if (hipStreamSynchronize(b->stream) != hipSuccess) return LBM_EHIP;
  int worst = LBM_OK;
  for (lbm_solver* s : b->members) {
    int rc = lbm_synchronize(s);
    if (rc && !worst) worst = rc;
  }
  return worst;
}

int lbm_batch_set_graphs(lbm_batch* b, int steps_per_graph) {
  if (!b || steps_per_graph < 0) return LBM_EINVAL;
  drop_graph(b);
  b->graphs_enabled = steps_per_graph > 0;
  if (steps_per_graph > 0) b->graph_chunk = steps_per_graph;
  return LBM_OK;
}

int lbm_batch_timing(lbm_batch* b, int enable) {
  if (!b) return LBM_EINVAL;
  int rc = collect_timing(b);
  b->timing = enable != 0;
  b->kernel_ms = 0;
  b->launches = 0;
  return rc;
}

int lbm_batch_kernel_time(lbm_batch* b, double* ms, int64_t* launches) {
  if (!b) return LBM_EINVAL;
  int rc = collect_timing(b);
  if (ms) *ms = b->kernel_ms;
  if (launches) *launches = b->launches;
  return rc;
}

int lbm_batch_destroy(lbm_batch* b) {
  if (!b) return LBM_OK;
  int rc = hipStreamSynchronize(b->stream) == hipSuccess ? LBM_OK : LBM_EHIP;
  drop_graph(b);
  for (hipEvent_t e : b->ev_pool) (void)hipEventDestroy(e);
  if (b->join) (void)hipEventDestroy(b->join);
  if (b->fork) (void)hipEventDestroy(b->fork);
  if (b->side) (void)hipStreamDestroy(b->side);
  if (b->d_descs) (void)hipFree(b->d_descs);
  if (b->d_work) (void)hipFree(b->d_work);
  if (b->d_solves) (void)hipFree(b->d_solves);
  delete b;
  return rc;
}

}  // extern "C"

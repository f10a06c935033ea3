// The library's host side (api.cpp, batch.cpp, lattice.cpp) on a HIP runtime of
// plain host memory whose launches only record which steps they would do: see
// test_host_bookkeeping_cpu.py.  A launch, an allocation or a copy can be made
// to fail.  argv[1]: the check to run.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "internal.hpp"

using namespace lbm;

#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::printf("line %d: %s\n", __LINE__, #c);             \
      std::exit(1);                                           \
    }                                                         \
  } while (0)

// ------------------------------------------------------------ the runtime
static int g_fail_launch = -1, g_fail_malloc = -1;  // calls until one fails
static std::vector<std::string> g_log;              // launches and events, in order
static std::set<hipEvent_t> g_recorded;
static int g_pinned = 0;                            // pinned buffers allocated
static int g_coef_k = 0;                            // K of the last coefficient launch

static bool fails(int& counter) { return counter >= 0 && counter-- == 0; }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (fails(g_fail_malloc)) return hipErrorOutOfMemory;
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  ++g_pinned;
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  --g_pinned;
  std::free(p);
  return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(new int);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { delete reinterpret_cast<int*>(s); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(new int); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<int*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  g_log.push_back("record");
  g_recorded.insert(e);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) {
  g_log.push_back("wait");
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = 1;
  return g_recorded.count(a) && g_recorded.count(b) ? hipSuccess : hipErrorInvalidHandle;
}
}

// ------------------------------------------------------------- the kernels
// steps that a solve has done, by its state block; each must come once, in order
static std::map<const SolveState*, int64_t> g_done;

static hipError_t run(const char* name, const SolveDesc* descs, const WorkItem* work, int nwork,
                      int dn, int nsub, const KernelEvents& ev) {
  g_log.push_back(name);
  if (fails(g_fail_launch)) return hipErrorLaunchFailure;
  g_recorded.insert({ev.start, ev.stop});
  std::set<int> solves;
  for (int i = 0; i < nwork; ++i)
    if (!work || work[i].tile != kNoTile) solves.insert(work ? work[i].solve : 0);
  for (int i : solves) {
    const SolveState* st = descs[i].state;
    CHECK(st->step + dn == g_done[st]);
    g_done[st] += nsub;
  }
  return hipSuccess;
}

namespace lbm {
hipError_t launch_step(int, bool, bool, bool, int, bool, const SolveDesc* descs,
                       const WorkItem* work, int nwork, const KernelLattice&, int dn, bool,
                       hipStream_t, KernelEvents ev) {
  return run("step", descs, work, nwork, dn, 1, ev);
}
hipError_t launch_coef(int, bool, int k, bool, bool, const SolveDesc* descs, const WorkItem* work,
                       int nwork, const KernelLattice&, int dn, hipStream_t, KernelEvents ev) {
  g_coef_k = k;
  return run("coef", descs, work, nwork, dn, 1, ev);
}
hipError_t launch_column(int, bool, bool, bool, const ColumnShape& sh, const SolveDesc* descs,
                         const WorkItem* work, int nwork, const KernelLattice&, int dn, hipStream_t,
                         KernelEvents ev) {
  return run("column", descs, work, nwork, dn, sh.nsub, ev);
}
hipError_t launch_column_single(int, bool, bool, bool, const SolveDesc* descs, const WorkItem* work,
                                int nwork, const KernelLattice&, int dn, bool, hipStream_t,
                                KernelEvents ev) {
  return run("single", descs, work, nwork, dn, 1, ev);
}
hipError_t launch_advance(const SolveDesc* descs, const int32_t* solves, int count, int nsteps,
                          hipStream_t) {
  if (count <= 0 || nsteps <= 0) return hipSuccess;
  g_log.push_back("advance");
  for (int i = 0; i < count; ++i) descs[solves[i]].state->step += nsteps;
  return hipSuccess;
}
int read_out(const SolveDesc*, int, hipStream_t, int64_t, int, int32_t* unstable, double*, double*) {
  Readout* r = take_readout();
  *unstable = 0;
  give_readout(r);
  return LBM_OK;
}
void release_scratch(int) {}
}  // namespace lbm

// -------------------------------------------------------------- the checks
static lbm_params params(int geom, int nx, int ny, int wall, int64_t steps) {
  lbm_params p;
  CHECK(lbm_params_init(&p) == LBM_OK);
  p.lattice = 37;
  p.storage = LBM_STORE_F32_DEV;
  p.collision = LBM_COLL_REGULARIZED;
  p.geometry = geom;
  p.far = geom == LBM_GEOM_BOX ? LBM_FAR_EQ : LBM_FAR_WALL;
  p.wall = wall;
  p.accommodation = 1.0;
  p.nx = nx;
  p.ny = ny;
  if (geom == LBM_GEOM_BOX) {
    p.box_x0 = nx / 2;
    p.box_y0 = ny / 2;
    p.box_lx = p.box_ly = 5;
  }
  p.tau = 0.9;
  p.omega = 0.1;
  p.u0 = 1e-3;
  p.rho0 = 1;
  p.max_steps = steps;
  return p;
}

static lbm_solver* solver(const lbm_params& p) {
  lbm_solver* s = nullptr;
  CHECK(lbm_create(&p, nullptr, &s) == LBM_OK);
  return s;
}

// members of every kind of launch
static std::vector<lbm_solver*> members(int64_t steps) {
  return {solver(params(LBM_GEOM_PLATE, 4, 100, LBM_WALL_BB, steps)),
          solver(params(LBM_GEOM_BOX, 80, 70, LBM_WALL_BB, steps)),
          solver(params(LBM_GEOM_PLATE, 5, 60, LBM_WALL_DS, steps)),
          solver(params(LBM_GEOM_BOX, 40, 40, LBM_WALL_DS, steps)),
          solver(params(LBM_GEOM_PLATE, 70, 30, LBM_WALL_DS, steps)),
          solver(params(LBM_GEOM_BOX, 40, 44, LBM_WALL_BB, steps))};
}

// A launch set that could not be built is built by the next call.
static void check_refresh() {
  for (int n = 0; n < 3; ++n) {
    auto ms = members(50);
    lbm_batch* b = nullptr;
    CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
    for (lbm_solver* s : ms) CHECK(lbm_batch_add(b, s) == LBM_OK);
    g_fail_malloc = n;
    CHECK(lbm_batch_step(b, 3) == LBM_ENOMEM);
    g_fail_malloc = -1;
    CHECK(lbm_batch_step(b, 3) == LBM_OK);
    for (lbm_solver* s : ms) CHECK(s->steps == 3 && g_done[s->desc.state] == 3);
    lbm_batch_destroy(b);
    for (lbm_solver* s : ms) lbm_destroy(s);
    g_done.clear();
  }
}

// The n-th launch fails; the run then goes on to its end.  run() checks that no
// step is launched twice or left out.
static void check_launch() {
  const int64_t steps = 2500;
  for (int timing = 0; timing < 2; ++timing)
    for (int n = 0; n < 3000; n += 1 + n / 9) {
      auto ms = members(steps);
      lbm_batch* b = nullptr;
      CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
      for (lbm_solver* s : ms) CHECK(lbm_batch_add(b, s) == LBM_OK);
      CHECK(lbm_batch_timing(b, timing) == LBM_OK);
      g_fail_launch = n;
      CHECK(lbm_batch_step(b, steps) == LBM_EHIP);
      for (lbm_solver* s : ms)
        CHECK(s->steps == g_done[s->desc.state] && s->desc.state->step == s->steps);
      CHECK(lbm_batch_step(b, steps) == LBM_OK);
      for (lbm_solver* s : ms) CHECK(s->steps == steps && g_done[s->desc.state] == steps);
      lbm_batch_destroy(b);
      for (lbm_solver* s : ms) lbm_destroy(s);
      g_done.clear();
    }
  for (int n = 0; n < 2000; n += 1 + n / 5)
    for (lbm_solver* s : members(steps)) {
      g_fail_launch = n;
      int rc = lbm_step(s, steps);
      g_fail_launch = -1;
      CHECK(s->steps == g_done[s->desc.state] && s->desc.state->step == s->steps);
      CHECK(rc == (s->steps == steps ? LBM_OK : LBM_EHIP));
      if (s->steps < steps) CHECK(lbm_step(s, steps - s->steps) == LBM_OK);
      CHECK(s->steps == steps && g_done[s->desc.state] == steps);
      g_done.erase(s->desc.state);
      lbm_destroy(s);
    }
  // a loaded state is still the one to step from
  lbm_solver* s = solver(params(LBM_GEOM_BOX, 80, 70, LBM_WALL_BB, 9));
  std::vector<double> f((size_t)37 * 80 * 70, 0.0);
  CHECK(lbm_set_deviations(s, f.data(), f.size()) == LBM_OK);
  g_fail_launch = 0;
  g_log.clear();
  CHECK(lbm_step(s, 2) == LBM_EHIP && lbm_step(s, 2) == LBM_OK);
  CHECK(g_log[0] == "step" && g_log[1] == "step" && s->steps == 2);
  lbm_destroy(s);
}

// A tile that a member asks for is the tile of the batch's launch; with none
// asked for the launch's wavefronts count, full or not.
static void check_tile() {
  for (int nx : {20, 64, 65}) {
    lbm_params p = params(LBM_GEOM_PLATE, nx, 12000, LBM_WALL_BB, 9);
    p.ny = nx == 65 ? 6000 : 12000;
    p.representation = LBM_REPR_COEFFICIENTS_NOLOAD;
    lbm_solver *a = solver(p), *c = solver(params(LBM_GEOM_BOX, 80, 70, LBM_WALL_BB, 9));
    CHECK(lbm_step(a, 1) == LBM_OK && g_coef_k == 3);
    CHECK(lbm_step(c, 1) == LBM_OK && g_coef_k == 1);
    lbm_batch* b = nullptr;
    CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
    CHECK(lbm_batch_add(b, a) == LBM_OK && lbm_batch_add(b, c) == LBM_OK);
    CHECK(lbm_batch_step(b, 1) == LBM_OK && g_coef_k == 3);
    lbm_batch_destroy(b);
    lbm_destroy(a);
    lbm_destroy(c);
    g_done.clear();
  }
  for (int order = 0; order < 2; ++order) {
    lbm_params p = params(LBM_GEOM_BOX, 80, 70, LBM_WALL_BB, 9), q = p;
    p.tile = order ? 3 : 0;
    q.tile = order ? 0 : 3;
    lbm_solver *a = solver(p), *c = solver(q);
    lbm_batch* b = nullptr;
    CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
    CHECK(lbm_batch_add(b, a) == LBM_OK && lbm_batch_add(b, c) == LBM_OK);
    CHECK(lbm_batch_step(b, 1) == LBM_OK && g_coef_k == 3);
    lbm_batch_destroy(b);
    lbm_destroy(a);
    lbm_destroy(c);
    g_done.clear();
  }
}

// Calls of one step: a launch per kind of member and one advance, no events.
static void check_single() {
  auto ms = members(9);
  lbm_batch* b = nullptr;
  CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
  for (lbm_solver* s : ms) CHECK(lbm_batch_add(b, s) == LBM_OK);
  for (int k = 1; k < 4; ++k) {
    g_log.clear();
    CHECK(lbm_batch_step(b, 1) == LBM_OK);
    CHECK(g_log.size() == 7 && g_log.back() == "advance");
    for (lbm_solver* s : ms) CHECK(s->steps == k && s->desc.state->step == k);
  }
  lbm_batch_destroy(b);
  for (lbm_solver* s : ms) lbm_destroy(s);
}

// Column launches go beside those of other members from 4 steps, beside small
// members from 12.
static void check_beside() {
  for (int n : {200, 500}) {
    std::vector<lbm_solver*> ms = {solver(params(LBM_GEOM_PLATE, 4, 100, LBM_WALL_BB, 99)),
                                   solver(params(LBM_GEOM_BOX, n, n, LBM_WALL_BB, 99))};
    lbm_batch* b = nullptr;
    CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
    for (lbm_solver* s : ms) CHECK(lbm_batch_add(b, s) == LBM_OK);
    CHECK(lbm_batch_step(b, 1) == LBM_OK);
    for (int k : {2, 3, 4, 11, 12, 20}) {
      g_log.clear();
      CHECK(lbm_batch_step(b, k) == LBM_OK);
      const bool beside = std::count(g_log.begin(), g_log.end(), "wait") > 0;
      CHECK(beside == (k >= (n < 400 ? 12 : 4)));
    }
    lbm_batch_destroy(b);
    for (lbm_solver* s : ms) lbm_destroy(s);
    g_done.clear();
  }
}

// Read-outs share pinned buffers, freed with the last solver.
static void check_pinned() {
  for (int round = 0; round < 2; ++round) {
    auto ms = members(9);
    for (lbm_solver* s : ms) CHECK(lbm_synchronize(s) == LBM_OK);
    CHECK(g_pinned == 1);
    std::vector<Readout*> taken;
    for (int i = 0; i < 9; ++i) taken.push_back(take_readout());
    CHECK(g_pinned == 9);
    for (Readout* r : taken) give_readout(r);
    CHECK(g_pinned == 4);
    for (lbm_solver* s : ms) {
      CHECK(g_pinned == 4);
      lbm_destroy(s);
    }
    CHECK(g_pinned == 0);
  }
}

// A lattice stepped by the column kernel carries no force links and no work
// list, and the static limit counts it as if it did.
static void check_tables() {
  for (int ny : {100, 5000}) {
    lbm_params p = params(LBM_GEOM_PLATE, 4, ny, LBM_WALL_BB, 9);
    lbm_solver* s = solver(p);
    CHECK(s->lay.column && s->lay.nwork == 0 && s->desc.nlinks == 0);
    uint64_t bytes = 0;
    int64_t beyond = 0;
    CHECK(required_bytes(&p, &bytes, &beyond) == LBM_OK && bytes == s->lay.total);
    // 4 columns x 26 crossing populations of 15 velocities, a weight pattern for
    // each, a work item per 256 cells
    const int64_t list = ((ny * 4 + 255) / 256 + 7) / 8 * 8;
    CHECK(beyond == 4 * (int64_t)kAlign - 4 * 26 * (int64_t)sizeof(ForceLink) -
                        15 * (int64_t)sizeof(LinkWeights) - list * (int64_t)sizeof(WorkItem));
    CHECK(lbm_step(s, 9) == LBM_OK);
    g_done.erase(s->desc.state);
    lbm_destroy(s);
  }
}

// A timed step whose launch failed is not part of the kernel time.
static void check_timing() {
  for (int several = 0; several < 2; ++several) {
    auto all = members(9);
    std::vector<lbm_solver*> ms(all.begin(), all.begin() + (several ? all.size() : 1));
    lbm_batch* b = nullptr;
    CHECK(lbm_batch_create(nullptr, &b) == LBM_OK);
    for (lbm_solver* s : ms) CHECK(lbm_batch_add(b, s) == LBM_OK);
    CHECK(lbm_batch_timing(b, 1) == LBM_OK);
    CHECK(lbm_batch_step(b, 2) == LBM_OK);
    g_fail_launch = 0;
    CHECK(lbm_batch_step(b, 2) == LBM_EHIP);
    CHECK(lbm_batch_step(b, 1) == LBM_OK);
    double ms_ = 0;
    int64_t n = 0;
    CHECK(lbm_batch_kernel_time(b, &ms_, &n) == LBM_OK && n == 3 && ms_ == 3);
    lbm_batch_destroy(b);
    for (lbm_solver* s : all) lbm_destroy(s);
    g_done.clear();
    g_recorded.clear();
  }
}

// Every step that a solve may have has its entry of the drive table.
static void check_steps() {
  lbm_params p = params(LBM_GEOM_BOX, 80, 70, LBM_WALL_BB, (int64_t)1 << 32);
  uint64_t bytes = 0;
  CHECK(lbm_required_bytes(&p, &bytes) == LBM_OK);
  for (int64_t n : {(int64_t)0, ((int64_t)1 << 31) - 1, (int64_t)1 << 31, p.max_steps - 1})
    CHECK((int64_t)drive_index(n) == n);
  ++p.max_steps;
  CHECK(lbm_required_bytes(&p, &bytes) == LBM_EINVAL);
}

int main(int argc, char** argv) {
  const std::map<std::string, std::function<void()>> checks{{"refresh", check_refresh},
                                                             {"launch", check_launch},
                                                             {"tile", check_tile},
                                                             {"single", check_single},
                                                             {"beside", check_beside},
                                                             {"pinned", check_pinned},
                                                             {"tables", check_tables},
                                                             {"timing", check_timing},
                                                             {"steps", check_steps}};
  CHECK(argc == 2 && checks.count(argv[1]));
  checks.at(argv[1])();
  std::printf("ok\n");
  return 0;
}

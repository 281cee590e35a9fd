// The library's host code (vp_api.cpp) over memory that stands for a device: the HIP calls and the
// kernel launches it makes are replaced by functions that work on host memory, check what the
// tables they are given say, and fail on demand.  Run on the CPU by test_host_device.py, one check
// per name.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <tuple>
#include <vector>

#include "vp.h"
#include "vp_internal.h"

static int failures = 0;
#define CHECK(c)                                                                    \
  do {                                                                              \
    if (!(c)) {                                                                     \
      std::fprintf(stderr, "check failed: %s (line %d): %s\n", #c, __LINE__, vp_last_error()); \
      ++failures;                                                                   \
    }                                                                               \
  } while (0)

// name -> calls until (and including) the one that fails; negative: every call fails
static std::map<std::string, int> fail_at;
static bool fails(const char* name) {
  auto it = fail_at.find(name);
  if (it == fail_at.end() || it->second == 0) return false;
  return it->second < 0 || --it->second == 0;
}
static size_t pinned = 0, pinned_most = 0;
static std::map<void*, size_t> pinned_blocks;

// ---------------------------------------------------------------- HIP
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::aligned_alloc(256, (n + 255) & ~size_t(255));
  std::memset(*p, 0xee, n);
  return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (fails("hipHostMalloc")) return hipErrorOutOfMemory;
  *p = std::malloc(n);
  pinned_blocks[*p] = n;
  pinned += n;
  pinned_most = pinned > pinned_most ? pinned : pinned_most;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  pinned -= pinned_blocks.at(p);
  pinned_blocks.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (fails("hipMemcpyAsync")) return hipErrorUnknown;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 1; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorUnknown; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorUnknown; }
}

// ---------------------------------------------------------------- launches
// particles taken by the fused launches: (instance's Q, first particle) -> count
static std::map<std::pair<void*, long long>, long long> stepped;

namespace vpk {
int kin_capacity(long long n) { return (int)((n + kMinTile - 1) / kMinTile); }
WsLayout workspace_layout(int ng, int, int hist_cap, long long n) {
  WsLayout w{};
  size_t o = 0;
  auto take = [&](size_t b) { const size_t at = o; o = (o + b + 255) & ~size_t(255); return at; };
  w.acc = take(256); w.E = take(8 * ng); w.g = take(8 * ng); w.Ef = take(4 * ng); w.gf = take(4 * ng);
  w.Phi = take(16 * ng); w.bt = take(16 * ng); w.tw = take(8 * ng); w.inv_lam = take(8 * ng);
  w.cw = take(8 * kConsTapsMax); w.scal = take(sizeof(InstScal));
  w.hist = take((size_t)hist_cap * kHistFields * 8);
  w.kin = take((size_t)kRing * kin_capacity(n) * kKinFields * 8);
  w.total = o;
  return w;
}
hipError_t launch_upload(const UploadArgs& u, hipStream_t) {
  if (fails("launch_upload")) return hipErrorUnknown;
  for (int k = 0; k < u.nseg; ++k) std::memcpy(u.seg[k].dst, u.seg[k].src, 8 * u.seg[k].n8);
  for (int k = 0; k < u.nzero; ++k) std::memset(u.zero[k].dst, 0, 8 * u.zero[k].n8);
  return hipSuccess;
}
hipError_t launch_fill_zero(void* p, size_t n, hipStream_t) {
  if (fails("launch_fill_zero")) return hipErrorUnknown;
  std::memset(p, 0, n);
  return hipSuccess;
}
// Every tile is one of an instance in the table, within its particles and its numbers.
static hipError_t tiles(const char* name, const InstDev* insts, const Tile* t, int tile0, int n) {
  if (fails(name)) return hipErrorUnknown;
  for (int k = tile0; k < tile0 + n; ++k) {
    const InstDev& d = insts[t[k].inst];
    CHECK(d.Q != nullptr && t[k].begin >= 0 && t[k].count > 0 && t[k].begin + t[k].count <= d.n &&
          t[k].local >= 0 && t[k].local < d.ntiles);
  }
  return hipSuccess;
}
hipError_t launch_fused(int, int, const InstDev* insts, const Tile* t, int tile0, int n, int, int, bool,
                        int, bool, bool, bool, bool, bool, hipStream_t) {
  for (int k = tile0; k < tile0 + n; ++k) {
    const InstDev& d = insts[t[k].inst];
    stepped[{d.Q, t[k].begin}] += t[k].count;
    if (t[k].local == 0) {  // the step's record: K tells the step
      double* r = d.hist + (d.scal->step % d.hist_cap) * kHistFields;
      std::memset(r, 0, kHistFields * 8);
      r[0] = r[2] = (double)d.scal->step;
      d.scal->step += 1;
    }
  }
  return tiles("launch_fused", insts, t, tile0, n);
}
hipError_t launch_deposit(int, int, const InstDev* i, const Tile* t, int tile0, int n, int, int, int, hipStream_t) { return tiles("launch_deposit", i, t, tile0, n); }
hipError_t launch_gather_push(int, int, const InstDev* i, const Tile* t, int tile0, int n, int, int, double, double, hipStream_t) { return tiles("launch_gather_push", i, t, tile0, n); }
hipError_t launch_settle(int, int, const InstDev* i, const Tile* t, int tile0, int n, int, int, int, hipStream_t) { return tiles("launch_settle", i, t, tile0, n); }
hipError_t launch_diag(int, int, const InstDev* i, const Tile* t, int tile0, int n, int, int, int, hipStream_t) {
  i[t[tile0].inst].scal->Kd = 7.0;
  return tiles("launch_diag", i, t, tile0, n);
}
hipError_t launch_persist(int, int, int, const InstDev* i, const Tile* t, int n, int, bool, bool, bool, int, int, hipStream_t) { return tiles("launch_persist", i, t, 0, n); }
int persist_capacity(int, int, int, int, bool, bool, bool) { return 256; }
long long resident_capacity(int, bool, bool, int) { return 4096; }
int resident_ppt(long long) { return 4; }
hipError_t launch_resident(int, long long, const InstDev*, const int*, int, int, bool, bool, bool, int, int, hipStream_t) { return hipErrorUnknown; }
static hipError_t slots(const char* name, const InstDev* insts, const int* s, int first, int n) {
  if (fails(name)) return hipErrorUnknown;
  for (int k = 0; k < n; ++k) CHECK(insts[s ? s[k] : first + k].Q != nullptr);
  return hipSuccess;
}
hipError_t launch_solve(int, const InstDev* i, const int* s, int first, int n, int, bool, int, hipStream_t) { return slots("launch_solve", i, s, first, n); }
hipError_t launch_ring(int, const InstDev* i, const int* s, int n, int, int, hipStream_t) { return slots("launch_ring", i, s, 0, n); }
hipError_t launch_slot_scalars(const InstDev* i, const int* s, int first, int n, int, int, hipStream_t) { return slots("launch_slot_scalars", i, s, first, n); }
hipError_t launch_slot_status(const InstDev* i, const int* s, int n, long long* out, hipStream_t) {
  for (int k = 0; k < n; ++k) {
    out[2 * k] = i[s[k]].scal->step;
    out[2 * k + 1] = 0;
  }
  return slots("launch_slot_status", i, s, 0, n);
}
hipError_t launch_cell_index(const InstDev*, int, int, int*, long long, hipStream_t) { return hipSuccess; }
hipError_t launch_sort(int, const InstDev*, int, long long, int, int*, hipStream_t) { return hipSuccess; }
bool cluster_runs(long long, int, int) { return false; }
size_t cluster_bytes(long long, int, int) { return 0; }
ClusterWs cluster_layout(long long, int, int, bool) { return ClusterWs{}; }
hipError_t cluster_static_workspace(void**) { return hipErrorUnknown; }
hipError_t cluster_check_inputs(const double*, long long, const int*, int, const int*, long long, void*, const ClusterWs&, ClusterCheck*, hipStream_t) { return hipErrorUnknown; }
hipError_t cluster_run(const double*, const double*, const double*, long long, int, const int*, const int*, int, int, int, double, double, double, void*, const ClusterWs&, bool, double*, double*, double*, double*, double*, int*, double*, int*, hipStream_t) { return hipErrorUnknown; }
}  // namespace vpk

// ---------------------------------------------------------------- checks
struct Instance {
  vp_config cfg{};
  vp_particles parts{};
  std::vector<double> arrays;  // one small block: the particles themselves are not read
  void* ws = nullptr;
  explicit Instance(long long n, int hist_cap = 16, bool monopole = false) {
    cfg.n = n; cfg.ng = 64; cfg.precision = VP_FP64; cfg.L = 1.0; cfg.dt = 0.1;
    cfg.hist_cap = hist_cap; cfg.element_order = 1; cfg.monopole_only = monopole;
    arrays.resize(monopole ? 2 * n + 8 : 16);
    double* a = arrays.data();
    parts = {a, a + 1, a + 8, monopole ? a + 8 + n : a + 2, a + 3, nullptr, nullptr, nullptr};
    size_t b = 0;
    CHECK(vp_workspace_bytes(&cfg, &b) == VP_OK);
    ws = std::aligned_alloc(256, b);
  }
  Instance(const Instance&) = delete;
  ~Instance() { std::free(ws); }
};

// One step of the engine takes exactly the particles of these instances, each once.
static void check_step(vp_handle* h, const std::vector<const Instance*>& in) {
  stepped.clear();
  CHECK(vp_step(h, 1) == VP_OK);
  std::map<void*, long long> next;
  for (const auto& [at, count] : stepped) {  // in order of the first particle
    CHECK(next[at.first] == at.second);
    next[at.first] += count;
  }
  CHECK(next.size() == in.size());
  for (const Instance* i : in) CHECK(next[i->parts.Q] == i->cfg.n);
}

static void check_reads(vp_handle* h, int slot, int steps) {
  std::vector<vp_diag> d(steps);
  CHECK(vp_history(h, slot, 0, steps, d.data()) == VP_OK);
  for (int k = 0; k < steps; ++k) CHECK(d[k].step == k && d[k].K == k);
  CHECK(vp_diagnostics(h, slot, d.data(), nullptr) == VP_OK && d[0].K == 7.0 && d[0].step == steps);
  std::vector<double> grid(4 * 64);
  CHECK(vp_diagnostics(h, slot, d.data(), grid.data()) == VP_OK);
  int64_t st[8];
  int32_t fl[8];
  CHECK(vp_slot_status(h, 8, st, fl) == VP_OK && st[slot] == steps && fl[slot] == VP_SLOT_OCCUPIED);
}

// Admissions, reads and retirements where no pinned memory is to be had.
static void no_pinned_memory() {
  fail_at["hipHostMalloc"] = -1;
  Instance a(5000), b(700, 3000, true), c(1 << 20);
  vp_handle* h = nullptr;
  CHECK(vp_engine_create(VP_FP64, 8, nullptr, &h) == VP_OK);
  CHECK(vp_admit(h, 3, &a.cfg, a.parts, a.ws) == VP_OK);
  check_step(h, {&a});
  check_reads(h, 3, 1);
  CHECK(vp_admit(h, 0, &b.cfg, b.parts, b.ws) == VP_OK);
  CHECK(vp_admit(h, 5, &c.cfg, c.parts, c.ws) == VP_OK);
  check_step(h, {&a, &b, &c});
  for (int k = 0; k < 2899; ++k) CHECK(vp_step(h, 1) == VP_OK);
  check_reads(h, 0, 2900);  // a read-back above the pinned one's size
  CHECK(vp_retire(h, 3) == VP_OK);
  check_step(h, {&b, &c});
  vp_tuning t{256, 4, 2, 0, 33, 0, 0};
  CHECK(vp_set_tuning(h, &t) == VP_OK);
  check_step(h, {&b, &c});
  CHECK(vp_admit(h, 3, &a.cfg, a.parts, a.ws) == VP_OK);
  check_step(h, {&a, &b, &c});
  CHECK(pinned_most == 0);
  CHECK(vp_destroy(h) == VP_OK);
}

// The pinned block stays small where the tables are large.
static void large_tables() {
  Instance a(5000), c(1 << 26);
  vp_handle* h = nullptr;
  CHECK(vp_engine_create(VP_FP64, 8, nullptr, &h) == VP_OK);
  CHECK(vp_admit(h, 1, &a.cfg, a.parts, a.ws) == VP_OK);
  CHECK(vp_admit(h, 2, &c.cfg, c.parts, c.ws) == VP_OK);
  check_step(h, {&a, &c});
  vp_tuning t{256, 1, 4, 0, 33, 0, 0};  // 262144 tiles, 8 MiB
  CHECK(vp_set_tuning(h, &t) == VP_OK);
  check_step(h, {&a, &c});
  CHECK(vp_retire(h, 1) == VP_OK);
  check_step(h, {&c});
  CHECK(vp_admit(h, 1, &a.cfg, a.parts, a.ws) == VP_OK);
  check_step(h, {&a, &c});
  check_reads(h, 1, 1);
  CHECK(vp_retire(h, 2) == VP_OK);
  check_step(h, {&a});
  CHECK(pinned_most > 0 && pinned_most <= (size_t(4) << 20));
  CHECK(vp_destroy(h) == VP_OK);
  CHECK(pinned == 0);
}

// After an upload that failed, the next one brings every table.
static void failed_upload() {
  Instance a(5000), b(20000), c(9000);
  vp_handle* h = nullptr;
  CHECK(vp_engine_create(VP_FP64, 8, nullptr, &h) == VP_OK);
  CHECK(vp_admit(h, 1, &a.cfg, a.parts, a.ws) == VP_OK);
  check_step(h, {&a});
  fail_at["launch_upload"] = 1;
  CHECK(vp_admit(h, 2, &b.cfg, b.parts, b.ws) == VP_ERR_HIP);
  CHECK(vp_admit(h, 2, &b.cfg, b.parts, b.ws) == VP_OK);
  check_step(h, {&a, &b});
  vp_tuning t{256, 4, 2, 0, 33, 0, 0}, t2{1024, 2, 8, 0, 33, 0, 0};
  CHECK(vp_set_tuning(h, &t) == VP_OK);
  fail_at["launch_upload"] = 1;
  CHECK(vp_set_tuning(h, &t2) == VP_ERR_HIP);
  check_step(h, {&a, &b});
  CHECK(vp_admit(h, 3, &c.cfg, c.parts, c.ws) == VP_OK);
  check_step(h, {&a, &b, &c});
  fail_at["launch_upload"] = 1;
  CHECK(vp_retire(h, 1) == VP_ERR_HIP);
  check_step(h, {&b, &c});
  CHECK(vp_admit(h, 1, &a.cfg, a.parts, a.ws) == VP_OK);
  check_step(h, {&a, &b, &c});
  fail_at["launch_ring"] = 1;
  CHECK(vp_set_tuning(h, &t2) == VP_ERR_HIP);
  check_step(h, {&a, &b, &c});
  CHECK(vp_set_tuning(h, &t2) == VP_OK);
  check_step(h, {&a, &b, &c});
  CHECK(vp_destroy(h) == VP_OK);
}

// Whatever call of an admission fails, the slot stays empty and the others go on; a tuning that
// fails leaves the one before.
static void failed_admission() {
  Instance a(5000), b(20000, 16, true);
  for (const char* name : {"launch_fill_zero", "launch_upload", "launch_deposit", "launch_solve"})
    for (int call = 1; call <= (std::string(name) == "launch_fill_zero" ? 2 : 1); ++call) {
      vp_handle* h = nullptr;
      CHECK(vp_engine_create(VP_FP64, 8, nullptr, &h) == VP_OK);
      CHECK(vp_admit(h, 1, &a.cfg, a.parts, a.ws) == VP_OK);
      check_step(h, {&a});
      fail_at[name] = call;
      CHECK(vp_admit(h, 2, &b.cfg, b.parts, b.ws) == VP_ERR_HIP);
      CHECK(std::strstr(vp_last_error(), "made to fail") != nullptr);
      int32_t slots = 0;
      int64_t n = 0;
      CHECK(vp_occupancy(h, &slots, &n) == VP_OK && slots == 1 && n == a.cfg.n);
      CHECK(vp_retire(h, 2) == VP_ERR_STATE);
      check_step(h, {&a});
      check_reads(h, 1, 2);
      CHECK(vp_admit(h, 2, &b.cfg, b.parts, b.ws) == VP_OK);
      check_step(h, {&a, &b});
      CHECK(vp_destroy(h) == VP_OK);
    }
  vp_handle* h = nullptr;
  CHECK(vp_engine_create(VP_FP64, 8, nullptr, &h) == VP_OK);
  CHECK(vp_admit(h, 1, &a.cfg, a.parts, a.ws) == VP_OK);
  vp_tuning t{256, 4, 2, 0, 33, 0, 0}, bad{1024, 2, 8, 0, 33, 0, 0}, got{};
  CHECK(vp_set_tuning(h, &t) == VP_OK);
  fail_at["launch_upload"] = 1;
  CHECK(vp_set_tuning(h, &bad) == VP_ERR_HIP);
  CHECK(vp_get_tuning(h, &got) == VP_OK && std::memcmp(&got, &t, sizeof t) == 0);
  int32_t th = 0, ppt = 0, k = 0;
  CHECK(vp_step_launch(h, 1, 5, &th, &ppt, &k) == VP_OK && th == 256 && ppt == 4 && k == 1);
  check_step(h, {&a});
  bad.persistent = 1;
  CHECK(vp_admit(h, 2, &b.cfg, b.parts, b.ws) == VP_OK);
  Instance c(1 << 20);
  CHECK(vp_admit(h, 0, &c.cfg, c.parts, c.ws) == VP_OK);  // 512 tiles and more: not all resident
  CHECK(vp_set_tuning(h, &bad) == VP_ERR_ARG);
  CHECK(std::strstr(vp_last_error(), "the device holds 256") != nullptr);
  CHECK(vp_get_tuning(h, &got) == VP_OK && std::memcmp(&got, &t, sizeof t) == 0);
  check_step(h, {&a, &b, &c});
  CHECK(vp_destroy(h) == VP_OK);
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> checks = {{"no_pinned_memory", no_pinned_memory},
                                                    {"large_tables", large_tables},
                                                    {"failed_upload", failed_upload},
                                                    {"failed_admission", failed_admission}};
  if (argc == 2 && checks.count(argv[1])) {
    checks.at(argv[1])();
  } else {
    for (const auto& c : checks) std::printf("%s\n", c.first.c_str());
    return argc == 1 ? 0 : 2;
  }
  return failures == 0 ? 0 : 1;
}

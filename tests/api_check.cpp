// Host check of the library's host side (psatd_api.hip), built and run by
// test_api_host.py: the HIP runtime is replaced by one in host memory that
// tracks every allocation and can refuse one, and the kernel launches by
// checks of what they are given: that every list, box and spectral plane a
// launch reaches lies inside a live allocation.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <utility>
#include <vector>

namespace fake {

struct Block {
  size_t bytes;
  bool live;
};
std::map<uintptr_t, Block> blocks;  // never reused, so that a stale pointer shows
int mallocs_left = -1, copies_left = -1;  // calls until one is refused (-1: none)
size_t largest = 0;                 // largest allocation since reset

bool covers(const void* p, size_t bytes) {
  const uintptr_t a = (uintptr_t)p;
  auto it = blocks.upper_bound(a);
  if (it == blocks.begin()) return false;
  --it;
  return it->second.live && a + bytes <= it->first + it->second.bytes;
}

bool refuse(int& left) {
  if (left < 0) return false;
  return left-- == 0;
}

// The stream under capture, and whether this thread may still allocate and copy.
hipStream_t capturing = nullptr;
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
bool capture_broken = false;
bool unsafe_in_capture() {
  if (!capturing || mode == hipStreamCaptureModeRelaxed) return false;
  return capture_broken = true;
}

hipError_t Malloc(void** p, size_t bytes) {
  *p = nullptr;
  if (unsafe_in_capture()) return hipErrorStreamCaptureUnsupported;
  if (refuse(mallocs_left)) return hipErrorOutOfMemory;
  *p = std::aligned_alloc(256, (bytes + 255) & ~(size_t)255);
  blocks[(uintptr_t)*p] = {bytes, true};
  largest = std::max(largest, bytes);
  return hipSuccess;
}
hipError_t Free(void* p) {
  if (unsafe_in_capture()) return hipErrorStreamCaptureUnsupported;
  if (p) blocks.at((uintptr_t)p).live = false;
  return hipSuccess;
}
hipError_t Memcpy(void* d, const void* s, size_t bytes) {
  if (unsafe_in_capture()) return hipErrorStreamCaptureUnsupported;
  if (refuse(copies_left)) return hipErrorUnknown;
  if (bytes) std::memcpy(d, s, bytes);
  return hipSuccess;
}

hipError_t Synchronize(hipStream_t s) {
  if (!capturing || s != capturing) return hipSuccess;
  capture_broken = true;
  return hipErrorStreamCaptureUnsupported;
}
hipError_t ExchangeMode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}

alignas(256) unsigned char scratch_memory[64 << 20];
hipError_t SymbolAddress(void** p) {
  *p = scratch_memory;
  blocks[(uintptr_t)scratch_memory] = {sizeof(scratch_memory), true};
  return hipSuccess;
}

}  // namespace fake

#define hipMalloc(p, n) fake::Malloc((void**)(p), n)
#define hipFree(p) fake::Free(p)
#define hipMemcpy(d, s, n, kind) fake::Memcpy(d, s, n)
#define hipMemcpyAsync(d, s, n, kind, st) fake::Memcpy(d, s, n)
#define hipGetSymbolAddress(p, sym) fake::SymbolAddress(p)
#define hipGetDevice(d) (*(d) = 0, hipSuccess)
#define hipGetDeviceProperties(p, d) hipErrorInvalidDevice
#define hipGetLastError() hipSuccess
#define hipStreamCreateWithFlags(s, f) (*(s) = (hipStream_t)(uintptr_t)1, hipSuccess)
#define hipStreamDestroy(s) hipSuccess
#define hipStreamSynchronize(s) fake::Synchronize(s)
#define hipStreamBeginCapture(s, m) hipSuccess
#define hipStreamEndCapture(s, g) hipSuccess
#define hipGraphInstantiate(x, g, a, b, c) hipSuccess
#define hipGraphLaunch(x, s) hipSuccess
#define hipGraphDestroy(g) hipSuccess
#define hipGraphExecDestroy(x) hipSuccess
#define hipThreadExchangeStreamCaptureMode(m) fake::ExchangeMode(m)

#include "psatd_api.hip"

namespace {

int g_fail = 0;
#define CHECK(c, ...)                      \
  do {                                     \
    if (!(c)) {                            \
      std::fprintf(stderr, __VA_ARGS__);   \
      std::fprintf(stderr, " (%s)\n", #c); \
      ++g_fail;                            \
      return;                              \
    }                                      \
  } while (0)

std::string g_launch_error;  // what the first launch out of bounds reached
std::string g_trace;         // the launches of a call
std::vector<std::pair<const void*, std::vector<unsigned char>>> g_reads;  // lists they were given

void reach(const void* p, size_t bytes, const char* what) {
  if (!fake::covers(p, bytes)) {
    if (g_launch_error.empty()) g_launch_error = what;
    return;
  }
  const unsigned char* b = (const unsigned char*)p;
  g_reads.push_back({p, {b, b + bytes}});
}

size_t csize(const DevPlan& p) { return p.f64 ? 16 : 8; }

void spectral(const DevPlan& p, const void* spec, int64_t first, int64_t elems) {
  if (first < 0 || !fake::covers((const char*)spec + first * (int64_t)csize(p), elems * csize(p)))
    if (g_launch_error.empty()) g_launch_error = "workspace";
}

void planes(const DevPlan& p, const PlaneRec* list, int at, int n, bool fwd, int64_t sbias, const void* spec) {
  reach(p.box, p.nsub * sizeof(BoxD), "boxes");
  reach(list + at, n * sizeof(PlaneRec), "planes");
  if (!g_launch_error.empty()) return;
  for (int i = at; i < at + n; ++i) {
    const PlaneRec& r = list[i];
    if (r.box < 0 || r.box >= p.nsub || r.z < 0 || r.z >= (fwd ? p.box[r.box].P[2] : p.box[r.box].n[2])) {
      g_launch_error = "plane record";
      return;
    }
    const BoxD& b = p.box[r.box];
    const int64_t pl = (int64_t)b.P[1] * b.H;
    if (fwd && !p.split) reach(p.pullp + r.p0, (r.p1 - r.p0) * sizeof(PullPiece), "pull pieces");
    for (int f = 0; f < (fwd ? 9 : 6); ++f)
      spectral(p, spec, fwd ? b.sb - sbias + f * b.sv + ring_slot(b, r.z) * b.pp : result_plane(b, sbias, f, r.z), pl);
  }
}

void ztiles(const DevPlan& p, const ZLaunch& l, int64_t sbias, const void* spec) {
  reach(p.box, p.nsub * sizeof(BoxD), "boxes");
  reach(p.tiles + l.u0, l.nu * sizeof(ZItem), "z tiles");
  if (!g_launch_error.empty()) return;
  for (int i = l.u0; i < l.u0 + l.nu; ++i) {
    const ZItem& t = p.tiles[i];
    if (t.box < 0 || t.box >= p.nsub || t.q0 < 0 || t.q0 >= p.box[t.box].P[1] * p.box[t.box].H) {
      g_launch_error = "z tile";
      return;
    }
    const BoxD& b = p.box[t.box];
    for (int f = 0; f < 9; ++f) spectral(p, spec, b.sb - sbias + f * b.sv + t.q0, 1);
  }
}

void note(const char* k, int n) { g_trace += std::string(k) + " " + std::to_string(n) + "\n"; }

}  // namespace

namespace psatd {

hipError_t launch_fill(const DevPlan&, void* const*, int ncomp, hipStream_t) {
  note("fill", ncomp);
  return hipSuccess;
}
hipError_t launch_sum(const DevPlan&, void* const*, hipStream_t) {
  note("sum", 3);
  return hipSuccess;
}
hipError_t launch_fwd(const DevPlan& p, const XyLaunch& l, int64_t sbias, void* const*, int nf, int, void* spec,
                      hipStream_t) {
  planes(p, p.fwd, l.f0, l.nf, true, sbias, spec);
  note("fwd", nf * l.nf);
  return hipSuccess;
}
hipError_t launch_upd(const DevPlan& p, const ZLaunch& l, int64_t sbias, void* spec, hipStream_t) {
  ztiles(p, l, sbias, spec);
  note("upd", l.nu);
  return hipSuccess;
}
hipError_t launch_upd_reg(const DevPlan& p, void*, hipStream_t) {
  reach(p.box, p.nsub * sizeof(BoxD), "boxes");
  note("upd_reg", p.nzg);
  return hipSuccess;
}
hipError_t launch_inv(const DevPlan& p, const XyLaunch& l, int64_t sbias, const void* spec, void* const*, int nf,
                      hipStream_t) {
  planes(p, p.inv, l.i0, l.ni, false, sbias, spec);
  note(l.half ? "inv in halves" : "inv", nf * l.ni);
  return hipSuccess;
}
hipError_t launch_heat_z(const DevPlan& p, const ZLaunch& l, void* spec, double, double, hipStream_t) {
  ztiles(p, l, 0, spec);
  note("heat", l.nu);
  return hipSuccess;
}
hipError_t launch_x_fwd(const DevPlan& p, const XyLaunch& l, void* const*, int nf, void* spec, hipStream_t) {
  planes(p, p.fwd, l.f0, l.nf, true, 0, spec);
  note("x_fwd", nf * l.nf);
  return hipSuccess;
}
hipError_t launch_y(const DevPlan& p, const XyLaunch& l, int dir, int nf, void* spec, hipStream_t) {
  planes(p, dir < 0 ? p.fwd : p.inv, dir < 0 ? l.c0 : l.d0, dir < 0 ? l.nc : l.nd, dir < 0, 0, spec);
  note(dir < 0 ? "y_fwd" : "y_inv", nf * (dir < 0 ? l.nc : l.nd));
  return hipSuccess;
}
hipError_t launch_x_inv(const DevPlan& p, const XyLaunch& l, const void* spec, void* const*, hipStream_t) {
  planes(p, p.inv, l.i0, l.ni, false, 0, spec);
  note("x_inv", 6 * l.ni);
  return hipSuccess;
}
hipError_t launch_scatter(const DevPlan&, const void* const*, void* const*, hipStream_t) { return hipSuccess; }
hipError_t launch_gather(const DevPlan&, const void* const*, void* const*, hipStream_t) { return hipSuccess; }
hipError_t launch_modk(const KEntry*, int, int, int, double*, hipStream_t) { return hipSuccess; }
hipError_t prepare_kernels(bool, int, int, int, int, int, int) { return hipSuccess; }

}  // namespace psatd

namespace {

// N^3 grid in k^3 equal boxes with guards g.
psatd_plan_t cubes(int64_t N, int k, int32_t g, int prec) {
  std::vector<int64_t> lo, n;
  std::vector<int32_t> gu;
  for (int z = 0; z < k; ++z)
    for (int y = 0; y < k; ++y)
      for (int x = 0; x < k; ++x)
        for (int c : {x, y, z}) {
          lo.push_back(c * N / k);
          n.push_back(N / k);
          gu.push_back(g);
        }
  const int64_t gn[3] = {N, N, N};
  const double gd[3] = {1, 1, 1};
  psatd_plan_t p = nullptr;
  if (psatd_plan(&p, gn, gd, k * k * k, lo.data(), n.data(), gu.data(), 8, 0.5, 1.0, prec, PSATD_J_REPLICATED,
                 nullptr) != PSATD_OK)
    std::fprintf(stderr, "plan: %s\n", psatd_last_error(nullptr));
  return p;
}

alignas(16) unsigned char field[16];
void* const F[3] = {field, field, field};  // never read: the launches are checks

// The launches of a call, or why it failed.
std::string trace(const std::function<psatd_status()>& call) {
  g_trace.clear();
  g_launch_error.clear();
  g_reads.clear();
  const psatd_status st = call();
  if (st != PSATD_OK) return "status " + std::to_string(st);
  if (!g_launch_error.empty()) return "out of bounds: " + g_launch_error;
  return g_trace;
}
std::string step(psatd_plan_t p) { return trace([&] { return psatd_step(p, F, F, F); }); }
bool ok(const std::string& t) { return t.find("fwd") != std::string::npos && t.find("out of") == std::string::npos; }

std::vector<int32_t> knobs(psatd_plan_t p) {
  std::vector<int32_t> v(PSATD_NTUNE);
  for (int k = 0; k < PSATD_NTUNE; ++k) psatd_get_tuning(p, k, &v[k]);
  return v;
}

// A batched plan's own workspace holds one batch (psatd_workspace_bytes), an
// unbatched one's at most the pitched planes; a caller's may be as small as
// psatd_workspace_bytes says.
void check_workspace(int prec) {
  for (int per : {1, 3, 0}) {
    psatd_plan_t p = cubes(48, 2, 8, prec);
    CHECK(p && psatd_set_tuning(p, PSATD_TUNE_BATCH_BOXES, per) == PSATD_OK, "workspace: plan");
    int64_t need = 0;
    CHECK(psatd_workspace_bytes(p, &need) == PSATD_OK, "workspace: size");
    fake::largest = 0;
    CHECK(ok(step(p)), "workspace, batches of %d: %s", per, step(p).c_str());
    const int64_t most = per ? need : p->h.lists.elems * (int64_t)(2 * real_size(p->h.prec));
    CHECK((int64_t)fake::largest <= std::max<int64_t>(most, need), "batches of %d: plan takes %zu bytes, needs %lld",
          per, fake::largest, (long long)need);
    void* own = nullptr;
    CHECK(fake::Malloc(&own, need) == hipSuccess && psatd_set_workspace(p, own, need) == PSATD_OK,
          "workspace: caller's");
    CHECK(ok(step(p)), "caller workspace, batches of %d: %s", per, step(p).c_str());
    psatd_destroy(p);
  }
  std::printf("workspace ok\n");
}

// The knobs that remake the work lists, each with a value other than the default.
struct Knob {
  int32_t key, value;
};
const Knob kListKnobs[] = {{PSATD_TUNE_Z_PENCILS, 4}, {PSATD_TUNE_SPLIT_XY, 1}, {PSATD_TUNE_BATCH_BOXES, 3},
                           {PSATD_TUNE_FUSE_EB, 1},   {PSATD_TUNE_XY_THREADS, 1024}, {PSATD_TUNE_Z_THREADS, 1024}};

// A knob whose lists cannot be allocated or copied to the device leaves the plan as it was.
void check_failures(int prec) {
  for (const Knob& k : kListKnobs)
    for (int which = 0; which < 4; ++which) {  // the first or the second allocation or copy
      const int copy = which & 1, nth = which >> 1;
      psatd_plan_t p = cubes(48, 2, 8, prec);
      // lists shorter than any that the knobs make, so that stale ones show
      CHECK(p && psatd_set_tuning(p, PSATD_TUNE_Z_PENCILS, 8) == PSATD_OK, "failures: plan");
      const std::string before = step(p);
      const std::vector<int32_t> was = knobs(p);
      CHECK(ok(before), "failures: %s", before.c_str());
      (copy ? fake::copies_left : fake::mallocs_left) = nth;
      const psatd_status st = psatd_set_tuning(p, k.key, k.value);
      const bool tried = (copy ? fake::copies_left : fake::mallocs_left) < 0;
      fake::mallocs_left = fake::copies_left = -1;
      CHECK(tried == (st != PSATD_OK), "knob %d: a refused upload is reported", k.key);
      if (tried) {
        CHECK(st == (copy ? PSATD_E_HIP : PSATD_E_NOMEM), "knob %d: status %d", k.key, st);
        CHECK(knobs(p) == was, "knob %d: a failed call keeps the knobs", k.key);
        const std::string after = step(p);
        CHECK(after == before, "knob %d: after a failed call: %s", k.key, after.c_str());
      }
      CHECK(psatd_set_tuning(p, k.key, k.value) == PSATD_OK && ok(step(p)), "knob %d: %s", k.key, step(p).c_str());
      psatd_destroy(p);
    }
  std::printf("failures ok\n");
}

// What a step's launches were given stays as it was through later tuning calls:
// they may not have run yet (another stream), or run again (a captured graph).
void check_lists_stay(int prec) {
  auto live = [] {
    size_t n = 0;
    for (const auto& b : fake::blocks) n += b.second.live;
    return n;
  };
  const size_t outside = live();
  psatd_plan_t p = cubes(48, 2, 8, prec);
  const std::vector<int32_t> first = knobs(p);
  CHECK(ok(trace([&] { return psatd_step_noalloc(p, F, F, F); })), "lists: step");
  const auto given = g_reads;
  size_t blocks = 0;
  for (int round = 0; round < 3; ++round) {
    for (const Knob& k : kListKnobs) {
      CHECK(psatd_set_tuning(p, k.key, k.value) == PSATD_OK && ok(step(p)), "lists: knob %d", k.key);
      for (const auto& g : given)
        CHECK(fake::covers(g.first, g.second.size()) && !std::memcmp(g.first, g.second.data(), g.second.size()),
              "lists: rewritten or freed by knob %d", k.key);
      CHECK(psatd_set_tuning(p, k.key, first[k.key]) == PSATD_OK, "lists: knob %d back", k.key);
    }
    for (int k : {PSATD_TUNE_FUSE_EB, PSATD_TUNE_XY_THREADS, PSATD_TUNE_Z_PENCILS, PSATD_TUNE_PULL_EB})
      CHECK(psatd_set_tuning(p, k, first[k]) == PSATD_OK, "lists: knob %d back", k);
    if (round == 1) blocks = fake::blocks.size();
  }
  CHECK(fake::blocks.size() == blocks, "lists: settings that come back allocate again");
  psatd_destroy(p);
  CHECK(live() == outside, "lists: memory not given back");
  std::printf("lists ok\n");
}

// The knobs that only choose among launches may be set while a stream, the plan's
// own too, is being captured.
void check_capture(int prec) {
  psatd_plan_t p = cubes(48, 2, 8, prec);
  const hipStream_t st = (hipStream_t)(uintptr_t)2;
  CHECK(psatd_set_stream(p, st) == PSATD_OK, "capture: stream");
  fake::capturing = st;
  for (const Knob& k : kListKnobs) {
    CHECK(ok(trace([&] { return psatd_step_noalloc(p, F, F, F); })), "capture: step");
    CHECK(psatd_set_tuning(p, k.key, k.value) == PSATD_OK && !fake::capture_broken, "capture: knob %d", k.key);
    if (k.key == PSATD_TUNE_SPLIT_XY) CHECK(psatd_set_tuning(p, k.key, 0) == PSATD_OK, "capture: unsplit");
    if (k.key == PSATD_TUNE_BATCH_BOXES) CHECK(psatd_set_tuning(p, k.key, 0) == PSATD_OK, "capture: unbatched");
  }
  CHECK(fake::mode == hipStreamCaptureModeGlobal, "capture: the thread's mode is given back");
  fake::capturing = nullptr;
  psatd_destroy(p);
  std::printf("capture ok\n");
}

}  // namespace

int main() {
  check_workspace(PSATD_F32_VALU);
  check_workspace(PSATD_F64);
  check_failures(PSATD_F32_VALU);
  check_failures(PSATD_F64);
  check_lists_stay(PSATD_F32_VALU);
  check_lists_stay(PSATD_F64);
  check_capture(PSATD_F32_VALU);
  check_capture(PSATD_F64);
  return g_fail ? 1 : 0;
}

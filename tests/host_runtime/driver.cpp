// The host code of the C ABI on a runtime of this file's own (memory from malloc,
// copies at once, graphs and events as empty handles) and with launchers that only
// record (launch_stubs.hip): what the stepping calls allocate, launch and wait for.
// Usage: driver SCENARIO; prints "ok" and exits 0.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

#include "../../include/rmrt.h"
#include "record.hpp"

// ---------------------------------------------------------------------------
// runtime
// ---------------------------------------------------------------------------
static std::map<void*, size_t> live;   // device and pinned allocations
static size_t live_bytes = 0;
static int allocations = 0, fail_at = 0;   // the fail_at-th allocation from here on fails
static int waits = 0;                      // stream and device synchronisations
static int event_waits = 0, fail_event_at = 0;

static hipError_t take(void** p, size_t n) {
  if (fail_at > 0 && ++allocations == fail_at) {
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  *p = calloc(1, n ? n : 1);
  live[*p] = n;
  live_bytes += n;
  return hipSuccess;
}
static hipError_t give(void* p) {
  auto it = live.find(p);
  if (it == live.end()) {
    fprintf(stderr, "freed what was not allocated\n");
    exit(1);
  }
  live_bytes -= it->second;
  live.erase(it);
  free(p);
  return hipSuccess;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return take(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return take(p, n); }
hipError_t hipFree(void* p) { return give(p); }
hipError_t hipHostFree(void* p) { return give(p); }
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = (size_t)256 << 30;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipDeviceSynchronize(void) { return ++waits, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return ++waits, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char symbol[1 << 16];
  return *p = symbol, hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = nullptr, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *e = nullptr, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphUpload(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
  return fail_event_at > 0 && ++event_waits == fail_event_at ? hipErrorLaunchFailure : hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
}

// ---------------------------------------------------------------------------
// contexts
// ---------------------------------------------------------------------------
#define CHECK(cond)                                                              \
  do {                                                                           \
    if (!(cond)) {                                                               \
      fprintf(stderr, "%s: line %d: %s\n", where.c_str(), __LINE__, #cond);      \
      exit(1);                                                                   \
    }                                                                            \
  } while (0)

struct Form {
  const char* name;
  int lattice, storage, pattern, nx, ny, nz, domains;   // domains 0: a single one
};
static const Form forms[] = {
    {"tiles AA", RMRT_Q9, RMRT_F32DEV, RMRT_AA, 512, 512, 1, 0},  {"tiles AB", RMRT_Q9, RMRT_F64, RMRT_AB, 512, 512, 1, 0},
    {"sweep AA", RMRT_Q19, RMRT_F32DEV, RMRT_AA, 128, 128, 96, 0}, {"sweep AB", RMRT_Q19, RMRT_F64, RMRT_AB, 128, 128, 96, 0},
    {"batch AA", RMRT_Q9, RMRT_F32DEV, RMRT_AA, 256, 200, 1, 3},  {"batch AB", RMRT_Q9, RMRT_F64, RMRT_AB, 256, 200, 1, 3},
};

struct Runner {
  rmrt_params p;
  rmrt_ctx* c = nullptr;
  rmrt_batch* b = nullptr;
  char f[8];   // the launchers touch no populations
  std::string where;
  explicit Runner(const Form& fm) : where(fm.name) {
    memset(&p, 0, sizeof(p));
    p.lattice = fm.lattice;
    p.equation = RMRT_NSE;
    p.storage = fm.storage;
    p.pattern = fm.pattern;
    p.n[0] = fm.nx;
    p.n[1] = fm.ny;
    p.n[2] = fm.nz;
    for (int a = 0; a < 3; ++a) p.dx[a] = 1.0;
    p.dt = 1.0;
    p.cs2 = p.nu_b = p.s_hi = p.w_corner = -1.0;
    p.nu = 0.05;
    p.rho0 = 1.0;
    for (double& v : p.nu_tensor) v = -1.0;
    for (double& v : p.nu_b_axis) v = -1.0;
    const bool ab = fm.pattern == RMRT_AB;
    const double rho = 1.0;
    int rc;
    if (fm.domains == 0) {
      rc = rmrt_init(&c, &p, f, ab ? f + 1 : nullptr, nullptr, &rho, &rho, 0, nullptr);
    } else {
      rmrt_params ps[3] = {p, p, p};
      void* f0[3] = {f, f, f};
      void* f1[3] = {f + 1, f + 1, f + 1};
      rc = rmrt_batch_create(&b, fm.domains, ps, f0, ab ? f1 : nullptr, nullptr, nullptr);
    }
    if (rc != RMRT_OK) fprintf(stderr, "%s\n", rmrt_last_error());
    CHECK(rc == RMRT_OK);
  }
  int step(int n) { return c ? rmrt_step(c, n, nullptr) : rmrt_batch_step(b, n, nullptr); }
  int tune() {
    int k;
    return c ? rmrt_tune(c, 2, nullptr, &k) : rmrt_batch_autotune(b, 2, nullptr, &k);
  }
  int launches_of(int n, int* k) {
    return c ? rmrt_step_launches(c, n, k) : rmrt_batch_step_launches(b, n, k);
  }
  int pin() {
    if (b) return rmrt_batch_set_config(b, 0);
    int cap, fl;
    rmrt_get_launch(c, &cap, &fl);
    return rmrt_set_launch(c, cap, fl);
  }
  // the launches of a call of n steps that is captured afresh; true with passes
  bool passes(int n) {
    launches.clear();
    CHECK(step(n) == RMRT_OK);
    int steps = 0, np = 0;
    for (const Launch& l : launches) {
      steps += l.steps;
      np += l.kind != 0;
    }
    CHECK(steps == n && np % 2 == 0);
    return np > 0;
  }
  ~Runner() {
    if (c) rmrt_free(c);
    if (b) rmrt_batch_free(b);
  }
};

// The first call of four steps or more without one of its allocations: single
// steps, and nothing kept that only passes use.
static void out_of_memory() {
  for (const Form& fm : forms) {
    int tried = 0;
    for (bool reached = true; reached; ++tried) {
      const std::string where = std::string(fm.name) + ", allocation " + std::to_string(tried + 1);
      {
        Runner r(fm);
        const size_t before = live_bytes;
        allocations = 0;
        fail_at = tried + 1;
        const bool passes = r.passes(8);
        reached = allocations >= fail_at;
        fail_at = 0;
        CHECK(passes == !reached);
        CHECK(passes || live_bytes == before);
        CHECK(r.passes(16) == passes);
      }
      CHECK(live.empty());
    }
    const std::string where = fm.name;
    CHECK(tried >= 2);
  }
}

// The first call of four steps or more waits for nothing; the preparing call, after
// which steps may come on any stream, does.
static void no_wait() {
  for (const Form& fm : forms) {
    const std::string where = fm.name;
    Runner r(fm), prepared(fm);
    waits = 0;
    CHECK(r.passes(8));
    CHECK(waits == 0);
    CHECK((prepared.c ? rmrt_step_prepare(prepared.c, 8, nullptr) : rmrt_batch_step_prepare(prepared.b, 8, nullptr)) == RMRT_OK);
    CHECK(waits > 0);
    waits = 0;
    CHECK(prepared.step(8) == RMRT_OK);
    CHECK(waits == 0);
  }
}

// Tuning that fails leaves a context on passes, or on the single steps that it was
// kept on; tuning that ends puts it on passes.
static void failed_tuning() {
  for (const Form& fm : forms)
    for (int pinned = 0; pinned < 2; ++pinned)
      for (int k : {1, 3, 0}) {
        const std::string where = std::string(fm.name) + (pinned ? ", pinned" : "") + ", event " + std::to_string(k);
        Runner r(fm);
        if (pinned) CHECK(r.pin() == RMRT_OK);
        event_waits = 0;
        fail_event_at = k;
        CHECK((r.tune() == RMRT_OK) == (k == 0));
        fail_event_at = 0;
        CHECK(r.passes(8) == (k == 0 || !pinned));
        CHECK(r.passes(2) == false);
      }
}

// The launches that a context reports for a call are the ones that the call makes.
static void counted_launches() {
  for (const Form& fm : forms)
    for (int pinned = 0; pinned < 2; ++pinned)
      for (int n : {1, 2, 3, 4, 5, 6, 7, 8, 11, 13, 14, 20, 37, 100, 256, 300}) {
        const std::string where = std::string(fm.name) + ", steps " + std::to_string(n);
        Runner r(fm);
        if (pinned) CHECK(r.pin() == RMRT_OK);
        int k = -1;
        CHECK(r.launches_of(n, &k) == RMRT_OK && k == n);   // nothing set up yet
        CHECK((r.c ? rmrt_step_prepare(r.c, n, nullptr) : rmrt_batch_step_prepare(r.b, n, nullptr)) == RMRT_OK);
        for (int again = 0; again < 2; ++again) {   // an even and, after odd calls, an odd step count
          Runner same(fm);                          // (calls captured afresh)
          if (pinned) CHECK(same.pin() == RMRT_OK);
          if (again) CHECK(same.step(1) == RMRT_OK && r.step(1) == RMRT_OK);
          launches.clear();
          CHECK(same.step(n) == RMRT_OK);
          CHECK(r.launches_of(n, &k) == RMRT_OK && k == (int)launches.size());
          CHECK(!pinned || k == n);
        }
        CHECK(r.launches_of(-1, &k) == RMRT_EINVAL);
        CHECK(r.launches_of(0, &k) == RMRT_OK && k == 0);
      }
}

// A call on rD2Q9 that takes no passes sets none up; a later one that does finds them.
static void only_for_passes() {
  const Form wide[] = {
      {"tiles AA, wide", RMRT_Q9, RMRT_F32DEV, RMRT_AA, 1500, 700, 1, 0},
      {"tiles AB, wide", RMRT_Q9, RMRT_F64, RMRT_AB, 1024, 512, 1, 0},
      {"batch AA, wide", RMRT_Q9, RMRT_F32DEV, RMRT_AA, 1500, 1024, 1, 3},
      forms[1], forms[5],
  };
  for (const Form& fm : wide) {
    const std::string where = fm.name;
    Runner r(fm);
    CHECK(r.step(1) == RMRT_OK);   // calls of four steps from an odd one: three from an even one
    for (int n : {2, 3, 4, 5, 4}) {
      const size_t before = live_bytes;
      CHECK(r.passes(n) || live_bytes == before);
    }
    CHECK(r.passes(24));
  }
}

int main(int argc, char** argv) {
  const std::string s = argc > 1 ? argv[1] : "";
  if (s == "out_of_memory") out_of_memory();
  else if (s == "no_wait") no_wait();
  else if (s == "failed_tuning") failed_tuning();
  else if (s == "counted_launches") counted_launches();
  else if (s == "only_for_passes") only_for_passes();
  else return fprintf(stderr, "unknown scenario\n"), 1;
  printf("ok\n");
  return 0;
}

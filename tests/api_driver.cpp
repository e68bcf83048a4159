// The C ABI's host side (bdrs_api.hip compiled by the host compiler) on a
// simulated runtime: device memory is host memory, a launch only records what
// it would have read and written.  One scenario per run, named on the command
// line; prints "ok" at the end.
//
// The simulated stream counts its unfinished launches, so a call that returns
// before its results are there is seen.  While it is under capture launches go
// into the capture and a wait is refused.
#include "bdrs_host.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

using namespace bdrs;

namespace {

int g_pending = 0;         // launches and copies enqueued and not yet waited for
bool g_capturing = false;  // the stream is under capture
int g_captured = 0;        // launches that went into the capture

#define EXPECT(cond)                                                              \
  do {                                                                            \
    if (!(cond)) {                                                                \
      std::printf("%s:%d: %s  [%s]\n", __FILE__, __LINE__, #cond, bdrs_last_error()); \
      std::exit(1);                                                               \
    }                                                                             \
  } while (0)

hipError_t launched() {
  ++(g_capturing ? g_captured : g_pending);
  return hipSuccess;
}

}  // namespace

// ---------------------------------------------------------------------------
// runtime
// ---------------------------------------------------------------------------
extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "none" : "simulated"; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorNotSupported; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return ++g_pending, hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return ++g_pending, hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  if (g_capturing) return hipErrorStreamCaptureUnsupported;
  return g_pending = 0, hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
// an event stands for the launches that were pending when it was recorded
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t) new int(0), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete (int*)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return *(int*)e = g_pending, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) {
  g_pending -= *(int*)e < g_pending ? *(int*)e : g_pending;
  return *(int*)e = 0, hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
namespace bdrs_host {
bool tuned_splits(int, int, int, int*, int*) { return false; }
}  // namespace bdrs_host

namespace bdrs {
int choose_splits(int, int ntiles_in) { return ntiles_in < 2 ? 1 : 2; }
hipError_t launch_pack(const LaunchCtx&, bool, const double*, double) { return launched(); }
hipError_t launch_pack_state(const LaunchCtx&, bool, double, bool) { return launched(); }
hipError_t launch_repair_pack(const LaunchCtx&) { return launched(); }
hipError_t launch_prologue(const LaunchCtx&) { return launched(); }
hipError_t launch_repack(const LaunchCtx&) { return launched(); }
hipError_t launch_sweep(const LaunchCtx&, bool, bool, int, double, int) { return launched(); }
hipError_t launch_sweep_bary(const LaunchCtx&, int, double) { return launched(); }
hipError_t launch_finish(const LaunchCtx&, bool, FinishKind, int, double*, int) { return launched(); }
hipError_t launch_advance(Ctrl* c, int n, hipStream_t) { return c->k += n, launched(); }
hipError_t launch_cert_reduce(const LaunchCtx& c) {
  // a finite certificate of the iteration before the counter
  const double rec[8] = {(double)(c.ctrl->k - 1), 0.1, 0.5, 1.0, 0.1, 0.9, 1.0, 0.0};
  std::memcpy(c.cert_out, rec, sizeof rec);
  return launched();
}
hipError_t launch_repair_reduce(const LaunchCtx&) { return launched(); }
hipError_t launch_round_reduce(const LaunchCtx& c) {
  for (int i = 8; i < 12; ++i) c.plan_stats[i] = 1.0;
  return launched();
}
hipError_t launch_plan_stats(const LaunchCtx&) { return launched(); }
hipError_t launch_export_factors(const LaunchCtx&, bool, const double*, double*, double*, double*, double*) {
  return launched();
}
hipError_t launch_plan_entries(const LaunchCtx&, const double*, const double*, const double*, const double*, double,
                               long long, long long, double*) {
  return launched();
}
hipError_t launch_count_tiles(const LaunchCtx&, int) { return launched(); }
hipError_t launch_scatter(const StateVecs&, hipStream_t) { return launched(); }
hipError_t launch_gather(const StateVecs&, hipStream_t) { return launched(); }
hipError_t launch_hints_out(const LaunchCtx&, int*, int*) { return launched(); }
hipError_t launch_hints_in(const LaunchCtx&, const int*, const int*) { return launched(); }
hipError_t launch_sweep_batch(const BatchItem*, int, const LaunchCtx*, int, bool, bool, int, hipStream_t) {
  return launched();
}
hipError_t launch_finish_batch(const BatchItem*, int, const LaunchCtx*, int, FinishKind, int, hipStream_t) {
  return launched();
}
hipError_t launch_advance_batch(const LaunchCtx*, int, int, hipStream_t) { return launched(); }
hipError_t launch_cert_batch(const BatchItem*, int, const int*, int, const LaunchCtx*, double*, hipStream_t) {
  return launched();
}
}  // namespace bdrs

// ---------------------------------------------------------------------------
// scenarios
// ---------------------------------------------------------------------------
namespace {

constexpr int kM = 130, kN = 70, kDim = 2;

struct Problem {
  std::vector<float> x, y;
  std::vector<double> r, c, w, out;
  std::vector<char> ws;
  bdrs_solver s = nullptr;
  explicit Problem(unsigned flags = 0) {
    for (int i = 0; i < kM * kDim; ++i) x.push_back((float)((i * 37) % 101) / 101.f);
    for (int i = 0; i < kN * kDim; ++i) y.push_back((float)((i * 53) % 97) / 97.f);
    r.assign(kM, 1.0 / kM);
    c.assign(kN, 1.0 / kN);
    w.assign(kM, 0.0);
    out.assign(kM, 0.0);
    bdrs_params p{};
    p.m = kM, p.n = kN, p.dim = kDim;
    p.x = x.data(), p.y = y.data(), p.r = r.data(), p.c = c.data();
    p.cost_scale = 0.5, p.eta = 1.0, p.lambda = 1.0, p.omega = 1.0;
    p.flags = flags | BDRS_F_NO_GRAPH;
    p.stream = (void*)&ws;  // a stream of its own, not the default one
    size_t bytes = 0;
    EXPECT(bdrs_workspace_size(&p, &bytes) == BDRS_OK);
    ws.resize(bytes + 256);
    p.workspace = (void*)(((uintptr_t)ws.data() + 255) / 256 * 256);
    p.workspace_bytes = bytes;
    EXPECT(bdrs_create(&p, &s) == BDRS_OK);
    EXPECT(bdrs_step(s, 3) == BDRS_OK);
  }
  ~Problem() { (void)bdrs_destroy(s); }
};

// A call that hands results back in caller memory has waited for them.
void results_are_there() {
  Problem p;
  for (int transpose = 0; transpose < 2; ++transpose) {
    EXPECT(bdrs_step(p.s, 1) == BDRS_OK && g_pending > 0);
    EXPECT(bdrs_lse(p.s, transpose, 0.1, p.w.data(), p.out.data()) == BDRS_OK);
    EXPECT(g_pending == 0);
  }
}

// A call that has to wait refuses a stream under capture and leaves nothing in it.
void refused_under_capture() {
  Problem p;
  g_capturing = true;
  for (int transpose = 0; transpose < 2; ++transpose) {
    EXPECT(bdrs_lse(p.s, transpose, 0.1, p.w.data(), p.out.data()) == BDRS_E_DEVICE);
    EXPECT(g_captured == 0);
  }
  g_capturing = false;
  EXPECT(bdrs_lse(p.s, 0, 0.1, p.w.data(), p.out.data()) == BDRS_OK);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "results_are_there") results_are_there();
  else if (name == "refused_under_capture") refused_under_capture();
  else return 2;
  std::printf("ok\n");
  return 0;
}

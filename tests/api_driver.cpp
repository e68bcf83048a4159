// The C ABI's host side (bdrs_api.hip compiled by the host compiler) on a
// simulated runtime: device memory is host memory, a launch only records what
// it would have read and written.  One scenario per run, named on the command
// line; prints "ok" at the end.
//
// The simulated stream counts its unfinished launches, so a call that returns
// before its results are there is seen.  While it is under capture launches go
// into the capture and a wait is refused.  Every sweep of the state checks that
// the packed weights it reads are the state's, and any launch, copy or wait can
// be made to fail.
#include "bdrs_host.h"

#include <cmath>
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
int g_fail_at = 0;         // the call into the runtime that fails (counted down; 0: none)
bool g_fail_on = false;    // ... and all after it
double g_round_cost = 1.0; // what the rounding's reduction gives
// whose weights the sides hold, and sweeps of the state that read others
bool g_rows_state = false, g_cols_state = false;
int g_wrong = 0;

#define EXPECT(cond)                                                              \
  do {                                                                            \
    if (!(cond)) {                                                                \
      std::printf("%s:%d: %s  [%s]\n", __FILE__, __LINE__, #cond, bdrs_last_error()); \
      std::exit(1);                                                               \
    }                                                                             \
  } while (0)

bool fails() {
  if (g_fail_at == 0 || --g_fail_at > 0) return false;
  if (g_fail_on) g_fail_at = 1;
  return true;
}

hipError_t launched() {
  if (fails()) return hipErrorUnknown;
  ++(g_capturing ? g_captured : g_pending);
  return hipSuccess;
}

// f is what the launch does if it does not fail (into a capture: nothing yet)
template <typename F>
hipError_t launched(F f) {
  const hipError_t e = launched();
  if (e == hipSuccess && !g_capturing) f();
  return e;
}

void state_sweep(bool transpose) { g_wrong += transpose ? !g_rows_state : !g_cols_state; }
void packed_by(FinishKind kind) {
  if (kind == kFinishRow) g_rows_state = true;
  if (kind == kFinishCol || kind == kFinishColCert) g_cols_state = true;
}
// a finite certificate of the iteration before the counter
void certify(const LaunchCtx& c, double* out) {
  const double rec[8] = {(double)(c.ctrl->k - 1), 0.1, 0.5, 1.0, 0.1, 0.9, 1.0, 0.0};
  std::memcpy(out, rec, sizeof rec);
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
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { return *p = (void*)symbol, hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return launched([=] { std::memcpy(d, s, n); });
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  return launched([=] { std::memset(d, v, n); });
}
hipError_t hipStreamSynchronize(hipStream_t) {
  if (fails()) return hipErrorUnknown;
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
hipError_t launch_pack(const LaunchCtx&, bool transpose, const double*, double) {
  return launched([=] { (transpose ? g_rows_state : g_cols_state) = false; });
}
hipError_t launch_pack_state(const LaunchCtx&, bool transpose, double, bool) {
  return launched([=] { (transpose ? g_rows_state : g_cols_state) = false; });
}
hipError_t launch_repair_pack(const LaunchCtx&) {
  return launched([] { g_cols_state = false; });
}
hipError_t launch_prologue(const LaunchCtx&) {
  return launched([] { g_cols_state = true; });
}
hipError_t launch_repack(const LaunchCtx& c) {
  return launched([&] {
    g_cols_state = true;
    if (c.ctrl->k > 0) g_rows_state = true;
  });
}
hipError_t launch_sweep(const LaunchCtx&, bool transpose, bool, int, double eps_arg, int) {
  return launched([=] {
    if (eps_arg <= 0.0) state_sweep(transpose);
  });
}
hipError_t launch_sweep_bary(const LaunchCtx&, int, double) { return launched(); }
hipError_t launch_finish(const LaunchCtx&, bool transpose, FinishKind kind, int, double*, int) {
  return launched([=] {
    if (kind == kFinishCertOnly) state_sweep(transpose);
    packed_by(kind);
  });
}
hipError_t launch_advance(Ctrl* c, int n, hipStream_t) {
  return launched([=] { c->k += n; });
}
hipError_t launch_cert_reduce(const LaunchCtx& c) {
  return launched([&] { certify(c, c.cert_out); });
}
hipError_t launch_repair_reduce(const LaunchCtx&) { return launched(); }
hipError_t launch_round_reduce(const LaunchCtx& c) {
  return launched([&] {
    for (int i = 8; i < 12; ++i) c.plan_stats[i] = g_round_cost;
  });
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
hipError_t launch_sweep_batch(const BatchItem*, int, const LaunchCtx*, int, bool transpose, bool, int, hipStream_t) {
  return launched([=] { state_sweep(transpose); });
}
hipError_t launch_finish_batch(const BatchItem*, int, const LaunchCtx*, int, FinishKind kind, int, hipStream_t) {
  return launched([=] { packed_by(kind); });
}
hipError_t launch_advance_batch(const LaunchCtx* descs, int count, int n, hipStream_t) {
  return launched([=] {
    for (int i = 0; i < count; ++i) descs[i].ctrl->k += n;
  });
}
hipError_t launch_cert_batch(const BatchItem*, int, const int* probs, int nprobs, const LaunchCtx* descs,
                             double* records, hipStream_t) {
  return launched([=] {
    for (int i = 0; i < nprobs; ++i) certify(descs[probs[i]], records + i * kCertSlots);
  });
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

// What a program does next: every sweep of the state reads the state's weights.
bdrs_status follow(Problem& p, int how) {
  bdrs_cert ce;
  int32_t status;
  switch (how) {
    case 0: return bdrs_step(p.s, 1);
    case 1: return bdrs_certificate(p.s, &ce);
    case 2: return bdrs_solve(p.s, 0.0, 1, 2, 2, &ce);
    default: return bdrs_batch_solve_static(&p.s, 1, 0.0, 1, 2, 1, &ce, &status);
  }
}

bdrs_status use(Problem& p, int call) {
  bdrs_plan_stats ps;
  bdrs_round_stats rs;
  bdrs_plan_export ex;
  bdrs_cert ce;
  double* out = p.out.data();
  switch (call) {
    case 0: return bdrs_lse(p.s, 0, 0.1, p.w.data(), out);
    case 1: return bdrs_lse(p.s, 1, 0.1, p.w.data(), out);
    case 2: return bdrs_plan(p.s, nullptr, out, nullptr, &ps);
    case 3: return bdrs_round(p.s, &rs);
    case 4: return bdrs_export_plan(p.s, BDRS_PLAN_ROUNDED, out, nullptr, nullptr, nullptr, &ex);
    case 5: return bdrs_export_plan(p.s, BDRS_PLAN_REPAIRED, out, nullptr, nullptr, nullptr, &ex);
    default: return bdrs_certificate(p.s, &ce);
  }
}

// A call that replaces the packed weights and ends early, wherever it does,
// leaves a solver whose next call sweeps the state's weights; if only one call
// into the runtime failed, the state's weights are there when it returns (a graph
// of iterations may be replayed next).
void weights_after_an_error() {
  for (int on = 0; on < 2; ++on)
  for (int call = 0; call < 7; ++call)
    for (int how = 0; how < 4; ++how) {
      const unsigned flags = call == 6 && how < 3 ? BDRS_F_REPAIR : 0;  // (not supported in batches)
      for (int n = 1;; ++n) {
        Problem p(flags);
        g_fail_at = n;
        g_fail_on = on != 0;
        const bdrs_status st = use(p, call);
        const bool failed = st != BDRS_OK;
        g_fail_at = 0;
        g_fail_on = false;
        EXPECT(st == (failed ? BDRS_E_DEVICE : BDRS_OK));
        EXPECT(on || (g_rows_state && g_cols_state));
        const bdrs_status next = follow(p, how);
        EXPECT(next == BDRS_OK || next == BDRS_NOT_CONVERGED);
        EXPECT(g_wrong == 0);
        if (!failed) break;
      }
    }
}

// The same where the call itself finds its result unusable.
void weights_after_a_numeric_error() {
  for (int how = 0; how < 4; ++how) {
    Problem p;
    g_round_cost = NAN;
    EXPECT(use(p, 3) == BDRS_E_NUMERIC);
    g_round_cost = 1.0;
    EXPECT(g_rows_state && g_cols_state);
    const bdrs_status next = follow(p, how);
    EXPECT(next == BDRS_OK || next == BDRS_NOT_CONVERGED);
    EXPECT(g_wrong == 0);
  }
}

// Weights restored inside a capture are not restored until it is replayed.
void weights_after_a_capture() {
  Problem p;
  g_fail_at = 4;  // the sweep's epilogue and what follows it
  g_fail_on = true;
  EXPECT(use(p, 0) == BDRS_E_DEVICE);
  g_fail_at = 0;
  g_fail_on = false;
  EXPECT(!g_cols_state);
  g_capturing = true;
  EXPECT(bdrs_step(p.s, 1) == BDRS_OK && g_captured > 0);
  g_capturing = false;
  EXPECT(bdrs_step(p.s, 1) == BDRS_OK);
  EXPECT(g_wrong == 0);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "results_are_there") results_are_there();
  else if (name == "refused_under_capture") refused_under_capture();
  else if (name == "weights_after_an_error") weights_after_an_error();
  else if (name == "weights_after_a_numeric_error") weights_after_a_numeric_error();
  else if (name == "weights_after_a_capture") weights_after_a_capture();
  else return 2;
  std::printf("ok\n");
  return 0;
}

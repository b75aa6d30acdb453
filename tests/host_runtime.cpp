// The library's host runtime (csrc/gmco_api.hip) on the CPU: a stand-in for the
// HIP runtime whose device work waits in a queue until the host synchronises,
// and stand-ins for the kernels, under the calls that a scenario makes.  Every
// scenario prints what it saw as one JSON line.
//
//     host_runtime <scenario> [numbers]
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "gmco_internal.h"

using gmco::few_chunk;

// ---- the device: a queue of work, run in order ----
static std::deque<std::function<void()>> g_queue;
static void later(std::function<void()> f) { g_queue.push_back(std::move(f)); }
static bool run_one() {
  if (g_queue.empty()) return false;
  auto f = std::move(g_queue.front());
  g_queue.pop_front();
  f();
  return true;
}
static void drain() {
  while (run_one()) {
  }
}

static double g_clock = 0.0;  // ms, advanced by the kernels
static std::map<void*, double> g_events;
static std::map<void*, size_t> g_device, g_pinned;
static long g_pins = 0, g_unpins = 0;
static size_t g_pinned_bytes = 0, g_pinned_peak = 0;
static bool g_no_pinning = false;

static void* map_bytes(size_t n) {
  void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  return p == MAP_FAILED ? nullptr : p;
}

extern "C" {
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void** p, size_t n) {
  *p = map_bytes(n);
  if (!*p) return hipErrorOutOfMemory;
  g_device[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  drain();
  munmap(p, g_device[p]);
  g_device.erase(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (g_no_pinning && n > 4096) return hipErrorOutOfMemory;
  *p = map_bytes(n);
  g_pinned[*p] = n;
  g_pins += 1;
  g_pinned_bytes += n;
  if (g_pinned_bytes > g_pinned_peak) g_pinned_peak = g_pinned_bytes;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  drain();
  munmap(p, g_pinned[p]);
  g_unpins += 1;
  g_pinned_bytes -= g_pinned[p];
  g_pinned.erase(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  later([=] { std::memcpy(d, s, n); });
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  later([=] { std::memset(d, v, n); });
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  drain();
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  drain();
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) {
  run_one();
  return g_queue.empty() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(new double(0.0));
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {  // (its memory stays: work that waits may name it)
  g_events.erase(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  later([=] { g_events[e] = g_clock; });
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) {
  drain();
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = (float)(g_events.at(b) - g_events.at(a));
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
}

// ---- the kernels ----
static float x_value(size_t p, int l) { return 0.25f + (float)(p % 977) + 0.001f * (float)l; }
static bool g_case_ok = true;       // the uploaded case, as the set-up kernel sees it
static const gmco_case* g_case = nullptr;
static long g_evals = 0, g_fail_at = -1;  // evaluations launched; the one that fails
static int g_live = 0;                    // rounds with running plans

namespace gmco {
hipError_t launch_dose_setup(const double* dwell_xyz, const double* pt_xyz, const double*, const int* perm, int M,
                             int K, int Mp, int Kp, int, int, int, double, double*, float*, void*, void*, float*,
                             double* scratch, double* t_bar, hipStream_t) {
  later([=] {
    for (size_t i = 0; i < dose_scratch(Mp, Kp); ++i) scratch[i] = -1.0;  // (nothing else is there)
    g_case_ok = std::memcmp(dwell_xyz, g_case->dwell_xyz, (size_t)K * 24) == 0 &&
                std::memcmp(pt_xyz, g_case->point_xyz, (size_t)M * 24) == 0;
    int last = -1, group = -1;  // stable order by group
    for (int i = 0; i < M && g_case_ok; ++i) {
      const int s = perm[i], g = s >= 0 && s < M ? g_case->group[s] : -1;
      g_case_ok = g > group || (g == group && s > last);
      group = g;
      last = s;
    }
    *t_bar = 1.0;
  });
  return hipSuccess;
}
hipError_t launch_init_plans(int P, int Pp, int K, int Kp, const double*, const double*, const double*, int, int,
                             const int*, const int*, float* xt, float* x, float*, double*, PlanState* ps,
                             hipStream_t) {
  later([=] {
    for (int p = 0; p < Pp; ++p) {
      ps[p] = PlanState{};
      ps[p].status = p < P ? ST_INIT : ST_INACTIVE;
      for (int l = 0; l < K && p < P; ++l) x[(size_t)p * Kp + l] = xt[(size_t)p * Kp + l] = x_value(p, l);
    }
  });
  return hipSuccess;
}
hipError_t launch_x32_to_device(const float* x, int P, int, int K, int Kp, float* xe, hipStream_t) {
  later([=] {
    for (int p = 0; p < P; ++p) std::memcpy(xe + (size_t)p * Kp, x + (size_t)p * K, (size_t)K * 4);
  });
  return hipSuccess;
}
hipError_t launch_finish_eval_f32(const float*, const double*, const float* x, int, int P, int, int K, int Kp,
                                  double* F, float* g, hipStream_t) {
  later([=] {
    for (int p = 0; p < P; ++p) {
      F[p] = p + 0.5;
      for (int l = 0; l < K; ++l) g[(size_t)p * K + l] = 2.f * x[(size_t)p * Kp + l];
    }
  });
  return hipSuccess;
}
hipError_t launch_metrics(const MetricsArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_metrics_final(const MetricsArgs& m, hipStream_t) {
  later([=] {
    for (int p = 0; p < m.P; ++p) {
      m.out[p].F64 = p + 0.25;
      m.out[p].iterations = p;
    }
  });
  return hipSuccess;
}
// A run whose plans all stop in round g_live - 1; a running evaluation takes 1 ms,
// an empty one 0.01, an update a tenth of that.
hipError_t launch_eval(const EvalArgs& a, int, hipStream_t) {
  if (g_evals++ == g_fail_at) return hipErrorLaunchFailure;
  const int nact = a.flag && a.round >= g_live ? 0 : a.P;
  later([=] {
    g_clock += nact > 0 ? 1.0 : 0.01;
    if (a.flag == nullptr) return;
    if (a.host_word != nullptr)
      *a.host_word = ((unsigned long long)(a.round + 1) << 32) | (unsigned)nact;
    *a.work += nact;
    if (a.work2 != nullptr) *a.work2 += nact;
  });
  return hipSuccess;
}
hipError_t launch_resume(PlanState* ps, const float*, float*, int*, int*, unsigned long long* work, int Pp, int, int,
                         int, hipStream_t) {
  later([=] {
    work[0] = work[1] = 0;
    for (int p = 0; p < Pp; ++p) ps[p].nevals0 = ps[p].nevals;
  });
  return hipSuccess;
}
hipError_t launch_update(const UpdateArgs& u, hipStream_t) {
  const int live = g_live;
  later([=] {
    g_clock += u.round < live ? 0.1 : 0.001;
    for (int p = 0; p < u.P && u.round < live; ++p) {  // plan 0 stops last
      if (p == 0 || u.round < live / 2) u.ps[p].nevals += 1;
      if (u.round == live - 1) u.ps[p].status = ST_CONVERGED;
    }
  });
  return hipSuccess;
}
hipError_t launch_dose64(const double*, const float*, int, int, int, int, double*, hipStream_t) { return hipSuccess; }
// not reached by any scenario
hipError_t launch_select(const gmco_plan_metrics*, int, int, const gmco_select_opts&, int*, int*, int*, int*,
                         hipStream_t) { std::abort(); }
hipError_t launch_features(const double*, const double*, const int*, const int*, const int*, int, int, unsigned*,
                           float*, hipStream_t) { std::abort(); }
hipError_t launch_dose_rate(const double*, const double*, const double*, const int*, int, int, int, int, double*,
                            hipStream_t) { std::abort(); }
hipError_t launch_widen_fp8(const void*, const float*, int, int, double*, hipStream_t) { std::abort(); }
hipError_t launch_pick_start(const double*, const double*, const float*, int, int, float*, float*, int*, int*,
                             hipStream_t) { std::abort(); }
hipError_t launch_finish_eval(const float*, const double*, const float*, int, int, int, int, int, double*, double*,
                              hipStream_t) { std::abort(); }
hipError_t launch_x_to_device(const double*, int, int, int, int, float*, hipStream_t) { std::abort(); }
hipError_t launch_eval_grouped(const EvalArgs*, const int*, int, int, int, int, int, hipStream_t) { std::abort(); }
hipError_t launch_update_grouped(const UpdateArgs*, int, int, int, int, int, hipStream_t) { std::abort(); }
hipError_t launch_learned_inputs(const double*, const float*, int, int, float*, hipStream_t) { std::abort(); }
hipError_t launch_learned_start(const float*, int, int, int, int, const double*, double, float*, hipStream_t) {
  std::abort();
}
int mlp_inputs(const gmco_mlp*) { std::abort(); }
int mlp_outputs(const gmco_mlp*) { std::abort(); }
int mlp_device(const gmco_mlp*) { std::abort(); }
hipError_t mlp_forward_device(gmco_mlp*, int, const float*, float*, hipStream_t) { std::abort(); }
}  // namespace gmco

// ---- scenarios ----
#define CHECK(call)                                                            \
  do {                                                                         \
    const int rc_ = (call);                                                    \
    if (rc_ != GMCO_OK) {                                                      \
      std::fprintf(stderr, "%s: %d %s\n", #call, rc_, gmco_last_error(g_ctx)); \
      std::exit(1);                                                            \
    }                                                                          \
  } while (0)

static gmco_ctx* g_ctx = nullptr;

struct Case {
  std::vector<double> dwell, pts;
  std::vector<int32_t> group;
  double params[16];
  gmco_case c{};
  Case(int K, int M) : dwell(3 * K), pts(3 * (size_t)M), group(M) {
    for (size_t i = 0; i < dwell.size(); ++i) dwell[i] = 0.01 * i;
    for (size_t i = 0; i < pts.size(); ++i) pts[i] = 1.0 + 1e-6 * i;
    for (int i = 0; i < M; ++i) group[i] = (i * 7) % 4;
    for (int j = 0; j < 4; ++j) {
      const double row[4] = {1.0, 5.0, 10.0, 1.0};
      std::memcpy(params + 4 * j, row, sizeof(row));
    }
    c.n_dwells = K;
    c.dwell_xyz = dwell.data();
    c.n_points = M;
    c.point_xyz = pts.data();
    c.group = group.data();
    c.n_groups = 4;
    c.group_params = params;
    c.prescription_gy = 15.0;
  }
};

static void start(const Case& cs, int P) {
  gmco_opts o{0, GMCO_DTYPE_F32, 1, P};
  CHECK(gmco_create(&g_ctx, &o));
  g_case = &cs.c;
  CHECK(gmco_load_case(g_ctx, &cs.c));
  std::vector<double> W((size_t)P * 4, 0.25);
  CHECK(gmco_set_weights(g_ctx, P, W.data(), nullptr));
}

// Every call that brings results to the host, four times over.
static int copies(int P, int K, int M, bool pinning) {
  g_no_pinning = !pinning;
  Case cs(K, M);
  start(cs, P);
  const size_t n = (size_t)P * K;
  std::vector<double> x(n), F(P), g(n), t(n);
  for (size_t i = 0; i < n; ++i) x[i] = 0.5 + 0.25 * (double)(i % 4099);
  std::vector<gmco_plan_metrics> m(P);
  bool ok = g_case_ok;
  std::string pins;
  for (int rep = 0; rep < 4; ++rep) {
    std::fill(F.begin(), F.end(), -1.0);
    std::fill(g.begin(), g.end(), -1.0);
    std::memset(m.data(), 0xff, m.size() * sizeof(m[0]));
    CHECK(gmco_evaluate(g_ctx, x.data(), F.data(), g.data()));
    for (int p = 0; p < P; ++p) ok = ok && F[p] == p + 0.5;
    for (size_t i = 0; i < n; ++i) ok = ok && g[i] == (double)(2.f * (float)x[i]);
    CHECK(gmco_get_dwell_times(g_ctx, t.data()));
    for (int p = 0; p < P; ++p)
      for (int l = 0; l < K; ++l) ok = ok && t[(size_t)p * K + l] == (double)x_value(p, l) * (double)x_value(p, l);
    CHECK(gmco_get_weights_x(g_ctx, t.data()));
    for (int p = 0; p < P; ++p)
      for (int l = 0; l < K; ++l) ok = ok && t[(size_t)p * K + l] == (double)x_value(p, l);
    CHECK(gmco_get_metrics(g_ctx, m.data()));
    for (int p = 0; p < P; ++p) ok = ok && m[p].F64 == p + 0.25 && m[p].iterations == p;
    pins += (rep ? ", " : "") + std::to_string(g_pins);
  }
  // a value that is not finite is refused wherever it stands
  for (size_t at : {size_t(0), n / 2, n - 1}) {
    const double keep = x[at];
    x[at] = -1.0 / 0.0;
    ok = ok && gmco_evaluate(g_ctx, x.data(), F.data(), g.data()) == GMCO_EINVAL;
    x[at] = keep;
  }
  const size_t peak = g_pinned_peak;
  CHECK(gmco_destroy(g_ctx));
  std::printf("{\"ok\": %d, \"pins\": [%s], \"peak\": %zu, \"left\": %zu}\n", ok ? 1 : 0, pins.c_str(), peak,
              g_pinned_bytes);
  return 0;
}

static gmco_run run_options() {
  gmco_run r{};
  r.max_iter = 1000;
  r.c1 = 1e-4;
  r.beta = 0.5;
  r.max_ls = 5;
  r.dtype = -1;
  return r;
}

// A run of which an evaluation fails to launch while the report of no running
// plan is on its way, and a run after it.
static int failed_launch(int live, int fail_at, int live2) {
  Case cs(5, 40);
  start(cs, 3);
  gmco_run r = run_options();
  gmco_run_info info{};
  g_live = live;
  g_fail_at = fail_at;
  const int rc = gmco_optimize(g_ctx, &r, &info);
  const size_t pending = g_queue.size();
  g_live = live2;
  g_fail_at = -1;
  CHECK(gmco_optimize(g_ctx, &r, &info));
  CHECK(gmco_destroy(g_ctx));
  std::printf("{\"rc\": %d, \"pending\": %zu, \"rounds\": %d, \"converged\": %d, \"work\": %g}\n", rc, pending,
              info.rounds, info.n_converged, info.eval_work);
  return 0;
}

// Sampled timing of two runs one after the other.
static int timing(int live, int every) {
  Case cs(5, 40);
  start(cs, 3);
  gmco_run r = run_options();
  r.time_kernels = every;
  std::string out;
  for (int run = 0; run < 2; ++run) {
    gmco_run_info info{};
    g_live = live + run;
    CHECK(gmco_optimize(g_ctx, &r, &info));
    char line[200];
    std::snprintf(line, sizeof(line), "%s[%d, %.6f, %.6f, %.6f, %d]", run ? ", " : "", info.timed_launches,
                  info.timed_work, info.eval_ms, info.update_ms, info.rounds);
    out += line;
  }
  CHECK(gmco_destroy(g_ctx));
  std::printf("{\"runs\": [%s]}\n", out.c_str());
  return 0;
}

static int checks(int live, int check_every) {
  Case cs(5, 40);
  start(cs, 3);
  gmco_run r = run_options();
  r.check_every = check_every;
  gmco_run_info info{};
  g_live = live;
  CHECK(gmco_optimize(g_ctx, &r, &info));
  CHECK(gmco_destroy(g_ctx));
  std::printf("{\"rounds\": %d, \"converged\": %d}\n", info.rounds, info.n_converged);
  return 0;
}

// The chunks of ranges of up to n blocks: in order, whole, none too long.
template <int NB>
static bool chunks_ok(int nblk) {
  const int nch = (nblk + NB - 1) / NB;
  bool ok = few_chunk<NB>(nblk, 0) == 0 && few_chunk<NB>(nblk, nch) == nblk;
  for (int c = 0; c < nch && ok; ++c) {
    const int n = few_chunk<NB>(nblk, c + 1) - few_chunk<NB>(nblk, c);
    ok = few_chunk<NB>(nblk, c) >= 0 && n >= 1 && n <= NB;
  }
  return ok;
}

static int few_chunks() {
  std::string bad;
  for (int n : {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 20, 63, 64, 65, 1000, 1250, 46341, 65536, 65537, 80265, 100003, 131072,
                1000000, 67108863})
    if (!chunks_ok<2>(n) || !chunks_ok<3>(n)) bad += (bad.empty() ? "" : ", ") + std::to_string(n);
  std::printf("{\"bad\": [%s]}\n", bad.c_str());
  return 0;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  auto arg = [&](int i) { return i < argc ? std::atoi(argv[i]) : 0; };
  if (what == "copies") return copies(arg(2), arg(3), arg(4), arg(5) != 0);
  if (what == "failed_launch") return failed_launch(arg(2), arg(3), arg(4));
  if (what == "timing") return timing(arg(2), arg(3));
  if (what == "checks") return checks(arg(2), arg(3));
  if (what == "few_chunks") return few_chunks();
  return 2;
}

// The library's host code on a HIP runtime that lives in host memory, so that what it does when
// the runtime refuses something can be tested without a GPU.  Streams are in order and done at
// once; the "chain" writes made-up counters and candidates where the descriptors say.
// fake_hip SCENARIO prints "ok" or what went wrong.
#include "lst_api.hip"

#include <set>

namespace {
hipError_t g_last = hipSuccess;
size_t g_refuse = SIZE_MAX;   // pinned allocations of this size and above fail
size_t g_pinned = 0, g_pinned_max = 0, g_pinned_calls = 0;
std::map<void *, size_t> g_host;
std::set<hipStream_t> g_streams;
bool g_record_fails = false;
bool g_capturing = false;     // the one graph: a chain over these descriptors
lst::Ws *g_graph_ws = nullptr;
int g_graph_B = 0;
int g_bad_stream_calls = 0, g_waits = 0, g_d2h = 0;
hipError_t ret(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}
// what the made-up chain finds: candidates of four hits each, per event
int g_candidates = 10;
int g_chains = 0;
}  // namespace

hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, n ? n : 1); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  ++g_pinned_calls;
  if (n >= g_refuse) return ret(hipErrorOutOfMemory);
  *p = calloc(1, n);
  g_host[*p] = n;
  g_pinned += n;
  g_pinned_max = std::max(g_pinned_max, g_pinned);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  g_pinned -= g_host[p];
  g_host.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost) ++g_d2h;
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return ret(g_record_fails ? hipErrorInvalidValue : hipSuccess); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); g_streams.insert(*s); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { g_streams.erase(s); free((void *)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (s && !g_streams.count(s)) ++g_bad_stream_calls;
  else ++g_waits;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { g_capturing = true; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { g_capturing = false; *g = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  lst::enqueue_chain(lst::DevGeom{}, g_graph_ws, g_graph_B, lst::Ws{}, nullptr, nullptr, nullptr, nullptr);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return hipSuccess; }

namespace lst {
const char *const kSiteNames[] = {"fixed", "shaped", "unshaped"};
const int kNumSites = 3;
bool site_tunable(int s) { return s > 0; }
bool site_shaped(int s) { return s == 1; }
void launch_module_windows(const int *, const float *, const float *, const float *, const float *, int, double, float4 *,
                           hipStream_t) {}
void launch_tc_export(const Ws *, int, int, int *, int *, int *, int *, hipStream_t) {}
void enqueue_chain(const DevGeom &, Ws *d, int B, const Ws &, hipStream_t, const KernelTimer *, const int *, const Ws *value) {
  ++g_chains;
  if (g_capturing) {
    g_graph_ws = d;
    g_graph_B = B;
    return;
  }
  for (int i = 0; i < B; ++i) {
    if (value) d[i] = value[i];
    const Ws &w = d[i];
    const int n = g_candidates, nh = 4 * n;
    memset(w.ctr, 0, sizeof(int) * C_COUNT);
    w.ctr[C_NTC] = n;
    w.ctr[C_NTCHITS] = nh;
    for (int k = 0; k < n; ++k) w.tc_out[k] = 3;
    for (int k = 0; k <= n; ++k) w.tc_out[n + k] = 4 * k;
    for (int k = 0; k < nh; ++k) w.tc_out[2 * n + 1 + k] = 7 * k + i;
    if (w.h_ctr) memcpy(w.h_ctr, w.ctr, sizeof(int) * C_COUNT);
    if (w.h_tc && 2 * n + 1 + nh <= w.h_tc_cap) memcpy(w.h_tc, w.tc_out, sizeof(int) * (2 * n + 1 + nh));
  }
}
}  // namespace lst

namespace {
#define CHECK(x)                                                     \
  do {                                                               \
    if (!(x)) {                                                      \
      printf("%s (line %d): %s\n", #x, __LINE__, lst_last_error()); \
      return 1;                                                      \
    }                                                                \
  } while (0)

lst_geometry geometry() {
  static int zero[2] = {0, 0}, off[3] = {0, 0, 0}, tgt[1] = {0};
  static float r[2] = {25.f, 26.f}, l0[2] = {1.f, 1.f}, l1[2] = {10.f, 10.f}, up[2] = {26.f, 27.f};
  lst_geometry_desc d{};
  d.n_modules = 2; d.subdet = zero; d.layer = zero; d.side = zero; d.type = zero;
  d.pos_lo = r; d.pos_up = up; d.lmin = l0; d.lmax = l1; d.map_offsets = off; d.map_targets = tgt;
  lst_geometry g = nullptr;
  if (lst_load_geometry(&d, &g) != LST_OK) printf("geometry: %s\n", lst_last_error());
  return g;
}

// An event of n hits and s seeds (its arrays are never read) and a workspace for B of them.
struct Call {
  std::vector<float> f;
  std::vector<int> i;
  lst_event_desc ev{};
  void *ws = nullptr;
  size_t bytes = 0;
  Call(lst_geometry g, int B, int n, int s) : f(n + 4 * s + 1), i(n + 4 * s + 1) {
    ev.n_hits = n; ev.n_seeds = s;
    ev.x = ev.y = ev.z = ev.px = ev.py = ev.pz = f.data();
    ev.module = ev.sensor = ev.q = ev.hits4 = i.data();
    std::vector<int32_t> nh(B, n), ns(B, s);
    lst_batch_workspace_bytes(g, B, nh.data(), ns.data(), nullptr, &bytes);
    ws = aligned_alloc(256, (bytes + 255) / 256 * 256);
  }
  ~Call() { free(ws); }
};

// The candidates of `e` are the chain's for event i.
bool candidates_ok(lst_event e, int i) {
  int32_t n = -1, nh = -1;
  if (lst_get_track_candidates(e, &n, &nh, nullptr, nullptr, nullptr) != LST_OK) return false;
  if (n != g_candidates || nh != 4 * n) return false;
  std::vector<int32_t> type(n), off(n + 1), hits(nh);
  if (lst_get_track_candidates(e, &n, &nh, type.data(), off.data(), hits.data()) != LST_OK) return false;
  for (int k = 0; k < n; ++k)
    if (type[k] != 3 || off[k + 1] != 4 * (k + 1)) return false;
  for (int k = 0; k < nh; ++k)
    if (hits[k] != 7 * k + i) return false;
  return true;
}

int plain() {
  lst_geometry g = geometry();
  Call c(g, 3, 500, 20);
  std::vector<lst_event_desc> evs(3, c.ev);
  lst_event e[3];
  CHECK(lst_enqueue_batch(g, 3, evs.data(), nullptr, c.ws, c.bytes, nullptr, e) == LST_OK);
  for (int i = 0; i < 3; ++i) {
    CHECK(lst_event_wait(e[i]) == LST_OK);
    CHECK(candidates_ok(e[i], i));
  }
  for (auto x : e) lst_release_event(x);
  return 0;
}

int refused() {
  lst_geometry g = geometry();
  g_refuse = 4096;  // the counters' and the descriptor's buffers are smaller
  Call c(g, 1, 500, 20);
  lst_event e = nullptr;
  CHECK(lst_enqueue_event(g, &c.ev, nullptr, c.ws, c.bytes, nullptr, &e) == LST_OK);
  CHECK(lst_event_wait(e) == LST_OK);
  g_refuse = SIZE_MAX;
  CHECK(candidates_ok(e, 0));
  lst_release_event(e);
  lst_plan p = nullptr;
  size_t bytes = 0;
  CHECK(lst_plan_workspace_bytes(g, 1, 500, 20, nullptr, &bytes) == LST_OK);
  void *ws = aligned_alloc(256, (bytes + 255) / 256 * 256);
  CHECK(lst_plan_create(g, 1, 500, 20, nullptr, ws, bytes, nullptr, &p) == LST_OK);
  g_refuse = 4096;
  CHECK(lst_plan_run(p, 1, &c.ev, nullptr, &e) == LST_OK);
  CHECK(hipGetLastError() == hipSuccess);
  CHECK(lst_event_wait(e) == LST_OK);
  g_refuse = SIZE_MAX;
  CHECK(candidates_ok(e, 0));
  lst_release_event(e);
  lst_plan_release(p);
  free(ws);
  return 0;
}

// no pinned buffer while the results are read
int unstaged() {
  lst_geometry g = geometry();
  g_candidates = 60000;
  Call c(g, 1, 500, 20);  // (made-up candidates: more than its result buffer holds)
  lst_capacity cap{};
  lst_default_capacity(500, 20, &cap);
  cap.t5 = 70000;
  size_t bytes = 0;
  CHECK(lst_workspace_bytes(g, 500, 20, &cap, &bytes) == LST_OK);
  void *ws = aligned_alloc(256, (bytes + 255) / 256 * 256);
  lst_event e = nullptr;
  CHECK(lst_enqueue_event(g, &c.ev, &cap, ws, bytes, nullptr, &e) == LST_OK);
  CHECK(lst_event_wait(e) == LST_OK);
  g_refuse = 0;
  CHECK(candidates_ok(e, 0));
  CHECK(g_d2h > 0 && hipGetLastError() == hipSuccess);
  lst_release_event(e);
  free(ws);
  return 0;
}

// a result that no size class of the pool holds goes straight to the caller
int unpooled() {
  lst_geometry g = geometry();
  g_candidates = 400000;  // 9.6 MB
  lst_capacity cap{};
  lst_default_capacity(500, 20, &cap);
  cap.t5 = 400000;
  size_t bytes = 0;
  CHECK(lst_workspace_bytes(g, 500, 20, &cap, &bytes) == LST_OK);
  Call c(g, 1, 500, 20);
  void *ws = aligned_alloc(256, (bytes + 255) / 256 * 256);
  lst_event e = nullptr;
  CHECK(lst_enqueue_event(g, &c.ev, &cap, ws, bytes, nullptr, &e) == LST_OK);
  CHECK(lst_event_wait(e) == LST_OK);
  const size_t before = g_pinned_calls;
  CHECK(candidates_ok(e, 0));
  CHECK(g_pinned_calls == before);
  lst_release_event(e);
  free(ws);
  return 0;
}

// An enqueue that fails after its launches: the chain may still write to the pinned buffers, so they
// are given back after a wait, and the stream, the program's own, may be gone by then.
int failed() {
  lst_geometry g = geometry();
  Call c(g, 1, 500, 20);
  hipStream_t st;
  CHECK(hipStreamCreateWithFlags(&st, 0) == hipSuccess);
  lst_event e = nullptr;
  g_record_fails = true;
  CHECK(lst_enqueue_event(g, &c.ev, nullptr, c.ws, c.bytes, st, &e) == LST_E_DEVICE && e);
  g_record_fails = false;
  CHECK(lst_event_wait(e) == LST_E_DEVICE);
  const int at_enqueue = g_waits;
  CHECK(hipStreamDestroy(st) == hipSuccess);
  lst_release_event(e);
  CHECK(g_bad_stream_calls == 0 && at_enqueue == 1);
  return 0;
}

// Host memory that held events take: little for small ones, bounded for many, and enough for the
// batches that are meant to fit.
int room() {
  lst_geometry g = geometry();
  {
    Call c(g, 1, 1400, 0);
    lst_event e = nullptr;
    CHECK(lst_enqueue_event(g, &c.ev, nullptr, c.ws, c.bytes, nullptr, &e) == LST_OK);
    CHECK(g_pinned <= 65536 && e->ws().h_tc && e->ws().h_tc_cap >= 4000);
    lst_release_event(e);
  }
  for (int n : {1400, 530000}) {  // a thousand events held at once
    Call c(g, 1, n, 0);
    std::vector<lst_event> held(1000);
    for (auto &e : held) CHECK(lst_enqueue_event(g, &c.ev, nullptr, c.ws, c.bytes, nullptr, &e) == LST_OK);
    CHECK(g_pinned <= (n == 1400 ? 40u << 20 : 136u << 20));  // (64 MiB of freed ones may be kept)
    CHECK(n != 530000 || (held[0]->ws().h_tc && !held[999]->ws().h_tc));
    CHECK(lst_event_wait(held[0]) == LST_OK && candidates_ok(held[0], 0));
    CHECK(lst_event_wait(held[999]) == LST_OK && candidates_ok(held[999], 0));
    for (auto e : held) lst_release_event(e);
  }
  // ints that the candidates of PU200 events take: 144k; a buffer that they do not fit in is not taken
  for (int B : {1, 4, 8, 9, 32}) {
    Call c(g, B, 530000, 8900);
    std::vector<lst_event_desc> evs(B, c.ev);
    std::vector<lst_event> e(B);
    CHECK(lst_enqueue_batch(g, B, evs.data(), nullptr, c.ws, c.bytes, nullptr, e.data()) == LST_OK);
    for (int i = 0; i < B; ++i) {
      const lst::Ws &w = e[i]->ws();
      CHECK(B > 4 ? !w.h_tc && !e[i]->batch->h_tc : w.h_tc && w.h_tc_cap >= 144000);
      CHECK(i == 0 || !w.h_tc || w.h_tc >= e[i - 1]->ws().h_tc + e[i - 1]->ws().h_tc_cap);
      CHECK(!w.h_tc || (size_t)(w.h_tc + w.h_tc_cap - e[i]->batch->h_tc) * sizeof(int) <= e[i]->batch->h_tc_bytes);
      CHECK(lst_event_wait(e[i]) == LST_OK && candidates_ok(e[i], i));
    }
    for (auto x : e) lst_release_event(x);
  }
  CHECK(host_pool().results_bytes == 0);
  return 0;
}

// A site whose launch reads no shape is timed as it is.
int tune() {
  lst_geometry g = geometry();
  Call c(g, 1, 500, 20);
  int32_t shape[3] = {0, 64, 128};
  CHECK(lst_set_launch_config(g, 3, shape) == LST_OK);
  float ms[3];
  CHECK(lst_autotune(g, 1, &c.ev, nullptr, c.ws, c.bytes, nullptr, 2, ms) == LST_OK);
  CHECK(ms[0] == -1.0f && ms[1] > 0.0f && ms[2] > 0.0f);
  CHECK(g_chains == 3 * 2 + 2);
  CHECK(lst_get_launch_config(g, 3, shape) == LST_OK && shape[0] == 0 && shape[2] == 128);
  return 0;
}
}  // namespace

int main(int argc, char **argv) {
  const std::map<std::string, int (*)()> scenarios = {{"plain", plain}, {"refused", refused}, {"unstaged", unstaged},
                                                          {"unpooled", unpooled}, {"failed", failed}, {"room", room}, {"tune", tune}};
  const int rc = scenarios.at(argv[1])();
  if (rc == 0) printf("ok\n");
  return rc;
}

// Stand-in for the HIP runtime and for the kernel launches of the library's
// host side (csrc/tnsim_abi.cpp), so that its ordering can be checked without a
// GPU: every stream is a queue that a thread of its own works off, slowly, in
// order; device memory is host memory; a blocking copy runs at once, as one on
// the null stream does beside a non-blocking stream.  The launches do just
// enough for the host code to go its way: a gate's Jacobi takes the number of
// sweeps that the scenario sets, a gradient entry counts its adjoint launches.
//
// usage: fake_hip gradient | replan | qr; prints "ok" or what went wrong.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../include/tnsim.h"
#include "../paper_2601_04422_amd/csrc/tnsim_internal.h"

using namespace tn;
typedef std::function<void()> Job;

static void pause_us(int us) { std::this_thread::sleep_for(std::chrono::microseconds(us)); }
static std::atomic<int> destroyed_in_flight{0};

struct Stream {
  std::mutex mu;
  std::condition_variable cv;
  std::deque<Job> q;
  uint64_t issued = 0, done = 0;
  std::vector<Job> *capture = nullptr;
  bool stop = false;
  std::thread worker{[this] { run(); }};
  void run() {
    std::unique_lock<std::mutex> l(mu);
    for (;;) {
      cv.wait(l, [&] { return stop || !q.empty(); });
      if (q.empty()) return;
      Job j = std::move(q.front());
      q.pop_front();
      l.unlock();
      j();
      l.lock();
      done++;
      cv.notify_all();
    }
  }
  void add(Job j) {
    if (capture) {
      capture->push_back(std::move(j));
      return;
    }
    std::lock_guard<std::mutex> l(mu);
    q.push_back(std::move(j));
    issued++;
    cv.notify_all();
  }
  void wait(uint64_t seq) {
    std::unique_lock<std::mutex> l(mu);
    cv.wait(l, [&] { return done >= seq; });
  }
  void sync() { wait(issued); }
  bool idle() {
    std::lock_guard<std::mutex> l(mu);
    return done == issued;
  }
  ~Stream() {
    {
      std::lock_guard<std::mutex> l(mu);
      stop = true;
      cv.notify_all();
    }
    worker.join();
  }
};
struct Event {
  Stream *s = nullptr;
  uint64_t seq = 0;
};
struct Graph {
  std::vector<Job> jobs;
};
struct Exec {
  std::vector<Job> jobs;
  std::atomic<int> in_flight{0};
};

static Stream null_stream;
static Stream *S(hipStream_t st) { return st ? (Stream *)st : &null_stream; }
static void noop(hipStream_t st) {
  S(st)->add([] { pause_us(5); });
}

// ---------------------------------------------------------------- runtime
extern "C" {
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { return *p = (void *)s, hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return *p = calloc(1, n), hipSuccess; }
hipError_t hipFree(void *p) { return free(p), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return *p = calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void *p) { return free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  null_stream.sync();
  return memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  S(st)->add([=] { memcpy(d, s, n); });
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  return *s = (hipStream_t) new Stream, hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return delete S(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return S(s)->sync(), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Event *ev = (Event *)e;
  Stream *on = ev->s;
  const uint64_t seq = ev->seq;
  S(s)->add([=] { on->wait(seq); });
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t) new Event, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete (Event *)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  Event *ev = (Event *)e;
  S(st)->add([] {});
  ev->s = S(st);
  ev->seq = S(st)->issued;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  return ((Event *)e)->s->wait(((Event *)e)->seq), hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  Event *ev = (Event *)e;
  std::lock_guard<std::mutex> l(ev->s->mu);
  return ev->s->done >= ev->seq ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  return S(s)->capture = new std::vector<Job>, hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
  Graph *gr = new Graph{std::move(*S(s)->capture)};
  delete S(s)->capture;
  S(s)->capture = nullptr;
  return *g = (hipGraph_t)gr, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  Exec *e = new Exec;
  e->jobs = ((Graph *)g)->jobs;
  return *x = (hipGraphExec_t)e, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete (Graph *)g, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  // an executable in flight is reported and left alone
  if (((Exec *)x)->in_flight)
    destroyed_in_flight++;
  else
    delete (Exec *)x;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st) {
  Exec *e = (Exec *)x;
  e->in_flight++;
  S(st)->add([=] {
    pause_us(2000);
    for (auto &j : e->jobs) j();
    e->in_flight--;
  });
  return hipSuccess;
}
}  // extern "C"

// ---------------------------------------------------------------- launches
// sweeps that the gate on sites (i, i + 1) takes
static int sweeps_of(int i) { return i % 4 == 0 ? 2 : 6; }

static int group_updates = 0, empty_updates = 0;

namespace tn {
int small_class(int, int, int) { return 0; }
void launch_fetch(hipStream_t st, void *host, const void *dev, size_t n, uint32_t *flag, uint32_t v) {
  S(st)->add([=] {
    memcpy(host, dev, n);
    __atomic_store_n(flag, v, __ATOMIC_RELEASE);
  });
}
void launch_fill_zero(hipStream_t st, void *p, size_t n) {
  S(st)->add([=] { memset(p, 0, n); });
}
void launch_copy_list(hipStream_t st, const CopyItem *items, int n) {
  for (int k = 0; k < n; k++) {
    const CopyItem c = items[k];
    S(st)->add([=] {
      for (uint32_t r = 0; r < c.rows; r++)
        memcpy((char *)c.dst + 8ull * r * c.dpitch, (const char *)c.src + 8ull * r * c.spitch,
               8ull * c.words);
    });
  }
}
void launch_gate_init(hipStream_t st, const GateDesc *d, int ng) {
  S(st)->add([=] {
    for (int g = 0; g < ng; g++) *d[g].sc = SlotScalars{};
  });
}
void launch_begin_sweep(hipStream_t st, const GateDesc *d, int ng) {
  S(st)->add([=] {
    for (int g = 0; g < ng; g++) d[g].sc->rot = ++d[g].sc->sweeps < sweeps_of(d[g].i);
  });
}
void launch_gather_sc(hipStream_t st, const GateDesc *d, int ng, SlotScalars *out) {
  S(st)->add([=] {
    for (int g = 0; g < ng; g++) out[g] = *d[g].sc;
  });
}
void launch_trunc(hipStream_t st, const GateDesc *d, int ng) {
  S(st)->add([=] {
    for (int g = 0; g < ng; g++) {
      d[g].sc->k = 1;
      d[g].sc->N = d[g].sc->W = 1.0;
      d[g].dimsDev[d[g].i + 1] = 1;
    }
  });
}
void launch_angle_grad(hipStream_t st, const double *, const Mat4 &, int, double *grad) {
  S(st)->add([=] {
    pause_us(3000);
    *grad += 1.0;
  });
}
void launch_smp_relabel(hipStream_t st, int, const int *, const int *, int *) { noop(st); }
double launch_probe(hipStream_t st, int, int, int, double *) { return noop(st), 1.0; }
#define NOOP(name, ...) \
  void name(hipStream_t st, __VA_ARGS__) { noop(st); }
typedef const GateDesc *D;
typedef const double2 *In;
NOOP(launch_init_state, void *const *, int, int, double *const *, int)
NOOP(launch_put, double2 *, double2)
NOOP(launch_apply_1q, const Gate1Desc *, int, int)
NOOP(launch_apply_1q_args, const Gate1Desc *, int, int)
NOOP(launch_convert, const void *, int, void *, int, size_t)
NOOP(launch_copy_state, int, const int *, void *const *, int, void *const *, int, double *const *,
     double *const *, size_t)
NOOP(launch_prop_merge, In, void *, int, int, int, int, int, const Mat4x4 &)
NOOP(launch_setup_slots, D, int, int, int)
NOOP(launch_theta, D, int, int, int, int)
NOOP(launch_colnorm, D, int, int)
NOOP(launch_small, D, int, bool, bool)
NOOP(launch_gram, D, int, int, int, int, bool, bool)
NOOP(launch_eig, D, int, int, int, int, bool, bool)
NOOP(launch_rot, D, int, int, int, int, int, int, bool)
NOOP(launch_qr_panel, D, int, int, int, int, bool, bool)
NOOP(launch_qr_update, D, int, int, int, int, int, bool, bool)
NOOP(launch_qr_tgroup, D, int, int, int)
void launch_qr_update_group(hipStream_t st, D, int, int stage, int, int, int max_cols, int, bool) {
  group_updates++;
  empty_updates += stage == 1 && max_cols <= 0;
  noop(st);
}
NOOP(launch_qr_r1h, D, int, int)
NOOP(launch_qr_r2h, D, int, int)
NOOP(launch_qr_gather, D, int, int, int)
NOOP(launch_wb_left, D, int, int, int)
NOOP(launch_wb_right, D, int, int, int, int)
NOOP(launch_gemm_gen, const GemmArgs &)
NOOP(launch_fill_c, double2 *, size_t, double2)
NOOP(launch_svd_adj_mid, In, double2 *, const double *, const double *, int, int, double)
NOOP(launch_herm_sum, In, double2 *, int)
NOOP(launch_weight_adj, In, In, double2 *, const double *, double *, int, int)
NOOP(launch_weight_apply, In, double2 *, const double *, int, int)
NOOP(launch_gate_adj, double2 *, int, int, const Mat16 &)
NOOP(launch_1q_adj, double2 *, const void *, int, int, int, const Mat4 &, double *)
NOOP(launch_dot_re, In, const void *, int, size_t, double *)
NOOP(launch_sigma_bar, const double *, const double *, const double *, double, int, double *)
NOOP(launch_gather_basis, In, int, const int *, const double *, double2 *, double *, int)
NOOP(launch_sort_all, const double *, int, int *)
NOOP(launch_pauli_phys, In, double2 *, int, int, double2, double2, double2, double2)
NOOP(launch_zgemm, ZgemmKind, const ZgemmArgs &, int, int)
NOOP(launch_smp_init, int, int, int *, double *, int *, double2 *, double2 *, int *)
NOOP(launch_smp_prob, In, In, int, int, const int *, double *)
NOOP(launch_smp_decide, int, int, int, const double *, const double *, const int *, int *, int *,
     uint8_t *, double *, int *)
NOOP(launch_smp_scan, const int *, int *, int *)
NOOP(launch_smp_parent, int *, const int *, const double *, const int *, int, int *, double *)
NOOP(launch_smp_add, In, size_t, double2 *)
NOOP(launch_amp_step, In, double2 *, double2 *, const void *, int, int, int, int)
}  // namespace tn

// ---------------------------------------------------------------- scenarios
static void *dev_alloc(size_t bytes) { return aligned_alloc(256, (bytes + 255) / 256 * 256); }
static int bad(const char *what) { return printf("%s\n", what), 1; }

static tnsim_gate gate2(int i) {
  tnsim_gate g{};
  g.q0 = i;
  g.q1 = i + 1;
  for (int e = 0; e < 4; e++) g.m[5 * e].re = 1.0;
  return g;
}

// Rotations on every qubit, then a two-qubit gate: on a stream of its own the
// gradient holds every adjoint's contribution, and nothing that uses the
// workspace is under way when the call returns.
static int gradient(tnsim_mps h, const tnsim_config &cfg, Stream &st) {
  const int n = cfg.n_qubits;
  std::vector<tnsim_gate> gates;
  std::vector<int32_t> param, axis(n, 1);
  std::vector<double> angles(n, 0.3), grad(n, -1.0);
  for (int q = 0; q < n; q++) {
    tnsim_gate g{};
    g.q0 = q;
    g.q1 = -1;
    gates.push_back(g);
    param.push_back(q);
  }
  gates.push_back(gate2(0));
  param.push_back(-1);
  const int32_t seg = 0;
  const std::string z(n, 'Z');
  const char *pauli = z.c_str();
  const double one = 1.0;
  double loss;
  const size_t bytes = tnsim_grad_workspace_bytes(&cfg, 1, (int)gates.size(), n);
  void *ws = dev_alloc(bytes);
  if (tnsim_forward_checkpointed(h, ws, bytes, gates.data(), (int)gates.size(), param.data(),
                                 axis.data(), angles.data(), n, &seg, 1, &pauli, &one, 1, &loss))
    return bad("forward failed");
  if (tnsim_backward(h, 1.0, grad.data())) return bad("backward failed");
  if (!st.idle()) return bad("work on the workspace under way after tnsim_backward");
  for (double g : grad)
    if (g != 1.0) return bad("the gradient was read before its adjoints had run");
  free(ws);
  return 0;
}

// Gates that converge at different sweeps: the launches are planned anew while
// the next sweep is in flight, whose captured graph has to stay until it is done.
static int replan(tnsim_mps h, const tnsim_config &cfg) {
  std::vector<tnsim_gate> layer;
  for (int i = 0; i + 1 < cfg.n_qubits; i += 2) layer.push_back(gate2(i));
  for (int k = 0; k < 3; k++)
    if (tnsim_apply_layer(h, layer.data(), (int)layer.size())) return bad("layer failed");
  int32_t rec[6 * 8], cnt;
  tnsim_last_batch(h, rec, 8, &cnt);
  for (int g = 0; g < cnt; g++)
    if (rec[6 * g + 5] != sweeps_of(rec[6 * g])) return bad("wrong sweep counts");
  return destroyed_in_flight ? bad("a graph in flight was destroyed") : 0;
}

// Preconditioned gates of one group of reflectors: Q1's T factor is computed,
// nothing is launched for Q2, which is not applied.
static int qr(tnsim_mps h) {
  const tnsim_gate g = gate2(2);
  if (tnsim_apply_layer(h, &g, 1)) return bad("layer failed");
  if (group_updates == 0) return bad("no factors for U");
  return empty_updates ? bad("a factor of Q2 that nothing reads") : 0;
}

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  tnsim_config cfg{};
  cfg.n_qubits = 8;
  cfg.chi_max = 8;
  cfg.svd_precondition = what == "qr";
  Stream st;
  const size_t bytes = tnsim_mps_arena_bytes(&cfg);
  void *arena = dev_alloc(bytes);
  memset(arena, 0, bytes);
  tnsim_mps h = nullptr;
  if (tnsim_mps_create(&cfg, arena, bytes, &st, &h)) return bad("create failed");
  const int r = what == "gradient" ? gradient(h, cfg, st)
                : what == "replan" ? replan(h, cfg)
                : what == "qr"     ? qr(h)
                                   : bad("usage: fake_hip gradient | replan | qr");
  tnsim_mps_destroy(h);
  free(arena);
  if (!r) printf("ok\n");
  return r;
}

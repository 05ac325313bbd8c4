// pf_graph_run of small windkessel filters on a stream that its caller is
// capturing, over the CPU stand-in runtime (fake_hip.cpp): refused, with
// nothing recorded into the capture, and the ancestors that were pending
// before are still written out by the next run.  The kernel stubs count their
// calls by name.  And which calls wait for the capture of a graph: a handle's
// first run of each tuning; a later one only where its remainder is shorter
// than every graph there is.
//   driver_capture refused | first | ladder
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

#include "pf.h"

static std::map<std::string, int> g_calls;
extern "C" void note_kernel(const char* name) { ++g_calls[name]; }
extern "C" void fake_trace(std::string* out);

#define CHECK_(c)                                          \
  do {                                                     \
    if (!(c)) {                                            \
      printf("FAIL %s (%s)\n", #c, pf_last_error());       \
      exit(1);                                             \
    }                                                      \
  } while (0)

static void refused() {
  const int B = 2, T = 8, K = 3;
  const std::vector<int64_t> np = {300, 70};
  const std::vector<int32_t> idx = {0};
  std::vector<double> obs(T, 95.0), q((size_t)T * K + 1, 100.0), theta;
  const double a = std::exp(-0.01 / 1.5);
  for (int b = 0; b < B; ++b)
    for (double v : {a, 1.0 - a, 0.03, 0.5, 90.0, 15.0}) theta.push_back(v);
  pf_config c{};
  c.model = PF_MODEL_WK;
  c.precision = PF_FP64;
  c.layout = PF_LAYOUT_PLAIN;
  c.d = 1;
  c.K = K;
  c.T = T;
  c.h = 0.01;
  c.n_obs = 1;
  c.obs_idx = idx.data();
  c.obs_sd = 1.0;
  c.obs = obs.data();
  c.q = q.data();
  c.B = B;
  c.n_theta = 6;
  c.n_particles = np.data();
  c.theta = theta.data();
  const size_t n = pf_workspace_bytes(&c);
  CHECK_(n > 0);
  void* ws = aligned_alloc(256, (n + 255) / 256 * 256);
  hipStream_t s;
  CHECK_(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
  pf_handle* h = nullptr;
  CHECK_(pf_init(&c, ws, n, s, &h) == PF_OK);
  CHECK_(pf_step(h) == PF_OK);
  CHECK_(pf_resample(h) == PF_OK);  // the ancestors are pending as marks now
  const auto before = g_calls;
  CHECK_(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) == hipSuccess);
  CHECK_(pf_graph_run(h, 2) == PF_E_DEVICE);
  CHECK_(g_calls == before);
  hipGraph_t g;
  CHECK_(hipStreamEndCapture(s, &g) == hipSuccess);
  CHECK_(hipGraphDestroy(g) == hipSuccess);
  // the refused call moved nothing on: the run writes the marks out first
  CHECK_(pf_graph_run(h, 2) == PF_OK);
  CHECK_(g_calls["launch_tile_anc"] == B);
  CHECK_(g_calls["launch_small_run"] == 1);
  // nothing pending as marks after it
  CHECK_(pf_graph_run(h, 5) == PF_OK);
  CHECK_(g_calls["launch_tile_anc"] == B);
  CHECK_(pf_graph_run(h, 1) == PF_E_STATE);  // t = T
  CHECK_(pf_destroy(h) == PF_OK);
  CHECK_(hipStreamDestroy(s) == hipSuccess);
  free(ws);
}

static void ladder() {
  for (int layout : {PF_LAYOUT_PLAIN, PF_LAYOUT_BATCHED}) {
    const int B = 3, T = 300, d = 4;
    const std::vector<int64_t> np = {300, 70, 1000};
    const std::vector<int32_t> idx = {0, 1, 2, 3};
    const std::vector<double> obs((size_t)T * d, 0.5), theta = {8.0, 0.1, 7.0, 0.2, 9.0, 0.1};
    pf_config c{};
    c.model = PF_MODEL_L96;
    c.precision = PF_FP32_MIXED;
    c.layout = layout;
    c.d = d;
    c.K = 2;
    c.T = T;
    c.h = 0.05;
    c.n_obs = d;
    c.obs_idx = idx.data();
    c.obs_sd = 0.5;
    c.obs = obs.data();
    c.B = B;
    c.n_theta = 2;
    c.n_particles = np.data();
    c.theta = theta.data();
    const size_t n = pf_workspace_bytes(&c);
    CHECK_(n > 0);
    void* ws = aligned_alloc(256, (n + 255) / 256 * 256);
    pf_handle* h = nullptr;
    CHECK_(pf_init(&c, ws, n, nullptr, &h) == PF_OK);
    // (the plain layout has no groups to tune)
    for (int groups = 1; groups <= (layout == PF_LAYOUT_BATCHED ? 2 : 1); ++groups) {
      CHECK_(pf_set_tuning(h, 512, groups) == PF_OK);
      CHECK_(pf_reset(h, 0) == PF_OK);
      const int G = groups;  // graphs of each length
      auto run = [&](int len) {
        std::string tr;
        fake_trace(&tr);
        CHECK_(pf_graph_run(h, len) == PF_OK);
        fake_trace(&tr);
        return tr;
      };
      auto waits = [](const std::string& tr) { return tr.find('L'); };
      auto launches = [](const std::string& tr) { return std::count(tr.begin(), tr.end(), 'L'); };
      std::string tr = run(10);  // graphs of 8 and 2
      CHECK_(waits(tr) == (size_t)(2 * G) && launches(tr) == 2 * G);
      tr = run(100);  // 12 of 8 and 2 of 2; 64, 32 and 4 captured behind them
      CHECK_(waits(tr) == 0 && launches(tr) == 14 * G && tr.size() == (size_t)(17 * G));
      tr = run(101);  // the graph of 1 is waited for
      CHECK_(waits(tr) == (size_t)G && launches(tr) == 4 * G && tr.size() == (size_t)(5 * G));
      tr = run(89);  // 64, 8, 8, 8, 1; 16 captured behind them
      CHECK_(waits(tr) == 0 && launches(tr) == 5 * G && tr.size() == (size_t)(6 * G));
    }
    CHECK_(pf_destroy(h) == PF_OK);
    free(ws);
  }
}

// A first run on a stream that its caller is capturing: refused before a
// capture of the handle's own is begun or anything is waited for (the stand-in
// stops at either), and the caller's capture goes on.
static void first() {
  for (int layout : {PF_LAYOUT_PLAIN, PF_LAYOUT_BATCHED}) {
    const int B = 3, T = 9, d = 4;
    const std::vector<int64_t> np = {300, 70, 1000};
    const std::vector<int32_t> idx = {0, 1, 2, 3};
    const std::vector<double> obs((size_t)T * d, 0.5), theta = {8.0, 0.1, 7.0, 0.2, 9.0, 0.1};
    pf_config c{};
    c.model = PF_MODEL_L96;
    c.precision = PF_FP64;
    c.layout = layout;
    c.d = d;
    c.K = 2;
    c.T = T;
    c.h = 0.05;
    c.n_obs = d;
    c.obs_idx = idx.data();
    c.obs_sd = 0.5;
    c.obs = obs.data();
    c.B = B;
    c.n_theta = 2;
    c.n_particles = np.data();
    c.theta = theta.data();
    const size_t n = pf_workspace_bytes(&c);
    CHECK_(n > 0);
    void* ws = aligned_alloc(256, (n + 255) / 256 * 256);
    hipStream_t s;
    CHECK_(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    pf_handle* h = nullptr;
    CHECK_(pf_init(&c, ws, n, s, &h) == PF_OK);
    CHECK_(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) == hipSuccess);
    CHECK_(pf_graph_run(h, 3) == PF_E_DEVICE);
    hipGraph_t g;
    CHECK_(hipStreamEndCapture(s, &g) == hipSuccess);
    CHECK_(hipGraphDestroy(g) == hipSuccess);
    CHECK_(pf_graph_run(h, 9) == PF_OK);
    CHECK_(pf_destroy(h) == PF_OK);
    CHECK_(hipStreamDestroy(s) == hipSuccess);
    free(ws);
  }
}

int main(int, char** argv) {
  if (std::string(argv[1]) == "refused") refused();
  else if (std::string(argv[1]) == "first") first();
  else ladder();
  printf("done\n");
  return 0;
}

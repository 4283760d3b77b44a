// Drives the exchange calls that take the two internal streams (streams and
// events made on first use, batches alternating between the lanes) from several
// threads at once, each with its own plan: the pencil schedule, and batches
// that a group cannot join.  Built like drive.cpp.
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "lace.h"

#define CHECK(x)                                                        \
  do {                                                                  \
    int rc_ = (x);                                                      \
    if (rc_ != LACE_OK) {                                               \
      std::fprintf(stderr, "%s:%d %s -> %d\n", __FILE__, __LINE__, #x, rc_); \
      std::exit(3);                                                     \
    }                                                                   \
  } while (0)

static void worker(int t, int reps) {
  const lace_precision precs[4] = {LACE_FP32_GAMMA, LACE_FP32, LACE_FP64,
                                   LACE_FP64_GAMMA};
  std::vector<int32_t> m;
  for (int z = -2; z <= 2; ++z)
    for (int y = -2; y <= 2; ++y)
      for (int x = -2; x <= 2; ++x) { m.push_back(x); m.push_back(y); m.push_back(z); }
  lace_cell_desc cell = {};
  cell.L = 10.0; cell.n = 8; cell.n_pw = (int64_t)m.size() / 3;
  cell.miller = m.data();
  lace_plan* plan = nullptr;
  CHECK(lace_plan_create(&cell, 1, precs[t % 4], &plan));
  // pairs per batch of 8, 36, 64 slots: 16, 3 and 2 batches share the energy
  // cells of a set
  for (int rep = 0; rep < reps; ++rep)
    for (int ppb : {8, 36, 64})
      for (int z = 0; z < 3; ++z) {
        const int n = 72;
        CHECK(lace_set_tuning(plan, 0, ppb, 0, z, 0));
        size_t wsb = 0;
        CHECK(lace_workspace_size(plan, 0, n, 0, &wsb));
        void* ws = std::calloc(wsb, 1);
        void* psi = std::calloc(16 * cell.n_pw * n, 1);
        void* w = std::calloc(16 * cell.n_pw * n, 1);
        double e = 0.0;
        int64_t kept = 0;
        CHECK(lace_apply_exchange(plan, 0, psi, n, 0.05, nullptr, nullptr, 0, w, &e,
                                  &kept, nullptr, ws, wsb, nullptr));
        CHECK(lace_apply_exchange_virtual(plan, 0, psi, n - 4, 4, 0.1, w, &e, nullptr,
                                          ws, wsb, nullptr));
        std::free(ws);
        std::free(psi);
        std::free(w);
      }
  CHECK(lace_plan_destroy(plan));
}

int main(int argc, char** argv) {
  const int threads = argc > 1 ? std::atoi(argv[1]) : 4;
  const int reps = argc > 2 ? std::atoi(argv[2]) : 2;
  std::vector<std::thread> th;
  for (int t = 0; t < threads; ++t) th.emplace_back(worker, t, reps);
  for (auto& x : th) x.join();
  std::printf("two lanes: %d threads x %d reps ok\n", threads, reps);
  return 0;
}

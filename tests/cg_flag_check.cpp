// CPU check of the CG scalars that a grid's blocks form for themselves (paper_2506_09435_amd/csrc/reduce.h):
// one block's 256 threads run as host threads, with the done flag as each of its four waves may have read
// it while another block set it.  Every combination must end in one decision for the whole block: all
// threads go on with the same alpha, the exact quotient, where no wave saw the flag, and all leave where
// one did; on a breakdown of p.Ap all leave.  Prints "ok" on success.
#include <pthread.h>

#include <cmath>
#include <cstdio>
#include <thread>
#include <vector>

#include "fnpf_internal.h"

// the device's names on the host: thread indices, the block's barrier, the wave's shuffle, shared memory
#undef __shared__
#define __shared__ static
struct Index {
  unsigned x;
};
static thread_local Index tIdx, bIdx;
#define threadIdx tIdx
#define blockIdx bIdx
static pthread_barrier_t g_block, g_wave[4];
static double g_lane[256];
static void sync_block() { pthread_barrier_wait(&g_block); }
#define __syncthreads sync_block
static double shfl_xor(double v, int o, int) {
  const int t = (int)tIdx.x;
  g_lane[t] = v;
  pthread_barrier_wait(&g_wave[t / 64]);
  const double r = g_lane[t ^ o];
  pthread_barrier_wait(&g_wave[t / 64]);
  return r;
}
#define __shfl_xor shfl_xor

#include "reduce.h"

using namespace fnpf;

struct Outcome {
  bool live;
  double alpha;
};

static std::vector<Outcome> run(int block, int waves, const std::vector<double> &partial, double rz, PcgScalars &sc) {
  std::vector<Outcome> out(256);
  std::vector<std::thread> th;
  for (int t = 0; t < 256; ++t)
    th.emplace_back([&, t] {
      tIdx.x = t;
      bIdx.x = block;
      const PartialLoads<1> pq(partial.data(), (int)partial.size());
      double alpha = 0.0;
      out[t].live = cg_alpha(pq, (waves >> (t / 64)) & 1, rz, &sc, alpha);
      out[t].alpha = alpha;
    });
  for (auto &x : th) x.join();
  return out;
}

int main() {
  int fails = 0;
  pthread_barrier_init(&g_block, nullptr, 256);
  for (auto &b : g_wave) pthread_barrier_init(&b, nullptr, 64);
  const double rz = 3.0;
  std::vector<double> partial(300);
  double sum = 0.0;
  for (size_t k = 0; k < partial.size(); ++k) sum += partial[k] = 1.0 + (double)(k % 7);   // exact in any order
  for (int waves = 0; waves < 16; ++waves) {
    PcgScalars sc{};
    for (const Outcome &o : run(1, waves, partial, rz, sc))
      if (o.live != (waves == 0) || (o.live && o.alpha != rz / sum)) ++fails;
    if (sc.alpha != 0.0 || sc.done != 0) ++fails;   // only the first block stores
  }
  {
    PcgScalars sc{};
    for (const Outcome &o : run(0, 0, partial, rz, sc))
      if (!o.live || o.alpha != rz / sum) ++fails;
    if (sc.alpha != rz / sum || sc.rz != rz || sc.pq != sum || sc.done != 0 || sc.breakdown != 0) ++fails;
  }
  for (const double bad : {-5000.0, 1e301, (double)INFINITY, (double)NAN}) {
    std::vector<double> p = partial;
    p[17] = bad;
    for (int block = 0; block < 2; ++block) {
      PcgScalars sc{};
      for (const Outcome &o : run(block, 0, p, rz, sc))
        if (o.live) ++fails;
      if (block == 0 && (sc.done != 1 || sc.breakdown != (bad == bad ? 1 : 2) || sc.alpha != 0.0)) ++fails;
    }
  }
  std::printf(fails == 0 ? "ok\n" : "FAILED %d\n", fails);
  return fails == 0 ? 0 : 1;
}

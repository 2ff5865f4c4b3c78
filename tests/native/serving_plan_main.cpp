// Host-only driver: the plan that a call launches.  Where it is the register-fragment kernel's form for five heads per pass, its
// fragments and partials fit the workspace, every head is in a pass, and its workgroups deal every tile once.
#include <stdio.h>
#include <string.h>

#include <vector>

#include "../../paper_2510_00636_amd/csrc/ea_common.h"

static int failures = 0;
#define CHECK(cond, ...)                                                         \
  do {                                                                           \
    if (!(cond) && ++failures <= 20) {                                           \
      fprintf(stderr, "%s:%d: check failed: %s: ", __FILE__, __LINE__, #cond);   \
      fprintf(stderr, __VA_ARGS__);                                              \
      fprintf(stderr, "\n");                                                     \
    }                                                                            \
  } while (0)

int main() {
  int five = 0;
  for (int d : {64, 128, 256})
    for (int G = 1; G <= 64; ++G)
      for (int units : {1, 2, 8, 33, 192, 600})
        for (int64_t n : {(int64_t)1, (int64_t)63, (int64_t)64, (int64_t)65, (int64_t)1500, (int64_t)4608, (int64_t)60000})
          for (int flags = 0; flags < 4; ++flags) {
            const bool fp8 = flags & 1, from_stats = flags & 2;
            if (fp8 && d == 64) continue;
            ea_params p;
            memset(&p, 0, sizeof p);
            p.batch = 1; p.n_q_heads = G * units; p.n_kv_heads = units; p.head_dim = d; p.dtype = EA_BF16;
            p.q_is_rotated = 1; p.horizon_T = 512;
            ea::Dims dims;
            CHECK(ea::check_params(&p, &dims) == EA_OK, "d %d G %d", d, G);
            dims.kv_fp8 = fp8;
            const ea::WsLayout L = ea::make_ws_layout(dims, n, 64);
            const ea::ScorePlan sp = ea::serving_score_plan(dims, n, 256, from_stats);
            CHECK((size_t)units * sp.unit_frags * 1024 <= L.post - L.frags, "d %d G %d units %d n %ld fragments", d, G, units, (long)n);
            CHECK((size_t)dims.qheads() * sp.npart * 8 <= L.lse - L.part, "d %d G %d units %d n %ld partials", d, G, units, (long)n);
            if (!sp.five) continue;
            ++five;
            const int64_t ntiles = (n + ea::kHwTile - 1) / ea::kHwTile;
            CHECK(!sp.hw && d == 128 && n >= ea::kHwTile && sp.GH == 5 && sp.passes * 5 >= G && sp.passes * 5 < G + 5, "G %d", G);
            CHECK(sp.nfrag == 5 * 20 + 8 && sp.unit_frags == sp.passes * sp.nfrag, "G %d: %d fragments", G, sp.unit_frags);
            CHECK(sp.pg == ea::kHwTile && sp.npart == ntiles && !sp.lse_pass, "n %ld: %d partials", (long)n, sp.npart);
            CHECK(sp.nchunk >= 1 && sp.nchunk <= ntiles, "n %ld: %d workgroups", (long)n, sp.nchunk);
            // every tile once: two by a workgroup's number and the rest drawn, or all of them drawn
            const int ways = ea::hw_ways(sp.nchunk);
            std::vector<int> seen(ntiles, 0);
            for (int way = 0; way < ways; ++way)
              for (int raw = 0; ea::hw_tile(raw, way, ways, (int)ntiles) >= 0; ++raw) ++seen[ea::hw_tile(raw, way, ways, (int)ntiles)];
            for (int64_t t = 0; t < ntiles; ++t) CHECK(seen[t] == 1, "n %ld: tile %ld", (long)n, (long)t);
          }
  CHECK(five > 100, "%d plans", five);
  // shapes of which one kernel is the faster one by 3 % or more (G, units, keys, 8-bit, behind statistics, five),
  const struct { int G, units; int64_t n; int fp8, stats, five; } measured[] = {
      {5, 8, 20000, 0, 0, 1}, {5, 192, 4608, 0, 0, 1}, {5, 320, 1500, 0, 0, 1}, {9, 32, 4608, 0, 0, 1}, {9, 8, 60000, 0, 0, 0},
      {5, 32, 4608, 1, 0, 1}, {5, 32, 32768, 1, 0, 0}, {13, 4, 131072, 0, 0, 1}, {9, 8, 25000, 0, 1, 1}, {5, 8, 12000, 0, 1, 1},
      {4, 8, 20000, 0, 0, 0}, {3, 40, 5000, 0, 1, 0}, {5, 8, 63, 0, 0, 0}, {5, 16, 60000, 0, 0, 0}, {5, 150, 4608, 0, 0, 1},
      {5, 320, 6940, 0, 0, 0}, {5, 300, 9000, 0, 1, 0}, {14, 200, 4608, 0, 0, 0}, {18, 140, 4000, 0, 1, 0}, {14, 230, 3000, 0, 0, 1},
      {18, 100, 5000, 0, 0, 1}, {20, 72, 13303, 0, 1, 0}, {40, 33, 6000, 0, 0, 0}, {20, 75, 2500, 0, 0, 1}, {30, 63, 6000, 0, 0, 1},
      // and those that the GPU test of this form means to reach it with, either way
      {5, 36, 4100, 0, 0, 1}, {5, 36, 4097, 0, 1, 1}, {5, 300, 1030, 0, 0, 1}, {5, 40, 4160, 0, 1, 1}, {9, 9, 16449, 0, 0, 1},
      {9, 9, 16449, 1, 0, 1}, {10, 9, 16449, 0, 0, 1}, {10, 9, 16449, 0, 1, 1}, {10, 9, 16449, 1, 0, 1}, {10, 100, 1030, 0, 0, 1},
      {10, 100, 1030, 1, 0, 1}, {13, 200, 64, 0, 0, 1}, {13, 200, 64, 1, 0, 1}, {15, 150, 1030, 0, 1, 1}, {10, 64, 2049, 0, 0, 0}};
  for (const auto& m : measured) {
    ea_params p;
    memset(&p, 0, sizeof p);
    p.batch = m.units; p.n_q_heads = m.G; p.n_kv_heads = 1; p.head_dim = 128; p.dtype = EA_BF16;
    p.q_is_rotated = 1; p.horizon_T = 512;
    ea::Dims dims;
    CHECK(ea::check_params(&p, &dims) == EA_OK, "G %d", m.G);
    dims.kv_fp8 = m.fp8;
    CHECK(ea::serving_score_plan(dims, m.n, 256, m.stats).five == m.five, "G %d, %d units x %ld keys", m.G, m.units, (long)m.n);
  }
  if (failures) {
    fprintf(stderr, "%d check(s) failed\n", failures);
    return 1;
  }
  printf("serving plans fit\n");
  return 0;
}

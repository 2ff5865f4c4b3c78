// Host-only driver: whatever kernel a call's score plan names, its fragments and partials fit the workspace, and the
// tiles that the register-fragment kernel deals out (two to every workgroup by its number and the rest by counters, one
// per residue class; with spare workgroups all of them by counters) are every tile of a head once.
#include <initializer_list>
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
  int registers = 0;
  for (int d : {64, 128, 256})
    for (int G = 1; G <= 64; ++G)
      for (int units : {1, 2, 3, 8, 33, 192, 600})
        for (int64_t n : {(int64_t)1, (int64_t)63, (int64_t)64, (int64_t)65, (int64_t)4608, (int64_t)131072})
          for (int fp8 = 0; fp8 <= (d >= 128); ++fp8)
            for (bool from_stats : {false, true})
              for (int cu : {64, 256, 304}) {
                ea_params p;
                memset(&p, 0, sizeof p);
                p.batch = 1; p.n_q_heads = G * units; p.n_kv_heads = units; p.head_dim = d; p.dtype = EA_BF16;
                p.q_is_rotated = 1; p.horizon_T = 512;
                ea::Dims dims;
                CHECK(ea::check_params(&p, &dims) == EA_OK, "d %d G %d", d, G);
                dims.kv_fp8 = fp8;
                const ea::WsLayout L = ea::make_ws_layout(dims, n, 64);
                const ea::ScorePlan sp = ea::choose_score_plan(dims, n, cu, from_stats);
                if (!sp.hw) {     // fragments of a pass: the heads' triangles, and a tile of extra rows on k and on k^2 per five heads
                  CHECK(sp.nfrag == sp.GH * ea::frags_per_head(d) + (sp.GH > 5 ? 2 : 1) * d / 16 && sp.unit_frags == sp.passes * sp.nfrag,
                        "d %d G %d: %d fragments", d, G, sp.nfrag);
                  CHECK(sp.lds_bytes <= 160 * 1024, "d %d G %d: %zu bytes of LDS", d, G, sp.lds_bytes);
                }
                CHECK((size_t)units * sp.unit_frags * 1024 <= L.post - L.frags, "d %d G %d units %d n %ld fragments", d, G, units, (long)n);
                CHECK((size_t)dims.qheads() * sp.npart * 8 <= L.lse - L.part, "d %d G %d units %d n %ld partials", d, G, units, (long)n);
                if (!sp.hw) continue;
                ++registers;
                const int64_t ntiles = (n + ea::kHwTile - 1) / ea::kHwTile;
                CHECK(n >= ea::kHwTile && d == 128 && sp.nchunk >= 1 && sp.nchunk <= ntiles, "n %ld: %d workgroups", (long)n, sp.nchunk);
                CHECK(sp.passes * 4 >= G && sp.passes * 4 < G + 4, "G %d: %d passes", G, sp.passes);
              }
  CHECK(registers > 1000, "%d plans", registers);
  // shapes at d = 128 of which one kernel is the faster one by 5 % or more
  const struct { int G, units; int64_t n; int fp8, hw; } measured[] = {
      {1, 300, 2000, 1, 0}, {1, 64, 9000, 1, 0}, {1, 20, 20000, 1, 0}, {1, 192, 700, 0, 0}, {1, 8, 9000, 0, 1}, {1, 1, 4608, 1, 1},
      {2, 300, 2000, 1, 0}, {2, 3, 131072, 1, 0}, {3, 64, 9000, 1, 0}, {4, 8, 131072, 0, 1}, {4, 192, 4608, 0, 1},
      {5, 32, 4608, 0, 0}, {5, 192, 700, 0, 0}, {5, 192, 4608, 0, 0}, {5, 8, 2000, 0, 1}, {6, 192, 2000, 0, 0}, {6, 20, 4608, 1, 1},
      {9, 8, 9000, 0, 1}, {9, 2, 131072, 0, 0}, {10, 100, 700, 0, 0}, {13, 100, 700, 0, 1}, {13, 20, 9000, 1, 1}, {40, 51, 1459, 1, 0}};
  for (const auto& m : measured) {
    ea_params p;
    memset(&p, 0, sizeof p);
    p.batch = m.units; p.n_q_heads = m.G; p.n_kv_heads = 1; p.head_dim = 128; p.dtype = EA_BF16;
    p.q_is_rotated = 1; p.horizon_T = 512;
    ea::Dims dims;
    CHECK(ea::check_params(&p, &dims) == EA_OK, "G %d", m.G);
    dims.kv_fp8 = m.fp8;
    CHECK(ea::choose_score_plan(dims, m.n, 256).hw == m.hw, "G %d, %d units x %ld keys, fp8 %d", m.G, m.units, (long)m.n, m.fp8);
    // operands from the statistics change the choice one way only, and not from 192 heads on
    const int with = ea::choose_score_plan(dims, m.n, 256, true).hw;
    CHECK(with >= m.hw && (dims.qheads() < ea::kStatsFragsMin || with == m.hw), "G %d, %d units x %ld keys", m.G, m.units, (long)m.n);
  }
  // the tile counters of up to 32 passes: every one a word of its own behind kTicketSlot in the unit's third histogram,
  // those of a pass on lines of their own
  std::vector<int> taken(ea::kSelBins, 0);
  static_assert(ea::kTicketSlot % 32 == 0, "lines of 128 bytes");
  for (int pass = 0; pass < 32; ++pass) {
    std::vector<int> lines;
    for (int way = 0; way < ea::kTicketWays; ++way) {
      const int word = ea::kTicketSlot + ea::ticket_word(pass, way);
      CHECK(word < ea::kSelBins && !taken[word]++, "pass %d way %d: word %d", pass, way, word);
      for (int line : lines) CHECK(line != word / 32, "pass %d way %d: line %d", pass, way, line);
      lines.push_back(word / 32);
    }
  }
  // spans of fp32 caches: those of the cheapest of all cuts
  for (int heads : {1, 4, 28, 32, 500, 4096})
    for (int slots : {128, 512, 1024})
      for (int64_t n : {(int64_t)1, (int64_t)64, (int64_t)65, (int64_t)1024, (int64_t)5003, (int64_t)16000, (int64_t)70001, (int64_t)131072, (int64_t)1 << 20, (int64_t)1 << 26}) {
        const int64_t steps = (n + 63) / 64;
        int64_t best = 0, best_cost = 0;
        for (int64_t c = 1; c <= steps && c <= 1024; ++c) {
          const int64_t per = (steps + c - 1) / c, cost = (heads * c + slots - 1) / slots * (2 * per + 1);
          if (best == 0 || cost < best_cost) { best = c; best_cost = cost; }
        }
        CHECK(ea::f32_span(heads, n, slots) == (steps + best - 1) / best * 64, "%d heads x %ld keys, %d slots", heads, (long)n, slots);
      }
  // the deal, played with the kernel's own functions: a workgroup works through what it is given until the first tile
  // that is none; draws that it made ahead are lost with it
  for (int nchunk = 1; nchunk <= 600; nchunk += nchunk < 80 ? 1 : 37)
    for (int ntiles : {nchunk, nchunk + 1, nchunk + 7, 2 * nchunk - 1, 2 * nchunk, 3 * nchunk + 5, 17 * nchunk + 3, 2048})
      for (bool spare : {false, true}) {
        if (ntiles < nchunk) continue;
        const int ways = ea::hw_ways(nchunk);
        CHECK(ways >= 1 && ways <= ea::kTicketWays && (ways == 1 || nchunk / ways >= 8), "%d workgroups: %d counters", nchunk, ways);
        std::vector<int> counter(ways, 0), scored(ntiles, 0);
        struct Workgroup { int way, dealt; std::vector<int> queue; bool done; };
        std::vector<Workgroup> wgs;
        auto draw = [&](Workgroup& w) { w.queue.push_back(ea::hw_tile(w.dealt + counter[w.way]++, w.way, ways, ntiles)); };
        for (int c = 0; c < nchunk; ++c) {
          const ea::HwDeal x = ea::hw_deal(c, nchunk, ways);
          Workgroup w{x.way, spare ? 0 : 2 * x.peers, {}, false};
          if (spare) { draw(w); draw(w); }
          else {
            w.queue.push_back(ea::hw_tile(x.nth, x.way, ways, ntiles));
            w.queue.push_back(ea::hw_tile(x.peers + x.nth, x.way, ways, ntiles));
          }
          if (spare || w.queue[0] >= 0) { draw(w); draw(w); }      // two ahead
          wgs.push_back(w);
        }
        int round = 0;
        for (bool busy = true; busy; ++round) {
          busy = false;
          for (int c = 0; c < nchunk; ++c) {
            Workgroup& w = wgs[(c + 13 * round) % nchunk];
            if (w.done) continue;
            const int t = w.queue.front();
            w.queue.erase(w.queue.begin());
            if (t < 0) { w.done = true; continue; }
            ++scored[t];
            draw(w);
            busy = true;
          }
        }
        for (int t = 0; t < ntiles; ++t) CHECK(scored[t] == 1, "%d workgroups, %d tiles, spare %d: tile %d %d times", nchunk, ntiles, spare, t, scored[t]);
      }
  for (int nchunk = 1; nchunk <= 600; ++nchunk) {
    const int ways = ea::hw_ways(nchunk);
    std::vector<std::vector<int>> members(ways);
    for (int chunk = 0; chunk < nchunk; ++chunk) {
      const ea::HwDeal x = ea::hw_deal(chunk, nchunk, ways);
      CHECK(x.way >= 0 && x.way < ways && x.nth == (int)members[x.way].size(), "workgroup %d of %d", chunk, nchunk);
      members[x.way].push_back(x.peers);
    }
    for (const auto& m : members)
      for (int peers : m) CHECK(peers == (int)m.size(), "%d workgroups: %d peers of %zu", nchunk, peers, m.size());
  }
  if (failures) return 1;
  printf("score plans fit\n");
  return 0;
}

// Internal definitions shared by the host shim and the HIP kernels of libea.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "../../include/ea.h"

namespace ea {

constexpr int kHwTile = 64;          // keys per iteration of the register-fragment score kernel
constexpr int kNW128 = 8;            // wavefronts per workgroup of the d = 128 score kernel
constexpr int kMaxWindow = 4096;
constexpr int64_t kMaxN = (int64_t)1 << 26;   // cached rows per head the launch grids cover
constexpr int kSelBins = 2048;        // radix-select digit width: 11 + 11 + 10 bits
constexpr int kSelBlock = 4096;       // scores per workgroup in the select passes
constexpr int kLseBlock = 2048;       // keys per softmax partial when the partials are taken from the stored logits
constexpr int kCompactRows = 96;     // destination rows per workgroup chunk in ea_compact (not a power of two on purpose)
// rows of 128 bytes (8-bit caches at d = 128, 16-bit at d = 64) come twice as many to a chunk: the
// same 24 KiB per workgroup for its ticket, its flags and its index loads
constexpr int compact_rows(int row_bytes) { return row_bytes <= 128 ? 2 * kCompactRows : kCompactRows; }

struct Dims {
  int B, Hq, Hkv, G, D, half;
  int dtype, rope_layout, q_is_rotated, ddof, T;
  float eps;
  int kv_fp8;     // 1: K and V rows are e4m3 bytes (dtype then describes q_win only)
  int units() const { return B * Hkv; }
  int qheads() const { return B * Hq; }
  int esize() const { return kv_fp8 ? 1 : dtype == EA_BF16 ? 2 : 4; }    // of a cached element
};

// How the matrix-core score kernel is tiled for one (d, G): heads per pass, passes, waves.
struct ScorePlan {
  int GH;       // query heads whose Sigma fragments are LDS-resident in one pass
  int passes;   // ceil(G / GH); K is streamed once per pass
  int NW;       // wavefronts per workgroup
  int nfrag;    // 1 KiB fragments per (unit, pass) (LDS-fragment kernels; at d = 256 with two heads those of the extra rows are in registers)
  int unit_frags;   // 1 KiB fragments per unit
  int nchunk;   // workgroups per (unit, pass)
  int spare;    // 1: more workgroups than CUs; the ones dispatched late join heads that still have tiles
  int hw;       // 1: the register-fragment kernel (one wavefront per query head, d = 128, four heads per pass)
  int five;     // 1: its form for five heads per pass, on the LDS-fragment kernels' layout of the fragments
  int pg;       // keys per softmax partial (max, sum exp): partial j covers keys [j*pg, (j+1)*pg)
  int npart;    // partials per query head = ceil(n / pg)
  int lse_pass; // 1: pass A leaves only logits; the partials are taken from them by a pass of their own
  size_t lds_bytes;
};

// Paged caches: K and V are pools [num_blocks][Hkv][bs][d]; logical block j of sequence b is pool
// block table[b * max_blocks + j]; bs = 1 << sh.  table == nullptr: contiguous tensors.
struct PageMap {
  const int32_t* table;
  int sh, max_blocks, hkv;
  long long num_blocks;
};

struct WsLayout {
  size_t tab, qproj, mu, sigma, frags, post, logits, vnorm, part, lse, scores, idx, base, hist, pool_hist, blk, flags, total;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// rows_only: the call only moves cache rows, so p->dtype may also be EA_FP8_E4M3
ea_status check_params(const ea_params* p, Dims* d, bool rows_only = false);
// the LDS-fragment kernels' plan, and the plan of the kernel that serves the call; from_stats: the
// operands come from the statistics kernel of the same call where it can make them (stats_makes_frags)
ScorePlan make_score_plan(const Dims& d, int64_t n, int num_cu);
ScorePlan choose_score_plan(const Dims& d, int64_t n, int num_cu, bool from_stats = false);
// what a call launches: that plan, or on its fragments the register-fragment kernel's form for five heads
ScorePlan serving_score_plan(const Dims& d, int64_t n, int num_cu, bool from_stats);
constexpr int kStatsFragsMin = 192;           // query heads from which one workgroup takes a whole head and makes its operands
WsLayout make_ws_layout(const Dims& d, int64_t n, int64_t window);

// Free words of the third radix histogram (its last digit has 1024 bins): the emit pass's block counter of
// every unit, unit 0's status word at kStatusSlot, the score kernel's tile counters of every unit from
// kTicketSlot on.  The launch that clears the histograms clears them all.
constexpr int kStatusSlot = 1030;
constexpr int kTicketSlot = 1056;
constexpr int kTicketWays = 8;       // tile counters per (unit, pass)
// Where counter `way` of a pass stands among them: neighbours on different lines of 128 bytes, of which there are 31.
// Next to each other, eight of them on one line dealt a tile every 23 ns whatever the chip did.  Operands + score, one
// unit x 131072 keys, before and now: d = 128, G = 1 51 and 29 us, 8 77 and 44, 12 80 and 60, 16 81 and 69; d = 64, G = 8
// 113 and 35; d = 256, G = 2 99 and 60; two units, d = 128, G = 5 79 and 56; from eight units on the same.
#ifdef __HIPCC__
__host__ __device__
#endif
constexpr int ticket_word(int pass, int way) {
  return (pass * kTicketWays + way) % 31 * 32 + (pass * kTicketWays + way) / 31;
}
// Status bits (see ea_debug_status)
constexpr uint32_t kStatusBadScore = 1u;      // ea_select met a negative or NaN score
constexpr uint32_t kStatusCompactWait = 2u;   // in-place ea_compact, or a block of ea_select, gave up waiting: stores skipped
constexpr uint32_t kStatusBadIndex = 4u;      // ea_compact met an idx list that is not strictly ascending in [j, n)
constexpr int kBaselineChunks = 256;          // most row chunks per head in the KeyDiff mean
constexpr int kCompactTicketStride = 64;      // words per (unit, tensor) at the head of the flag region

// Workgroups of 256 threads of the table launch, which makes one entry per (sample, channel pair) and clears
// the scratch words of the stages behind it: enough for the entries, and for at most kClearWords words each.
// The entries alone leave all of the clearing to one workgroup at a window of two samples: 24 sequences x 8 heads x
// 4608 pairs (5.7 MB to clear) took 442 us with head-adaptive budgets, 402 without, at windows of 2; now 283 and 242.
// (1024, 4096 and 8192 words per workgroup measure the same.)
constexpr size_t kClearWords = 2048;
inline size_t table_blocks(int64_t w, int half, size_t clear_words) {
  const size_t entries = ((size_t)w * half + 255) / 256, clearing = (clear_words + kClearWords - 1) / kClearWords;
  return entries > clearing ? entries : clearing;
}

// KeyDiff, rows per workgroup in multiples of 128 (16 rows at a time, eight loads in flight).  Its passes are cut
// into about 1024 workgroups, as far as the heads are long enough: the first one is bound by the loads a CU
// keeps in flight (8 heads x 65536 rows at d = 128: 121 us in both passes with 4096 rows per workgroup of the
// first, 1.6 TB/s, 56 with 512).
constexpr int64_t kKeydiffWgs = 1024;
inline int64_t keydiff_spread(int64_t n, int64_t units) {
  const int64_t rows = (n * units / kKeydiffWgs + 127) / 128 * 128;
  return rows < 128 ? 128 : rows;
}
// The first pass: stretches of up to 4096 rows where they are 600 workgroups or more already (300 heads x 5000 rows,
// two of 2500 each or four of 1280: 134 and 141 us for fp32 keys at d = 64; 700 x 4000, one or two of 2048: 280 and 289;
// 256 x 32768, eight of 4096 or four of 8192: 819 and 834; but 500 x 2500, one or two of 1280: 116 and 110, 192 x 4608,
// two or five: 88 and 81).  No more chunks than the scratch holds, and a head's chunks of one size but for what
// rounding to 128 rows leaves.
inline int keydiff_rows(int64_t n, int64_t units) {
  int64_t rows = units * ((n + 4095) / 4096) >= 600 ? 4096 : keydiff_spread(n, units);
  const int64_t least = ((n + kBaselineChunks - 1) / kBaselineChunks + 127) / 128 * 128;
  if (rows < least) rows = least;
  const int64_t nchunk = (n + rows - 1) / rows;
  return (int)(((n + nchunk - 1) / nchunk + 127) / 128 * 128);
}

// The tiles of a (unit, pass) of the register-fragment kernel: `ways` counters deal those of a residue class each.  Which
// class a workgroup takes part in, its number among those that do, and how many do.
// Of the two workgroups on a CU the one that came first gets the issue slots that both want and is up to a third faster,
// so a counter has to serve first and second ones alike (and every die): the residue goes round by one from each group of
// `ways` workgroups to the next.  With the residue chunk % ways the first ones of a CU were done after 69 us and the
// second ones after 95 (8-bit cache, 8 units x 131072 keys); now all within 6 us of each other.
struct HwDeal { int way, nth, peers; };
#ifdef __HIPCC__
__host__ __device__
#endif
inline HwDeal hw_deal(int chunk, int nchunk, int ways) {
  HwDeal x;
  x.nth = chunk / ways;
  x.way = (chunk + x.nth) % ways;
  const int groups = nchunk / ways;
  x.peers = groups + ((x.way + ways - groups % ways) % ways < nchunk % ways ? 1 : 0);
  return x;
}

// How many counters a (unit, pass) of nchunk workgroups uses, at least eight workgroups each; and the tile with number `raw`
// of residue class `way`, the last tile of the head first, -1 past the first one.
#ifdef __HIPCC__
__host__ __device__
#endif
inline int hw_ways(int nchunk) { return nchunk < 16 ? 1 : nchunk < 8 * kTicketWays ? nchunk / 8 : kTicketWays; }
#ifdef __HIPCC__
__host__ __device__
#endif
inline int hw_tile(int raw, int way, int ways, int ntiles) {
  const int t = ntiles - 1 - (raw * ways + way);
  return t < 0 ? -1 : t;
}

// Keys per workgroup of k_score_f32_whole, whole 64 of them, a head in at most 1024 spans.  The workgroups that fit the chip
// at once do the same amount each, so what counts is rounds of them x (tiles per wavefront + what a workgroup pays at
// its start).  Of the cuts with the same steps of 64 keys per span the one into fewest spans is looked at: 90 instead of
// 1024 of them for 131072 keys, with the same result.
inline int64_t f32_span(int64_t heads, int64_t n, int64_t slots) {
  const int64_t steps = (n + 63) / 64;
  int64_t best = steps, best_cost = 0;
  for (int64_t c = 1, per = steps; c <= 1024; c = (steps + per - 2) / (per - 1)) {
    per = (steps + c - 1) / c;
    const int64_t cost = (heads * c + slots - 1) / slots * (2 * per + 1);
    if (best_cost == 0 || cost < best_cost) { best = per; best_cost = cost; }
    if (per == 1) break;
  }
  return best * 64;
}

// fragments per head of the triangular Sigma tiling, and per pass
inline int frags_per_head(int D) { int njt = D / 32; return njt * (njt + 1); }
// those of the extra rows of a pass of GH heads: a tile of 16 rows for up to five of them, on k and on k^2
inline int extra_frags_of(int D, int GH) { return (GH > 5 ? 2 : 1) * D / 16; }

}  // namespace ea

// Host-only part of libea: argument validation, tiling plans, workspace layout, and the two
// host helpers of the ABI.  Nothing here touches the GPU, so it is testable without one.
#include <math.h>

#include "ea_common.h"

namespace ea {

ea_status check_params(const ea_params* p, Dims* d, bool rows_only) {
  if (!p) return EA_ERR_INVALID_ARG;
  if (p->batch < 1 || p->n_kv_heads < 1 || p->n_q_heads < 1) return EA_ERR_INVALID_ARG;
  if (p->n_q_heads % p->n_kv_heads != 0) return EA_ERR_INVALID_ARG;
  if (p->cov_ddof != 0 && p->cov_ddof != 1) return EA_ERR_INVALID_ARG;
  if (p->rope_layout != 0 && p->rope_layout != 1) return EA_ERR_INVALID_ARG;
  if (p->q_is_rotated != 0 && p->q_is_rotated != 1) return EA_ERR_INVALID_ARG;
  if (p->horizon_T < 1) return EA_ERR_INVALID_ARG;
  if (!(p->epsilon >= 0.0f) || !isfinite(p->epsilon)) return EA_ERR_INVALID_ARG;
  const bool fp8 = p->dtype == EA_FP8_E4M3;
  if (p->dtype != EA_F32 && p->dtype != EA_BF16 && !(fp8 && rows_only)) return EA_ERR_UNSUPPORTED;
  if (p->head_dim != 64 && p->head_dim != 128 && p->head_dim != 256) return EA_ERR_UNSUPPORTED;
  if (fp8 && p->head_dim == 64) return EA_ERR_UNSUPPORTED;
  int G = p->n_q_heads / p->n_kv_heads;
  if (G > 64) return EA_ERR_UNSUPPORTED;
  if ((int64_t)p->batch * p->n_q_heads > (1 << 20)) return EA_ERR_UNSUPPORTED;
  d->B = p->batch;
  d->Hq = p->n_q_heads;
  d->Hkv = p->n_kv_heads;
  d->G = G;
  d->D = p->head_dim;
  d->half = p->head_dim / 2;
  d->dtype = fp8 ? (int)EA_BF16 : p->dtype;
  d->kv_fp8 = fp8 ? 1 : 0;
  d->rope_layout = p->rope_layout;
  d->q_is_rotated = p->q_is_rotated;
  d->ddof = p->cov_ddof;
  d->T = p->horizon_T;
  d->eps = p->epsilon;
  return EA_OK;
}

// Of the workgroups that k_score_mfma's launch starts with, one per CU, how many the head with the fewest has (its
// order: transposed over the eight dies where the grid is a multiple of eight, units innermost).
static int least_served(int units, int64_t grid, int num_cu) {
  int count[512] = {};
  if (units > 512) return 0;
  for (int64_t b = 0; b < num_cu && b < grid; ++b) ++count[(grid % 8 == 0 ? (b % 8) * (grid / 8) + b / 8 : b) % units];
  int least = count[0];
  for (int u = 1; u < units; ++u) least = count[u] < least ? count[u] : least;
  return least;
}

// Heads per pass: as many as fit the 160 KiB of LDS with their fragments, next to the per-wave staging buffers; of the
// template instances (GH) the smallest that covers ceil(G / passes) of them.
ScorePlan make_score_plan(const Dims& d, int64_t n, int num_cu) {
  ScorePlan s;
  s.hw = 0;
  s.five = 0;
  s.spare = 0;
  s.lse_pass = 0;
  const int NF = frags_per_head(d.D);
  const size_t lds_max = 160 * 1024, slack = 1024;
  const int inst64[] = {1, 2, 4, 8}, inst128[] = {1, 2, 3, 4, 5}, inst256[] = {1};
  const int* inst = d.D == 64 ? inst64 : d.D == 128 ? inst128 : inst256;
  const int ninst = d.D == 64 ? 4 : d.D == 128 ? 5 : 1;
  s.NW = d.D == 256 ? 4 : d.D == 128 ? kNW128 : 8;
  const size_t stage = (size_t)s.NW * 16 * d.D * 2;
  int ghmax = 1;
  for (int i = 0; i < ninst; ++i)
    if ((size_t)(inst[i] * NF + extra_frags_of(d.D, inst[i])) * 1024 + stage + slack <= lds_max) ghmax = inst[i];
  s.passes = (d.G + ghmax - 1) / ghmax;
  int need = (d.G + s.passes - 1) / s.passes;
  s.GH = ghmax;
  for (int i = ninst - 1; i >= 0; --i)
    if (inst[i] >= need) s.GH = inst[i];
  s.nfrag = s.GH * NF + extra_frags_of(d.D, s.GH);
  s.unit_frags = s.passes * s.nfrag;
  s.lds_bytes = (size_t)s.nfrag * 1024 + stage + slack;
  if (d.D == 256 && d.G >= 2) {
    // two query heads per pass: their triangular fragments in LDS (144 KiB), the extra tile's in
    // registers, K staged through 4 KiB per wave: exactly the 160 KiB a workgroup may have
    s.GH = 2;
    s.passes = (d.G + 1) / 2;
    s.nfrag = 2 * NF + extra_frags_of(d.D, 2);
    s.unit_frags = s.passes * s.nfrag;
    s.lds_bytes = (size_t)2 * NF * 1024 + (size_t)s.NW * 4096;
  }
  // A CU holds one workgroup.  Up to half as many units as CUs: every unit gets its share of the CUs, rounded down.
  // Where that leaves a wavefront at most three tiles, only as many workgroups as finish in the same number of tiles
  // per wavefront: more of them load fragments and draw tickets for nothing.  score, with the share and with fewer: d = 256,
  // G = 1, 32 x 1500 36.0 and 31.9 us, 8 x 5000 30.6 and 29.4; G = 2, 8 x 9999 48.0 and 46.2; d = 128, G = 5, 32 x 4608 47.9
  // and 46.9.  In one pass not for fewer than eight units, at d = 64 than 32 (d = 256, G = 1, one x 100000 38.7 and 44.9; d = 64,
  // G = 8, 8 x 9999 28.9 and 30.1), and not with more tiles per wavefront (one x 360443 53.1 and 62.9).
  // In several passes also with four to seven tiles, for heads of 40 workgroups and more that lose more than a few of them
  // (d = 64, G = 16, 3 x 91387 70.9 and 66.1; d = 256, G = 8, 3 x 45691 177 and 159).  There not all workgroups are on the chip
  // at once, and a head that the first ones leave out starts late: the smaller launch has to serve every head as the share
  // does, and keep a grid of a multiple of eight (d = 256, G = 8, one x 180219, 256 and not 235: 196 and 203).  Few long heads
  // at d = 256 in two passes keep their share (6 x 12091, G = 4, 65.4 and 68.4) unless nearly half of the workgroups go
  // (3 x 11963, G = 4, 52.8 and 44.4).
  //
  // More units: one workgroup per (unit, pass) job, and where these leave the last round of CUs to 85 % full
  // or less, spare ones behind them, three per job (two while the units do not exceed the CUs: fewer CUs are
  // idle then): a CU whose head is done takes one of them and joins a head that still has tiles (tickets deal
  // them).  query_stats + score in a row at d = 128, without and with: 304 units, G = 4, n = 4608 319 and 265 us;
  // 384 units, G = 5, 421 and 382; 160 units in two passes 277 and 234.  Not on heads of under 1024 keys.  (From
  // seven rounds on the last one is always more than 85 % of the whole.)  With fewer jobs than CUs it does not
  // pay at d <= 128: 192 CUs at the clock the chip then grants do what 256 do (192 units 203 and 200 us, the whole
  // decode-time pass 415 and 420).  At d = 256, one wavefront per SIMD, it does once the head is long enough for
  // the fragments that a spare workgroup loads first, 72 KiB per query head, the longer the fewer CUs are idle.
  // score, two query heads per pass, without and with: 160 units x 1024 keys 94.4 and 98.5 us, x 1500 119 and 118,
  // x 4000 242 and 211; 200 units x 1500 133 and 144, x 4000 261 and 260, x 9000 512 and 493; one query head, 200 units
  // x 1024 72.2 and 74.1, x 2000 118 and 113.
  const int64_t ntiles = (n + 31) / 32, most = (ntiles + s.NW - 1) / s.NW;       // every wavefront with a tile at least
  const int64_t jobs = (int64_t)d.units() * s.passes;
  int64_t wgs = num_cu / d.units();
  if (wgs > 1024) wgs = 1024;
  if (wgs < 2) {
    const int64_t rounds = (jobs + num_cu - 1) / num_cu;
    const int64_t least = jobs > num_cu ? 1024 : s.GH * (jobs * 4 > (int64_t)num_cu * 3 ? 2000 : 640);
    s.spare = jobs * 20 < rounds * num_cu * 17 && n >= 1024 && n >= least && (jobs > num_cu || d.D == 256);
    wgs = !s.spare ? 1 : wgs == 1 ? 3 : 4;
  } else {
    const int64_t per_wave = (ntiles + wgs * s.NW - 1) / (wgs * s.NW), fewer = (ntiles + per_wave * s.NW - 1) / (per_wave * s.NW);
    bool take = per_wave <= 3 || (per_wave < 8 && wgs >= 40 && fewer * 20 <= wgs * 19);
    if (s.passes == 1) take = per_wave <= 3 && d.units() >= (d.D == 64 ? 32 : 8);
    if (d.D == 256 && s.passes == 2 && d.units() >= 2 && d.units() <= 6) take = take && fewer * 5 < wgs * 3;
    if (take && fewer < wgs && s.passes > 1)
      take = least_served(d.units(), jobs * fewer, num_cu) * 10 >= least_served(d.units(), jobs * wgs, num_cu) * 9 &&
             ((jobs * wgs) % 8 != 0 || (jobs * fewer) % 8 == 0);
    if (take) wgs = fewer;
  }
  if (wgs > most) wgs = most;
  if (wgs < 2) s.spare = 0;
  s.nchunk = (int)wgs;
  s.lse_pass = 1;
  s.pg = kLseBlock;
  s.npart = (int)((n + s.pg - 1) / s.pg);
  return s;
}

// How the register-fragment kernel cuts the keys of its (unit, pass) jobs.
static void deal_register_workgroups(const Dims& d, int64_t n, int num_cu, ScorePlan* s) {
  // Two workgroups per CU.  Where whole ones for every (unit, pass) leave more than a twentieth of them out, one more for
  // each, as in make_score_plan: 192 units x 4608, G = 4, two and three per unit 138 and 132 us; G = 7 251 and 230;
  // 384 jobs (G = 6) 248 and 227, 576 (G = 9) 375 and 337.
  const int64_t ntiles = (n + kHwTile - 1) / kHwTile;
  const int64_t jobs = (int64_t)d.units() * s->passes, slots = 2 * (int64_t)num_cu;
  int64_t wgs = slots / jobs;
  if (wgs < 8) {
    const int64_t rounds = (jobs + slots - 1) / slots, used = wgs ? wgs * jobs : jobs;
    s->spare = n >= 1024 && used * 20 < rounds * slots * 19;
    wgs = s->spare ? (wgs ? wgs + 1 : 2) : wgs;
  }
  if (wgs > 1024) wgs = 1024;
  if (wgs > ntiles) wgs = ntiles;
  if (wgs < 1) wgs = 1;
  if (wgs < 2) s->spare = 0;
  s->nchunk = (int)wgs;
  s->pg = kHwTile;
  s->npart = (int)ntiles;
}

// The register-fragment kernel (d = 128): four query heads per pass, one wavefront each, two workgroups of four
// wavefronts on a CU, whatever the cache layout.
static ScorePlan register_plan(const Dims& d, int64_t n, int num_cu) {
  ScorePlan s;
  s.hw = 1;
  s.five = 0;
  s.GH = 4;
  s.passes = (d.G + 3) / 4;
  s.NW = 4;
  s.spare = 0;
  s.lse_pass = 0;
  s.lds_bytes = 0;
  // the fragments of the unit's heads, then those of the extra rows of every pass
  s.nfrag = 0;
  s.unit_frags = d.G * frags_per_head(128) + s.passes * extra_frags_of(128, 4);
  deal_register_workgroups(d, n, num_cu, &s);
  return s;
}

// Which of the two kernels serves a call that both can: the lines are where operands + score took as long with either, over
// 2400 shapes, when this kernel's workgroups stood in the transposed order (see transposed_order) and it alone had its operands
// from the statistics.  Since then calls on both sides of them have become faster, and over 280 shapes most of those that
// the other kernel would serve better by more than 3 % lie outside: compress, G = 3, 128 x 2585 111 and 97, 64 x 447 40 and 36,
// 256 x 419 of G = 2 63 and 58; inside, 8-bit G = 10, 2 x 52097 82 and 88.
// Figures: us with the LDS-fragment kernel and with this one, 8-bit rows behind the bar.
static bool registers_serve(const Dims& d, int64_t n, int num_cu, const ScorePlan& lds, const ScorePlan& hw, bool from_stats) {
  // As many passes, and every wavefront (or all but the last pass's fourth) with a head: this one.  G = 4, 8 x 16384 38
  // and 31, 192 x 4608 150 and 140, 64 x 9000 85 and 86; G = 7, 8 x 45000 104 and 104; G = 12, 64 x 9000 186 and 175
  if (hw.passes <= lds.passes && hw.passes * 4 - d.G <= (hw.passes > 1)) return true;
  // Else wavefronts without a head, or a pass more, have to be paid for by the cheaper start: 20 KiB of fragments per
  // wavefront, not 36 and more per query head through LDS, and no pass of its own for the partials.  So only calls of few
  // (tile, pass) pairs, the fewer the more is lost on each:
  //   idle wavefronts: G = 1, 8 x 9000 24 and 22, 20 x 20000 48 and 49, 8-bit 20 x 2000 20 and 17, x 4608 21 and 22;
  //     G = 2, 8-bit 8 x 20000 29 and 28, 3 x 131072 41 and 47; G = 6, 20 x 9000 60 and 56, 64 x 9000 128 and 141
  //   a pass more: G = 5, 20 x 2000 35 and 30, x 4608 37 and 40; G = 9, 8 x 9000 47 and 42, x 20000 63 and 68; G = 13 to 15,
  //     20 x 9000 98 and 93, 12 x 40000 203 and 210; G = 17 and more, 12 x 12000 128 and 120, 6 x 40000 135 and 145
  const int64_t tiles = (int64_t)d.units() * ((n + kHwTile - 1) / kHwTile);
  const bool more = hw.passes > lds.passes;
  int64_t most = hw.passes > 1 ? 6000 : 5000;
  if (more) most = lds.passes == 1 ? 2300 : lds.passes == 2 ? 6800 : lds.passes == 3 ? 20000 : 12000;
  else if (d.kv_fp8 && d.G <= 2) most = d.G == 1 ? 1100 : 2800;
  // (in a compress call of fewer heads than kStatsFragsMin further out: the statistics make either kernel's operands; with the lines
  // of a score call, the whole pass of G = 3, 40 x 5000 93.8 us and 90.7 with these, G = 6, 20 x 12000 132 and 128, 16 x 12000
  // 112 and 110)
  const bool saves = from_stats && d.qheads() < kStatsFragsMin;
  if (saves) most += most / 2 + 1000;
  if (tiles * hw.passes > most) return false;
  if (d.units() <= 32 || saves || tiles * hw.passes <= 330) return true;
  // More units fill the chip with either.  One pass: very short heads, and where the LDS-fragment kernel leaves a fifth of the
  // CUs out.  G = 2, 64 x 350 25 and 24, x 700 27 and 29, 100 x 700 31 and 28.
  const int64_t share = num_cu / d.units();
  if (hw.passes == 1) return tiles <= 390 || (share >= 2 && share * d.units() * 5 <= num_cu * 4);
  // Several: where its workgroups take one round, fill three quarters of it and, with a job each, not more than seven eighths
  // (above that some of them run after the others): G = 9, 64 x 2500 82 and 77, 100 x 2500 116 and 130; G = 14, 100 x 700
  // 129 and 88, 128 x 2500 199 and 208; G = 18, 80 x 700 102 and 88, 100 x 700 133 and 151; G = 28, compress, 61 x 778 163
  // and 143.  But G = 5, 64 x 700 37 and 42, and G = 6, 64 x 700, where a workgroup has less than three tiles, 39 and 43.
  const int64_t each = hw.nchunk - hw.spare, wgs = d.units() * hw.passes * each, slots = 2 * (int64_t)num_cu;
  if (more ? lds.passes == 1 : hw.npart < 3 * each) return false;
  return wgs <= slots && wgs * 4 >= slots * 3 && (each > 1 || wgs * 8 <= slots * 7);
}

ScorePlan choose_score_plan(const Dims& d, int64_t n, int num_cu, bool from_stats) {
  const ScorePlan lds = make_score_plan(d, n, num_cu);
  if (d.D != 128 || d.dtype != EA_BF16 || n < kHwTile) return lds;
  const ScorePlan hw = register_plan(d, n, num_cu);
  return registers_serve(d, n, num_cu, lds, hw, from_stats) ? hw : lds;
}

// Where the LDS-fragment kernel would take five heads per pass, the register-fragment one does too, on tensors and on block pools
// alike (a cache's scores do not hang on its layout).  In a row both do the same
// work at the clock that the chip grants; this one starts sooner (26 KiB of fragments per wavefront, not 108 through LDS), leaves
// the softmax partials on its way, and cuts the keys finer.  query_stats + score, us with the LDS-fragment kernel and with
// this one, block pools behind the bar: G = 5, 8 x 20000 53 and 48 | 53 and 51, 64 x 9000 119 and 109 | 117 and 117, 100 x 20000 327
// and 298 | 334 and 319, 150 x 4608 173 and 156; G = 10, 64 x 2900 111 and 98 | 112 and 101; G = 18, 100 x 5000 391 and 339.
// Not where that is all there is:
//   one pass whose workgroups fill the chip with the other kernel, too: 16 x 60000 147 and 153 | 155 and 162, 32 x 131072 544 and
//     562 (but 8 x 60000, 7500 tiles, 92 and 89 | 90 and 94); over more than a few 8-bit rows 128 x 2000 80.9 and 82.1, 32 x 32768
//     142 and 147;
//   two passes over long heads: G = 9, 8 x 20000 73.0 and 71.6, 8 x 60000 138 and 143, 8-bit 128 and 129.
// Nor where its two workgroups per job share out the chip worse than the other kernel's three, which takes heads of some length:
//   one pass, jobs for every CU: 320 x 1500 170 and 168, x 4000 258 and 274, x 13000 610 and 684; 300 x 9000 441 and 498;
//   three and more, a little more than one per CU or than two: 280 to 320 jobs over heads x 6000 up to 12 % more, x 13000 17 % (G = 40,
//     33 units; G = 20, 75), x 2500 even, 350 jobs even; G = 14, 180 x 4608 465 and 483, 200 x 4608 491 and 517; G = 18, 140 x 4000
//     426 and 459 (but G = 14, 230 x 3000 479 and 460).
// In a compress call it comes before the one of four heads per pass, whose lines are drawn further out there (registers_serve):
// the whole pass, us, that one and this one: G = 5, 8 x 12000 73.2 and 69.7, 20 x 5000 73.5 and 68.7; G = 9, 8 x 25000 140 and
// 131; G = 10, 16 x 12000 130 and 123.
ScorePlan serving_score_plan(const Dims& d, int64_t n, int num_cu, bool from_stats) {
  ScorePlan s = choose_score_plan(d, n, num_cu);
  const int64_t tiles = (int64_t)d.units() * ((n + kHwTile - 1) / kHwTile);
  const int64_t jobs = (int64_t)d.units() * s.passes, share = num_cu / d.units();
  const bool filled = share == 0 || share * d.units() * 10 >= (int64_t)num_cu * 9;
  bool long_call = s.passes == 2 && tiles * 2 > 12000;
  if (s.passes == 1) long_call = (d.kv_fp8 && tiles > 2600) || (filled && tiles > 10000) || (jobs >= num_cu && n > 2000);
  else if (s.passes > 2) long_call = (n > 3000 && jobs > num_cu && jobs * 3 < 4 * num_cu) || (n > 2000 && jobs > 2 * num_cu && jobs * 2 < 5 * num_cu);
  if (s.hw || d.D != 128 || d.dtype != EA_BF16 || s.GH != 5 || n < kHwTile || long_call)
    return choose_score_plan(d, n, num_cu, from_stats);
  s.five = 1;
  s.NW = 4;
  s.spare = 0;
  s.lse_pass = 0;
  s.lds_bytes = 0;
  deal_register_workgroups(d, n, num_cu, &s);
  return s;
}

WsLayout make_ws_layout(const Dims& d, int64_t n, int64_t window) {
  WsLayout w;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = align_up(o + bytes, 256);
    return at;
  };
  const size_t qh = (size_t)d.qheads(), un = (size_t)d.units();
  // the fragments: those of whichever kernel needs more of them, whatever the cache layout
  int unit_frags = make_score_plan(d, n, 256).unit_frags;
  if (d.D == 128 && register_plan(d, n, 256).unit_frags > unit_frags) unit_frags = register_plan(d, n, 256).unit_frags;
  const size_t frags_per_unit = (size_t)unit_frags * 1024;
  w.tab = take((size_t)window * d.half * 2 * sizeof(float));
  w.qproj = take(qh * (size_t)window * d.D * sizeof(float));   // projected queries of ea_query_stats_hidden
  w.mu = take(qh * d.D * sizeof(float));
  w.sigma = take(qh * d.D * d.D * sizeof(float));
  w.frags = take(un * frags_per_unit);
  w.post = take(qh * 2 * sizeof(float));
  w.logits = take(qh * (size_t)n * 8);          // fp32 logits (bf16 path) or fp64 (fp32 path)
  w.vnorm = take(un * (size_t)n * sizeof(float));
  // (max, sum exp) partials: float2 per fixed block of keys (bf16 path), double2 per chunk (fp32 path)
  size_t part_bytes = qh * (((size_t)n + 31) / 32) * 8;     // the finest block any plan uses
  if (part_bytes < qh * 1024 * 16) part_bytes = qh * 1024 * 16;
  w.part = take(part_bytes);
  w.lse = take(qh * sizeof(double));
  w.scores = take(un * (size_t)n * sizeof(float));
  w.idx = take(un * (size_t)n * sizeof(int32_t));
  w.base = take(un * kBaselineChunks * d.D * sizeof(float));    // KeyDiff partial sums
  w.hist = take(un * 3 * kSelBins * sizeof(uint32_t) + 256);
  w.pool_hist = take((size_t)d.B * 3 * kSelBins * sizeof(uint32_t));    // of a sequence's heads taken together
  size_t nblk = ((size_t)n + kSelBlock - 1) / kSelBlock;
  w.blk = take(un * nblk * 2 * sizeof(uint32_t));
  size_t nch = ((size_t)n + kCompactRows - 1) / kCompactRows;
  w.flags = take(2 * un * (nch + kCompactTicketStride) * sizeof(uint32_t));   // ticket counters, then flags
  w.total = o;
  return w;
}

}  // namespace ea

extern "C" {

size_t ea_workspace_bytes(const ea_params* p, int64_t n, int64_t window) {
  ea::Dims d;
  if (ea::check_params(p, &d, true) != EA_OK) return 0;
  if (n < 1 || n > ea::kMaxN || window < 1 || window > ea::kMaxWindow) return 0;
  return ea::make_ws_layout(d, n, window).total;
}

int64_t ea_n_keep(int64_t n, double ratio) {
  if (n < 0 || !(ratio >= 0.0) || !(ratio <= 1.0)) return -1;
  return (int64_t)((double)n * (1.0 - ratio));
}

const char* ea_status_string(ea_status s) {
  switch (s) {
    case EA_OK: return "ok";
    case EA_ERR_INVALID_ARG: return "invalid argument";
    case EA_ERR_UNSUPPORTED: return "unsupported configuration";
    case EA_ERR_WORKSPACE: return "workspace too small";
    case EA_ERR_DEVICE: return "device launch failed";
  }
  return "unknown status";
}

}  // extern "C"

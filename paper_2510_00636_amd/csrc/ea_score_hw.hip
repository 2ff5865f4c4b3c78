// Score pass A at d = 128 with the Sigma fragments held in REGISTERS, four query heads per pass (Eq. 7 of the paper:
// l_g = mu_g.k/sqrt(d) + k^T Sigma_g k/(2d) for every cached key).
//
// The LDS-fragment kernel (ea_score_mfma.h) reads one 1 KiB fragment from LDS per matrix-core instruction; with four SIMDs
// that is the whole LDS bandwidth of a CU at the matrix cores' peak, and a workgroup starts with 96 KiB of them.  Here a
// workgroup is four wavefronts, one per query head: each keeps its head's 20 triangular fragments and the 8 of the extra
// rows in registers, and the four share ONE tile of 64 keys per iteration, converted to fp16 once.  Two workgroups fit a CU.
//
//   * K tile: each wavefront loads 16 rows of the tile after next (coalesced 16-byte loads, in flight for a whole
//     iteration), converts those that arrived bf16 / e4m3 -> fp16 and writes them to LDS as 16-byte chunks; lane
//     (c, q) = (l % 16, l / 16) reads chunk 4 b + q of key 16 m + c as its B operand of k-step b for key group m.
//   * V rows: same split; squared norms straight from the coalesced registers.
//   * quadratic form: v_mfma_f32_16x16x32_f16, A = 16 output channels x 32 input channels of M, every fragment used for
//     two key groups in a row; a lane gets back channels it holds of the same keys, so k.(M k) is 4 FMAs per tile.
//   * extra rows (fp16 head / tail of mu_g on k, rounding residual of diag(Sigma_g) on k^2): wavefront w computes those of
//     all four heads for key group w; they go through LDS and every wavefront picks up its own head's an iteration later.
//   * softmax partials: (max, sum exp) per tile of 64 keys, so that the finalize pass combines the same numbers in the
//     same order on every run, whichever workgroup scored the tile.
//
// What bounds it: instruction issue (88 matrix and 300 to 350 vector instructions per wavefront and tile, 2100 cycles of the
// issue port; two wavefronts per SIMD take 4900 for one each) and the clock, which falls with what the operands make the matrix cores
// draw: 2.4 GHz in a copy, 1.9 for one call of 4 x 8 heads x 131072 keys after a pause, 1.7 with such calls in a row.  Of the
// 16-bit forms the 16x16x32 one then gets most done (random data 1900 TFLOP/s, 32x32x16 1660, bf16 1440; zeros 2450), and
// every zero in the operands helps, which is why the fragments on the diagonal are folded onto their triangle too (8-bit
// cache, 8 x 131072 keys: 115 -> 112.5 us).  Against the kernel it
// replaces (32x32x16, tiles of 32 keys, four fragments re-read from LDS; contiguous bf16 only) and, for 8-bit caches and
// block pools, the LDS-fragment one: operands + score, 8 heads of 4 x 131072 keys 155 -> 128 us, 8-bit 120 -> 110, x 16384
// 38 -> 31, keys only x 32768 46 -> 43, pools of 16-row blocks x 20011 44 -> 39.
//
// FIVE: five query heads per pass, each wavefront with a head of its own and a quarter of the fifth one's triangle; the extra
// rows' fragments then stand in LDS, and the fifth head's logits and softmax partials are the wavefronts' in turn.  In a
// row it does what the LDS-fragment kernel does (8 heads of 5 x 131072 keys 155 and 156 us: the clock), but it starts
// sooner and leaves no partials to another launch: x 20000 54.4 -> 50.9, 192 x 4608 184 -> 177, 320 x 1500 171 -> 163; where
// which of them is taken stands at serving_score_plan.
//
// Scales and the meaning of `post` are those of k_prep_frags (ea_stats.hip).
#include "ea_score_mfma.h"

namespace ea {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// The 40 steps of an iteration (52 for five heads), two 16x16x32 instructions with the same fragment each: the output tiles 0 .. 7 of the
// quadratic form of keys 0-15 and 16-31, then of keys 32-47 and 48-63.  Tile j takes the k-steps 0 .. j / 2.

// Sums over the four groups of 16 lanes of four values per lane: value m, complete, in the lanes of group m.
__device__ __forceinline__ float sum_groups(const float (&p)[4]) {
  auto merge32 = [](float x, float y) {      // lower half: x of both halves, upper half: y of both
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  const float e = merge32(p[0], p[2]), o = merge32(p[1], p[3]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(e), __float_as_uint(o), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}


// Maxima of lane l and lane l ^ 16, l ^ 32, or another lane of the row of 16; the median of x, y and infinity is one
// instruction where fmaxf, which first quiets a signalling operand, makes three.
__device__ __forceinline__ float max_of(float x, float y) {
  float inf = INFINITY;
  asm("" : "+s"(inf));                    // (or the compiler makes the longer form of it)
  return __builtin_amdgcn_fmed3f(x, y, inf);
}
__device__ __forceinline__ float max_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_of(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_of(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int CTRL>
__device__ __forceinline__ float max_dpp(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true);
  return max_of(x, __int_as_float(y));
}

// FIVE heads per pass: every wavefront also multiplies a quarter of the fifth head's triangle, output tiles w and 7 - w of
// wavefront w: one or two k-steps of the first and three or four of the second, taken as two and four (a step that the
// tile does not have multiplies zeros), as tiles 8 and 9 of the schedule and fragments 20 .. 25 of the wavefront.
struct HwStep { int sub, tile, kt, frag, set; };
template <bool FIVE> constexpr int kHwTiles = FIVE ? 10 : 8;         // output tiles per pair of key groups
template <bool FIVE> constexpr int kHwSteps = FIVE ? 26 : 20;        // and steps
template <bool FIVE>
constexpr int hw_end(int u) {              // last step of tile u of the iteration (u = 0 .. 2 kHwTiles - 1)
  int e = -1;
  for (int i = 0; i <= u; ++i) {
    const int j = i % kHwTiles<FIVE>;
    e += j < 8 ? j / 2 + 1 : j == 8 ? 2 : 4;
  }
  return e;
}
template <bool FIVE>
constexpr HwStep hw_step(int f) {
  int u = 0;
  while (hw_end<FIVE>(u) < f) ++u;
  const int first = u == 0 ? 0 : hw_end<FIVE>(u - 1) + 1, j = u % kHwTiles<FIVE>, kt = f - first;
  return HwStep{u / kHwTiles<FIVE>, j, kt, (j < 8 ? j / 2 * (j / 2 + 1) + j % 2 * (j / 2 + 1) : j == 8 ? 20 : 22) + kt, u % 4};
}

// MODE kHwNoV: the caller has weights of its own, V is not read.  kHwNorms: neither, nor a softmax; the quadratic forms
// leave as norms sqrt(k^T M k) (the rows are values then, M = W_o^T W_o, mu = 0).
constexpr int kHwScores = 0, kHwNoV = 1, kHwNorms = 2;

template <bool FP8, bool PAGED, int MODE, bool FIVE>
__global__ __launch_bounds__(256, 2) void k_score_hw(ScoreArgs a) {
  constexpr int NKS = 4, NF = 20, GH = FIVE ? 5 : 4;
  constexpr int HT = kHwTiles<FIVE>, HS = kHwSteps<FIVE>;
  constexpr int RB = FP8 ? 128 : 256;        // bytes of a row
  constexpr int NL = FP8 ? 2 : 4;            // wave-wide loads of a wavefront's 16 rows
  constexpr int S = kHwTile;                 // slots between the 16-byte chunks of a row in LDS
  // fp16 K tile [16-byte chunk of the row][key ^ chunk]: double buffered.  The swizzle keeps both the staging writes (16
  // chunks of a row) and the operand reads (16 keys of four chunks) free of bank conflicts.
  __shared__ u32x4 s_k[2][16 * S];
  constexpr int SP = 68;                     // pitch of the extra rows: the four rows a wavefront touches at once in different banks
  __shared__ float s_p[2][16 * SP];          // extra rows: [buffer][row][key]
  __shared__ int s_tk[8];                    // ring of tiles, by ordinal
  // FIVE: fragments of the extra rows (registers otherwise); the wavefronts' parts of the fifth head's form: [buffer][wavefront][key]
  __shared__ u32x4 s_x[FIVE ? 2 * NKS * 64 : 1];
  __shared__ float s_q5[2][FIVE ? 4 * S : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q = lane >> 4;  // matrix-core column (key of a group of 16) and group of rows / channels
  const int lrow = FP8 ? lane >> 3 : lane >> 4, lch = FP8 ? lane & 7 : lane & 15;

  int bid = blockIdx.x;
  if (a.transposed && (gridDim.x & 7u) == 0) bid = (bid & 7) * (int)(gridDim.x >> 3) + (bid >> 3);
  int unit = bid % a.units;
  const int t2 = bid / a.units;
  int chunk = t2 % a.nchunk, pass = t2 / a.nchunk;
  if (a.spare) {                             // more workgroups than the chip holds: see k_score_mfma
    chunk = t2 / a.passes;
    pass = t2 % a.passes;
    unit = (unit + 3 * chunk) % a.units;
  }
  const int g0 = pass * GH;
  constexpr bool kV = MODE == kHwScores;
  const bool do_v = pass == 0;
  const int n = (int)a.n;
  const int ntiles = (n + kHwTile - 1) / kHwTile;

  // Tiles of a (unit, pass): the first two of a workgroup by its number, the others as they are drawn from its counter,
  // the last tile of the head first (see k_score_mfma).
  const int ways = hw_ways(a.nchunk);
  const HwDeal deal = hw_deal(chunk, a.nchunk, ways);
  const int way = deal.way, nth = deal.nth, peers = deal.peers;
  uint32_t* tk = a.tickets + (size_t)unit * a.ticket_stride + ticket_word(pass, way);
  auto tile_of = [&](int raw) { return hw_tile(raw, way, ways, ntiles); };
  int t_cur = tile_of(nth), t_n1 = tile_of(peers + nth);
  const int dealt = a.spare ? 0 : 2 * peers; // tiles of the class that are dealt by number
  uint32_t draw2 = 0, draw3 = 0;
  if (a.spare) {                             // all tiles are drawn: a workgroup may come when there are none left
    if (tid == 0) {
      const uint32_t d0 = atomicAdd(tk, 1u), d1 = atomicAdd(tk, 1u);
      draw2 = atomicAdd(tk, 1u);
      draw3 = atomicAdd(tk, 1u);
      s_tk[0] = tile_of((int)d0);
      s_tk[1] = tile_of((int)d1);
    }
    __syncthreads();
    t_cur = __builtin_amdgcn_readfirstlane(s_tk[0]);
    t_n1 = __builtin_amdgcn_readfirstlane(s_tk[1]);
  }
  if (t_cur < 0) return;                     // it came too late; or (short heads) its class has fewer tiles than workgroups
  if (!a.spare && tid == 0) {
    draw2 = atomicAdd(tk, 1u);
    draw3 = atomicAdd(tk, 1u);
  }

  const char* kbase = (const char*)a.k + (PAGED ? (size_t)0 : (size_t)unit * a.n_cap * RB);
  const char* vbase = (const char*)a.v + (PAGED ? (size_t)0 : (size_t)unit * a.n_cap * RB);
  // byte offset of this lane's 16 bytes in load j, from the first of the wavefront's 16 rows
  const uint32_t row_off = (uint32_t)lrow * RB, ch_off = (uint32_t)lch * 16;
  // first row of tile t (contiguous: the last one is moved back to end at row n)
  auto base_row = [&](int t) -> int { return t < 0 ? 0 : PAGED ? t * kHwTile : min(t * kHwTile, n - kHwTile); };
  // where the wavefront's 16 rows of tile t start, in bytes
  auto rows_at = [&](int t) -> size_t {
    const int row = base_row(t) + 16 * w;
    if constexpr (!PAGED) return (size_t)row * RB;
    // (a wavefront's rows lie inside one block; past the end of the head: its last 16 rows)
    else return paged_row(a.pm, unit, min(row, (n - 1) & ~15)) * RB;
  };
  // PAGED: rows past the end of the head become its last row again: of the 16 rows, those that are loaded
  struct Lim { int lo, hi; };
  auto rows_left = [&](int t) -> Lim {
    const int row = base_row(t) + 16 * w, last = (n - 1) & ~15, hi = min(n - 1 - min(row, last), 15);
    return Lim{row > last ? hi : 0, hi};
  };

  u32x4 rawK[NL], rawV[NL];
  auto lane_off = [&](int j, const Lim& lim) -> uint32_t {
    if constexpr (!PAGED) return row_off + ch_off;          // + j KiB as an immediate
    else return (uint32_t)max(lim.lo, min(j * (16 / NL) + lrow, lim.hi)) * RB + ch_off;
  };
  auto load_k = [&](int j, size_t at, const Lim& lim) __attribute__((always_inline)) {
    rawK[j] = __builtin_nontemporal_load((const u32x4*)(kbase + at + (PAGED ? 0 : j * 1024) + lane_off(j, lim)));
  };
  auto load_v = [&](int j, size_t at, const Lim& lim) __attribute__((always_inline)) {   // later passes: the same 16 rows of the head
    rawV[j] = __builtin_nontemporal_load((const u32x4*)(vbase + (do_v ? at : 0) + (PAGED ? 0 : j * 1024) + lane_off(j, lim)));
  };
  {
    const size_t at = rows_at(t_cur);
    const Lim lim = rows_left(t_cur);
#pragma unroll
    for (int j = 0; j < NL; ++j) load_k(j, at, lim);
    if constexpr (kV) {
#pragma unroll
      for (int j = 0; j < NL; ++j) load_v(j, at, lim);
    }
  }

  // this head's fragments (and this wavefront's of the fifth head), and those of the extra rows
  half8 F[FIVE ? NF + 6 : NF], X[FIVE ? 1 : 2 * NKS];
  {
    // (five heads per pass: the layout of the LDS-fragment kernels)
    const u32x4* src = a.frags + ((size_t)unit * a.unit_frags + (FIVE ? pass * (5 * NF + 2 * NKS) : g0 * NF)) * 64;
    const u32x4* ext = FIVE ? src + 5 * NF * 64 : a.frags + ((size_t)unit * a.unit_frags + a.G * NF + pass * 2 * NKS) * 64;
    const bool mine = g0 + w < a.G;          // a wavefront without a head multiplies zeros, which cost the clock least
#pragma unroll
    for (int i = 0; i < NF; ++i)
      F[i] = mine ? __builtin_bit_cast(half8, src[(w * NF + i) * 64 + lane]) : (half8)(_Float16)0.f;
    if constexpr (FIVE) {
      const int j0 = w, j1 = 7 - w;
      const u32x4* fifth = src + 4 * NF * 64;
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        const int j = i < 2 ? j0 : j1, kt = i < 2 ? i : i - 2, h = j / 2 + 1;
        F[NF + i] = g0 + 4 < a.G && kt < h ? __builtin_bit_cast(half8, fifth[((j / 2 + j % 2) * h + kt) * 64 + lane]) : (half8)(_Float16)0.f;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) s_x[i * 256 + tid] = ext[i * 256 + tid];
    } else {
#pragma unroll
      for (int i = 0; i < 2 * NKS; ++i) X[i] = __builtin_bit_cast(half8, ext[i * 64 + lane]);
    }
  }
  const float ks = (FP8 && a.kscale) ? a.kscale[unit] : 1.0f;
  const float vs2 = (FP8 && a.vscale) ? a.vscale[unit] * a.vscale[unit] : 1.0f;
  // post[2g] = 1 / (2 d sM_g), post[2g+1] = 1 / (sqrt(d) smu_g)
  float pq_mine = 0.f, sc_mine = 0.f;        // sc: of the extra rows that this lane adds up (4 q + w: head, tail, residual, nothing)
  if (g0 + w < a.G) {
    pq_mine = a.post[((size_t)unit * a.G + g0 + w) * 2 + 0] * (ks * ks);
    sc_mine = a.post[((size_t)unit * a.G + g0 + w) * 2 + 1] * ks;
    sc_mine = q < 2 ? sc_mine : q == 2 ? 256.0f * pq_mine : 0.f;
  }
  float pq5 = 0.f, sc5 = 0.f;                // of the fifth head
  const bool five = FIVE && g0 + 4 < a.G;
  if (five) {
    auto scalar = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
    pq5 = scalar(a.post[((size_t)unit * a.G + g0 + 4) * 2 + 0] * (ks * ks));
    sc5 = scalar(a.post[((size_t)unit * a.G + g0 + 4) * 2 + 1] * ks);
    pq_mine = scalar(pq_mine);
  }

  float* dump = a.dump;                                     // at least n floats; contents never read
  const bool mine = g0 + w < a.G;                           // this wavefront has a head
  float* lg_out = mine ? a.logits + ((size_t)unit * a.G + g0 + w) * a.n : dump;
  float* vn_eff = do_v ? a.vnorm + (size_t)unit * a.n : dump;
  float2* part_out = a.part + ((size_t)unit * a.G + g0 + (mine ? w : 0)) * a.npart;

  // K chunk j of the raw rows -> fp16 -> LDS
  const int row0 = 16 * w + lrow, chunk0 = FP8 ? 2 * lch : lch;
  auto stage_k = [&](int j, int buf) __attribute__((always_inline)) {
    const int row = row0 + j * (16 / NL);
    if constexpr (FP8) {
      half8 lo, hi;
      fp8x16_to_half8x2(rawK[j], lo, hi);
      s_k[buf][chunk0 * S + (row ^ chunk0)] = __builtin_bit_cast(u32x4, lo);
      s_k[buf][(chunk0 + 1) * S + (row ^ (chunk0 + 1))] = __builtin_bit_cast(u32x4, hi);
    } else {
      s_k[buf][chunk0 * S + (row ^ chunk0)] = __builtin_bit_cast(u32x4, bf16x8_to_half8(rawK[j]));
    }
  };
  auto square_v = [&](int j) __attribute__((always_inline)) -> float {
    return FP8 ? sumsq_fp8x16(rawV[j]) : sumsq_bf16x8(rawV[j]);
  };
  // The sums over the lanes of a row; this lane ends up with load lch & 3 (FP8: lch / 4): the first steps of the
  // butterfly hand half of the loads to each side.
  auto reduce_v = [&](const float (&s)[NL]) __attribute__((always_inline)) -> float {
    float x;
    if constexpr (FP8) {
      const bool o4 = lane & 4;
      x = dpp_add_of<0x141>(o4 ? s[1] : s[0], o4 ? s[0] : s[1]);
      x = dpp_add<0xB1>(x);
      x = dpp_add<0x4E>(x);
    } else {
      const bool o1 = lane & 1, o2 = lane & 2;
      const float a0 = dpp_add_of<0xB1>(o1 ? s[1] : s[0], o1 ? s[0] : s[1]);
      const float a1 = dpp_add_of<0xB1>(o1 ? s[3] : s[2], o1 ? s[2] : s[3]);
      x = dpp_add_of<0x4E>(o2 ? a1 : a0, o2 ? a0 : a1);
      // 4 lanes of a quad hold 4 loads; the quads of a row of 16 hold parts of the same sums: rotations by 4 and 8
      x = dpp_add<0x124>(x);
      x = dpp_add<0x128>(x);
    }
    return x;
  };
  const int vn_row = 16 * w + (FP8 ? lch >> 2 : lch & 3) * (16 / NL) + lrow;
  auto out_value = [&](float lg) __attribute__((always_inline)) -> float {
    if constexpr (MODE != kHwNorms) return lg;
    const float x = lg * 256.f;              // 2 d
    return x > 0.f ? sqrtf(x) : 0.f;
  };
  // keys past the end (PAGED) hold the last key again: same value, same place
  auto out_row = [&](int row) -> int { return PAGED ? min(row, n - 1) : row; };

  {
#pragma unroll
    for (int j = 0; j < NL; ++j) stage_k(j, 0);
    if constexpr (kV) {
      float sv[NL];
#pragma unroll
      for (int j = 0; j < NL; ++j) sv[j] = square_v(j);
      const float x = reduce_v(sv);
      vn_eff[out_row(base_row(t_cur) + vn_row)] = __builtin_amdgcn_sqrtf(FP8 ? x * vs2 : x);
    }
    const size_t at = rows_at(t_n1);
    const Lim lim = rows_left(t_n1);
#pragma unroll
    for (int j = 0; j < NL; ++j) load_k(j, at, lim);
    if constexpr (kV) {
#pragma unroll
      for (int j = 0; j < NL; ++j) load_v(j, at, lim);
    }
  }
  if (tid == 0) {
    s_tk[2] = tile_of(dealt + (int)draw2);
    s_tk[3] = tile_of(dealt + (int)draw3);
  }
  __syncthreads();

  float quad[4] = {0.f, 0.f, 0.f, 0.f};      // of the previous tile, by group of 16 keys
  int t_prev = -1;
  uint32_t pend = 0;                         // wavefront 0, lane 0: the draw waiting to be published
  int s = 0;
  // lane's B operand of k-step b for key group m: s_k[.][kh_idx[b] + 16 m]
  int kh_idx[NKS];
#pragma unroll
  for (int b = 0; b < NKS; ++b) kh_idx[b] = (4 * b + q) * S + (c16 ^ (4 * b + q));
  // (the last rows are the fifth head's: what the fourth group of lanes adds nothing of is its own head's, too)
  const int p_out = 4 * q * SP + 16 * w + c16;
  auto row_in = [&](int l) { return (4 * (FIVE ? min(l >> 4, 2) : l >> 4) + w) * SP + (l & 15); };
  const int p_in = row_in(lane);
  // FIVE: the fifth head's logit of key `lane` of tile t, from the buffers of its iteration
  auto fifth_logit = [&](int pb, int lane) __attribute__((always_inline)) -> float {
    const float* qp = s_q5[pb] + lane;
    const float* ep = s_p[pb] + 12 * SP + lane;
    const float quad5 = (qp[0] + qp[S]) + (qp[2 * S] + qp[3 * S]);
    return fmaf(quad5, pq5, fmaf(ep[0] + ep[SP], sc5, ep[2 * SP] * (256.0f * pq5)));
  };
  // PAGED: the keys of the head's last tile to the lanes that have them where that tile ends at row n, so that the partial is
  // the same sum, in the same order, on either cache layout.
  auto to_end = [&](float x, int t) __attribute__((always_inline)) -> float {
    if constexpr (!PAGED) return x;
    const int here = min(n - base_row(t), kHwTile);
    return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (lane + here), __float_as_int(x)));
  };
  // logit of key `lane` and softmax partial of a finished tile, where that is not spread over the steps
  auto finish_row = [&](float lg, int t, float* lg_to, float2* part_to, bool here) __attribute__((always_inline)) {
    const int row = base_row(t) + lane;
    lg_to[out_row(row)] = out_value(lg);
    if constexpr (MODE != kHwNorms) {
      const bool valid = PAGED ? row < n : row >= t * kHwTile;
      lg = to_end(valid ? lg : -INFINITY, t);
      float m = lg;
      m = max_dpp<0x140>(max_dpp<0x141>(max_dpp<0x4E>(max_dpp<0xB1>(max_xor32(max_xor16(m))))));
      float e = expf(lg - m);
      e = sum_halves(sum_xor16(dpp_add<0x140>(dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(e))))));
      if (here && lane == 0) part_to[t] = make_float2(m, e);
    }
  };
  float* lg5_out = five ? a.logits + ((size_t)unit * a.G + g0 + 4) * a.n : dump;
  float2* part5_out = a.part + ((size_t)unit * a.G + g0 + (five ? 4 : 0)) * a.npart;

  // One body, the buffers by a number that the compiler does not know: unrolled for the two of them, the loop gets two
  // exits, and the paths that then join in front of it make every wavefront wait there for all the loads in flight.
  do {
    const int PB = s & 1;
    constexpr floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    half8 K[2][2][NKS], Kx[NKS];
    // (FIVE has no registers to keep the four addresses in; they differ from the first in two bits of the key's place)
    int k_at = kh_idx[0];
    if constexpr (FIVE) asm volatile("" : "+v"(k_at));
    auto k_index = [&](int kt) __attribute__((always_inline)) { return FIVE ? (k_at ^ (4 * kt)) + 4 * kt * S : kh_idx[kt]; };
    auto read_k = [&](int m, int kt) __attribute__((always_inline)) {
      return __builtin_bit_cast(half8, s_k[PB][k_index(kt) + 16 * m]);
    };
    auto read_pair = [&](auto sub_, auto kt_) __attribute__((always_inline)) {
      constexpr int sub = decltype(sub_)::value, kt = decltype(kt_)::value;
      K[sub][0][kt] = read_k(2 * sub, kt);
      K[sub][1][kt] = read_k(2 * sub + 1, kt);
    };
    read_pair(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    read_pair(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
#pragma unroll
    for (int b = 0; b < NKS; ++b) Kx[b] = read_k(w, b);
    float lp[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) lp[m] = s_p[PB ^ 1][p_in + 16 * m];
    const int t_n2 = __builtin_amdgcn_readfirstlane(s_tk[(s + 2) & 7]);
    const size_t at_n2 = rows_at(t_n2);
    const Lim lim_n2 = rows_left(t_n2);
    __builtin_amdgcn_sched_barrier(0);

    floatx4 acc[4][2], ex;
    half8 sq;
    float dot[4] = {0.f, 0.f, 0.f, 0.f}, dot5[4] = {0.f, 0.f, 0.f, 0.f};
    uint2 k5[2][2];                          // FIVE: this lane's channels of output tiles w and 7 - w, both key groups
    half8 xf[FIVE ? 2 * NKS : 1];
    float sv[NL], lg = 0.f, lm = 0.f, le = 0.f, vn = 0.f;
    const int row_prev = base_row(t_prev) + lane;
    auto dots = [&](auto u_, auto h_) __attribute__((always_inline)) {     // rows 2 h, 2 h + 1 of the tile, both groups
      constexpr int u = decltype(u_)::value, h = decltype(h_)::value, sub = u / HT, j = u % HT;
      static_for<2>([&](auto v_) {
        constexpr int v = 2 * h + decltype(v_)::value;
        if constexpr (j < 8) {
          dot[2 * sub] = fmaf(acc[u % 4][0][v], (float)K[sub][0][j / 2][4 * (j % 2) + v], dot[2 * sub]);
          dot[2 * sub + 1] = fmaf(acc[u % 4][1][v], (float)K[sub][1][j / 2][4 * (j % 2) + v], dot[2 * sub + 1]);
        } else {
          typedef _Float16 half4 __attribute__((ext_vector_type(4)));
          dot5[2 * sub] = fmaf(acc[u % 4][0][v], (float)__builtin_bit_cast(half4, k5[j - 8][0])[v], dot5[2 * sub]);
          dot5[2 * sub + 1] = fmaf(acc[u % 4][1][v], (float)__builtin_bit_cast(half4, k5[j - 8][1])[v], dot5[2 * sub + 1]);
        }
      });
      if constexpr (j < 8) asm volatile("" : "+v"(dot[2 * sub]), "+v"(dot[2 * sub + 1]));
      else asm volatile("" : "+v"(dot5[2 * sub]), "+v"(dot5[2 * sub + 1]));
    };
    __builtin_amdgcn_s_setprio(1);
    static_for<2 * HS + 3>([&](auto f_) {
      constexpr int f = decltype(f_)::value;
      if constexpr (f < 2 * HS) {
        constexpr HwStep st = hw_step<FIVE>(f);
#pragma unroll
        for (int m = 0; m < 2; ++m)
          acc[st.set][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(F[st.frag], K[st.sub][m][st.kt], st.kt == 0 ? zero4 : acc[st.set][m], 0, 0, 0);
      }
      // -- extra rows of key group w
      if constexpr (FIVE && f < 2 * NKS) xf[f] = __builtin_bit_cast(half8, s_x[(f / 2 + f % 2 * NKS) * 64 + lane]);
      if constexpr (f >= 2 && f < 2 + 2 * NKS) {
        constexpr int b = (f - 2) / 2;
        if constexpr (f % 2 == 0) {
          const half8 t = Kx[b] * (_Float16)0.0625f;
          // saturate instead of overflowing for |k| > 4096: infinity times a zero residual is NaN
          sq = __builtin_elementwise_min(t * t, (half8)(_Float16)65504.0f);
          ex = __builtin_amdgcn_mfma_f32_16x16x32_f16(FIVE ? xf[FIVE ? 2 * b : 0] : X[FIVE ? 0 : b], Kx[b], b == 0 ? zero4 : ex, 0, 0, 0);
        } else {
          ex = __builtin_amdgcn_mfma_f32_16x16x32_f16(FIVE ? xf[FIVE ? 2 * b + 1 : 0] : X[FIVE ? 0 : NKS + b], sq, ex, 0, 0, 0);
        }
      }
      if constexpr (f == 12) {
#pragma unroll
        for (int v = 0; v < 4; ++v) s_p[PB][p_out + v * SP] = ex[v];
      }
      // -- operands, a few steps ahead of their first use
      if constexpr (f == 2) read_pair(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
      if constexpr (f == 6) read_pair(std::integral_constant<int, 0>{}, std::integral_constant<int, 3>{});
      if constexpr (f == (FIVE ? HS - 2 : HS - 4)) read_pair(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{});
      if constexpr (f == (FIVE ? HS : HS - 2)) read_pair(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
      if constexpr (f == HS + 2) read_pair(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
      if constexpr (f == HS + 6) read_pair(std::integral_constant<int, 1>{}, std::integral_constant<int, 3>{});
      if constexpr (FIVE) {                  // (tiles 8 and 9 start at steps 20 and 22 of a pair of key groups)
        if constexpr (f % HS == 17 || f % HS == 19) {
          constexpr int i = f % HS == 17 ? 0 : 1, sub = f / HS;
          const int j = i == 0 ? w : 7 - w;  // the lane's four channels of output tile j
          const uint2* at = reinterpret_cast<const uint2*>(s_k[PB]) + k_index(j >> 1) * 2 + (j & 1) + 64 * sub;
          k5[i][0] = at[0];
          k5[i][1] = at[32];
        }
      }
      // -- the previous tile's logits, key `lane` of 64
      if constexpr (f == 0) {
        float p[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) p[m] = fmaf(quad[m], pq_mine, lp[m] * sc_mine);
        lg = sum_groups(p);
      }
      if constexpr (f == 2) {
        char* dst = (char*)(t_prev >= 0 ? lg_out : dump);
        *(float*)(dst + (uint32_t)(4 * out_row(row_prev))) = out_value(lg);
        const bool valid = PAGED ? row_prev < n : row_prev >= t_prev * kHwTile;
        lg = to_end(valid ? lg : -INFINITY, t_prev);
        if constexpr (!PAGED) lm = lg;
      }
      if constexpr (PAGED && f == 5) lm = lg;
      // -- its softmax partial: max and sum over the 64 lanes, one step of the butterflies at a time
      if constexpr (MODE != kHwNorms) {
        if constexpr (f == 5) lm = max_xor16(lm);
        if constexpr (f == 6) lm = max_xor32(lm);
        if constexpr (f == 7) lm = max_dpp<0xB1>(lm);
        if constexpr (f == 9) lm = max_dpp<0x4E>(lm);
        if constexpr (f == 11) lm = max_dpp<0x141>(lm);
        if constexpr (f == 13) lm = max_dpp<0x140>(lm);
        if constexpr (f == 15) le = expf(lg - lm);
        if constexpr (f == 18) le = dpp_add<0xB1>(le);
        if constexpr (f == 19) le = dpp_add<0x4E>(le);
        if constexpr (f == 21) le = dpp_add<0x141>(le);
        if constexpr (f == 23) le = dpp_add<0x140>(le);
        if constexpr (f == 25) le = sum_xor16(le);
        if constexpr (f == 27) le = sum_halves(le);
      }
      // -- staging of the next tile, each chunk requested again for the one after it
      constexpr int L0 = 2 * HS - 10;
      if constexpr (f >= L0 && f < L0 + 2 * NL && (f & 1) == 0) {
        constexpr int j = (f - L0) / 2;
        stage_k(j, PB ^ 1);
        load_k(j, at_n2, lim_n2);
      }
      if constexpr (kV && f >= L0 + 1 && f < L0 + 1 + 2 * NL && (f & 1) == 1) {
        constexpr int j = (f - L0 - 1) / 2;
        sv[j] = square_v(j);
        load_v(j, at_n2, lim_n2);
      }
      if constexpr (kV && f == L0 + 9) vn = reduce_v(sv);
      if constexpr (kV && f == L0 + 10) *(float*)((char*)vn_eff + (uint32_t)(4 * out_row(base_row(t_n1) + vn_row))) = __builtin_amdgcn_sqrtf(FP8 ? vn * vs2 : vn);
      // -- dot products of finished output tiles with k
      static_for<2 * HT>([&](auto u_) {
        constexpr int u = decltype(u_)::value, e = hw_end<FIVE>(u);
        if constexpr (f == e + 2) dots(u_, std::integral_constant<int, 0>{});
        if constexpr (f == e + 3) dots(u_, std::integral_constant<int, 1>{});
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_s_setprio(0);
    // ---- tail: the parts that need a branch
    if constexpr (FIVE) {
      s_q5[PB][w * S + lane] = sum_groups(dot5);
      // the fifth head's previous tile, by the wavefronts in turn
      if (five && t_prev >= 0 && w == (s & 3)) finish_row(fifth_logit(PB ^ 1, lane), t_prev, lg5_out, part5_out, true);
    }
    if (MODE != kHwNorms && t_prev >= 0 && mine && lane == 0) part_out[t_prev] = make_float2(lm, le);
    if (tid == 0) {
      if (s >= 1) s_tk[(s + 3) & 7] = tile_of(dealt + (int)pend);
      pend = atomicAdd(tk, 1u);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) quad[m] = dot[m];
    t_prev = t_cur;
    t_cur = t_n1;
    t_n1 = t_n2;
    ++s;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  } while (t_cur >= 0);
  // the last tile's logits
  if (t_prev >= 0) {
    const int pb = (s - 1) & 1;
    int l = lane;
    if constexpr (FIVE) asm volatile("" : "+v"(l));          // (the addresses once more, not kept in registers through the loop)
    float p[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) p[m] = fmaf(quad[m], pq_mine, s_p[pb][row_in(l) + 16 * m] * sc_mine);
    finish_row(sum_groups(p), t_prev, lg_out, part_out, mine);
    if (five && w == (s & 3)) finish_row(fifth_logit(pb, l), t_prev, lg5_out, part5_out, true);
  }
}

template <bool FIVE>
static void launch_score_hw_heads(const ScoreArgs& a, bool fp8, hipStream_t st) {
  const int grid = a.units * a.nchunk * a.passes;
  if (a.pm.table) k_score_hw<false, true, kHwScores, FIVE><<<grid, 256, 0, st>>>(a);
  else if (fp8) k_score_hw<true, false, kHwScores, FIVE><<<grid, 256, 0, st>>>(a);
  else if (a.norms_out) k_score_hw<false, false, kHwNorms, FIVE><<<grid, 256, 0, st>>>(a);
  else if (a.skip_v) k_score_hw<false, false, kHwNoV, FIVE><<<grid, 256, 0, st>>>(a);
  else k_score_hw<false, false, kHwScores, FIVE><<<grid, 256, 0, st>>>(a);
}

hipError_t launch_score_hw(const ScoreArgs& a, const ScorePlan& sp, bool fp8, hipStream_t st) {
  if (sp.five) launch_score_hw_heads<true>(a, fp8, st);
  else launch_score_hw_heads<false>(a, fp8, st);
  return hipGetLastError();
}

}  // namespace ea

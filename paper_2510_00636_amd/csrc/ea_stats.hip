// Query statistics (Eq. 5-6) and the conversion of (mu, Sigma) into matrix-core operands.
//
// The window queries are mapped by one linear map per (sample, channel pair),
//     u~_s = R-bar R(p_s)^T q_s ,
// and mu = mean_s u~_s, Sigma = cov_s u~_s.  This equals R-bar m and R-bar S R-bar^T of
// Eq. 6 because mean and covariance commute with a fixed linear map; it lets one kernel
// produce Sigma directly.  Angles and the averaged rotation are evaluated in fp64: at
// position 1e5 an fp32 angle is already off by ~1e-2 rad.
#include <hip/hip_runtime.h>

#include "ea_kernels.h"
#include "ea_lanes.h"

namespace ea {

// ---------------------------------------------------------------------------------------
// tab[s][c] = (A, Bc): the 2x2 block  [[A, -Bc], [Bc, A]] = R-bar_c * Rot(-p_s theta_c).
// R-bar_c = mean_{j<T} Rot((t_next + j) theta_c) has the closed form of a Dirichlet kernel:
//   mean_j exp(i (t_next + j) theta) = exp(i theta (t_next + (T-1)/2)) sin(T theta/2) / (T sin(theta/2)).
//
// Where channel pair c of a sample stands in its row: the eight pairs 8 g + e of a group g are what a thread of the
// statistics kernels takes, two of them per 16-byte load, so that the loads of all groups side by side are one piece of
// memory: [e / 2][g][e % 2].  In the pairs' order a wavefront's load touched 64 pieces of 64 bytes (decode-time pass, 40
// heads, 359.4 and 357.8 us; 24 x 32 heads, w = 512, 134.3 and 133.5).
__host__ __device__ constexpr int table_slot(int c, int half) { return (c % 8 / 2 * (half / 8) + c / 8) * 2 + c % 2; }

__global__ void k_rope_table(const double* __restrict__ inv_freq, long long q_pos0,
                             long long t_next, int T, int w, int half, int q_is_rotated,
                             float2* __restrict__ tab, uint32_t* __restrict__ clear,
                             size_t clear_words) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  // riding along: zero the counters / histograms / flags of the later stages (one launch less)
  for (size_t i = gid; i < clear_words; i += (size_t)gridDim.x * blockDim.x) clear[i] = 0u;
  if (gid >= (size_t)w * half) return;
  int i = (int)gid;
  int s = i / half, c = i - s * half;
  // R-bar and the way back to position 0 in one angle: one sine and cosine instead of two, and of a smaller number
  const double th = inv_freq[c], sh = sin(0.5 * th), back = q_is_rotated ? (double)(q_pos0 + s) : 0.0;
  const bool flat = T == 1 || fabs(sh) < 1e-300;
  const double amp = flat ? 1.0 : sin(0.5 * th * (double)T) / ((double)T * sh);
  double co, si;
  sincos(th * ((double)t_next + (flat ? 0.0 : 0.5 * (double)(T - 1)) - back), &si, &co);
  tab[(size_t)s * half + table_slot(c, half)] = make_float2((float)(amp * co), (float)(amp * si));
}

// ---------------------------------------------------------------------------------------
// Sigma is symmetric, so only its 32 x 32 tiles on and above the diagonal are computed (3 of 4 at
// d = 64, 10 of 16 at d = 128, 36 of 64 at d = 256) and every tile above the diagonal is stored
// twice, once transposed.  A head's tiles are dealt to StatsTiling<D>::PARTS workgroups (1 / 2 / 4), each
// of which reads the window ONCE, in chunks of up to 64 or 32 samples: every thread issues all its
// 16-byte query loads and table loads of a chunk together (one memory latency per chunk instead
// of one per sample; the next chunk's loads go out before the current chunk's arithmetic), maps
// them to u~, subtracts the head's first sample u~_0 and writes the result to LDS; the four
// wavefronts then add the chunk's outer products to their accumulator tiles with fp32
// matrix-core instructions, two samples per instruction.
// With x = u~ - u~_0,
//     mean  = u~_0 + (1/w) sum_s x_s
//     Sigma = (1/(w - ddof)) (sum_s x_s x_s^T - w xbar xbar^T)
// exactly; the shift keeps |x| at the scale of the spread, so the subtraction of the second
// term costs no accuracy even for channels whose mean is many standard deviations from zero.
// Column sums are formed on the way in (each thread keeps the sums of the 16 channels of its
// items, all of one channel group) and combined in a fixed order, so results are reproducible.
// The fp32 matrix-core work is what bounds the kernel for long windows (64 cycles per pair of
// samples and tile): the triangle and the even deal over workgroups are what keep it short.

// fp32 windows: samples per LDS chunk.  A thread keeps its share of the next chunk in registers, 32 of them per item of
// 16 channels: with chunks of 64 samples that is 64 at d = 128 and 128 at d = 256, where a CU then holds one workgroup.
constexpr int stats_f32_chunk(int D) { return D == 64 ? 64 : 32; }
template <int D, int PARTS_ = 0> struct StatsTiling {
  static constexpr int NCT = D / 32;                       // 32-column tiles across Sigma
  static constexpr int NT = NCT * (NCT + 1) / 2;           // tiles on and above the diagonal
  static constexpr int PARTS = PARTS_ > 0 ? PARTS_ : D <= 64 ? 1 : (D <= 128 ? 2 : 4);
  static constexpr int TP = (NT + PARTS - 1) / PARTS;      // tiles per workgroup
  // A workgroup's first 4 WHOLE tiles go one (or WHOLE) to each wavefront; the SHARED tiles left
  // over are each split four ways by samples and the four partial tiles added at the end, so
  // every wavefront carries the same matrix-core load.
  static constexpr int WHOLE = TP >= 4 ? TP / 4 : 1;
  static constexpr int SHARED = TP >= 4 ? TP % 4 : 0;
  static constexpr int SLOTS = WHOLE + SHARED;             // accumulator tiles per wavefront
};

// Channels of pair e of channel group g: ja for the first, jb for the second element of the pair.
template <int D>
__device__ __forceinline__ int stats_ja(int layout, int g, int e) { return layout ? 2 * (8 * g + e) : 8 * g + e; }
template <int D>
__device__ __forceinline__ int stats_jb(int layout, int g, int e) { return layout ? 2 * (8 * g + e) + 1 : 8 * g + e + D / 2; }

// One item = one sample's channel group g: 8 pairs (qa[e], qb[e]) of the query row and their 2x2
// blocks tb[e] of the table row.  An item is fetched as raw words (bf16 rows stay packed, half
// the registers, while the loads are in flight) and unpacked where it is used.
template <bool BF16>
struct StatsRaw {
  uint4 w[BF16 ? 2 : 4];
  float4 t[4];
};
template <int D, bool BF16>
__device__ __forceinline__ void stats_fetch_item(const void* __restrict__ q_win, size_t row, int g, int layout,
                                                 const float2* __restrict__ tabrow, StatsRaw<BF16>& raw) {
  constexpr int HALF = D / 2;
  // half-split: channels 8g.. and HALF+8g..; interleaved: 16 consecutive channels = 8 pairs
  const size_t oa = row + (layout ? 16 * g : 8 * g), ob = row + (layout ? 16 * g + 8 : HALF + 8 * g);
  if (BF16) {
    raw.w[0] = *reinterpret_cast<const uint4*>((const uint16_t*)q_win + oa);
    raw.w[1] = *reinterpret_cast<const uint4*>((const uint16_t*)q_win + ob);
  } else {
    raw.w[0] = *reinterpret_cast<const uint4*>((const float*)q_win + oa);
    raw.w[1] = *reinterpret_cast<const uint4*>((const float*)q_win + oa + 4);
    raw.w[BF16 ? 0 : 2] = *reinterpret_cast<const uint4*>((const float*)q_win + ob);
    raw.w[BF16 ? 1 : 3] = *reinterpret_cast<const uint4*>((const float*)q_win + ob + 4);
  }
  const float4* tp = reinterpret_cast<const float4*>(tabrow) + g;
#pragma unroll
  for (int e = 0; e < 4; ++e) raw.t[e] = tp[e * (HALF / 8)];     // see table_slot
}
template <bool BF16>
__device__ __forceinline__ void stats_unpack_item(const StatsRaw<BF16>& raw, int layout, float (&qa)[8],
                                                  float (&qb)[8], float2 (&tb)[8]) {
  float xa[8], xb[8];
  if (BF16) {
    const uint32_t wa[4] = {raw.w[0].x, raw.w[0].y, raw.w[0].z, raw.w[0].w};
    const uint32_t wb[4] = {raw.w[1].x, raw.w[1].y, raw.w[1].z, raw.w[1].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xa[2 * e] = __uint_as_float(wa[e] << 16);
      xa[2 * e + 1] = __uint_as_float(wa[e] & 0xffff0000u);
      xb[2 * e] = __uint_as_float(wb[e] << 16);
      xb[2 * e + 1] = __uint_as_float(wb[e] & 0xffff0000u);
    }
  } else {
    const uint4 a0 = raw.w[0], a1 = raw.w[1], b0 = raw.w[BF16 ? 0 : 2], b1 = raw.w[BF16 ? 1 : 3];
    const uint32_t wa[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    const uint32_t wb[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) { xa[e] = __uint_as_float(wa[e]); xb[e] = __uint_as_float(wb[e]); }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // pair e of the group: (xa[e], xb[e]) half-split; (x[2e], x[2e+1]) of the 16 interleaved
    qa[e] = layout ? (e < 4 ? xa[2 * e] : xb[2 * e - 8]) : xa[e];
    qb[e] = layout ? (e < 4 ? xa[2 * e + 1] : xb[2 * e - 7]) : xb[e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    tb[2 * e] = make_float2(raw.t[e].x, raw.t[e].y);
    tb[2 * e + 1] = make_float2(raw.t[e].z, raw.t[e].w);
  }
}
// u~ - shift: the 2x2 block of the table applied to one pair.  The products with the pair's second channel are
// rounded on their own, those with its first are not, and nothing else is contracted: written out, so that the
// bits of the statistics, and with them every score, do not hang on what the compiler makes of the code around
// it, and one rule for every channel, layout and instance, so that the first sample less the shift, which is
// the first sample, is zero.
__device__ __forceinline__ void stats_rotate(float2 t, float qa, float qb, float sha, float shb, float& xa, float& xb) {
#pragma clang fp contract(off)
  const float pa = t.y * qb, pb = t.x * qb;
  xa = fmaf(t.x, qa, -pa) - sha;
  xb = fmaf(t.y, qa, pb) - shb;
}

// Sums over the lanes that share a channel group (stride G8), of eight values each: on return v[0 .. n) of a lane are those of
// the values stats_sum_at(lane, 0 .. n), n = stats_sums(G8).  Every step but the first of G8 = 4 hands half of the values to
// each side.
template <int G8> constexpr int stats_sums = G8 <= 8 ? 1 : 2;
template <int G8>
__device__ __forceinline__ int stats_sum_at(int lane, int i) {
  const int hi = lane >> 5, mid = lane >> 4 & 1, lo = lane >> 3 & 1;
  return G8 <= 8 ? 4 * hi + 2 * mid + lo : 4 * i + 2 * hi + mid;
}
template <int G8>
__device__ __forceinline__ void stats_lane_sums(float (&v)[8], int lane) {
  if (G8 <= 4) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += __shfl_xor(v[e], 4);
  }
  constexpr int N = G8 <= 8 ? 4 : 8;
  if (G8 <= 8) {
    const bool odd = lane & 8;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = dpp_add_of<0x128>(odd ? v[2 * e + 1] : v[2 * e], odd ? v[2 * e] : v[2 * e + 1]);
  }
#pragma unroll
  for (int e = 0; e < N / 2; ++e) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[2 * e]), __float_as_uint(v[2 * e + 1]), false, false);
    v[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int e = 0; e < N / 4; ++e) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2 * e]), __float_as_uint(v[2 * e + 1]), false, false);
    v[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}

typedef float floatx16_t __attribute__((ext_vector_type(16)));

// Register budget: four workgroups per CU at d = 64, two at d = 256, three at 128 (137 registers), without spills: a
// kernel that needs scratch memory costs some 10 us more per launch when several streams are in use.  Reading
// operands under "inside the window" and "my tile" and waiting for each pair bounded it (28 heads, d = 128,
// w = 200 29 us).  With the operands requested a step ahead and chunks of 64 samples a long window of few heads
// took 18, but at d = 256 one workgroup per CU was left (200 heads x 64 samples 54 -> 59 us, 800 x 16 112 -> 132) and
// short windows of very many heads lost at d = 128 (2000 x 16: 64 -> 70).  Chunks of 32: 16.9, 42, 90 and 57.
template <int D, bool BF16>
__global__ __launch_bounds__(256, (D == 64 ? 4 : 2)) void k_stats(const void* __restrict__ q_win, int w, int layout,
                                               int ddof, const float2* __restrict__ tab,
                                               float* __restrict__ mu, float* __restrict__ sigma) {
  constexpr int HALF = D / 2, G8 = HALF / 8;          // groups of 8 channel pairs per sample
  constexpr int WC = stats_f32_chunk(D);
  constexpr int ITEMS = WC * G8 / 256;          // (sample, group) items per thread and chunk
  typedef StatsTiling<D> TL;
  constexpr int NCT = TL::NCT, TPW = TL::SLOTS;
  static_assert(256 % G8 == 0 && ITEMS >= 1, "one channel group per thread");
  extern __shared__ __align__(16) float s_dyn[];
  float* s_u = s_dyn;                                 // [WC][D]   x = u~ - u~_0 of the chunk
  float* s_part = s_dyn + WC * D;               // [4][D]          column sums per wavefront
  float* s_shift = s_part + 4 * D;                    // [D]             u~_0
  float* s_xbar = s_shift + D;                        // [D]             (1/w) sum_s x_s
  const int head = blockIdx.x, part = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);        // wave-uniform: tile numbers stay scalar
  const size_t qbase = (size_t)head * w * D;
  const int nchunks = (w + WC - 1) / WC;
  const int g = tid % G8;                             // the channel group of all this thread's items

  // the first chunk's loads go out before anything waits on memory
  StatsRaw<BF16> raw[ITEMS];
  auto load_chunk = [&](int ch) __attribute__((always_inline)) {
    const int s0 = ch * WC, ns = min(WC, w - s0);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int sl = (tid + it * 256) / G8;
      if (sl < ns)
        stats_fetch_item<D, BF16>(q_win, qbase + (size_t)(s0 + sl) * D, g, layout,
                                  tab + (size_t)(s0 + sl) * HALF, raw[it]);
    }
  };
  load_chunk(0);
  // u~_0 of the head, kept in LDS (every thread reads its own group's 16 values per item)
  if (tid < G8) {
    float qa[8], qb[8];
    float2 tb[8];
    StatsRaw<BF16> raw0;
    stats_fetch_item<D, BF16>(q_win, qbase, g, layout, tab, raw0);
    stats_unpack_item<BF16>(raw0, layout, qa, qb, tb);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float ua, ub;
      stats_rotate(tb[e], qa[e], qb[e], 0.f, 0.f, ua, ub);
      s_shift[stats_ja<D>(layout, g, e)] = ua;
      s_shift[stats_jb<D>(layout, g, e)] = ub;
    }
  }
  __syncthreads();
  float suma[8], sumb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { suma[e] = 0.f; sumb[e] = 0.f; }

  // Outer products on the matrix cores in fp32: v_mfma_f32_32x32x2_f32 adds, for two samples at a
  // time, the 32 x 32 block  x[rows] x[cols]^T.  Lane l feeds row (or column) l % 32 of sample
  // l / 32 of the pair; wavefront `wave` owns the column tiles wave, wave + 4, ...
  const int r32 = lane & 31, hh = lane >> 5;
  // this wavefront's tiles: number wave + 4 t of the workgroup's share for the whole ones, then the
  // shared ones; rows of the triangle in order
  int t_rb[TPW], t_ct[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int local = t < TL::WHOLE ? wave + 4 * t : 4 * TL::WHOLE + (t - TL::WHOLE);
    int idx = part * TL::TP + local, rb = 0;
    const bool ok = local < TL::TP && idx < TL::NT;
    if (!ok) idx = 0;
#pragma unroll
    for (int r = 0; r < NCT; ++r)
      if (idx >= NCT - rb && rb == r) { idx -= NCT - rb; ++rb; }
    t_rb[t] = ok ? rb : -1;
    t_ct[t] = rb + idx;
  }
  floatx16_t acc[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

  for (int ch = 0; ch < nchunks; ++ch) {
    const int s0 = ch * WC, ns = min(WC, w - s0);
    if (ch > 0) __syncthreads();                      // the previous chunk has been consumed
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int sl = (tid + it * 256) / G8;
      if (sl < ns) {
        float qa[8], qb[8], xa[8], xb[8];
        float2 tb[8];
        stats_unpack_item<BF16>(raw[it], layout, qa, qb, tb);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          stats_rotate(tb[e], qa[e], qb[e], s_shift[stats_ja<D>(layout, g, e)],
                       s_shift[stats_jb<D>(layout, g, e)], xa[e], xb[e]);
          suma[e] += xa[e];
          sumb[e] += xb[e];
        }
        if (layout == 0) {                            // half-split: two runs of 8 consecutive channels
          float4* pa = reinterpret_cast<float4*>(s_u + sl * D + 8 * g);
          float4* pb = reinterpret_cast<float4*>(s_u + sl * D + HALF + 8 * g);
          pa[0] = make_float4(xa[0], xa[1], xa[2], xa[3]);
          pa[1] = make_float4(xa[4], xa[5], xa[6], xa[7]);
          pb[0] = make_float4(xb[0], xb[1], xb[2], xb[3]);
          pb[1] = make_float4(xb[4], xb[5], xb[6], xb[7]);
        } else {                                      // interleaved: 16 consecutive channels
          float4* pi = reinterpret_cast<float4*>(s_u + sl * D + 16 * g);
#pragma unroll
          for (int e = 0; e < 4; ++e) pi[e] = make_float4(xa[2 * e], xb[2 * e], xa[2 * e + 1], xb[2 * e + 1]);
        }
      } else if (sl < ((ns + 15) & ~15)) {            // past the window's end, as far as a step of eight pairs goes: zeros
        float4* z = reinterpret_cast<float4*>(s_u + sl * D + 16 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    __syncthreads();
    if (ch + 1 < nchunks) load_chunk(ch + 1);         // in flight during the matrix-core loop
    // Eight sample pairs per step, the operands of the next step requested before the instructions of this one
    // (samples past the window's end are zero rows in LDS); of a shared tile's pairs, two of every eight are
    // this wavefront's.  A tile that it does not have (d = 64) is computed as tile 0 and not stored.
    constexpr int PS = 8;
    const int npair = (ns + 1) / 2;
    float av[2][PS][TL::WHOLE], bv[2][PS][TL::WHOLE], as[2][2][TL::SHARED + 1], bs[2][2][TL::SHARED + 1];
    auto read_step = [&](int sp, int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < PS; ++u) {
        const float* row = s_u + (2 * (sp + u) + hh) * D + r32;
#pragma unroll
        for (int t = 0; t < TL::WHOLE; ++t) {
          av[buf][u][t] = row[max(t_rb[t], 0) * 32];
          bv[buf][u][t] = row[t_ct[t] * 32];
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float* row = s_u + (2 * (sp + 2 * wave + u) + hh) * D + r32;
#pragma unroll
        for (int t = 0; t < TL::SHARED; ++t) {
          as[buf][u][t] = row[t_rb[TL::WHOLE + t] * 32];
          bs[buf][u][t] = row[t_ct[TL::WHOLE + t] * 32];
        }
      }
    };
    auto multiply_step = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < PS; ++u)
#pragma unroll
        for (int t = 0; t < TL::WHOLE; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[buf][u][t], bv[buf][u][t], acc[t], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < TL::SHARED; ++t)
          acc[TL::WHOLE + t] =
              __builtin_amdgcn_mfma_f32_32x32x2f32(as[buf][u][t], bs[buf][u][t], acc[TL::WHOLE + t], 0, 0, 0);
    };
    read_step(0, 0);
    for (int sp = 0; sp < npair; sp += 2 * PS) {
      read_step(min(sp + PS, WC / 2 - PS), 1);
      multiply_step(0);
      if (WC > 4 * PS) read_step(min(sp + 2 * PS, WC / 2 - PS), 0);
      if (sp + PS < npair) multiply_step(1);
    }
  }
  if (TL::SHARED > 0) {
    // the four partial tiles of every shared tile, added in wavefront order by wavefront 0
    static_assert(TL::SHARED * 4 * 16 * 64 <= WC * D, "partial tiles fit in the chunk buffer");
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TL::SHARED; ++r)
#pragma unroll
      for (int v = 0; v < 16; ++v) s_u[((r * 4 + wave) * 16 + v) * 64 + lane] = acc[TL::WHOLE + r][v];
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int r = 0; r < TL::SHARED; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float* pp = s_u + (r * 4 * 16 + v) * 64 + lane;
          acc[TL::WHOLE + r][v] = (pp[0] + pp[16 * 64]) + (pp[2 * 16 * 64] + pp[3 * 16 * 64]);
        }
    }
  }

  // column sums: lanes that share a channel group (stride G8) first, then the four wavefronts
  stats_lane_sums<G8>(suma, lane);
  stats_lane_sums<G8>(sumb, lane);
#pragma unroll
  for (int i = 0; i < stats_sums<G8>; ++i) {
    const int e = stats_sum_at<G8>(lane, i);
    s_part[wave * D + stats_ja<D>(layout, g, e)] = suma[i];
    s_part[wave * D + stats_jb<D>(layout, g, e)] = sumb[i];
  }
  __syncthreads();
  const float invw = 1.0f / (float)w;
  for (int c = tid; c < D; c += 256) {
    const float xb = ((s_part[c] + s_part[D + c]) + (s_part[2 * D + c] + s_part[3 * D + c])) * invw;
    s_xbar[c] = xb;
    if (part == 0) mu[(size_t)head * D + c] = s_shift[c] + xb;
  }
  __syncthreads();
  // accumulator register v of lane (r32, hh) is row 8 (v / 4) + 4 hh + v % 4, column r32 of the tile
  const float fw = (float)w, inv = 1.0f / (float)(w - ddof);
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    if (t_rb[t] >= 0 && (t < TL::WHOLE || wave == 0)) {
      const int i0 = t_rb[t] * 32, j = t_ct[t] * 32 + r32;
      const float xj = s_xbar[j];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = i0 + 8 * (v / 4) + 4 * hh + v % 4;
        acc[t][v] = (acc[t][v] - fw * s_xbar[i] * xj) * inv;
        sigma[((size_t)head * D + i) * D + j] = acc[t][v];
      }
      if (t_rb[t] != t_ct[t]) {                          // four rows in a row: 16 bytes of the transposed tile
#pragma unroll
        for (int c = 0; c < 4; ++c)
          *reinterpret_cast<float4*>(sigma + ((size_t)head * D + j) * D + i0 + 8 * c + 4 * hh) =
              make_float4(acc[t][4 * c], acc[t][4 * c + 1], acc[t][4 * c + 2], acc[t][4 * c + 3]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Matrix-core operands for the score kernel, made by k_prep_frags from (mu, Sigma) in memory or by the
// statistics kernel itself.
//
// The quadratic form k^T Sigma k is evaluated as sum_j (sum_c k_c M[c][j]) k_j where M folds
// the pair (c, j) and (j, c) onto one side: M[c][j] = Sigma[c][j] + Sigma[j][c] when c < j, and 0 the other way
// round, so the form is that of any Sigma, symmetric or not.  Blocks of 32 x 32 channels that are all zeros are
// simply not stored, which removes 3/8 of the matrix-core work at d = 128.  M is scaled by a power of
// two into fp16 range and rounded to fp16; the rounding error of its diagonal (the dominant
// error term, since k_c^2 never cancels) is kept as a residual row that multiplies k_c^2 in
// an extra accumulator tile.  mu is split into an fp16 head and tail in the same tile.
// A fragment is 1 KiB, 64 lanes x 8 halves; what a lane holds say frag_item and extra_item below.
__device__ __forceinline__ float scale_for(float maxabs) {
  if (!(maxabs > 0.f) || !isfinite(maxabs)) return 1.0f;
  int e;
  frexpf(maxabs, &e);                 // maxabs = f * 2^e, f in [0.5, 1)
  int sh = 13 - e;                    // scaled max in [2^12, 2^13)
  sh = max(-100, min(100, sh));
  return ldexpf(1.0f, sh);
}

__device__ __forceinline__ uint4 pack_half8(const _Float16 (&h)[8]) {
  uint4 pk;
  pk.x = (uint32_t)__builtin_bit_cast(uint16_t, h[0]) | ((uint32_t)__builtin_bit_cast(uint16_t, h[1]) << 16);
  pk.y = (uint32_t)__builtin_bit_cast(uint16_t, h[2]) | ((uint32_t)__builtin_bit_cast(uint16_t, h[3]) << 16);
  pk.z = (uint32_t)__builtin_bit_cast(uint16_t, h[4]) | ((uint32_t)__builtin_bit_cast(uint16_t, h[5]) << 16);
  pk.w = (uint32_t)__builtin_bit_cast(uint16_t, h[6]) | ((uint32_t)__builtin_bit_cast(uint16_t, h[7]) << 16);
  return pk;
}

// Where FUSED instances write: the operands of the score kernel instead of mu and Sigma.
struct FragsOut {
  uint4* frags;
  float* post;
  int G, GH, passes, nfrag, unit_frags, hw;
};
// First fragment of query head gq of a unit, and of the extra rows of a pass: passes of `nfrag` fragments each, or (hw)
// all of a unit's heads, then the extra rows of every pass.
__device__ __forceinline__ size_t head_frags(const FragsOut& fo, int unit, int gq, int NF) {
  const int pass = gq / fo.GH;
  return (size_t)unit * fo.unit_frags + (fo.hw ? gq * NF : pass * fo.nfrag + (gq - pass * fo.GH) * NF);
}
__device__ __forceinline__ size_t extra_frags(const FragsOut& fo, int unit, int pass, int NF, int nks) {
  return (size_t)unit * fo.unit_frags + (fo.hw ? fo.G * NF + pass * 2 * nks : pass * fo.nfrag + fo.GH * NF);
}

// What lane l of fragment f of a head holds: eight entries of M, output channel `out`, input channels from `in0` on.
// Fragments are 16 x 32 operands: k-step b is the channels 32 b .. 32 b + 31, lane l's key operand the eight from
// 32 b + 8 (l / 16) on, output tile j has the rows 4 q + v for channel 32 (j / 2) + 8 q + 4 (j % 2) + v, so that a lane gets
// back channels it holds, and takes the k-steps 0 .. j / 2.  The zeros of the block on the diagonal cost the clock
// less than the same form spread over all of it.
struct FragItem { int out, in0; };
__device__ __forceinline__ FragItem frag_item(int f, int l) {
  FragItem x;
  int j = 0;
  while (f >= j / 2 + 1) { f -= j / 2 + 1; ++j; }
  const int m = l & 15;
  x.out = j / 2 * 32 + 8 * (m >> 2) + 4 * (j & 1) + (m & 3);
  x.in0 = 32 * f + 8 * (l >> 4);
  return x;
}
// M's entry for input channel `in` and output channel `out` out of Sigma[out][in] and Sigma[in][out].  Both are
// taken: a caller's Sigma need not be symmetric, and inside a 32 x 32 tile on the diagonal the statistics kernels'
// two differ by rounding.
__device__ __forceinline__ float folded_entry(int in, int out, float val, float mirrored) {
  return in < out ? val + mirrored : in == out ? val : 0.f;
}
// What lane l of extra fragment fe (tile, then on k or on k^2, then k-step) holds: eight channels from `c0` on of kind 0
// (fp16 head of mu), 1 (its tail) or 2 (rounding residual of the diagonal) of head g of the pass, or nothing (g < 0).
// Rows 4 kind + g for four heads per tile; a fifth head of five in rows 12, 13 and 14.
struct ExtraItem { int g, kind, c0; };
constexpr int extra_tiles(int GH) { return GH > 5 ? 2 : 1; }
template <int D>
__device__ __forceinline__ ExtraItem extra_item(int GH, int fe, int l) {
  constexpr int NK = D / 32;
  const int m = l & 15, tile = fe / (2 * NK);
  const bool is_res = fe / NK % 2 != 0;
  int g = -1, kind = -1;
  if (m < 12) { g = 4 * tile + (m & 3); kind = m >> 2; }
  else if (GH == 5 && m < 15) { g = 4; kind = m - 12; }
  if (g >= GH || (kind == 2) != is_res) g = -1;
  return ExtraItem{g, kind, 32 * (fe % NK) + 8 * (l >> 4)};
}

// ---------------------------------------------------------------------------------------
// The same statistics for bf16 windows with the outer products on the fp16 matrix cores.
//
// fp32 matrix-core instructions run at the rate of the vector units (and do not overlap with
// vector work), which made the kernel above the largest stage of a decode-time pass (512-sample
// windows).  Here every shifted sample x = u~ - u~_0 is scaled by a power of two s and split into
// two fp16 numbers, x s = hi + lo (hi = x s rounded toward zero to fp16, lo = the remainder
// rounded to fp16: 21 significant bits together), and
//     sum_s x x^T  =  (1/s^2) sum_s (hi hi^T + hi lo^T + lo hi^T)  + O(2^-21)
// runs as three v_mfma_f32_32x32x16_f16 per tile and 16 samples (96 cycles instead of 512), with
// fp32 accumulation.  The samples are the contraction index, so the chunk is staged transposed:
// two planes [channel][chunk of 64 or 32 samples] of fp16 with a row pitch of 8 more (conflict-free
// 16-byte reads).
// s is taken from the largest |x| of the head's first chunk (that chunk lands in [16, 32)), which
// leaves a factor 2048 of headroom for later samples before fp16 overflows (an overflow shows as
// non-finite statistics, and then as the NaN-score bit of the status word).  Mean, column sums,
// the shift and the final algebra are those of k_stats, in fp32.
typedef _Float16 stats_half8 __attribute__((ext_vector_type(8)));
typedef _Float16 stats_half2 __attribute__((ext_vector_type(2)));
// samples per staged chunk: 64, and 32 at d = 256 (registers: a thread keeps its share of the next
// chunk's queries and table rows in flight during the matrix-core loop)
constexpr int stats_split_chunk(int D) { return D >= 256 ? 32 : 64; }

// What bounds it at the decode-time shape (960 heads, w = 512, two workgroups of four wavefronts per CU) is the work
// between the barriers of a chunk, 5000 cycles of which 1000 are matrix instructions and the rest the conversions, the
// issue of the next chunk's loads (a CU's address unit takes 64 bytes per clock, and the table is two thirds of them) and
// LDS; then the 14000 of the first chunk and the end.  In calls of few heads it is the latter two: a workgroup of a window
// of 128 samples takes 24000 cycles, 12000 of them behind its last chunk, when every entry of Sigma is an LDS round trip of
// its own and sums and maxima over the lanes go through LDS as well; 18000 without those (one layer of 32 heads 13.1 -> 10.8
// us, decode-time shape 93 -> 82, 32 heads without operands 9.2 -> 7.4).
// FUSED (d <= 128): Sigma leaves as the fragments that k_prep_frags would have made of it, tile by tile.  One workgroup per
// head: they are the same bit for bit.  Two (OWN below): each makes those of its own tiles, the same up to the head's power of
// two.
template <int D, int LAYOUT, int PARTS = 0, bool FUSED = false>
__global__ __launch_bounds__(256, (D <= 128 && !(D == 128 && (PARTS == 1 || FUSED)) ? 3 : 2)) void k_stats_split(const void* __restrict__ q_win, int w,
                                                                         int ddof,
                                                                         const float2* __restrict__ tab,
                                                                         float* __restrict__ mu,
                                                                         float* __restrict__ sigma, FragsOut fo) {
  constexpr int HALF = D / 2, G8 = HALF / 8, layout = LAYOUT;   // the channel pairing is a compile-time constant:
                                                                // every LDS address below is a base plus an immediate
  constexpr int WC = stats_split_chunk(D);            // samples per chunk
  constexpr int ITEMS = WC * G8 / 256;                // consecutive samples per thread and chunk
  constexpr int P = WC + 8;                           // halves per channel row of a plane
  // Rows eight channels apart start 0 or 32 banks apart whatever the (16-byte aligned) pitch, and
  // those are the rows the lanes of one staging write go to (one channel of every group): the
  // 16-byte column blocks of a row are therefore XOR-swizzled by the row's channel group, which
  // spreads the groups over the blocks (writes conflict-free at d = 128, two-way at d = 256) and
  // leaves the 16 lanes of a matrix-operand read (two groups of equal swizzle) in one block.
  constexpr int NB = WC / 8;                          // column blocks per row
  constexpr int BW = G8 >= 16 ? 1 : 16 / G8;          // blocks one wave-wide staging write spans
  auto swz_of_group = [](int gg) { return ITEMS >= 2 ? ((gg >> 1) * BW) % NB : 0; };
  auto group_of_channel = [](int c) { return LAYOUT ? c / 16 : (c % HALF) / 8; };
  typedef StatsTiling<D, PARTS> TL;
  constexpr int NCT = TL::NCT, TPW = TL::SLOTS;
  static_assert(ITEMS >= 1 && 256 % G8 == 0, "one channel group per thread");
  static_assert(TL::SHARED * 4 * 16 * 64 * 4 <= 2 * D * P * 2, "partial tiles fit in the planes");
  extern __shared__ __align__(16) float s_dyn[];
  _Float16* s_hi = reinterpret_cast<_Float16*>(s_dyn);            // [D][P]
  _Float16* s_lo = s_hi + D * P;                                   // [D][P]
  float* s_part = reinterpret_cast<float*>(s_lo + D * P);          // [4][D] column sums per wavefront
  float* s_shift = s_part + 4 * D;                                 // [D] u~_0
  float* s_xbar = s_shift + D;                                     // [D]
  float* s_max = s_xbar + D;                                       // [4]
  float* s_sq = s_max + 4;                                         // OWN: [4][D] sums of squares per wavefront
  const int head = blockIdx.x, part = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t qbase = (size_t)head * w * D;
  const int nchunks = (w + WC - 1) / WC;
  const int g = tid % G8, sl_t = ITEMS * (tid / G8);   // this thread's channel group and first sample of a chunk

  StatsRaw<true> raw[ITEMS];
  auto load_chunk = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int sa = min(ch * WC + sl_t + it, w - 1);   // no load under a condition: past the end, the last sample again
      stats_fetch_item<D, true>(q_win, qbase + (size_t)sa * D, g, layout, tab + (size_t)sa * HALF, raw[it]);
    }
  };
  load_chunk(0);
  if (tid < G8) {
    float qa[8], qb[8];
    float2 tb[8];
    StatsRaw<true> raw0;
    stats_fetch_item<D, true>(q_win, qbase, g, layout, tab, raw0);
    stats_unpack_item<true>(raw0, layout, qa, qb, tb);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float ua, ub;
      stats_rotate(tb[e], qa[e], qb[e], 0.f, 0.f, ua, ub);
      s_shift[stats_ja<D>(layout, g, e)] = ua;
      s_shift[stats_jb<D>(layout, g, e)] = ub;
    }
  }
  __syncthreads();
  // OWN: two workgroups of a head, each making the fragments of its own tiles; the scale of the head's fragments comes from
  // sums of squares, which both take of all channels
  constexpr bool OWN = FUSED && TL::PARTS == 2;
  float suma[8], sumb[8], sqa[8], sqb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { suma[e] = sumb[e] = sqa[e] = sqb[e] = 0.f; }

  const int r32 = lane & 31, kg = lane >> 5;
  int t_rb[TPW], t_ct[TPW];
  // A whole head at d = 128: two tiles per wavefront, next to each other in the triangle's order and of one row of
  // tiles (the row operand is read once for both), and as shared ones the tiles that are left, numbers 4 and 9:
  // those that a head split over two workgroups adds up from partial sums as well, so that Sigma has the same
  // bits either way.  (With the last two tiles shared, one pair of eight had two rows, and the second form of
  // the loop that it needed took 8 to 10 registers more than there are.)
  constexpr bool kPairs = D == 128 && PARTS == 1;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    int local = t < TL::WHOLE ? (kPairs ? 2 * wave + t : wave + 4 * t) : 4 * TL::WHOLE + (t - TL::WHOLE);
    if constexpr (kPairs) local = t < TL::WHOLE ? (local < 4 ? local : local + 1) : t == TL::WHOLE ? 4 : 9;
    int idx = part * TL::TP + local, rb = 0;
    const bool ok = local < TL::TP && idx < TL::NT;
    if (!ok) idx = 0;
#pragma unroll
    for (int r = 0; r < NCT; ++r)
      if (idx >= NCT - rb && rb == r) { idx -= NCT - rb; ++rb; }
    t_rb[t] = ok ? rb : -1;
    t_ct[t] = rb + idx;
  }
  floatx16_t acc[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
  // Where a lane's operand of tile block b (channels 32 b + r32) and step ks starts: the swizzle of
  // channel 32 b + r32 is U(b) ^ L(r32), L living in bits of its own, so the address is a part that is the
  // same for all lanes plus one of two lane parts.
  constexpr int LM = 1 | (LAYOUT ? 0 : D == 64 ? 4 : D == 128 ? 2 : 1);          // lane-dependent bits of the block number
  const int lswz = kg ^ (LAYOUT ? 0 : swz_of_group(r32 / 8));
  auto operand_at = [&](int blk, int ks) __attribute__((always_inline)) {
    const int u = (2 * ks) ^ (swz_of_group(group_of_channel(blk * 32)));
    return (blk * 32 * P + ((u & ~LM) << 3)) + (r32 * P + ((lswz ^ (u & LM)) << 3));
  };

  // x = u~ - u~_0 of item `it` of the chunk in flight: [0, 8) the first,
  // [8, 16) the second channels of the group's pairs.  Nothing in it sits under a condition: a shift
  // read inside "if (inside the chunk)" was a branch and an LDS round trip per element.
  auto item_x = [&](int it, const float (&sh)[16], float (&x)[16]) __attribute__((always_inline)) {
    float qa[8], qb[8];
    float2 tb[8];
    stats_unpack_item<true>(raw[it], layout, qa, qb, tb);
#pragma unroll
    for (int e = 0; e < 8; ++e) stats_rotate(tb[e], qa[e], qb[e], sh[e], sh[8 + e], x[e], x[8 + e]);
  };

  float scale = 1.0f;
  for (int ch = 0; ch < nchunks; ++ch) {
    const int ns = min(WC, w - ch * WC);
    // ---- this thread's samples of the chunk, then at once the requests for the next chunk: they
    //      travel during the conversion, the barriers and the matrix-core loop below
    float xs[ITEMS][16];
    {
      float sh[16];                                   // this thread's channels of u~_0, as four 16-byte reads
      const float4* pa = reinterpret_cast<const float4*>(s_shift + (layout ? 16 * g : 8 * g));
      const float4* pb = reinterpret_cast<const float4*>(s_shift + (layout ? 16 * g + 8 : HALF + 8 * g));
      const float4 f[4] = {pa[0], pa[1], pb[0], pb[1]};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float y[4] = {f[c].x, f[c].y, f[c].z, f[c].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = 4 * c + i;                    // half-split: as they come; interleaved: pairs
          sh[layout ? (m & 1) * 8 + (m >> 1) : m] = y[i];
        }
      }
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) item_x(it, sh, xs[it]);
    }
    if (ns < WC) {                                    // zeros past the chunk's end
#pragma unroll
      for (int it = 0; it < ITEMS; ++it)
#pragma unroll
        for (int c16 = 0; c16 < 16; ++c16) xs[it][c16] = sl_t + it < ns ? xs[it][c16] : 0.f;
    }
    // (nothing moves across: loads in front of the last use of the registers they go to cost 50 copies per chunk)
    __builtin_amdgcn_sched_barrier(0);
    load_chunk(ch + 1);                               // (behind the last chunk: its last sample)
    if (ch == 0) {
      // the head's scale: a power of two that puts the first chunk's largest |x| into [16, 32)
      float amax = 0.f;
#pragma unroll
      for (int it = 0; it < ITEMS; ++it)
#pragma unroll
        for (int c16 = 0; c16 < 16; ++c16) amax = fmaxf(amax, fabsf(xs[it][c16]));
      amax = wave_max(amax);
      if (lane == 0) s_max[wave] = amax;
      __syncthreads();
      const float m = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
      if (m > 0.f && m < INFINITY) {
        int ex;
        frexpf(m, &ex);                               // m = f 2^ex, f in [0.5, 1)
        scale = ldexpf(1.0f, max(-100, min(100, 5 - ex)));
      }
    } else {
      __syncthreads();                                // the previous chunk has been consumed
    }
    // ---- fp16 (hi, lo) of x * scale into the transposed planes, column sums on the way
#pragma unroll
    for (int it = 0; it < ITEMS; it += 2) {
#pragma unroll
      for (int c16 = 0; c16 < 16; ++c16) {
        const int e = c16 & 7;
        const int c = c16 < 8 ? stats_ja<D>(layout, g, e) : stats_jb<D>(layout, g, e);
        const float x0 = xs[it][c16];
        const float y0 = x0 * scale;
        if constexpr (ITEMS >= 2) {
          const float x1 = xs[it + 1][c16];
          if (c16 < 8) suma[e] += x0 + x1; else sumb[e] += x0 + x1;
          if constexpr (OWN) {
            if (c16 < 8) sqa[e] = fmaf(x0, x0, fmaf(x1, x1, sqa[e])); else sqb[e] = fmaf(x0, x0, fmaf(x1, x1, sqb[e]));
          }
          const float y1 = x1 * scale;
          const stats_half2 h = __builtin_bit_cast(stats_half2, __builtin_amdgcn_cvt_pkrtz(y0, y1));
          const stats_half2 l = {(_Float16)(y0 - (float)h[0]), (_Float16)(y1 - (float)h[1])};
          const int col = ((((sl_t + it) >> 3) ^ swz_of_group(g)) << 3) + ((sl_t + it) & 7);
          *reinterpret_cast<stats_half2*>(s_hi + c * P + col) = h;
          *reinterpret_cast<stats_half2*>(s_lo + c * P + col) = l;
        } else {
          if (c16 < 8) suma[e] += x0; else sumb[e] += x0;
          const stats_half2 h = __builtin_bit_cast(stats_half2, __builtin_amdgcn_cvt_pkrtz(y0, 0.f));
          s_hi[c * P + sl_t] = h[0];
          s_lo[c * P + sl_t] = (_Float16)(y0 - (float)h[0]);
        }
      }
    }
    __syncthreads();
    // ---- three matrix-core instructions per tile and 16 samples, one straight line (samples past the
    //      window's end are zeros in the planes), so that the operand reads of the next step travel
    //      under the matrix instructions of this one.  A tile that this wavefront does not have (d = 64)
    //      is computed as tile 0 and not stored.
    constexpr int KS = WC / 16;
    auto step = [&](int t, int ks) __attribute__((always_inline)) {
      const int oa = operand_at(max(t_rb[t], 0), ks), ob = operand_at(t_ct[t], ks);
      const stats_half8 ah = *reinterpret_cast<const stats_half8*>(s_hi + oa);
      const stats_half8 al = *reinterpret_cast<const stats_half8*>(s_lo + oa);
      const stats_half8 bh = *reinterpret_cast<const stats_half8*>(s_hi + ob);
      const stats_half8 bl = *reinterpret_cast<const stats_half8*>(s_lo + ob);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, acc[t], 0, 0, 0);
    };
    if constexpr (kPairs) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks > 0 && ks * 16 >= ns) break;           // a window's last samples fill no chunk
        const int oa = operand_at(t_rb[0], ks), ob = operand_at(t_ct[0], ks), oc = operand_at(t_ct[1], ks);
        const stats_half8 ah = *reinterpret_cast<const stats_half8*>(s_hi + oa);
        const stats_half8 al = *reinterpret_cast<const stats_half8*>(s_lo + oa);
        const stats_half8 bh = *reinterpret_cast<const stats_half8*>(s_hi + ob);
        const stats_half8 bl = *reinterpret_cast<const stats_half8*>(s_lo + ob);
        const stats_half8 ch2 = *reinterpret_cast<const stats_half8*>(s_hi + oc);
        const stats_half8 cl2 = *reinterpret_cast<const stats_half8*>(s_lo + oc);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, ch2, acc[1], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, cl2, acc[1], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, ch2, acc[1], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < TL::WHOLE; ++t) step(t, ks);
    }
    // a shared tile's steps go round the wavefronts: step number ch * KS + ks modulo 4
    if constexpr (TL::SHARED > 0) {
      static_assert(4 % KS == 0, "at most one step of a shared tile per wavefront and chunk");
      const int ks = (wave - ch * KS) & 3;
      if (KS == 4 || ks < KS) {
#pragma unroll
        for (int t = TL::WHOLE; t < TPW; ++t) step(t, ks);
      }
    }
  }
  if (TL::SHARED > 0) {
    // the four partial tiles of every shared tile, added in wavefront order by wavefront 0
    float* s_u = s_dyn;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TL::SHARED; ++r)
#pragma unroll
      for (int v = 0; v < 16; ++v) s_u[((r * 4 + wave) * 16 + v) * 64 + lane] = acc[TL::WHOLE + r][v];
    __syncthreads();
    // (shared tile r by wavefront 3 - r: the first ones come from the diagonal, which has more to do behind this)
#pragma unroll
    for (int r = 0; r < TL::SHARED; ++r)
      if (wave == 3 - r) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float* pp = s_u + (r * 4 * 16 + v) * 64 + lane;
          acc[TL::WHOLE + r][v] = (pp[0] + pp[16 * 64]) + (pp[2 * 16 * 64] + pp[3 * 16 * 64]);
        }
      }
  }
  auto mine = [&](int t) { return t_rb[t] >= 0 && (t < TL::WHOLE || wave == 3 - (t - TL::WHOLE)); };   // tiles to hand on

  // column sums: lanes that share a channel group (stride G8) first, then the four wavefronts
  stats_lane_sums<G8>(suma, lane);
  stats_lane_sums<G8>(sumb, lane);
  if constexpr (OWN) {
    stats_lane_sums<G8>(sqa, lane);
    stats_lane_sums<G8>(sqb, lane);
  }
#pragma unroll
  for (int i = 0; i < stats_sums<G8>; ++i) {
    const int e = stats_sum_at<G8>(lane, i);
    const int ca = wave * D + stats_ja<D>(layout, g, e), cb = wave * D + stats_jb<D>(layout, g, e);
    s_part[ca] = suma[i];
    s_part[cb] = sumb[i];
    if constexpr (OWN) {
      s_sq[ca] = sqa[i];
      s_sq[cb] = sqb[i];
    }
  }
  __syncthreads();
  const float invw = 1.0f / (float)w;
  for (int c = tid; c < D; c += 256) {
    const float xb = ((s_part[c] + s_part[D + c]) + (s_part[2 * D + c] + s_part[3 * D + c])) * invw;
    s_xbar[c] = xb;
    if (!FUSED && part == 0) mu[(size_t)head * D + c] = s_shift[c] + xb;
  }
  __syncthreads();
  // In the matrix-core product a lane's B operand is column r32 and its A rows come back as
  // accumulator register v = row 8 (v / 4) + 4 kg + v % 4: the tile's entry (row, column r32).
  const float fw = (float)w, inv = 1.0f / (float)(w - ddof), unscale = 1.0f / (scale * scale);
  auto sigma_entry = [&](float sum, float xi, float xj) {
#pragma clang fp contract(off)
    return fmaf(unscale, sum, -(xj * (fw * xi))) * inv;
  };
  // The entries of tile t, in the accumulators' place.  (All of xbar first: read next to the stores of the entries, which it
  // may alias, every entry was an LDS round trip of its own, 2200 cycles per tile.)
  auto finish_tile = [&](int t) __attribute__((always_inline)) {
    const float xj = s_xbar[t_ct[t] * 32 + r32];
    float xi[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float4 f = *reinterpret_cast<const float4*>(s_xbar + t_rb[t] * 32 + 8 * c + 4 * kg);
      xi[4 * c] = f.x; xi[4 * c + 1] = f.y; xi[4 * c + 2] = f.z; xi[4 * c + 3] = f.w;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = sigma_entry(acc[t][v], xi[v], xj);
  };
  auto row_of = [&](int v) { return 8 * (v / 4) + 4 * kg + v % 4; };      // in the tile, of accumulator register v
  // A tile above the diagonal is also stored transposed.  Straight from the accumulators that is
  // 64 separate 4-byte writes per instruction (a lane holds one column).  At d = 256 (28 of 36 tiles
  // are mirrored, 64 MB of Sigma per launch of the four-sequence shape) the tile takes a trip
  // through the wavefront's own patch of LDS (the planes are free by now) and leaves as rows; at
  // d <= 128 that costs the registers that keep three workgroups on a CU without scratch memory,
  // and the direct stores are the faster ones (5.6 against 10.4 us per layer at the decode shape).
  constexpr bool kViaLds = D >= 256;
  if constexpr (FUSED) {
    // Largest diagonal entry and largest mean.  OWN: the entry from the sums of squares, by every wavefront for itself
    // (the same for both workgroups of the head); else from the diagonal, in three steps.
    float mxS = 0.f, mxM = 0.f;
    for (int c = lane; c < D; c += 64) {
      if constexpr (OWN) {
        const float sq = (s_sq[c] + s_sq[D + c]) + (s_sq[2 * D + c] + s_sq[3 * D + c]);
        mxS = fmaxf(mxS, fabsf((sq - fw * s_xbar[c] * s_xbar[c]) * inv));
      }
      mxM = fmaxf(mxM, fabsf(s_shift[c] + s_xbar[c]));
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (!mine(t)) continue;
      finish_tile(t);
      if (!OWN && t_rb[t] == t_ct[t]) {
#pragma unroll
        for (int v = 0; v < 16; ++v) mxS = row_of(v) == r32 ? fmaxf(mxS, fabsf(acc[t][v])) : mxS;
      }
    }
    mxS = wave_max(mxS);
    mxM = wave_max(mxM);
    if constexpr (!OWN) {
      if (lane == 0) s_max[wave] = mxS;
      __syncthreads();
      mxS = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    }
    const float sM = scale_for(2.0f * mxS), smu = scale_for(mxM);
    constexpr int NF = NCT * (NCT + 1), nks = NCT;
    const int unit = head / fo.G, gq = head - unit * fo.G, pass = gq / fo.GH, gp = gq - pass * fo.GH;
    const int nhere = min(fo.GH, fo.G - pass * fo.GH);    // heads of this (unit, pass)
    uint4* out = fo.frags + head_frags(fo, unit, gq, NF) * 64;
    uint4* extra = fo.frags + extra_frags(fo, unit, pass, NF, nks) * 64;
    // the head's row of kind `kind` in the extra rows' fragments, see extra_item
    const int etile = D == 64 && fo.GH > 5 ? gp / 4 : 0;
    auto extra_row = [&](int kind) { return gp - 4 * etile < 4 ? 4 * kind + gp - 4 * etile : 12 + kind; };
    float* patch = s_dyn + wave * (32 * 33);
    static_assert(4 * 32 * 33 * 4 <= 2 * D * P * 2, "patches fit in the planes");
    // The tile (rows of block rb, columns of block ct) is fragments (2 ct, rb) and (2 ct + 1, rb), see frag_item: through
    // the wavefront's own patch of LDS.  On the diagonal also the residuals of the extra rows.
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (!mine(t)) continue;
      const int rb = t_rb[t], ct = t_ct[t];
#pragma unroll
      for (int v = 0; v < 16; ++v) patch[row_of(v) * 33 + r32] = acc[t][v];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int m = lane & 15, grp = lane >> 4;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int ol = 8 * (m >> 2) + 4 * jj + (m & 3);
        _Float16 h[8];
        float val[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) val[i] = patch[(8 * grp + i) * 33 + ol];    // Sigma[in][out]
        if (rb < ct) {                                   // (Sigma[out][in] too)
#pragma unroll
          for (int i = 0; i < 8; ++i) val[i] += val[i];
        } else {
          float other[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) other[i] = patch[ol * 33 + 8 * grp + i];
#pragma unroll
          for (int i = 0; i < 8; ++i) val[i] = folded_entry(8 * grp + i, ol, other[i], val[i]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) h[i] = (_Float16)(val[i] * sM);
        out[(ct * (ct + 1) + jj * (ct + 1) + rb) * 64 + lane] = pack_half8(h);
      }
      if (rb == ct && lane < 4) {
        _Float16 h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float x = patch[(8 * lane + i) * 34] * sM;
          h[i] = (_Float16)(x - (float)(_Float16)x);
        }
        extra[((2 * etile + 1) * nks + rb) * 64 + lane * 16 + extra_row(2)] = pack_half8(h);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    if (part == 0) {
      if (tid == 0) {
        fo.post[(size_t)head * 2 + 0] = 1.0f / (2.0f * (float)D * sM);
        fo.post[(size_t)head * 2 + 1] = 1.0f / (sqrtf((float)D) * smu);
      }
      if (tid < 8 * nks) {                               // head and tail of mu
        const int kind = tid / (4 * nks), b = tid / 4 % nks, grp = tid & 3;
        _Float16 h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int c = 32 * b + 8 * grp + i;
          const float x = (s_shift[c] + s_xbar[c]) * smu;
          const float hi = (float)(_Float16)x;
          h[i] = (_Float16)(kind == 0 ? hi : x - hi);
        }
        extra[(2 * etile * nks + b) * 64 + grp * 16 + extra_row(kind)] = pack_half8(h);
      }
      if (gp == 0) {                                     // rows that belong to no head, and heads that the last pass has room
        const uint4 z = make_uint4(0u, 0u, 0u, 0u);      // for but not
        for (int item = tid; item < extra_tiles(fo.GH) * 2 * nks * 64; item += 256) {
          const ExtraItem x = extra_item<D>(fo.GH, item >> 6, item & 63);
          if (x.g < 0 || x.g >= nhere) extra[item] = z;
        }
        if (!fo.hw)
          for (int item = nhere * NF * 64 + tid; item < fo.GH * NF * 64; item += 256) out[item] = z;
      }
    }
  } else if constexpr (!kViaLds) {
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (mine(t)) {
        const int i0 = t_rb[t] * 32, j = t_ct[t] * 32 + r32;
        finish_tile(t);
#pragma unroll
        for (int v = 0; v < 16; ++v) sigma[((size_t)head * D + i0 + row_of(v)) * D + j] = acc[t][v];
        if (t_rb[t] != t_ct[t]) {                        // four rows in a row: 16 bytes of the transposed tile
#pragma unroll
          for (int c = 0; c < 4; ++c)
            *reinterpret_cast<float4*>(sigma + ((size_t)head * D + j) * D + i0 + 8 * c + 4 * kg) =
                make_float4(acc[t][4 * c], acc[t][4 * c + 1], acc[t][4 * c + 2], acc[t][4 * c + 3]);
        }
      }
    }
  } else {
    float* s_tr = s_dyn + wave * (32 * 33);
    static_assert(4 * 32 * 33 * 4 <= 2 * D * P * 2, "transposition patches fit in the planes");
    __syncthreads();                 // every wavefront is done with the planes (and the partial tiles)
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (mine(t)) {
        const int i0 = t_rb[t] * 32, j0 = t_ct[t] * 32, j = j0 + r32;
        const bool mirror = t_rb[t] != t_ct[t];
        finish_tile(t);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          sigma[((size_t)head * D + i0 + row_of(v)) * D + j] = acc[t][v];
          if (mirror) s_tr[r32 * 33 + row_of(v)] = acc[t][v];         // [column][row]
        }
        if (mirror) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int jl = 2 * v + kg;                    // column of the tile = row of the transposed one
            sigma[((size_t)head * D + j0 + jl) * D + i0 + r32] = s_tr[jl * 33 + r32];
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// The operands from (mu, Sigma) in memory, a wavefront per fragment: it requests the fragment's entries and what its scale
// needs together and waits once.  (With the scales of a pass's heads in front of a barrier, and the fragments dealt to 16
// workgroups behind it, three trips to memory: one sequence of 32 heads 6.2 us, now 4.9; four 8.0 and 6.3; the literal pass,
// which prepares twice, 98.9 and 97.6.)
template <int D>
__global__ __launch_bounds__(256) void k_prep_frags(const float* __restrict__ mu, const float* __restrict__ sigma,
                                                    FragsOut fo, int shared_heads, uint32_t* __restrict__ clear,
                                                    size_t clear_words) {
  // mu == nullptr: zero means.  shared_heads > 0: one set of that many heads' Sigma for every sequence.
  // clear: counters of the score kernel and what stands around them, zeroed on the way (one launch less)
  for (size_t i = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x; i < clear_words;
       i += (size_t)gridDim.x * gridDim.y * 256)
    clear[i] = 0u;
  constexpr int NJT = D / 32, NF = NJT * (NJT + 1), NK = D / 32, PL = D / 64;
  const int G = fo.G, GH = fo.GH, passes = fo.passes, nextra = extra_tiles(GH) * 2 * NK;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int unit = blockIdx.x / passes, pass = blockIdx.x % passes;
  const int g0 = pass * GH;
  const int f = blockIdx.y * 4 + wave;
  if (f >= GH * NF + nextra) return;
  auto sigma_of = [&](int gq_) {
    const int head = unit * G + gq_;
    return sigma + (size_t)(shared_heads ? head % shared_heads : head) * D * D;
  };
  // Sigma is a covariance matrix, so |Sigma[a][b]| <= max_c Sigma[c][c]: the diagonal alone bounds every entry of M (<= 2x).
  auto load_diagonal = [&](int gq, float (&x)[PL]) __attribute__((always_inline)) {
    const float* S = sigma_of(gq);
#pragma unroll
    for (int i = 0; i < PL; ++i) x[i] = S[(size_t)(lane + 64 * i) * (D + 1)];
  };
  auto load_mean = [&](int gq, float (&x)[PL]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PL; ++i) x[i] = mu ? mu[((size_t)unit * G + gq) * D + lane + 64 * i] : 0.f;
  };
  auto largest = [&](const float (&x)[PL]) __attribute__((always_inline)) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < PL; ++i) m = fmaxf(m, fabsf(x[i]));
    return wave_max(m);
  };
  _Float16 h[8];
  uint4* out;
  if (f < GH * NF) {
    const int g = f / NF, gq = g0 + g;
    if (fo.hw && gq >= G) return;
    out = fo.frags + (head_frags(fo, unit, gq, NF) + (f - g * NF)) * 64 + lane;
    if (gq < G) {
      const FragItem x = frag_item(f - g * NF, lane);
      const float* S = sigma_of(gq);
      // the pair (c_in, c_out) and its mirror contribute the same product k_in * k_out: the row's run and the column's
      float diag[PL], mean[PL], mirrored[8];
      constexpr bool kShared = D >= 128;                  // (then a workgroup's four fragments are one head's)
      static_assert(!kShared || (NF % 4 == 0 && 2 * NK % 4 == 0), "one head per workgroup");
      __shared__ float s_max[4];
      const float4 lo = *reinterpret_cast<const float4*>(S + (size_t)x.out * D + x.in0);
      const float4 hi = *reinterpret_cast<const float4*>(S + (size_t)x.out * D + x.in0 + 4);
#pragma unroll
      for (int i = 0; i < 8; ++i) mirrored[i] = S[(size_t)(x.in0 + i) * D + x.out];
      if constexpr (kShared) diag[0] = (int)threadIdx.x < D ? S[(size_t)threadIdx.x * (D + 1)] : 0.f;
      else load_diagonal(gq, diag);
      const bool first = f == g * NF;                     // the wavefront that writes the head's factors
      if (first) load_mean(gq, mean);
      float mxS;
      if constexpr (kShared) {                            // (256 lines for every wavefront to itself: 64 heads of d = 256 11.0 us,
        const float m = wave_max(fabsf(diag[0]));         // now 9.2)
        if (lane == 0) s_max[wave] = m;
        __syncthreads();
        mxS = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
      } else {
        mxS = largest(diag);
      }
      const float sM = scale_for(2.0f * mxS);
      if (first) {
        const float sm = scale_for(largest(mean));
        if (lane == 0) {
          fo.post[((size_t)unit * G + gq) * 2 + 0] = 1.0f / (2.0f * (float)D * sM);
          fo.post[((size_t)unit * G + gq) * 2 + 1] = 1.0f / (sqrtf((float)D) * sm);
        }
      }
      const float val[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) h[i] = (_Float16)(folded_entry(x.in0 + i, x.out, val[i], mirrored[i]) * sM);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) h[i] = (_Float16)0.f;
    }
  } else {
    const int fe = f - GH * NF, nhere = min(GH, G - g0);
    const bool residual = fe / NK % 2 != 0;               // the fragment's rows: residuals of the diagonals, or heads and tails of the means
    out = fo.frags + (extra_frags(fo, unit, pass, NF, NK) + fe) * 64 + lane;
    const ExtraItem x = extra_item<D>(GH, fe, lane);
    float scale = 0.f, val[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) val[i] = 0.f;
    if (x.g >= 0 && x.g < nhere) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        val[i] = residual ? sigma_of(g0 + x.g)[(size_t)(x.c0 + i) * (D + 1)] : mu ? mu[((size_t)unit * G + g0 + x.g) * D + x.c0 + i] : 0.f;
    }
    float all[8][PL];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      if (g >= nhere) break;
      if (residual) load_diagonal(g0 + g, all[g]);
      else load_mean(g0 + g, all[g]);
    }
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      if (g >= nhere) break;
      const float m = largest(all[g]), sc = scale_for(residual ? 2.0f * m : m);
      if (x.g == g) scale = sc;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float m = val[i] * scale, hi = (float)(_Float16)m;
      h[i] = (_Float16)(x.g < 0 || x.g >= nhere ? 0.f : x.kind == 0 ? hi : m - hi);
    }
  }
  *out = pack_half8(h);
}

// ---------------------------------------------------------------------------------------
hipError_t launch_rope_table(const Dims& d, const double* inv_freq, int64_t q_pos0, int64_t t_next,
                             int w, float2* tab, uint32_t* clear, size_t clear_words, hipStream_t st) {
  k_rope_table<<<(unsigned)table_blocks(w, d.half, clear_words), 256, 0, st>>>(inv_freq, q_pos0, t_next, d.T, w, d.half,
                                                    d.q_is_rotated, tab, clear, clear_words);
  return hipGetLastError();
}

template <int D, bool BF16>
static hipError_t launch_stats_one(const Dims& d, const void* q_win, int w, const float2* tab,
                                   float* mu, float* sigma, hipStream_t st) {
  auto kern = k_stats<D, BF16>;
  const size_t lds = (size_t)(stats_f32_chunk(D) * D + 6 * D) * sizeof(float);
  static LdsOptIn opt;                    // one per kernel instance
  hipError_t e = opt.ensure(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  dim3 grid(d.qheads(), StatsTiling<D>::PARTS);
  kern<<<grid, 256, lds, st>>>(q_win, w, d.rope_layout, d.ddof, tab, mu, sigma);
  return hipGetLastError();
}

template <int D, int LAYOUT, int PARTS>
static hipError_t launch_stats_split_parts(const Dims& d, const void* q_win, int w, const float2* tab, float* mu,
                                           float* sigma, hipStream_t st) {
  auto kern = k_stats_split<D, LAYOUT, PARTS>;
  const size_t lds = (size_t)2 * D * (stats_split_chunk(D) + 8) * sizeof(_Float16) + (size_t)(6 * D + 4) * sizeof(float);
  static LdsOptIn opt;
  hipError_t e = opt.ensure(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  dim3 grid(d.qheads(), StatsTiling<D, PARTS>::PARTS);
  kern<<<grid, 256, lds, st>>>(q_win, w, d.ddof, tab, mu, sigma, FragsOut{});
  return hipGetLastError();
}
// Every workgroup of a head stages all of the head's samples, so a head split over two workgroups
// pays the staging twice: with enough heads to fill the chip (the decode-time shape: 960 per call)
// one workgroup takes all ten tiles of a d = 128 head.
constexpr int kStatsWholeHeadMin = 384;
template <int D, int LAYOUT>
static hipError_t launch_stats_split_one(const Dims& d, const void* q_win, int w, const float2* tab, float* mu,
                                         float* sigma, hipStream_t st) {
  if constexpr (D == 128) {
    if (d.qheads() >= kStatsWholeHeadMin) return launch_stats_split_parts<D, LAYOUT, 1>(d, q_win, w, tab, mu, sigma, st);
  }
  return launch_stats_split_parts<D, LAYOUT, 0>(d, q_win, w, tab, mu, sigma, st);
}
template <int D>
static hipError_t launch_stats_split(const Dims& d, const void* q_win, int w, const float2* tab, float* mu,
                                     float* sigma, hipStream_t st) {
  return d.rope_layout ? launch_stats_split_one<D, 1>(d, q_win, w, tab, mu, sigma, st)
                       : launch_stats_split_one<D, 0>(d, q_win, w, tab, mu, sigma, st);
}

hipError_t launch_stats(const Dims& d, const void* q_win, int w, const float2* tab, float* mu,
                        float* sigma, hipStream_t st) {
  const bool bf = d.dtype == EA_BF16;
  // bf16 windows: outer products on the fp16 matrix cores (split operands); fp32 windows: fp32 ones
  if (bf && d.D == 64) return launch_stats_split<64>(d, q_win, w, tab, mu, sigma, st);
  if (bf && d.D == 128) return launch_stats_split<128>(d, q_win, w, tab, mu, sigma, st);
  if (bf) return launch_stats_split<256>(d, q_win, w, tab, mu, sigma, st);
  if (d.D == 64) return launch_stats_one<64, false>(d, q_win, w, tab, mu, sigma, st);
  if (d.D == 128) return launch_stats_one<128, false>(d, q_win, w, tab, mu, sigma, st);
  return launch_stats_one<256, false>(d, q_win, w, tab, mu, sigma, st);
}

template <int D, int LAYOUT, int PARTS>
static hipError_t launch_stats_frags_one(const Dims& d, const void* q_win, int w, const float2* tab, const FragsOut& fo,
                                         hipStream_t st) {
  auto kern = k_stats_split<D, LAYOUT, PARTS, true>;
  const size_t lds = (size_t)2 * D * (stats_split_chunk(D) + 8) * sizeof(_Float16) + (size_t)(10 * D + 4) * sizeof(float);
  static LdsOptIn opt;
  hipError_t e = opt.ensure(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  const dim3 grid(d.qheads(), StatsTiling<D, PARTS>::PARTS);
  kern<<<grid, 256, lds, st>>>(q_win, w, d.ddof, tab, nullptr, nullptr, fo);
  return hipGetLastError();
}
template <int LAYOUT>
static hipError_t launch_stats_frags_layout(const Dims& d, const void* q_win, int w, const float2* tab, const FragsOut& fo,
                                            hipStream_t st) {
  if (d.D == 64) return launch_stats_frags_one<64, LAYOUT, 0>(d, q_win, w, tab, fo, st);
  if (d.qheads() < kStatsFragsMin) return launch_stats_frags_one<128, LAYOUT, 0>(d, q_win, w, tab, fo, st);
  return launch_stats_frags_one<128, LAYOUT, 1>(d, q_win, w, tab, fo, st);
}
hipError_t launch_stats_frags(const Dims& d, const ScorePlan& sp, const void* q_win, int w, const float2* tab,
                              uint4* frags, float* post, hipStream_t st) {
  const FragsOut fo{frags, post, d.G, sp.GH, sp.passes, sp.nfrag, sp.unit_frags, sp.hw};
  return d.rope_layout ? launch_stats_frags_layout<1>(d, q_win, w, tab, fo, st)
                       : launch_stats_frags_layout<0>(d, q_win, w, tab, fo, st);
}

hipError_t launch_prep_frags(const Dims& d, const ScorePlan& sp, const float* mu,
                             const float* sigma, uint4* frags, float* post, hipStream_t st, uint32_t* clear,
                             size_t clear_words, bool sigma_shared) {
  const int nfrag = sp.GH * frags_per_head(d.D) + extra_tiles(sp.GH) * 2 * (d.D / 32);
  dim3 grid(d.units() * sp.passes, (nfrag + 3) / 4);
  const int shared = sigma_shared ? d.Hq : 0;
  const FragsOut fo{frags, post, d.G, sp.GH, sp.passes, sp.nfrag, sp.unit_frags, sp.hw};
  if (d.D == 64) k_prep_frags<64><<<grid, 256, 0, st>>>(mu, sigma, fo, shared, clear, clear_words);
  else if (d.D == 128) k_prep_frags<128><<<grid, 256, 0, st>>>(mu, sigma, fo, shared, clear, clear_words);
  else k_prep_frags<256><<<grid, 256, 0, st>>>(mu, sigma, fo, shared, clear, clear_words);
  return hipGetLastError();
}

}  // namespace ea

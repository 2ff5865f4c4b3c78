// Scoring kernels: Eq. 7 (expected unnormalised attention, as a logit), Eq. 8 (softmax over
// all cached keys) and Eq. 9 with ||v|| and the GQA group mean.
//
//   pass A  k_score_mfma / k_score_hw / k_score_f32 : stream K and V once; per key the G logits
//           l_g = mu_g.k/sqrt(d) + k^T Sigma_g k/(2d) and ||v||.
//           (max, sum exp) per query head and fixed block of keys: k_score_hw and k_score_f32 keep
//           them on the way, for k_score_mfma k_lse_part takes them from the stored logits.
//   pass B  k_finalize : combine the pairs into log-sum-exp per head, then
//           score = (mean_g exp(l_g - lse_g) + eps) * ||v||.
#include "ea_lse.h"
#include "ea_score_mfma.h"

namespace ea {

// Consecutive workgroups run on different dies, and with as many heads as dies a head's are on one: its fragments, which every
// workgroup starts with, then come out of that die's L2, and its counters are near.  In the transposed order every head has
// workgroups on all dies, and all of them share the heads evenly, which is what counts in a long call.
// query_stats + score, us, transposed and plain; register-fragment kernel, G = 4: 8 x 20000 43.9 and 42.1, 16 x 3000 35.7 and 30.6,
// 32 x 20000 99.7 and 95.0, 8 x 131072 138 and 135, 64 x 60000 475 and 465, 12 and 20 heads (that eight does not divide) x 131072
// 196 and 197, 313 and 316; but 16 x 131072 246 and 249, 32 x 60000 241 and 244, x 131072 477 and 493; 8-bit rows 8 x 60000 67.1
// and 65.4, 64 x 32768 227 and 220, but 8 x 131072 113 and 116, 16 x 131072 207 and 213, 32 x 131072 399 and 406; block pools 8 x
// 60000 82.2 and 79.1, 32 x 60000 252 and 257.  Several passes: G = 6, 8 x 20000 60.9 and 58.5, 16 x 2000 38.9 and 35.4, but x 20000
// 88.1 and 99.5; G = 12, three heads x 8000 39.6 and 41.4.
// LDS-fragment kernel, one pass: d = 256, G = 1, 32 x 3000 54.1 and 53.3, 8 x 20000 59.5 and 60.4, 8 x 40000 81.1 and 83.0; G = 2, 8 x
// 12000 66.3 and 62.7, x 20000 81.8 and 78.9, x 40000 118 and 117; d = 64, G = 4, 16 x 12000 36.3 and 33.6, x 30000 51.4 and 48.5,
// 32 x 20000 60.5 and 59.1, x 32768 even; G = 8, 8 x 70000 70.9 and 71.7, 32 x 20000 79.2 and 79.4; in
// several passes plain is up to 16 % slower (d = 64, G = 16, one x 100000 48.7 and 56.6; d = 256, G = 8, 8 x 8000 104 and 119).
static bool transposed_order(const Dims& d, const ScorePlan& sp, int64_t n) {
  if (sp.spare) return false;                 // (their order is the order of coming)
  const int64_t units = d.units();
  if (!sp.hw && !sp.five) {
    if (d.D == 64) return sp.passes > 1 || n > 60000 || units * n > 600000;
    return sp.passes > 1 || n > 40000 || units * n > (d.D == 256 && sp.GH == 2 ? 320000 : 100000);
  }
  if (sp.passes == 1) return units <= 32 && units * sp.npart > (d.kv_fp8 ? 16000 : 30000);
  return units % 8 != 0 || units * sp.npart * sp.passes > 8500;
}

hipError_t launch_score_mfma(const Dims& d, const ScorePlan& sp, const void* k, const void* v,
                             int64_t n, int64_t n_cap, const uint4* frags, const float* post,
                             float* logits, float* vnorm, float2* part, uint32_t* tickets,
                             int ticket_stride, hipStream_t st, const PageMap* pm, const float* kscale,
                             const float* vscale, bool skip_v, float* norms_out) {
  ScoreArgs a;
  a.skip_v = skip_v ? 1 : 0;
  a.pm = pm ? *pm : PageMap{nullptr, 0, 0, 1, 0};
  a.kscale = kscale;
  a.vscale = vscale;
  a.k = (const u32x4*)k;
  a.v = (const u32x4*)v;
  a.n = n;
  a.n_cap = n_cap;
  a.frags = (const u32x4*)frags;
  a.post = post;
  // (the upper half of the logit scratch serves only fp32 caches)
  a.dump = norms_out ? logits : logits + (size_t)d.qheads() * n;
  a.norms_out = norms_out ? 1 : 0;
  a.logits = norms_out ? norms_out : logits;
  a.vnorm = vnorm;
  a.part = part;
  a.G = d.G;
  a.passes = sp.passes;
  a.nchunk = sp.nchunk;
  a.npart = sp.npart;
  a.spare = sp.spare;
  a.transposed = transposed_order(d, sp, n) ? 1 : 0;
  a.units = d.units();
  a.unit_frags = sp.unit_frags;
  a.tickets = tickets;
  a.ticket_stride = ticket_stride;
  if (sp.hw || sp.five) return launch_score_hw(a, sp, d.kv_fp8 != 0, st);
  if (d.kv_fp8) return launch_score_mfma_fp8(d.D, a, sp, st);
  switch (d.D) {
    case 64: return launch_score_mfma_d64(a, sp, st);
    case 128: return sp.GH <= 3 ? launch_score_mfma_d128(a, sp, st) : launch_score_mfma_d128b(a, sp, st);
    case 256: return launch_score_mfma_d256(a, sp, st);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------
// fp32 caches: everything in fp64 (the 1e-5 score tolerance of this path leaves no room for fp32
// accumulation of a d^2-term quadratic form), the quadratic form on the fp64 matrix cores.
//
// Y = M K^T runs as v_mfma_f64_16x16x4_f64: A = 16 output channels x 4 input channels of M, B = 4
// input channels x 16 keys.  Lane l = (r = l % 16, q = l / 16) owns the channels q*d/4 .. of key r as
// B operands; accumulator register v of the lane is row q + 4 v, and row rho of tile jt is the
// channel (rho % 4)*d/4 + 4 jt + rho / 4, so the lane gets back channels it holds and k.(M k) needs
// no data movement.  M folds the pair (c, j) and (j, c) of Sigma onto one side at the granularity
// of the 16-channel blocks fb(c) = (c mod d/4) / 4 (the sum of two fp32 numbers, exact in fp64):
// (d/16 + 1) / (2 d/16) of the dense work is left.  The rows of M of one output tile, a slab of up
// to d/16 KiB x 2, are put together in LDS from Sigma by the four wavefronts and then used by each
// for its 16 keys, which stay in registers as fp32.
//
// What bounds it is the matrix cores' fp64 rate (64 cycles per instruction, 37 us of the 63 that the first shape below
// takes) and the latency around it.  Slabs of M per step, in turn with their use, left the matrix cores idle 60 % of the
// time; at d = 64 and 128 all of M fits in LDS (k_score_f32_whole).  score, 28 query heads x 5003 keys at d = 128 83 -> 73
// us, x 12000 157 -> 136; 8 x 9000 59 -> 51; 32 x 16000 at d = 64 84 -> 68, 4 x 1024 13.3 -> 12.5.  (The next tiles' rows
// requested ahead: 1 to 2 us slower; three tiles at a time: no registers for it.)  At d = 256 M takes 272 KiB and comes in
// slabs (16 x 2000 72 us).
typedef double doublex4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256, 2) void k_score_f32(const float* __restrict__ k, const float* __restrict__ v, long long n,
                                                   long long n_cap, const float* __restrict__ mu,
                                                   const float* __restrict__ sigma, int G, int units, int span,
                                                   int nchunk, double* __restrict__ logits, float* __restrict__ vnorm,
                                                   double2* __restrict__ part) {
  constexpr int D = 256, QW = D / 4, NT = D / 16;
  __shared__ double s_a[NT * 4 * 64];       // fragments of a slab, [k-step][lane]
  __shared__ double s_mu[D];
  __shared__ double s_ms[4][2];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int unit = blockIdx.x % units;
  const int t2 = blockIdx.x / units;
  const int gq = t2 % G, chunk = t2 / G;
  const float* S = sigma + ((size_t)unit * G + gq) * D * D;
  const float* kb = k + (size_t)unit * n_cap * D;
  const float* vb = v + (size_t)unit * n_cap * D;
  const bool do_v = chunk % G == gq;        // the value norms of a span: dealt to the group's heads in turn
  const long long key_lo = (long long)chunk * span, key_hi = min(key_lo + (long long)span, n);
  double m_run = -INFINITY, s_run = 0.0;    // of the keys in this lane's slots r
  if (tid < D) s_mu[tid] = (double)mu[((size_t)unit * G + gq) * D + tid];
  __syncthreads();
  // Tile b of slab jt is one wavefront's: M's own side (c_out, c_in .. c_in + 3) and, for b < jt, the
  // mirrored entries (c_in, c_out ..), which are added to it in LDS.  (A second buffer, filled during the
  // matrix instructions of the slab in front, costs the third workgroup of a CU and gains nothing.)
  const int ms = (lane >> 2) & 3, mq = lane & 3;
  auto build_slab = [&](int jt) __attribute__((always_inline)) {
#pragma unroll 1
    for (int b = wave; b <= jt; b += 4) {
      const float4 own = *reinterpret_cast<const float4*>(S + (size_t)((r & 3) * QW + 4 * jt + (r >> 2)) * D + q * QW + 4 * b);
      const float4 mir = *reinterpret_cast<const float4*>(S + (size_t)(q * QW + 4 * b + ms) * D + mq * QW + 4 * jt);
      double* at = s_a + b * 256;
      at[lane] = own.x;
      at[64 + lane] = own.y;
      at[128 + lane] = own.z;
      at[192 + lane] = own.w;
      if (b < jt) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double* am = at + ms * 64 + q * 16 + mq;
        am[0] += (double)mir.x;
        am[4] += (double)mir.y;
        am[8] += (double)mir.z;
        am[12] += (double)mir.w;
      }
    }
  };
  for (long long key0 = key_lo; key0 < key_hi; key0 += 64) {
    float kf[QW];
    const long long key = key0 + wave * 16 + r;
    const float4* kp = reinterpret_cast<const float4*>(kb + min(key, n - 1) * D + q * QW);
#pragma unroll
    for (int x = 0; x < QW / 4; ++x) {
      const float4 f = kp[x];
      kf[4 * x] = f.x; kf[4 * x + 1] = f.y; kf[4 * x + 2] = f.z; kf[4 * x + 3] = f.w;
    }
    double lin = 0.0, quad = 0.0;
#pragma unroll
    for (int x = 0; x < QW; ++x) lin = fma(s_mu[q * QW + x], (double)kf[x], lin);
    asm volatile("" : "+v"(lin));
    static_for<NT>([&](auto jt_) {
      constexpr int jt = decltype(jt_)::value;
      // (keeps the compiler from holding the keys widened to 64 bits across the slabs: the conversions are
      // hidden by the matrix instructions, twice the registers are not)
#pragma unroll
      for (int x = 0; x < QW; ++x) asm volatile("" : "+v"(kf[x]));
      __syncthreads();                      // the previous slab has been consumed
      build_slab(jt);
      __syncthreads();
      doublex4 acc = doublex4{0.0, 0.0, 0.0, 0.0};
      // four k-steps at a time, the next four fragments on their way; nothing moves across the blocks
      // (left alone, the scheduler widens every key and fetches every fragment of the slab at once)
      double f[2][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) f[0][e] = s_a[e * 64 + lane];
      static_for<jt + 1>([&](auto b_) {
        constexpr int b = decltype(b_)::value;
        if constexpr (b < jt) {
#pragma unroll
          for (int e = 0; e < 4; ++e) f[(b + 1) & 1][e] = s_a[(4 * (b + 1) + e) * 64 + lane];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[b & 1][e], (double)kf[4 * b + e], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int x = 0; x < 4; ++x) quad = fma(acc[x], (double)kf[4 * jt + x], quad);
      asm volatile("" : "+v"(quad));       // dotted here, not at the end of all slabs
    });
    double lg = lin / sqrt((double)D) + quad / (2.0 * D);
    lg += __shfl_xor(lg, 16);
    lg += __shfl_xor(lg, 32);
    if (key < n) {
      if (q == 0) logits[((size_t)unit * G + gq) * n + key] = lg;
      const double mn = fmax(m_run, lg);
      s_run = s_run * exp(m_run - mn) + exp(lg - mn);
      m_run = mn;
    }
    if (do_v) {
      const float4* vp = reinterpret_cast<const float4*>(vb + min(key, n - 1) * D + q * QW);
      double ss = 0.0;
#pragma unroll
      for (int x = 0; x < QW / 4; ++x) {
        const float4 f = vp[x];
        ss = fma((double)f.x, (double)f.x, ss);
        ss = fma((double)f.y, (double)f.y, ss);
        ss = fma((double)f.z, (double)f.z, ss);
        ss = fma((double)f.w, (double)f.w, ss);
      }
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (q == 0 && key < n) vnorm[(size_t)unit * n + key] = (float)sqrt(ss);
    }
  }
  // (max, sum exp) of the span: the 16 key slots of each wavefront, then the four wavefronts
  double m = m_run, s = s_run;
  auto merge = [&](double m2, double s2) {
    const double mn = fmax(m, m2);
    if (mn == -INFINITY) s = 0.0;
    else s = s * exp(m - mn) + s2 * exp(m2 - mn);
    m = mn;
  };
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) merge(__shfl_xor(m, o), __shfl_xor(s, o));
  if (lane == 0) { s_ms[wave][0] = m; s_ms[wave][1] = s; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w) merge(s_ms[w][0], s_ms[w][1]);
    part[((size_t)unit * G + gq) * nchunk + chunk] = make_double2(m, s);
  }
}

// d = 64 and 128: all of the folded M, 20 or 72 KiB of it, stands in LDS from the start (one memory latency and one barrier
// per workgroup instead of one of each per slab and 64 or 128 keys), and the wavefronts then go their own ways through
// every fourth tile of 16 keys of the workgroup's span, two at a time.  Two workgroups fit a CU at d = 128.  Same
// arithmetic per key as above.
template <int D>
__global__ __launch_bounds__(256, D == 64 ? 4 : 2) void k_score_f32_whole(const float* __restrict__ k, const float* __restrict__ v, long long n,
                                                   long long n_cap, const float* __restrict__ mu,
                                                   const float* __restrict__ sigma, int G, int units, int span,
                                                   int nchunk, double* __restrict__ logits, float* __restrict__ vnorm,
                                                   double2* __restrict__ part) {
  constexpr int QW = D / 4, NT = D / 16, NB = NT * (NT + 1) / 2;
  extern __shared__ __align__(16) double s_m[];    // blocks (jt, b), b <= jt, of 4 fragments [lane] each, then mu
  double* s_mu = s_m + NB * 256;
  __shared__ double s_ms[4][2];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int unit = blockIdx.x % units;
  const int t2 = blockIdx.x / units;
  const int gq = t2 % G, chunk = t2 / G;
  const float* S = sigma + ((size_t)unit * G + gq) * D * D;
  const float* kb = k + (size_t)unit * n_cap * D;
  const float* vb = v + (size_t)unit * n_cap * D;
  const long long key_lo = (long long)chunk * span, key_hi = min(key_lo + (long long)span, n);
  {
    // block `at` of the triangle, jt rows down and b along: M's own side and, for b < jt, the mirrored entries
    constexpr int PER = (NB + 3) / 4;
    const int ms = (lane >> 2) & 3, mq = lane & 3;
    float4 own[PER], mir[PER];
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int at = min(wave + 4 * x, NB - 1);
      int jt = 0, b = at;
      while (b > jt) { b -= jt + 1; ++jt; }
      own[x] = *reinterpret_cast<const float4*>(S + (size_t)((r & 3) * QW + 4 * jt + (r >> 2)) * D + q * QW + 4 * b);
      mir[x] = *reinterpret_cast<const float4*>(S + (size_t)(q * QW + 4 * b + ms) * D + mq * QW + 4 * jt);
    }
    if (tid < D) s_mu[tid] = (double)mu[((size_t)unit * G + gq) * D + tid];
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int at = wave + 4 * x;
      if (at < NB) {
        double* to = s_m + at * 256;
        to[lane] = own[x].x;
        to[64 + lane] = own[x].y;
        to[128 + lane] = own[x].z;
        to[192 + lane] = own[x].w;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int at = wave + 4 * x;
      int jt = 0, b = at;
      while (b > jt) { b -= jt + 1; ++jt; }
      if (at < NB && b < jt) {
        double* am = s_m + at * 256 + ms * 64 + q * 16 + mq;
        am[0] += (double)mir[x].x;
        am[4] += (double)mir[x].y;
        am[8] += (double)mir[x].z;
        am[12] += (double)mir[x].w;
      }
    }
  }
  __syncthreads();
  double m_run = -INFINITY, s_run = 0.0;    // of the keys in this lane's slots r
  auto tiles = [&](auto kt_, long long key0) __attribute__((always_inline)) {      // tiles at key0 and key0 + 64
    constexpr int KT = decltype(kt_)::value;
    float kf[KT][QW];
    long long key[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      key[t] = key0 + t * 64 + r;
      const float4* kp = reinterpret_cast<const float4*>(kb + min(key[t], n - 1) * D + q * QW);
#pragma unroll
      for (int x = 0; x < QW / 4; ++x) {
        const float4 f = kp[x];
        kf[t][4 * x] = f.x; kf[t][4 * x + 1] = f.y; kf[t][4 * x + 2] = f.z; kf[t][4 * x + 3] = f.w;
      }
    }
    double lin[KT], quad[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) { lin[t] = 0.0; quad[t] = 0.0; }
#pragma unroll
    for (int x = 0; x < QW; ++x) {
      const double m = s_mu[q * QW + x];
#pragma unroll
      for (int t = 0; t < KT; ++t) lin[t] = fma(m, (double)kf[t][x], lin[t]);
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) asm volatile("" : "+v"(lin[t]));
    static_for<NT>([&](auto jt_) {
      constexpr int jt = decltype(jt_)::value, at = jt * (jt + 1) / 2;
      // (keeps the compiler from holding the keys widened to 64 bits across the tiles)
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int x = 0; x < QW; ++x) asm volatile("" : "+v"(kf[t][x]));
      doublex4 acc[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t) acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
      double f[2][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) f[0][e] = s_m[(at * 4 + e) * 64 + lane];
      static_for<jt + 1>([&](auto b_) {
        constexpr int b = decltype(b_)::value;
        if constexpr (b < jt) {
#pragma unroll
          for (int e = 0; e < 4; ++e) f[(b + 1) & 1][e] = s_m[((at + b + 1) * 4 + e) * 64 + lane];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < KT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[b & 1][e], (double)kf[t][4 * b + e], acc[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int x = 0; x < 4; ++x) quad[t] = fma(acc[t][x], (double)kf[t][4 * jt + x], quad[t]);
#pragma unroll
      for (int t = 0; t < KT; ++t) asm volatile("" : "+v"(quad[t]));
    });
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      double lg = lin[t] / sqrt((double)D) + quad[t] / (2.0 * D);
      lg += __shfl_xor(lg, 16);
      lg += __shfl_xor(lg, 32);
      if (key[t] < n) {
        if (q == 0) logits[((size_t)unit * G + gq) * n + key[t]] = lg;
        const double mn = fmax(m_run, lg);
        s_run = s_run * exp(m_run - mn) + exp(lg - mn);
        m_run = mn;
      }
      if (((key0 + t * 64) >> 4) % G == gq) {        // the value norms: dealt to the group's heads tile by tile
        const float4* vp = reinterpret_cast<const float4*>(vb + min(key[t], n - 1) * D + q * QW);
        double ss = 0.0;
#pragma unroll
        for (int x = 0; x < QW / 4; ++x) {
          const float4 f = vp[x];
          ss = fma((double)f.x, (double)f.x, ss);
          ss = fma((double)f.y, (double)f.y, ss);
          ss = fma((double)f.z, (double)f.z, ss);
          ss = fma((double)f.w, (double)f.w, ss);
        }
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        if (q == 0 && key[t] < n) vnorm[(size_t)unit * n + key[t]] = (float)sqrt(ss);
      }
    }
  };
  long long key0 = key_lo + wave * 16;
  for (; key0 + 64 < key_hi; key0 += 128) tiles(std::integral_constant<int, 2>{}, key0);
  if (key0 < key_hi) tiles(std::integral_constant<int, 1>{}, key0);
  // (max, sum exp) of the span: the 16 key slots of each wavefront, then the four wavefronts
  double m = m_run, s = s_run;
  auto merge = [&](double m2, double s2) {
    const double mn = fmax(m, m2);
    if (mn == -INFINITY) s = 0.0;
    else s = s * exp(m - mn) + s2 * exp(m2 - mn);
    m = mn;
  };
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) merge(__shfl_xor(m, o), __shfl_xor(s, o));
  if (lane == 0) { s_ms[wave][0] = m; s_ms[wave][1] = s; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w) merge(s_ms[w][0], s_ms[w][1]);
    part[((size_t)unit * G + gq) * nchunk + chunk] = make_double2(m, s);
  }
}

template <int D>
static hipError_t launch_f32_whole(const Dims& d, const float* k, const float* v, int64_t n, int64_t n_cap, const float* mu,
                                   const float* sigma, double* logits, float* vnorm, double2* part, int* nchunk_out,
                                   hipStream_t st) {
  constexpr int NT = D / 16;
  const size_t lds = (size_t)(NT * (NT + 1) / 2 * 256 + D) * sizeof(double);
  auto kern = k_score_f32_whole<D>;
  static LdsOptIn opt;
  hipError_t e = opt.ensure(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  const int64_t heads = d.qheads(), span = f32_span(heads, n, (int64_t)device_num_cu() * (D == 64 ? 4 : 2));
  const int nchunk = (int)((n + span - 1) / span);
  *nchunk_out = nchunk;
  kern<<<(unsigned)(heads * nchunk), 256, lds, st>>>(k, v, n, n_cap, mu, sigma, d.G, d.units(), (int)span, nchunk, logits, vnorm, part);
  return hipGetLastError();
}

hipError_t launch_score_f32(const Dims& d, const void* k, const void* v, int64_t n, int64_t n_cap,
                            const float* mu, const float* sigma, double* logits, float* vnorm,
                            double2* part, int* nchunk_out, hipStream_t st) {
  if (d.D == 64) return launch_f32_whole<64>(d, (const float*)k, (const float*)v, n, n_cap, mu, sigma, logits, vnorm, part, nchunk_out, st);
  if (d.D == 128) return launch_f32_whole<128>(d, (const float*)k, (const float*)v, n, n_cap, mu, sigma, logits, vnorm, part, nchunk_out, st);
  // 64 keys per workgroup and step, spans so that a head has at most 1024 partials
  int64_t span = (n + 1023) / 1024;
  span = (span + 63) / 64 * 64;
  const int nchunk = (int)((n + span - 1) / span);
  *nchunk_out = nchunk;
  if (d.D != 256) return hipErrorInvalidValue;
  k_score_f32<<<(unsigned)((int64_t)d.qheads() * nchunk), 256, 0, st>>>((const float*)k, (const float*)v, n, n_cap, mu, sigma, d.G,
                                                                   d.units(), (int)span, nchunk, logits, vnorm, part);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Pass B.  One workgroup = `rounds` x 1024 keys of one unit.  LT is the logit type (float: bf16
// caches, double: fp32 caches).  With hist0 != nullptr the first radix-select digit (top 11
// bits of the score's bit pattern) is histogrammed on the way out.
//
// The (max, sum exp) partials of pass A belong to fixed blocks of keys (partial j of a head
// covers the same keys in every run) and are combined here in index order, so the log-sum-exp,
// and with it every score, comes out bit-identical from run to run however pass A's tiles were
// dealt to workgroups.
// (max, sum exp) of one block of kLseBlock keys of one query head, from the logits pass A stored:
// the LDS-fragment kernels leave the softmax to this pass, so the partial of a block is the same
// number on every run whichever waves scored its keys (fixed reduction tree), and the score
// kernel's inner loop carries no exponentials or cross-lane reductions.  The logits were written
// a moment ago and are read from the caches.
__global__ __launch_bounds__(256) void k_lse_part(const float* __restrict__ logits, long long n, int npart,
                                                  float2* __restrict__ part) {
  constexpr int PER = kLseBlock / 256;
  __shared__ float s_red[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.x / npart, j = blockIdx.x - head * npart;
  const float* lp = logits + (size_t)head * n;
  const long long base = (long long)j * kLseBlock;
  float x[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {          // no load under a condition: indices past the end are clamped
    const long long i = base + it * 256 + tid;
    const float v = lp[min(i, n - 1)];
    x[it] = i < n ? v : -INFINITY;
  }
  float m = x[0];
#pragma unroll
  for (int it = 1; it < PER; ++it) m = fmaxf(m, x[it]);
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if (lane == 0) s_red[0][wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(s_red[0][0], s_red[0][1]), fmaxf(s_red[0][2], s_red[0][3]));   // a block holds a key: finite
  float s = 0.f;
#pragma unroll
  for (int it = 0; it < PER; ++it) s += expf(x[it] - m);
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) s_red[1][wave] = s;
  __syncthreads();
  if (tid == 0) part[(size_t)head * npart + j] = make_float2(m, (s_red[1][0] + s_red[1][1]) + (s_red[1][2] + s_red[1][3]));
}

// Heads with very many partials: one workgroup per query head reduces them once, ahead of
// pass B (otherwise every workgroup of pass B would walk the whole list).
template <typename LT>
__global__ __launch_bounds__(256) void k_lse(const typename LT2<LT>::type* __restrict__ part, int npart,
                                             LT* __restrict__ lse) {
  __shared__ LT s_m[4], s_s[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const typename LT2<LT>::type* p = part + (size_t)blockIdx.x * npart;
  LT m, s;
  gather_lt<LT>(p, npart, tid, 256, m, s);
  for (int o = 32; o >= 1; o >>= 1) {
    LT m2 = __shfl_xor(m, o), s2 = __shfl_xor(s, o);
    merge_lt<LT>(m, s, m2, s2);
  }
  if (lane == 0) { s_m[wave] = m; s_s[wave] = s; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w) merge_lt<LT>(m, s, s_m[w], s_s[w]);
    lse[blockIdx.x] = m + ea_log(s);
  }
}

template <typename LT>
__global__ __launch_bounds__(256) void k_finalize(const LT* __restrict__ logits,
                                                  const float* __restrict__ vnorm,
                                                  const typename LT2<LT>::type* __restrict__ part,
                                                  const LT* __restrict__ lse_in, int G, int npart,
                                                  long long n, float eps, int units, int rounds,
                                                  float* __restrict__ scores,
                                                  uint32_t* __restrict__ hist0,
                                                  const float* __restrict__ wnorm) {
  __shared__ LT s_lse[64];
  __shared__ uint32_t s_hist[kSelBins];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int unit = blockIdx.x % units;
  const long long blk = blockIdx.x / units;
  if (hist0)
    for (int i = tid; i < kSelBins; i += 256) s_hist[i] = 0;
  for (int g = wave; g < G; g += 4) {
    const LT v = lse_in ? lse_in[(size_t)unit * G + g]
                        : wave_lse<LT>(part + ((size_t)unit * G + g) * npart, npart, lane);
    if (lane == 0) s_lse[g] = v;
  }
  __syncthreads();
  const LT invG = (LT)1 / (LT)G;
  for (int rd = 0; rd < rounds; ++rd) {
    const long long base = (blk * rounds + rd) * 1024;
    if (base >= n) break;
    // The four keys of a thread go through the heads together and no load sits under a condition
    // (indices past the end are clamped): loads inside "if (i < n)" come back one at a time.
    long long ic[4];
    float vn[4];
    LT acc[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      ic[it] = min(base + it * 256 + tid, n - 1);
      vn[it] = vnorm[(size_t)unit * n + ic[it]];
      acc[it] = 0;
    }
    // Four heads' logits are requested together, then added in head order: one head at a time kept 16 KiB
    // in flight per CU, which is what bounded the pass (G = 4: 32 units x 131072 keys 25.3 -> 21.6 us; with norms per
    // query head 8 x 32768 11.2 -> 6.8).
    for (int g0 = 0; g0 < G; g0 += 4) {
      LT lv[4][4];
      float wv[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const size_t row = ((size_t)unit * G + min(g0 + j, G - 1)) * n;
#pragma unroll
        for (int it = 0; it < 4; ++it) lv[j][it] = logits[row + ic[it]];
        if (wnorm) {      // Eq. 9 with the output projection: every query head weighs by its own norm
#pragma unroll
          for (int it = 0; it < 4; ++it) wv[j][it] = wnorm[row + ic[it]];
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (g0 + j >= G) break;
        const LT lse = s_lse[g0 + j];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          if (wnorm) acc[it] += (ea_exp(lv[j][it] - lse) + (LT)eps) * (LT)wv[j][it];
          else acc[it] += ea_exp(lv[j][it] - lse);
        }
      }
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const long long i = base + it * 256 + tid;
      if (i < n) {
        float sc = wnorm ? (float)(acc[it] * invG) : (float)((acc[it] * invG + (LT)eps) * (LT)vn[it]);
        scores[(size_t)unit * n + i] = sc;
        if (hist0) {
          atomicAdd(&s_hist[__float_as_uint(sc) >> 21], 1u);
          if (__float_as_uint(sc) > 0x7f800000u)      // NaN (non-finite inputs): see ea_debug_status
            atomicOr(hist0 + 2 * kSelBins + kStatusSlot, kStatusBadScore);
        }
      }
    }
  }
  if (hist0) {
    __syncthreads();
    for (int i = tid; i < kSelBins; i += 256) {
      uint32_t c = s_hist[i];
      if (c) atomicAdd(&hist0[(size_t)unit * 3 * kSelBins + i], c);
    }
  }
}

// ||W_o^(g) v_i|| from the quadratic form pass A leaves in `logits` when it is run over the value
// rows with mu = 0 and Sigma = M_g = W_o^(g)^T W_o^(g):  logits = v^T M_g v / (2 d).
template <typename LT>
__global__ void k_wnorm(const LT* __restrict__ logits, size_t count, float two_d, float* __restrict__ wnorm) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) {
    const LT q = logits[i] * (LT)two_d;
    wnorm[i] = q > (LT)0 ? (float)sqrt(q) : 0.f;
  }
}

hipError_t launch_wnorm(const void* logits, int logits_f64, size_t count, int D, float* wnorm, hipStream_t st) {
  const unsigned grid = (unsigned)((count + 255) / 256);
  if (logits_f64)
    k_wnorm<double><<<grid, 256, 0, st>>>((const double*)logits, count, 2.0f * (float)D, wnorm);
  else
    k_wnorm<float><<<grid, 256, 0, st>>>((const float*)logits, count, 2.0f * (float)D, wnorm);
  return hipGetLastError();
}

constexpr int kLseInlineMax = 1024;   // more partials per head than this: reduce them in k_lse first (one short launch; every
                                      // finalize workgroup then reads G numbers instead of the list).  Operands + score, with
                                      // and without that launch: G = 3, 8 heads x 30000 keys (469 partials) 41.4 and 39.4 us,
                                      // whole pass of 8 x 20000 105.2 and 102.7; 8 x 131072 (2048) 127 and 132

hipError_t launch_finalize(const Dims& d, int64_t n, const void* logits, int logits_f64,
                           const float* vnorm, const void* part, int npart, void* lse, float* scores,
                           uint32_t* hist0, hipStream_t st, const float* wnorm, int lse_pass, const KeepOut* sel) {
  // 1024 keys per workgroup; four rounds of them (fewer histogram flushes) once that still leaves
  // a few thousand workgroups: the pass is bound by memory latency and wants the chip full
  const int rounds = (n + 1023) / 1024 * d.units() >= 4096 ? 4 : 1;
  const int64_t nblk = (n + 1024 * rounds - 1) / (1024 * rounds);
  const unsigned grid = (unsigned)(nblk * d.units());
  const bool pre = npart > kLseInlineMax;
  if (sel) {                       // short heads: their selection in the same launch
    if (lse_pass)
      k_lse_part<<<(unsigned)((size_t)d.qheads() * npart), 256, 0, st>>>((const float*)logits, n, npart, (float2*)part);
    return launch_finish_select(d, n, logits, logits_f64, vnorm, part, npart, scores, *sel, hist0, st);
  }
  if (logits_f64) {
    if (pre) k_lse<double><<<d.qheads(), 256, 0, st>>>((const double2*)part, npart, (double*)lse);
    k_finalize<double><<<grid, 256, 0, st>>>((const double*)logits, vnorm, (const double2*)part,
                                             pre ? (const double*)lse : nullptr, d.G, npart, n, d.eps,
                                             d.units(), rounds, scores, hist0, wnorm);
  } else {
    if (lse_pass)
      k_lse_part<<<(unsigned)((size_t)d.qheads() * npart), 256, 0, st>>>((const float*)logits, n, npart, (float2*)part);
    if (pre) k_lse<float><<<d.qheads(), 256, 0, st>>>((const float2*)part, npart, (float*)lse);
    k_finalize<float><<<grid, 256, 0, st>>>((const float*)logits, vnorm, (const float2*)part,
                                            pre ? (const float*)lse : nullptr, d.G, npart, n, d.eps,
                                            d.units(), rounds, scores, hist0, wnorm);
  }
  return hipGetLastError();
}

}  // namespace ea

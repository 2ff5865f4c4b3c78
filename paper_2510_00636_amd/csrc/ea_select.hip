// Top-k selection per KV head (Sec. 2.2 "Compression", Listing 1 top-k) as an exact radix
// select on the fp32 bit patterns (non-negative floats order like unsigned integers).
//
// Three histogram passes (11 + 11 + 10 bits) narrow down the bit pattern T of the n_keep-th
// largest score and the number q of scores equal to T that must still be kept; every
// workgroup re-derives the digits found so far from the shared histograms (a 2048-entry
// suffix scan, cheaper than another launch).  The emit pass then counts and writes the kept
// positions in ascending order: score > T, or == T among the first q such positions.
#include <hip/hip_runtime.h>

#include "ea_kernels.h"

namespace ea {

constexpr int kSelThreads = 256;
constexpr int kSelPer = kSelBlock / kSelThreads;   // 16 consecutive scores per thread

// zeroes p[0, count) and, if given, the single word *extra
__global__ void k_zero(uint32_t* p, size_t count, uint32_t* extra) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0;
  if (extra && i == 0) *extra = 0;
}

hipError_t launch_zero(uint32_t* p, size_t count, hipStream_t st, uint32_t* extra) {
  if (count == 0 && !extra) return hipSuccess;
  k_zero<<<(unsigned)((count + 255) / 256 + (count == 0)), 256, 0, st>>>(p, count, extra);
  return hipGetLastError();
}

// Bin b (counting down from the top) with  count(bins > b) < target <= count(bins >= b);
// *rem = target - count(bins > b).  Called by all 64 lanes of ONE wavefront; the result is
// uniform.  nbins is 2048 or 1024; lane l owns the nbins/64 bins just below nbins - l*nbins/64.
__device__ int find_bin_wave(const uint32_t* __restrict__ hist, int nbins, uint32_t target,
                             uint32_t* rem, int lane) {
  const int per = nbins / 64;                        // 32 or 16
  const int lo = nbins - per * (lane + 1);
  uint32_t loc[32];
  uint32_t sum = 0;
  const uint4* hp = reinterpret_cast<const uint4*>(hist + lo);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (4 * j < per) {
      const uint4 v = hp[j];
      loc[4 * j] = v.x; loc[4 * j + 1] = v.y; loc[4 * j + 2] = v.z; loc[4 * j + 3] = v.w;
      sum += v.x + v.y + v.z + v.w;
    } else {
      loc[4 * j] = loc[4 * j + 1] = loc[4 * j + 2] = loc[4 * j + 3] = 0;
    }
  }
  uint32_t incl = sum;                               // inclusive scan over lanes (lane 0 = top bins)
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  const uint32_t excl = incl - sum;
  const bool mine = excl < target && target <= incl;
  int b = 0;
  uint32_t r = 0;
  if (mine) {
    uint32_t cum = excl;
    b = lo;
    r = target - cum;
#pragma unroll
    for (int j = 31; j >= 0; --j) {                  // walk this lane's bins from the top down
      if (j < per) {
        if (target > cum && target <= cum + loc[j]) { b = lo + j; r = target - cum; }
        cum += loc[j];
      }
    }
  }
  const unsigned long long m = __ballot(mine);
  const int src = m ? __ffsll((long long)m) - 1 : 0;
  *rem = __shfl(r, src);
  return __shfl(b, src);
}

struct SelArgs {
  const float* scores;
  long long n;
  uint32_t n_keep;
  uint32_t* hist;    // [units][3][2048]; word [unit][2][kEmitTicket] deals the emit pass its blocks
  uint32_t* blk;     // [units][nblk], zero at launch: kEmitSeen | count == T << 13 | count > T of a block
  int32_t* idx;      // [units][n_keep]
  int nblk;
  uint32_t* status;  // status word
};

// Digits fixed by the histogram passes before pass P: wavefront 0 re-derives them (a few
// hundred cycles, cheaper than another launch) and the workgroup reads them from s_res.
template <int P>
__device__ void resolve(const SelArgs& a, int unit, uint32_t* s_res, uint32_t* prefix, uint32_t* rem) {
  if (P >= 1 && threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const uint32_t* h = a.hist + (size_t)unit * 3 * kSelBins;
    uint32_t r = a.n_keep, pre = 0;
    const int b0 = find_bin_wave(h, 2048, r, &r, lane);
    pre = (uint32_t)b0;
    if (P >= 2) { const int b1 = find_bin_wave(h + kSelBins, 2048, r, &r, lane); pre = (pre << 11) | (uint32_t)b1; }
    if (P >= 3) { const int b2 = find_bin_wave(h + 2 * kSelBins, 1024, r, &r, lane); pre = (pre << 10) | (uint32_t)b2; }
    if (lane == 0) { s_res[0] = pre; s_res[1] = r; }
  }
  __syncthreads();
  *prefix = P >= 1 ? s_res[0] : 0u;
  *rem = P >= 1 ? s_res[1] : a.n_keep;
  __syncthreads();
}

template <int P>
__global__ __launch_bounds__(kSelThreads) void k_sel_hist(SelArgs a) {
  __shared__ uint32_t s_hist[kSelBins];
  __shared__ uint32_t s_tmp[258];
  const int tid = threadIdx.x, unit = blockIdx.x;
  uint32_t prefix = 0, rem;
  resolve<P>(a, unit, s_tmp, &prefix, &rem);
  for (int i = tid; i < kSelBins; i += kSelThreads) s_hist[i] = 0;
  __syncthreads();
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  const long long base = (long long)blockIdx.y * kSelBlock;
  // All loads first and none under a condition (indices past the end are clamped): a load inside
  // "if (i < n)" is followed by a wait for it, one memory round trip per score.
  uint32_t uu[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) uu[j] = sc[min(base + j * kSelThreads + tid, a.n - 1)];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    const long long i = base + j * kSelThreads + tid;
    if (i < a.n) {
      const uint32_t u = uu[j];
      if (P == 0) {
        atomicAdd(&s_hist[u >> 21], 1u);
        // outside the domain (negative or NaN): the order of bit patterns is not the order of
        // values there; the selection still completes, the status word records it
        if (u > 0x7f800000u) atomicOr(a.status, kStatusBadScore);
      }
      if (P == 1 && (u >> 21) == prefix) atomicAdd(&s_hist[(u >> 10) & 2047u], 1u);
      if (P == 2 && (u >> 10) == prefix) atomicAdd(&s_hist[u & 1023u], 1u);
    }
  }
  __syncthreads();
  uint32_t* out = a.hist + ((size_t)unit * 3 + P) * kSelBins;
  for (int i = tid; i < kSelBins; i += kSelThreads) {
    const uint32_t c = s_hist[i];
    if (c) atomicAdd(&out[i], c);
  }
}

// Counting and writing in one launch.  A workgroup takes the next block of its unit by ticket, counts what its
// block keeps, publishes the two counts in one word and adds up those of the blocks in front of it: blocks
// with lower tickets, so their workgroups are running already and publish before they wait for anybody;
// every wait ends.  (A thread's spin budget for the whole sum keeps even a corrupted workspace from hanging: the
// block then writes nothing and the status word says so.)  Wavefront w holds 16 rows of 64 consecutive scores,
// so that loads and stores run along the lanes and positions are ballots.  Against a counting launch and an emit
// launch in which a thread read 16 consecutive scores (64 cache lines per load): 7.0 + 16.8 -> 16.8 us at 32 units x
// 131072, 5.4 + 7.4 -> 10.7 at 8, and a launch less (whole pass of 8 units x 20011: 132.4 -> 128.6 us).
// What lies in front of a block is (scores above T) + min(q, scores at T), whatever the order of the blocks, so a
// lane just adds up words, two in flight.  Scanning them in order, 64 at a time, had made whole selections of one long
// head slower than the two launches were: 2^22 scores 70.3 -> 76.2 us, 2^26 1489 -> 1815; now 70.6 and 915.  Four words
// in flight per lane are 6 % faster at 2^26 and 2 % slower at 8 heads x 2^20 (69.7 us), all four wavefronts at it 18 %
// slower there.
constexpr uint32_t kEmitTicket = 1026;     // free word of a unit's third histogram
constexpr uint32_t kEmitSeen = 1u << 31;
constexpr int kEmitSpinLimit = 1 << 20;

__global__ __launch_bounds__(kSelThreads) void k_sel_emit(SelArgs a) {
  constexpr int W = kSelThreads / 64, U = 2;
  __shared__ uint32_t s_tmp[258];
  __shared__ uint32_t s_w[2][W];
  __shared__ uint32_t s_front[3];
  __shared__ uint32_t s_blk;
  const int tid = threadIdx.x, lane = tid & 63, unit = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) s_blk = atomicAdd(a.hist + ((size_t)unit * 3 + 2) * kSelBins + kEmitTicket, 1u);
  __syncthreads();
  const int blk = __builtin_amdgcn_readfirstlane((int)s_blk);
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  const long long base = (long long)blk * kSelBlock + wave * (kSelBlock / W) + lane;    // of u[0]; u[j]: 64 j further
  uint32_t u[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) u[j] = sc[min(base + 64 * j, a.n - 1)];
  uint32_t T, q;
  resolve<3>(a, unit, s_tmp, &T, &q);
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    gt += __popcll(__ballot(base + 64 * j < a.n && u[j] > T));
    eq += __popcll(__ballot(base + 64 * j < a.n && u[j] == T));
  }
  if (lane == 0) { s_w[0][wave] = gt; s_w[1][wave] = eq; }
  __syncthreads();
  uint32_t* pub = a.blk + (size_t)unit * a.nblk;
  const int front = min(blk, a.nblk);       // (a counter that did not start at zero never leads past the unit's words)
  if (tid == 0 && blk < a.nblk) {
    uint32_t g = 0, e = 0;
    for (int w = 0; w < W; ++w) { g += s_w[0][w]; e += s_w[1][w]; }
    __hip_atomic_store(&pub[blk], kEmitSeen | (e << 13) | g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // scores above T and at T in the blocks in front of this one
  if (wave == 0) {
    uint32_t gf = 0, ef = 0;
    int spin = 0;
    for (int j0 = lane; j0 < front && spin < kEmitSpinLimit; j0 += U * 64) {
      uint32_t word[U];
#pragma unroll
      for (int x = 0; x < U; ++x)
        word[x] = j0 + 64 * x < front ? __hip_atomic_load(&pub[j0 + 64 * x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kEmitSeen;
#pragma unroll
      for (int x = 0; x < U; ++x) {
        while ((word[x] & kEmitSeen) == 0u && ++spin < kEmitSpinLimit) {
          __builtin_amdgcn_s_sleep(1);
          word[x] = __hip_atomic_load(&pub[j0 + 64 * x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        gf += word[x] & 0x1fffu;
        ef += (word[x] >> 13) & 0x1fffu;
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) { gf += __shfl_xor(gf, o); ef += __shfl_xor(ef, o); }
    const bool ok = __ballot(spin >= kEmitSpinLimit) == 0ull;
    if (lane == 0) {
      s_front[0] = gf;
      s_front[1] = ef;
      s_front[2] = ok;
      if (!ok) atomicOr(a.status, kStatusCompactWait);
    }
  }
  __syncthreads();
  if (!s_front[2]) return;
  // what lies in front of this wavefront
  uint32_t pos = s_front[0], eq_before = s_front[1];
  for (int w = 0; w < wave; ++w) { pos += s_w[0][w]; eq_before += s_w[1][w]; }
  pos += eq_before < q ? eq_before : q;
  int32_t* out = a.idx + (size_t)unit * a.n_keep;
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    const bool in = base + 64 * j < a.n;
    const unsigned long long ties = __ballot(in && u[j] == T);
    const bool keep = in && (u[j] > T || (u[j] == T && eq_before + __popcll(ties & below) < q));
    const unsigned long long mask = __ballot(keep);
    const uint32_t at = pos + __popcll(mask & below);
    if (keep && at < a.n_keep) out[at] = (int32_t)(base + 64 * j);
    pos += __popcll(mask);
    eq_before += __popcll(ties);
  }
}

// ---------------------------------------------------------------------------------------
// Short heads (n <= kSelSmallMax): one workgroup of 16 wavefronts per unit does all of the above in one
// launch.  The scores are read once and stay in registers, up to PER per thread: wavefront w holds 64 R
// consecutive positions (R = ceil(n / 1024)), lane l the l-th of each row of 64, so that positions are
// counted with ballots and the kept ones leave in order.  Same result as the multi-launch path, bit for bit.
//
// What bounds it is the chain of three histograms.  Scores crowd into a few bins of the first digit (four
// bins per factor of two), and LDS atomics on one address go one by one, so that digit's histogram is kept in
// four copies, copies of a bin in neighbouring banks.  Against the version that kept the scores in LDS and
// gave every thread a run of positions (bank conflicts of n / 1024 ways): 8 units x 16384 19.5 -> 14.4 us,
// 8 x 8000 11.4 -> 9.7, 8 x 1000 8.8 -> 7.4, 192 x 4608 10.1 -> 9.4.
constexpr int kSelSmallThreads = 1024;
constexpr int kSelCopies = 4;

template <int PER, bool HIST0>
__global__ __launch_bounds__(kSelSmallThreads) void k_sel_small(SelArgs a) {
  __shared__ uint32_t s_hist[kSelBins * kSelCopies];
  __shared__ uint32_t s_w[2][kSelSmallThreads / 64];
  __shared__ uint32_t s_res[2];
  const int tid = threadIdx.x, lane = tid & 63, unit = blockIdx.x, n = (int)a.n;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows = (n + kSelSmallThreads - 1) / kSelSmallThreads;      // <= PER
  const int base = wave * 64 * rows + lane;                            // position of u[it]: base + 64 it
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  uint32_t u[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) u[it] = sc[min(base + 64 * min(it, rows - 1), n - 1)];
  // u[it] is a score of the head and of this wavefront's share; `lim` is made opaque in front of every phase,
  // or the compiler keeps PER lane masks alive through all of them
  int lim = min(n - base, 64 * rows - lane);
  auto inside = [&](int it) { return 64 * it < lim; };

  uint32_t prefix = 0, rem = a.n_keep;
  bool bad = false;
#pragma unroll
  for (int P = 0; P < 3; ++P) {
    if (HIST0 && P == 0) {                          // the caller's first histogram
      if (wave == 0) {
        uint32_t r;
        const int b = find_bin_wave(a.hist + (size_t)unit * 3 * kSelBins, 2048, rem, &r, lane);
        if (lane == 0) { s_res[0] = (uint32_t)b; s_res[1] = r; }
      }
      for (int i = tid; i < kSelBins; i += kSelSmallThreads) s_hist[i] = 0;
      __syncthreads();
      prefix = s_res[0];
      rem = s_res[1];
      continue;
    }
    if (!(HIST0 && P == 1)) {
      for (int i = tid; i < (P == 0 ? kSelBins * kSelCopies : kSelBins); i += kSelSmallThreads) s_hist[i] = 0;
      __syncthreads();
    }
    asm volatile("" : "+v"(lim));
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      if (!inside(it)) continue;
      if (P == 0) {
        atomicAdd(&s_hist[(u[it] >> 21) * kSelCopies + (lane & (kSelCopies - 1))], 1u);
        bad |= u[it] > 0x7f800000u;
      }
      if (P == 1 && (u[it] >> 21) == prefix) atomicAdd(&s_hist[(u[it] >> 10) & 2047u], 1u);
      if (P == 2 && (u[it] >> 10) == prefix) atomicAdd(&s_hist[u[it] & 1023u], 1u);
    }
    __syncthreads();
    if (P == 0) {                                   // the copies of every bin, added up in place
      uint32_t sum[kSelBins / kSelSmallThreads];
#pragma unroll
      for (int j = 0; j < kSelBins / kSelSmallThreads; ++j) {
        const uint4 c = reinterpret_cast<const uint4*>(s_hist)[tid + j * kSelSmallThreads];
        sum[j] = c.x + c.y + c.z + c.w;
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kSelBins / kSelSmallThreads; ++j) s_hist[tid + j * kSelSmallThreads] = sum[j];
      __syncthreads();
    }
    if (wave == 0) {
      uint32_t r;
      const int b = find_bin_wave(s_hist, P == 2 ? 1024 : 2048, rem, &r, lane);
      if (lane == 0) { s_res[0] = (prefix << (P == 2 ? 10 : 11)) | (uint32_t)b; s_res[1] = r; }
    }
    __syncthreads();
    prefix = s_res[0];
    rem = s_res[1];
  }
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(a.status, kStatusBadScore);
  const uint32_t T = prefix, q = rem;             // threshold pattern, ties at T to keep

  // scores above T and at T per wavefront, then what lies in front of this wavefront
  asm volatile("" : "+v"(lim));
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    gt += __popcll(__ballot(inside(it) && u[it] > T));
    eq += __popcll(__ballot(inside(it) && u[it] == T));
  }
  if (lane == 0) { s_w[0][wave] = gt; s_w[1][wave] = eq; }
  __syncthreads();
  uint32_t pos = 0, eq_before = 0;
  for (int w = 0; w < wave; ++w) { pos += s_w[0][w]; eq_before += s_w[1][w]; }
  pos += eq_before < q ? eq_before : q;
  int32_t* out = a.idx + (size_t)unit * a.n_keep;
  const unsigned long long below = (1ull << lane) - 1ull;
  asm volatile("" : "+v"(lim));
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const unsigned long long ties = __ballot(inside(it) && u[it] == T);
    const bool keep = inside(it) && (u[it] > T || (u[it] == T && eq_before + __popcll(ties & below) < q));
    const unsigned long long kept = __ballot(keep);
    const uint32_t at = pos + __popcll(kept & below);
    if (keep && at < a.n_keep) out[at] = base + 64 * it;
    pos += __popcll(kept);
    eq_before += __popcll(ties);
  }
}

hipError_t launch_select(const Dims& d, const float* scores, int64_t n, int64_t n_keep, int32_t* idx,
                         uint32_t* hist, uint32_t* blk, bool hist0_done, hipStream_t st, uint32_t* status_hist) {
  SelArgs a;
  a.status = (status_hist ? status_hist : hist) + 2 * kSelBins + kStatusSlot;
  a.scores = scores;
  a.n = n;
  a.n_keep = (uint32_t)n_keep;
  a.hist = hist;
  a.blk = blk;
  a.idx = idx;
  a.nblk = (int)((n + kSelBlock - 1) / kSelBlock);
  static_assert(kSelSmallMax <= 16 * kSelSmallThreads, "scores per thread");
  if (select_in_one_launch(n)) {
#define EA_SMALL(PP)                                                                                  \
  if (hist0_done) k_sel_small<PP, true><<<d.units(), kSelSmallThreads, 0, st>>>(a);                   \
  else k_sel_small<PP, false><<<d.units(), kSelSmallThreads, 0, st>>>(a)
    if (n <= 4 * kSelSmallThreads) { EA_SMALL(4); }
    else if (n <= 8 * kSelSmallThreads) { EA_SMALL(8); }
    else { EA_SMALL(16); }
#undef EA_SMALL
    return hipGetLastError();
  }
  dim3 grid(d.units(), a.nblk);
  if (!hist0_done) k_sel_hist<0><<<grid, kSelThreads, 0, st>>>(a);
  k_sel_hist<1><<<grid, kSelThreads, 0, st>>>(a);
  k_sel_hist<2><<<grid, kSelThreads, 0, st>>>(a);
  k_sel_emit<<<grid, kSelThreads, 0, st>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Head-adaptive budgets (Sec. 2.2, "Head-Adaptive Compression"): the selection runs once over the
// pooled scores of a layer's KV heads, [H][n] read as one list of H*n, after every head's own
// `floor` best pairs have been lifted to +inf so that the pooled selection takes them first.
//
// One workgroup = kSelBlock scores of a head: copied into LDS, those on the head's list of its `n_mark` best
// (the stretch of it that lies in the block: two 64-ary searches) set to +inf, written out, and the first
// digit of the pooled list's radix select counted on the way: a copy, a marking and a histogram launch in one.
// (With it, one clearing launch instead of four and the heads' first digit taken from the finalize pass, the
// adaptive pass of 8 heads x 50001 keys went from 24 launches and 266 us to 18 and 253.)
__global__ __launch_bounds__(kSelThreads) void k_lift(const float* __restrict__ scores, const int32_t* __restrict__ top,
                                                      long long n, int n_mark, int Hkv, float* __restrict__ lifted,
                                                      uint32_t* __restrict__ pool_hist) {
  __shared__ float s_sc[kSelBlock];
  __shared__ uint32_t s_hist[kSelBins];
  __shared__ int s_j[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, unit = blockIdx.x;
  const long long base = (long long)blockIdx.y * kSelBlock;
  const int m = (int)min((long long)kSelBlock, n - base);
  const int32_t* list = top + (size_t)unit * n_mark;
  float x[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) x[j] = scores[(size_t)unit * n + min(base + j * kSelThreads + tid, n - 1)];
  for (int i = tid; i < kSelBins; i += kSelThreads) s_hist[i] = 0;
  if (wave < 2) {                                        // first list entry at or past the block's start, and past its end
    const long long key = wave == 0 ? base : base + m;
    int lo = 0, hi = n_mark;                             // entries below lo are < key, from hi on >= key
    while (lo < hi) {
      const int stride = (hi - lo + 63) / 64, at = lo + lane * stride;
      const unsigned long long ge = __ballot(at >= hi || list[min(at, n_mark - 1)] >= key);
      const int first = ge ? __ffsll((long long)ge) - 1 : 64;
      hi = first < 64 ? min(hi, lo + first * stride) : hi;
      if (first > 0) lo = lo + (first - 1) * stride + 1;
    }
    if (lane == 0) s_j[wave] = hi;
  }
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) s_sc[j * kSelThreads + tid] = x[j];
  __syncthreads();
  for (int j = s_j[0] + tid; j < s_j[1]; j += kSelThreads) {
    const long long at = list[j] - base;
    if (at >= 0 && at < m) s_sc[at] = INFINITY;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    const int i = j * kSelThreads + tid;
    if (i < m) {
      const float v = s_sc[i];
      lifted[(size_t)unit * n + base + i] = v;
      if (pool_hist) atomicAdd(&s_hist[__float_as_uint(v) >> 21], 1u);
    }
  }
  if (!pool_hist) return;
  __syncthreads();
  uint32_t* out = pool_hist + (size_t)(unit / Hkv) * 3 * kSelBins;
  for (int i = tid; i < kSelBins; i += kSelThreads) {
    const uint32_t c = s_hist[i];
    if (c) atomicAdd(&out[i], c);
  }
}

hipError_t launch_lift(const Dims& d, const float* scores, const int32_t* top, int64_t n, int64_t n_mark, float* lifted,
                       uint32_t* pool_hist, hipStream_t st) {
  const dim3 grid(d.units(), (unsigned)((n + kSelBlock - 1) / kSelBlock));
  k_lift<<<grid, kSelThreads, 0, st>>>(scores, top, n, (int)n_mark, d.Hkv, lifted, pool_hist);
  return hipGetLastError();
}

// kSplitChunks workgroups per (sequence, head): the head's stretch of the pooled ascending list is
// found by two binary searches (every workgroup repeats them: forty loads), then copied with the
// head's offset taken off, each workgroup one slice of it.
constexpr int kSplitChunks = 32;
__global__ __launch_bounds__(256) void k_split_pooled(const int32_t* __restrict__ flat, int H, long long n,
                                                      long long n_keep, int32_t* __restrict__ idx,
                                                      int32_t* __restrict__ lengths) {
  const int b = blockIdx.x / H, h = blockIdx.x % H, chunk = blockIdx.y;
  const long long total = (long long)H * n_keep;
  const int32_t* f = flat + (size_t)b * total;
  auto lower = [&](long long key) {
    long long lo = 0, hi = total;
    while (lo < hi) {
      const long long mid = (lo + hi) >> 1;
      if (f[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
  };
  const long long lo = lower((long long)h * n), hi = lower((long long)(h + 1) * n);
  if (threadIdx.x == 0 && chunk == 0) lengths[blockIdx.x] = (int32_t)(hi - lo);
  int32_t* out = idx + (size_t)blockIdx.x * n;
  const long long per = (hi - lo + kSplitChunks - 1) / kSplitChunks;
  const long long j0 = lo + chunk * per, j1 = min(hi, j0 + per);
  for (long long j = j0 + threadIdx.x; j < j1; j += 256) out[j - lo] = f[j] - (int32_t)(h * n);
}

hipError_t launch_split_pooled(const int32_t* flat, int B, int H, int64_t n, int64_t n_keep, int32_t* idx,
                               int32_t* lengths, hipStream_t st) {
  k_split_pooled<<<dim3(B * H, kSplitChunks), 256, 0, st>>>(flat, H, n, n_keep, idx, lengths);
  return hipGetLastError();
}

}  // namespace ea

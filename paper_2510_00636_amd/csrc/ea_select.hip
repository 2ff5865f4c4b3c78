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
#include "ea_lse.h"

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

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
#define EA_SCAN_STEP(CTRL, ROWS)                                                       \
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, ROWS == 0xf)
  EA_SCAN_STEP(0x111, 0xf);                          // lanes 1, 2, 4 and 8 to the left in the row of 16
  EA_SCAN_STEP(0x112, 0xf);
  EA_SCAN_STEP(0x114, 0xf);
  EA_SCAN_STEP(0x118, 0xf);
  EA_SCAN_STEP(0x142, 0xa);                          // the last lane of the row in front, into rows 1 and 3
  EA_SCAN_STEP(0x143, 0xc);                          // lane 31, into rows 2 and 3
#undef EA_SCAN_STEP
  return x;
}

// The digit search.  Bin b (counting down from the top) with  count(bins > b) < target <= count(bins >= b), and
// rem = target - count(bins > b), by all NT threads of a workgroup: thread t holds the PER bins below nbins - t * PER,
// the lowest of them first.  One barrier between the wavefronts' sums and one in front of the result.  (By one wavefront,
// 32 bins per lane, it took some 300 instructions in a row, 64 lines of cache or 64 lanes on the same banks of LDS per load,
// and as much code again for every digit: k_sel_hist 4.5 to 4.9 -> 3.9 us at 8 units x 20011, k_sel_emit 12.1 -> 9.8 at 8 x
// 131072.)
template <int NT>
struct BinSearch {
  uint32_t sum[NT / 64];
  uint32_t bin, rem;
};
template <int NT, int PER>
__device__ __forceinline__ void find_bin(BinSearch<NT>& s, const uint32_t (&cnt)[PER], uint32_t target, uint32_t* bin,
                                         uint32_t* rem) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) sum += cnt[j];
  const uint32_t incl = wave_scan(sum);
  if (lane == 63) s.sum[wave] = incl;
  if (tid == 0) { s.bin = 0u; s.rem = 0u; }          // (counters that do not add up to the target: as good as any)
  __syncthreads();
  uint32_t front = 0;                                // in the wavefronts in front of this one
  if constexpr (NT > 256) {
    front = wave_scan(lane < wave ? s.sum[lane % (NT / 64)] : 0u);
    front = __builtin_amdgcn_readlane(front, 63);
  } else {
#pragma unroll
    for (int w = 0; w < NT / 64 - 1; ++w) front += w < wave ? s.sum[w] : 0u;
  }
  front += incl - sum;                               // and in the lanes
  uint32_t r = target - front;
  if (front < target && r <= sum) {
    uint32_t b = PER - 1;
#pragma unroll
    for (int j = PER - 1; j >= 1; --j)
      if (b == (uint32_t)j && r > cnt[j]) { r -= cnt[j]; --b; }
    s.bin = (uint32_t)((NT - 1 - tid) * PER) + b;
    s.rem = r;
  }
  __syncthreads();
  *bin = s.bin;
  *rem = s.rem;
}
// this thread's bins of a histogram of NT * PER
template <int NT, int PER>
__device__ __forceinline__ void load_bins(const uint32_t* hist, uint32_t (&cnt)[PER]) {
  const uint32_t* p = hist + (NT - 1 - (int)threadIdx.x) * PER;
  if constexpr (PER % 4 == 0) {
#pragma unroll
    for (int j = 0; j < PER / 4; ++j) {
      const uint4 v = reinterpret_cast<const uint4*>(p)[j];
      cnt[4 * j] = v.x; cnt[4 * j + 1] = v.y; cnt[4 * j + 2] = v.z; cnt[4 * j + 3] = v.w;
    }
  } else if constexpr (PER == 2) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    cnt[0] = v.x; cnt[1] = v.y;
  } else {
#pragma unroll
    for (int j = 0; j < PER; ++j) cnt[j] = p[j];
  }
}

// The kept ones among 64 consecutive scores, a lane each: above T, or at T and one of the first q such of the head, to
// out[pos ..] in order.  pos, eq_before (scores at T in front): the same in all lanes, taken past the row.  Rows with a score
// at T are few, and the others are spared the counting of them.
// (Lane masks as numbers: kept as conditions they went through vector registers.)
__device__ __forceinline__ void emit_row(unsigned long long in, uint32_t u, uint32_t T, uint32_t q, uint32_t& pos,
                                         uint32_t& eq_before, int32_t* out, uint32_t n_keep, int at) {
  unsigned long long mask = __ballot(u > T) & in;
  const unsigned long long ties = __ballot(u == T) & in;
  if (ties != 0ull) {
    const uint32_t nth = eq_before + __builtin_amdgcn_mbcnt_hi((uint32_t)(ties >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ties, 0u));
    mask |= __ballot(nth < q) & ties;
    eq_before += __popcll(ties);
  }
  const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, pos));
  if (__builtin_amdgcn_inverse_ballot_w64(mask) && to < n_keep) out[to] = at;
  pos += __popcll(mask);
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

// Digits fixed by the histogram passes before pass P: every workgroup searches for them again (cheaper than a
// launch), the histograms requested ahead of everything else.
template <int P>
struct Digits {
  uint32_t c0[P >= 1 ? kSelBins / kSelThreads : 1], c1[P >= 2 ? kSelBins / kSelThreads : 1], c2[P >= 3 ? kSelBins / 2 / kSelThreads : 1];
  __device__ __forceinline__ void load(const SelArgs& a, int unit) {
    const uint32_t* h = a.hist + (size_t)unit * 3 * kSelBins;
    if constexpr (P >= 1) load_bins<kSelThreads>(h, c0);
    if constexpr (P >= 2) load_bins<kSelThreads>(h + kSelBins, c1);
    if constexpr (P >= 3) load_bins<kSelThreads>(h + 2 * kSelBins, c2);
  }
  // prefix: the digits' bits; rem: what is left of n_keep among the scores that start with them
  __device__ __forceinline__ void find(BinSearch<kSelThreads>* s, uint32_t n_keep, uint32_t* prefix, uint32_t* rem) {
    uint32_t pre = 0, r = n_keep, b;
    if constexpr (P >= 1) { find_bin<kSelThreads>(s[0], c0, r, &b, &r); pre = b; }
    if constexpr (P >= 2) { find_bin<kSelThreads>(s[1], c1, r, &b, &r); pre = (pre << 11) | b; }
    if constexpr (P >= 3) { find_bin<kSelThreads>(s[2], c2, r, &b, &r); pre = (pre << 10) | b; }
    *prefix = pre;
    *rem = r;
  }
};

template <int P>
__global__ __launch_bounds__(kSelThreads) void k_sel_hist(SelArgs a) {
  __shared__ uint32_t s_hist[kSelBins];
  __shared__ BinSearch<kSelThreads> s_find[P + 1];
  const int tid = threadIdx.x, unit = blockIdx.x;
  Digits<P> dig;
  dig.load(a, unit);
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  const long long base = (long long)blockIdx.y * kSelBlock;
  // All loads first and none under a condition (indices past the end are clamped): a load inside
  // "if (i < n)" is followed by a wait for it, one memory round trip per score.
  uint32_t uu[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) uu[j] = sc[min(base + j * kSelThreads + tid, a.n - 1)];
  for (int i = tid; i < kSelBins; i += kSelThreads) s_hist[i] = 0;
  uint32_t prefix = 0, rem;
  dig.find(s_find, a.n_keep, &prefix, &rem);
  if (P == 0) __syncthreads();                       // (else the search's barriers lie behind the zeros)
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
  __shared__ BinSearch<kSelThreads> s_find[3];
  __shared__ uint32_t s_w[2][W];
  __shared__ uint32_t s_front[3];
  __shared__ uint32_t s_blk;
  const int tid = threadIdx.x, lane = tid & 63, unit = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) s_blk = atomicAdd(a.hist + ((size_t)unit * 3 + 2) * kSelBins + kEmitTicket, 1u);
  Digits<3> dig;
  dig.load(a, unit);
  __syncthreads();
  const int blk = __builtin_amdgcn_readfirstlane((int)s_blk);
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  const long long base = (long long)blk * kSelBlock + wave * (kSelBlock / W) + lane;    // of u[0]; u[j]: 64 j further
  uint32_t u[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) u[j] = sc[min(base + 64 * j, a.n - 1)];
  // which lanes' u[j] are scores of the head, as a number
  const long long left = a.n - ((long long)blk * kSelBlock + wave * (kSelBlock / W));
  auto inside = [&](int j) -> unsigned long long {
    const int m = (int)min(max(left - 64 * j, 0ll), 64ll);
    return m >= 64 ? ~0ull : (1ull << m) - 1ull;
  };
  uint32_t T, q;
  dig.find(s_find, a.n_keep, &T, &q);
  T = __builtin_amdgcn_readfirstlane(T);
  q = __builtin_amdgcn_readfirstlane(q);
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    gt += __popcll(__ballot(u[j] > T) & inside(j));
    eq += __popcll(__ballot(u[j] == T) & inside(j));
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
  pos = __builtin_amdgcn_readfirstlane(pos);
  eq_before = __builtin_amdgcn_readfirstlane(eq_before);
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) emit_row(inside(j), u[j], T, q, pos, eq_before, out, a.n_keep, (int)(base + 64 * j));
}

// ---------------------------------------------------------------------------------------
// Short heads (n <= kSelSmallMax): one workgroup of 16 wavefronts per unit does all of the above in one
// launch.  The scores are read once and stay in registers, up to PER per thread: wavefront w holds 64 R
// consecutive positions (R = ceil(n / 1024)), lane l the l-th of each row of 64, so that positions are
// counted with ballots and the kept ones leave in order.  Same result as the multi-launch path, bit for bit.
//
// What bounds it is the issue of instructions on the one CU that a head gets (four wavefronts per SIMD), then the chain of
// three histograms.  So lane masks, counts and positions of whole rows are scalar, a row without a score at the threshold is
// spared the counting of ties, and the digits are searched for by all threads: 1000 -> 670 vector instructions per
// wavefront, 8 units x 16384 12.0 -> 8.5 us, 192 x 4608 10.3 -> 8.0, 2 x 1024 6.1 -> 4.5.  Scores crowd into a few bins of
// the first digit (four bins per factor of two), and LDS atomics on one address go one by one, so that digit's histogram is
// kept in four copies, copies of a bin in neighbouring banks.
constexpr int kSelSmallThreads = 1024;
constexpr int kSelCopies = 4;

// position of u[0] of a thread, and the rows per wavefront
struct SmallShare { int rows, base; };
__device__ __forceinline__ SmallShare small_share(int n) {
  const int rows = (n + kSelSmallThreads - 1) / kSelSmallThreads;
  return SmallShare{rows, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) * 64 * rows + ((int)threadIdx.x & 63)};
}

// The selection out of the registers of the workgroup, to out[0 .. n_keep).  HIST0: the caller's first histogram; else s_hist0 is
// LDS for it, kSelBins * kSelCopies words that are free again (`out` may be there) when the positions are written.
template <int PER, bool HIST0>
__device__ __forceinline__ void select_unit(const SelArgs& a, int unit, const uint32_t (&u)[PER], uint32_t* s_hist0, int32_t* out) {
  constexpr int NT = kSelSmallThreads;
  __shared__ __align__(16) uint32_t s_hist1[kSelBins], s_hist2[kSelBins / 2];
  __shared__ BinSearch<NT> s_find[3];
  __shared__ uint32_t s_w[2][NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, n = (int)a.n;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows = small_share(n).rows, base = small_share(n).base;
  uint32_t c0[kSelBins / NT], c1[kSelBins / NT], c2[kSelBins / 2 / NT];
  if (HIST0) load_bins<NT>(a.hist + (size_t)unit * 3 * kSelBins, c0);   // the caller's first histogram
  // Which lanes' u[it] are scores of the head and of this wavefront's share, as a number.  (What is the same for all lanes is
  // kept out of the vector instructions: on the one CU that a head gets, their number is what takes the time.)
  const int left = __builtin_amdgcn_readfirstlane(min(max(n - wave * 64 * rows, 0), 64 * rows));
  auto inside = [&](int it) -> unsigned long long {
    const int m = left - 64 * it;
    return m >= 64 ? ~0ull : m > 0 ? (1ull << m) - 1ull : 0ull;
  };
  if (!HIST0)
    for (int i = tid; i < kSelBins * kSelCopies; i += NT) s_hist0[i] = 0;
  for (int i = tid; i < kSelBins; i += NT) s_hist1[i] = 0;
  if (tid < kSelBins / 2) s_hist2[tid] = 0;

  uint32_t T, q, bin;                             // threshold pattern so far, what is left to keep among the scores that start with it
  bool bad = false;
  if (!HIST0) {
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      if (!__builtin_amdgcn_inverse_ballot_w64(inside(it))) continue;
      atomicAdd(&s_hist0[(u[it] >> 21) * kSelCopies + (lane & (kSelCopies - 1))], 1u);
      bad |= u[it] > 0x7f800000u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSelBins / NT; ++j) {     // the copies of every bin
      const uint4 c = reinterpret_cast<const uint4*>(s_hist0)[(NT - 1 - tid) * (kSelBins / NT) + j];
      c0[j] = c.x + c.y + c.z + c.w;
    }
  }
  find_bin<NT>(s_find[0], c0, a.n_keep, &T, &q);  // (its barriers lie behind the zeros)
#pragma unroll
  for (int it = 0; it < PER; ++it)
    if (__builtin_amdgcn_inverse_ballot_w64(__ballot((u[it] >> 21) == T) & inside(it))) atomicAdd(&s_hist1[(u[it] >> 10) & 2047u], 1u);
  __syncthreads();
  load_bins<NT>(s_hist1, c1);
  find_bin<NT>(s_find[1], c1, q, &bin, &q);
  T = (T << 11) | bin;
#pragma unroll
  for (int it = 0; it < PER; ++it)
    if (__builtin_amdgcn_inverse_ballot_w64(__ballot((u[it] >> 10) == T) & inside(it))) atomicAdd(&s_hist2[u[it] & 1023u], 1u);
  __syncthreads();
  load_bins<NT>(s_hist2, c2);
  find_bin<NT>(s_find[2], c2, q, &bin, &q);
  T = (T << 10) | bin;
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(a.status, kStatusBadScore);
  // T: threshold pattern, q: ties at T to keep

  T = __builtin_amdgcn_readfirstlane(T);
  q = __builtin_amdgcn_readfirstlane(q);
  // scores above T and at T per wavefront, then what lies in front of this wavefront
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    gt += __popcll(__ballot(u[it] > T) & inside(it));
    eq += __popcll(__ballot(u[it] == T) & inside(it));
  }
  if (lane == 0) { s_w[0][wave] = gt; s_w[1][wave] = eq; }
  __syncthreads();
  uint32_t pos = 0, eq_before = 0;
  for (int w = 0; w < wave; ++w) { pos += s_w[0][w]; eq_before += s_w[1][w]; }
  pos = __builtin_amdgcn_readfirstlane(pos + (eq_before < q ? eq_before : q));
  eq_before = __builtin_amdgcn_readfirstlane(eq_before);
#pragma unroll
  for (int it = 0; it < PER; ++it) emit_row(inside(it), u[it], T, q, pos, eq_before, out, a.n_keep, base + 64 * it);
}

template <int PER, bool HIST0>
__global__ __launch_bounds__(kSelSmallThreads) void k_sel_small(SelArgs a) {
  const SmallShare x = small_share((int)a.n);
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)blockIdx.x * a.n;
  __shared__ __align__(16) uint32_t s_hist0[HIST0 ? 1 : kSelBins * kSelCopies];
  uint32_t u[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) u[it] = sc[min(x.base + 64 * min(it, x.rows - 1), (int)a.n - 1)];
  select_unit<PER, HIST0>(a, blockIdx.x, u, s_hist0, a.idx + (size_t)blockIdx.x * a.n_keep);
}

// The finalize pass of a unit (k_finalize, the same numbers) in front of its selection.
template <typename LT, int PER>
__global__ __launch_bounds__(kSelSmallThreads) void k_finish_select(SelArgs a, const LT* __restrict__ logits,
                                                                    const float* __restrict__ vnorm,
                                                                    const typename LT2<LT>::type* __restrict__ part, int G,
                                                                    int npart, float eps, float* __restrict__ scores) {
  constexpr int NH = 4;                                  // heads' logits requested together
  __shared__ LT s_lse[64];
  const int lane = threadIdx.x & 63, unit = blockIdx.x, n = (int)a.n;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const SmallShare x = small_share(n);
  int at[PER];
  float vn[PER];
  LT acc[PER], lv[NH][PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    at[it] = min(x.base + 64 * min(it, x.rows - 1), n - 1);
    vn[it] = vnorm[(size_t)unit * n + at[it]];
    acc[it] = 0;
  }
  auto fetch = [&](int g0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NH; ++j)
#pragma unroll
      for (int it = 0; it < PER; ++it) lv[j][it] = logits[((size_t)unit * G + min(g0 + j, G - 1)) * n + at[it]];
  };
  fetch(0);
  for (int g = wave; g < G; g += kSelSmallThreads / 64) {
    const LT v = wave_lse<LT>(part + ((size_t)unit * G + g) * npart, npart, lane);
    if (lane == 0) s_lse[g] = v;
  }
  __syncthreads();
  for (int g0 = 0; g0 < G; g0 += NH) {
    if (g0 > 0) fetch(g0);
#pragma unroll
    for (int j = 0; j < NH; ++j) {
      if (g0 + j >= G) break;
      const LT lse = s_lse[g0 + j];
#pragma unroll
      for (int it = 0; it < PER; ++it) acc[it] += ea_exp(lv[j][it] - lse);
    }
  }
  const LT invG = (LT)1 / (LT)G;
  uint32_t u[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const float sc = (float)((acc[it] * invG + (LT)eps) * (LT)vn[it]);
    u[it] = __float_as_uint(sc);
    scores[(size_t)unit * n + at[it]] = sc;              // (rows past the share's end: its last one, or the head's, again)
  }
  __shared__ __align__(16) uint32_t s_hist0[kSelBins * kSelCopies];
  select_unit<PER, false>(a, unit, u, s_hist0, a.idx + (size_t)unit * a.n_keep);
}

hipError_t launch_finish_select(const Dims& d, int64_t n, const void* logits, int logits_f64, const float* vnorm, const void* part,
                                int npart, float* scores, const KeepOut& sel, uint32_t* hist, hipStream_t st) {
  SelArgs a = {};
  a.status = hist + 2 * kSelBins + kStatusSlot;
  a.n = n;
  a.n_keep = (uint32_t)sel.n_keep;
  a.idx = sel.idx;
  static_assert(kFinishMax <= 5 * kSelSmallThreads && kFinishMaxF32 <= 4 * kSelSmallThreads, "scores per thread");
#define EA_FINISH(LT, LT2T, PP) \
  k_finish_select<LT, PP><<<d.units(), kSelSmallThreads, 0, st>>>(a, (const LT*)logits, vnorm, (const LT2T*)part, d.G, npart, d.eps, scores)
  switch ((n + kSelSmallThreads - 1) / kSelSmallThreads * 2 + (logits_f64 ? 1 : 0)) {      // (a row too many costs 6 % of the pass)
    case 2: EA_FINISH(float, float2, 1); break;
    case 4: EA_FINISH(float, float2, 2); break;
    case 6: EA_FINISH(float, float2, 3); break;
    case 8: EA_FINISH(float, float2, 4); break;
    case 10: EA_FINISH(float, float2, 5); break;
    case 3: EA_FINISH(double, double2, 1); break;
    case 5: EA_FINISH(double, double2, 2); break;
    case 7: EA_FINISH(double, double2, 3); break;
    case 9: EA_FINISH(double, double2, 4); break;
    default: return hipErrorInvalidValue;
  }
#undef EA_FINISH
  return hipGetLastError();
}

hipError_t launch_select(const Dims& d, const float* scores, int64_t n, int64_t n_keep, int32_t* idx,
                         uint32_t* hist, uint32_t* blk, bool hist0_done, hipStream_t st) {
  SelArgs a;
  a.status = hist + 2 * kSelBins + kStatusSlot;
  a.scores = scores;
  a.n = n;
  a.n_keep = (uint32_t)n_keep;
  a.hist = hist;
  a.blk = blk;
  a.idx = idx;
  a.nblk = (int)((n + kSelBlock - 1) / kSelBlock);
  static_assert(kSelSmallMax <= 24 * kSelSmallThreads, "scores per thread");
  if (select_in_one_launch(n)) {
#define EA_SMALL(PP)                                                                                  \
  if (hist0_done) k_sel_small<PP, true><<<d.units(), kSelSmallThreads, 0, st>>>(a);                   \
  else k_sel_small<PP, false><<<d.units(), kSelSmallThreads, 0, st>>>(a)
    if (n <= 4 * kSelSmallThreads) { EA_SMALL(4); }
    else if (n <= 8 * kSelSmallThreads) { EA_SMALL(8); }
    else if (n <= 16 * kSelSmallThreads) { EA_SMALL(16); }
    else { EA_SMALL(24); }
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
// Head-adaptive budgets (Sec. 2.2, "Head-Adaptive Compression"): every KV head keeps its own `floor` best scores, and what
// is left of the layer's budget goes to the best of all the others, wherever they are.
//
// Both searches walk down the digits side by side, and neither list is ever written down: of a head's scores those above
// its floor's threshold are out of the pool, so its part in a pooled histogram is
//   where the pool's prefix lies below the head's:  all its scores with that prefix (counted into the pool's histogram),
//   where they are the same:                        the head's own histogram, cut off at the head's next digit,
//   where it lies above:                            nothing,
// and the first one is the sum of the heads' first histograms, cut off.  The emit pass then writes every head's list
// straight away: with T the pool's threshold and T_h the floor's it keeps what lies above the lower of them, and of
// the scores at it the first ones: the floor's share where that is T_h, the pool's where it is T, which depends on the
// scores at T in the heads in front.
// As two selections, with a copy of the scores in between (the floor's lifted to infinity) and a pooled list that was
// cut into the heads' afterwards, it took eight launches and 57 us behind the finalize pass at 8 heads x 50001 with a
// quarter of the budget by head; now four and 25 (whole pass 236 -> 203 us).  What bounds it now is the latency of the
// rounds through the histograms.
// A head's digits are found once, behind its counts.  With every block of the next launch finding those of all the heads that
// share the pool's prefix (most of them where the floors are close to the budget or the heads of one scale), select_adaptive took
// 88 us over 32 heads x 9000 of equal scale with nine tenths of the budget by head and 928 over 512 x 9000: now 34 and 156.
// (Two selections took 55 and 205.)
struct AdaptArgs {
  const float* scores;
  long long n;
  uint32_t floor, rest;   // scores that every head keeps, and that the layer keeps besides
  uint32_t* hist;         // [units][3][2048], the first one filled; see kPrefixSlot
  uint32_t* pool;         // [B][3][2048], zero at launch
  uint2* own;             // [units]: (threshold, rest of the floor) of a head, side by side: every block may read those in front
  uint32_t* blk;          // [units][nblk], zero at launch: kEmitSeen | kEmitPool | count == threshold << 13 | count > threshold
  int32_t* idx;           // [units][n]
  int32_t* lengths;       // [units]
  int B, H, nblk;
  uint32_t* status;
};
// Free words of a third histogram: (prefix, rest) after each of the first two digits, the unit's or the pool's, and how many of
// the head's blocks have counted the second and the third.  The former on a line without counters (the score kernel's are done
// with): next to the emit pass's, whose blocks all read them, select_adaptive
// took 199 us over 512 heads x 9000, and 137 so.
constexpr int kPrefixSlot = 1088, kCountedSlot = 1040;
constexpr uint32_t kNoPrefix = ~0u;        // no floor: above every prefix; nothing besides the floor: the same for the pool
constexpr uint32_t kEmitPool = 1u << 30;

__device__ __forceinline__ uint32_t* adapt_slot(uint32_t* hist, int level) { return hist + 2 * kSelBins + kPrefixSlot + 2 * level; }

// Digit P of a head by a workgroup, its histogram in LDS or (nullptr) in memory: the digit, and the head's part to the pool's histogram if
// it shares the pool's prefix: what lies below the bin of its floor's threshold, and of that bin all but the `rem` best.
template <int P>
__device__ __forceinline__ void adapt_cut(const AdaptArgs& a, int unit, uint32_t* hist, uint32_t* pool_hist, uint32_t prefix, uint32_t rem,
                                          bool pooled, const uint32_t* whole, BinSearch<kSelThreads>& s) {
  constexpr int PER = (P == 2 ? kSelBins / 2 : kSelBins) / kSelThreads, BITS = P == 2 ? 10 : 11;
  const uint32_t lo = (uint32_t)((kSelThreads - 1 - (int)threadIdx.x) * PER);
  uint32_t cnt[PER], bin = kNoPrefix;
#pragma unroll
  for (int i = 0; i < PER; ++i)                      // (P > 0: counted in this launch)
    cnt[i] = P == 0 ? hist[lo + i] : whole ? whole[lo + i] : __hip_atomic_load(&hist[P * kSelBins + lo + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (a.floor) find_bin<kSelThreads>(s, cnt, rem, &bin, &rem);
  if (threadIdx.x == 0) {
    const uint32_t pre = a.floor ? (prefix << BITS) | bin : kNoPrefix;
    if (P == 2) {
      a.own[unit] = make_uint2(pre, rem);
    } else {
      adapt_slot(hist, P)[0] = pre;
      adapt_slot(hist, P)[1] = rem;
    }
  }
  if (!pooled) return;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const uint32_t part = lo + i < bin ? cnt[i] : lo + i == bin ? cnt[i] - rem : 0u;
    if (part) atomicAdd(&pool_hist[P * kSelBins + lo + i], part);
  }
}

// The first digits, by a workgroup per head.
__global__ __launch_bounds__(kSelThreads) void k_adapt_first(AdaptArgs a) {
  __shared__ BinSearch<kSelThreads> s;
  adapt_cut<0>(a, blockIdx.x, a.hist + (size_t)blockIdx.x * 3 * kSelBins, a.pool + (size_t)(blockIdx.x / a.H) * 3 * kSelBins, 0u, a.floor, true, nullptr, s);
}

// Second (P == 1) and third histogram of the heads, where their floors' thresholds are, and of the pool.  The last block of a
// head that has counted finds the head's digit and adds its part to the pool's histogram.
template <int P>
__global__ __launch_bounds__(kSelThreads) void k_adapt_hist(AdaptArgs a) {
  constexpr int SHIFT = P == 1 ? 21 : 10;
  __shared__ uint32_t s_own[kSelBins], s_pool[kSelBins];
  __shared__ BinSearch<kSelThreads> s;
  __shared__ uint32_t s_counted;
  const int tid = threadIdx.x, unit = blockIdx.x, b = unit / a.H, h = unit - b * a.H;
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  const long long base = (long long)blockIdx.y * kSelBlock;
  uint32_t* hist = a.hist + (size_t)unit * 3 * kSelBins;
  uint32_t* pool_hist = a.pool + (size_t)b * 3 * kSelBins;
  uint32_t cnt[kSelBins / kSelThreads];
  load_bins<kSelThreads>(pool_hist + (P - 1) * kSelBins, cnt);
  uint32_t own = kNoPrefix, own_rem = 0u, pool = 0u, pool_rem = a.rest;
  if (a.floor) { own = adapt_slot(hist, P - 1)[0]; own_rem = adapt_slot(hist, P - 1)[1]; }
  if (P == 2) { pool = adapt_slot(pool_hist, 0)[0]; pool_rem = adapt_slot(pool_hist, 0)[1]; }
  uint32_t u[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) u[j] = sc[min(base + j * kSelThreads + tid, a.n - 1)];
  for (int i = tid; i < kSelBins; i += kSelThreads) s_own[i] = s_pool[i] = 0;
  if (a.rest) {
    uint32_t bin;
    find_bin<kSelThreads>(s, cnt, pool_rem, &bin, &pool_rem);
    pool = (pool << 11) | bin;
  } else {
    pool = kNoPrefix;
  }
  if (tid == 0 && blockIdx.y == 0 && h == 0) {           // for the launches behind this one
    adapt_slot(pool_hist, P - 1)[0] = pool;
    adapt_slot(pool_hist, P - 1)[1] = pool_rem;
  }
  __syncthreads();
  const bool counted = a.floor != 0u, pooled = a.rest != 0u && own > pool;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    if (base + j * kSelThreads + tid < a.n) {
      const uint32_t digit = P == 1 ? (u[j] >> 10) & 2047u : u[j] & 1023u;
      if (counted && (u[j] >> SHIFT) == own) atomicAdd(&s_own[digit], 1u);
      if (pooled && (u[j] >> SHIFT) == pool) atomicAdd(&s_pool[digit], 1u);
    }
  }
  __syncthreads();
  for (int i = tid; i < kSelBins / P; i += kSelThreads) {
    const uint32_t c = s_own[i], d = s_pool[i];
    if (c && a.nblk > 1) atomicAdd(&hist[P * kSelBins + i], c);
    if (d) atomicAdd(&pool_hist[P * kSelBins + i], d);
  }
  if (!counted) return;
  const bool shared = a.rest != 0u && own == pool;
  if (a.nblk == 1) {
    adapt_cut<P>(a, unit, hist, pool_hist, own, own_rem, shared, s_own, s);
    return;
  }
  // Every thread waits for its own counts, which are atomics of the whole chip and in their place when they are acknowledged; then
  // the block's mark; and the last block reads past its caches.  (Fences of that reach write back and empty the dies' L2 for
  // every block: select_adaptive, 32 heads x 32768, half of the budget by head, 52 us
  // and 39.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) s_counted = atomicAdd(hist + 2 * kSelBins + kCountedSlot + P, 1u);
  __syncthreads();
  if (s_counted != (uint32_t)a.nblk - 1u) return;
  adapt_cut<P>(a, unit, hist, pool_hist, own, own_rem, shared, nullptr, s);
}

// The heads' lists and lengths, see k_sel_emit: blocks by ticket in the order of (head, block), waiting for lower ones only.
__global__ __launch_bounds__(kSelThreads) void k_adapt_emit(AdaptArgs a) {
  constexpr int W = kSelThreads / 64, U = 2;
  constexpr int PER = kSelBins / 2 / kSelThreads;
  __shared__ BinSearch<kSelThreads> s;
  __shared__ uint32_t s_w[2][W];
  __shared__ uint32_t s_front[4];
  __shared__ uint32_t s_blk, s_share;
  const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.x % a.B;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t* pool_hist = a.pool + (size_t)b * 3 * kSelBins;
  if (tid == 0) {
    s_blk = atomicAdd(pool_hist + 2 * kSelBins + kEmitTicket, 1u);
    s_share = 0u;
  }
  uint32_t cnt[PER];
  load_bins<kSelThreads>(pool_hist + 2 * kSelBins, cnt);
  uint32_t pool = adapt_slot(pool_hist, 1)[0], pool_rem = adapt_slot(pool_hist, 1)[1];
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane((int)s_blk);
  if (ticket >= a.H * a.nblk) return;           // (a counter that did not start at zero)
  const int h = ticket / a.nblk, blk = ticket - h * a.nblk, unit = b * a.H + h;
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)unit * a.n;
  const long long base = (long long)blk * kSelBlock + wave * (kSelBlock / W) + lane;    // of u[0]; u[j]: 64 j further
  uint32_t u[kSelPer];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) u[j] = sc[min(base + 64 * j, a.n - 1)];
  const long long left = a.n - ((long long)blk * kSelBlock + wave * (kSelBlock / W));
  auto inside = [&](int j) -> unsigned long long {
    const int m = (int)min(max(left - 64 * j, 0ll), 64ll);
    return m >= 64 ? ~0ull : (1ull << m) - 1ull;
  };
  uint32_t own = kNoPrefix, own_rem = 0u;
  const uint2* owns = a.own + (size_t)b * a.H;           // of the sequence's first head
  if (a.floor) { own = owns[h].x; own_rem = owns[h].y; }
  if (a.rest) {
    uint32_t bin;
    find_bin<kSelThreads>(s, cnt, pool_rem, &bin, &pool_rem);
    pool = (pool << 10) | bin;
    const uint32_t lo = (uint32_t)((kSelThreads - 1 - tid) * PER);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (lo + i == bin && cnt[i] != pool_rem) s_share = 1u;     // not all of the pool's scores at its threshold are kept
  } else {
    pool = kNoPrefix;
  }
  const uint32_t T = __builtin_amdgcn_readfirstlane(min(own, pool));
  const bool at_pool = a.rest != 0u && T == pool;
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    gt += __popcll(__ballot(u[j] > T) & inside(j));
    eq += __popcll(__ballot(u[j] == T) & inside(j));
  }
  if (lane == 0) { s_w[0][wave] = gt; s_w[1][wave] = eq; }
  __syncthreads();
  uint32_t* pub = a.blk + (size_t)b * a.H * a.nblk;
  if (tid == 0) {
    uint32_t g = 0, e = 0;
    for (int w = 0; w < W; ++w) { g += s_w[0][w]; e += s_w[1][w]; }
    __hip_atomic_store(&pub[ticket], kEmitSeen | (at_pool ? kEmitPool : 0u) | (e << 13) | g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // in the head's blocks in front of this one: above T and at T; in the heads in front: at the pool's threshold
  if (wave == 0) {
    uint32_t gf = 0, ef = 0, pf = 0;
    int spin = 0;
    const int own0 = h * a.nblk;
    // (without a tie to share out the heads in front do not matter)
    const bool share = at_pool && s_share != 0u;
    if (share && a.floor)                                // at the pool's threshold, but of the floors of the heads in front
      for (int g = lane; g < h; g += 64) pf -= owns[g].x == pool ? owns[g].y : 0u;
    for (int j0 = (share ? 0 : own0) + lane; j0 < ticket && spin < kEmitSpinLimit; j0 += U * 64) {
      uint32_t word[U];
#pragma unroll
      for (int y = 0; y < U; ++y)
        word[y] = j0 + 64 * y < ticket ? __hip_atomic_load(&pub[j0 + 64 * y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kEmitSeen;
#pragma unroll
      for (int y = 0; y < U; ++y) {
        while ((word[y] & kEmitSeen) == 0u && ++spin < kEmitSpinLimit) {
          __builtin_amdgcn_s_sleep(1);
          word[y] = __hip_atomic_load(&pub[j0 + 64 * y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint32_t e = (word[y] >> 13) & 0x1fffu;
        if (j0 + 64 * y >= own0) { gf += word[y] & 0x1fffu; ef += e; }
        else if (word[y] & kEmitPool) pf += e;
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) { gf += __shfl_xor(gf, o); ef += __shfl_xor(ef, o); pf += __shfl_xor(pf, o); }
    const bool ok = __ballot(spin >= kEmitSpinLimit) == 0ull;
    if (lane == 0) {
      s_front[0] = gf;
      s_front[1] = ef;
      s_front[2] = pf;
      s_front[3] = ok;
      if (!ok) atomicOr(a.status, kStatusCompactWait);
    }
  }
  __syncthreads();
  if (!s_front[3]) return;
  // scores at T to keep: the floor's, and the pool's that the heads in front have left
  uint32_t q = T == own ? own_rem : 0u;
  if (at_pool) q = s_share == 0u ? (uint32_t)a.n : q + (s_front[2] < pool_rem ? pool_rem - s_front[2] : 0u);
  q = __builtin_amdgcn_readfirstlane(q);
  uint32_t pos = s_front[0], eq_before = s_front[1];
  for (int w = 0; w < W; ++w) {
    if (w == wave) break;
    pos += s_w[0][w];
    eq_before += s_w[1][w];
  }
  pos = __builtin_amdgcn_readfirstlane(pos + min(eq_before, q));
  eq_before = __builtin_amdgcn_readfirstlane(eq_before);
  int32_t* out = a.idx + (size_t)unit * a.n;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) emit_row(inside(j), u[j], T, q, pos, eq_before, out, (uint32_t)a.n, (int)(base + 64 * j));
  if (blk == a.nblk - 1 && tid == kSelThreads - 1) a.lengths[unit] = (int32_t)pos;
}

// Short layers without a floor: the pooled list of a sequence by one workgroup, into LDS, and from there to the heads.
// (select_adaptive, us, with the launches above and with this: 8 heads x 64 20.6 and 9.7, x 1000 21.2 and 10.8, 8 sequences of
// them 21.3 and 11.2; compress_layer_adaptive, 8 x 64 40.0 and 29.5, x 1000 44.4 and 40.7.)
constexpr int kAdaptSmallMax = kSelBins * kSelCopies, kAdaptSmallHeads = 2047;
static_assert(kAdaptSmallMax <= 8 * kSelSmallThreads, "scores per thread");
template <int PER>
__global__ __launch_bounds__(kSelSmallThreads) void k_adapt_small(SelArgs a, int H, int n, int32_t* __restrict__ lengths) {
  __shared__ __align__(16) uint32_t s_list[kAdaptSmallMax];
  __shared__ int s_start[kAdaptSmallHeads + 1];          // of a head's part of the list
  const int tid = threadIdx.x, b = blockIdx.x, kept = (int)a.n_keep;
  const SmallShare x = small_share((int)a.n);
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(a.scores) + (size_t)b * a.n;
  uint32_t u[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) u[it] = sc[min(x.base + 64 * min(it, x.rows - 1), (int)a.n - 1)];
  const int* list = reinterpret_cast<const int*>(s_list);
  select_unit<PER, false>(a, b, u, s_list, reinterpret_cast<int32_t*>(s_list));
  __syncthreads();
  for (int j = tid; j < kept; j += kSelSmallThreads) {
    const int h = list[j] / n, before = j > 0 ? list[j - 1] / n : -1;
    for (int g = before + 1; g <= h; ++g) s_start[g] = j;
    if (j == kept - 1)
      for (int g = h + 1; g <= H; ++g) s_start[g] = kept;
  }
  __syncthreads();
  for (int j = tid; j < kept; j += kSelSmallThreads) {
    const int h = list[j] / n;
    a.idx[((size_t)b * H + h) * n + (j - s_start[h])] = list[j] - h * n;
  }
  for (int h = tid; h < H; h += kSelSmallThreads) lengths[(size_t)b * H + h] = s_start[h + 1] - s_start[h];
}

hipError_t launch_select_adaptive(const Dims& d, const float* scores, int64_t n, int64_t n_keep, int64_t floor, int32_t* idx,
                                  int32_t* lengths, uint32_t* hist, uint32_t* pool_hist, uint32_t* blk, uint2* own,
                                  bool hist0_done, hipStream_t st) {
  if (n_keep == 0) return launch_zero((uint32_t*)lengths, d.units(), st);
  const int nblk = (int)((n + kSelBlock - 1) / kSelBlock);
  if (floor == 0 && d.Hkv * n <= kAdaptSmallMax && d.Hkv <= kAdaptSmallHeads) {
    SelArgs f = {};
    f.scores = scores;
    f.n = d.Hkv * n;
    f.n_keep = (uint32_t)(d.Hkv * n_keep);
    f.idx = idx;
    f.status = hist + 2 * kSelBins + kStatusSlot;
    if (f.n <= 2 * kSelSmallThreads) k_adapt_small<2><<<d.B, kSelSmallThreads, 0, st>>>(f, d.Hkv, (int)n, lengths);
    else if (f.n <= 4 * kSelSmallThreads) k_adapt_small<4><<<d.B, kSelSmallThreads, 0, st>>>(f, d.Hkv, (int)n, lengths);
    else k_adapt_small<8><<<d.B, kSelSmallThreads, 0, st>>>(f, d.Hkv, (int)n, lengths);
    return hipGetLastError();
  }
  AdaptArgs a;
  a.scores = scores;
  a.n = n;
  a.floor = (uint32_t)floor;
  a.rest = (uint32_t)((n_keep - floor) * d.Hkv);
  a.hist = hist;
  a.pool = pool_hist;
  a.own = own;
  a.blk = blk;
  a.idx = idx;
  a.lengths = lengths;
  a.B = d.B;
  a.H = d.Hkv;
  a.nblk = nblk;
  a.status = hist + 2 * kSelBins + kStatusSlot;
  const dim3 grid(d.units(), nblk);
  if (!hist0_done) {
    SelArgs f = {};
    f.scores = scores;
    f.n = n;
    f.n_keep = (uint32_t)n_keep;
    f.hist = hist;
    f.nblk = nblk;
    f.status = a.status;
    k_sel_hist<0><<<grid, kSelThreads, 0, st>>>(f);
  }
  k_adapt_first<<<d.units(), kSelThreads, 0, st>>>(a);
  k_adapt_hist<1><<<grid, kSelThreads, 0, st>>>(a);
  k_adapt_hist<2><<<grid, kSelThreads, 0, st>>>(a);
  k_adapt_emit<<<(unsigned)(d.units() * nblk), kSelThreads, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace ea

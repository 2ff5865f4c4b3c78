// Launch wrappers of the HIP kernels (one translation unit per stage).
#pragma once
#include <hip/hip_runtime.h>

#include "ea_common.h"

namespace ea {

// pool row of logical row `row` of unit (b, h); a table entry outside the pool is clamped into it,
// so a malformed table can never send an access outside the allocation
__device__ __forceinline__ size_t paged_row(const PageMap& m, int unit, int row) {
  const int b = unit / m.hkv, h = unit - b * m.hkv;
  long long blk = m.table[(size_t)b * m.max_blocks + (row >> m.sh)];
  blk = blk < 0 ? 0 : (blk >= m.num_blocks ? m.num_blocks - 1 : blk);
  return ((size_t)(blk * m.hkv + h) << m.sh) + (size_t)(row & ((1 << m.sh) - 1));
}

// ea_stats.hip
hipError_t launch_rope_table(const Dims& d, const double* inv_freq, int64_t q_pos0, int64_t t_next,
                             int w, float2* tab, uint32_t* clear, size_t clear_words, hipStream_t st);
hipError_t launch_stats(const Dims& d, const void* q_win, int w, const float2* tab, float* mu,
                        float* sigma, hipStream_t st);
// the two of them in one for bf16 windows: mu and Sigma stay on the chip, the operands are those
// launch_prep_frags makes of what launch_stats writes.  At d = 64 a head is one workgroup's either
// way.  At d = 128 two workgroups that share a head each make the fragments of their own tiles of Sigma, in either score
// kernel's layout (whole pass, 8 heads x 16384, 94.5 -> 91.2 us with the
// histogram of the finalize pass, x 3000 57.3 -> 53.7; 32 x 9000 138 -> 132); from 192 heads on a head is one workgroup's
// (whole pass, n = 4608, w = 512, us, two workgroups per head and one: 32 query heads 45.8 and 49.6, 128 69.4 and 73.0, 160 82.4
// and 80.0, 192 89.5 and 89.0, 288 125 and 121, 512 181 and 167, 960 308 and 281).  At d = 256 Sigma's tiles stay apart.
// One workgroup: the same operands bit for bit.  Two: up to the power of two by which a head's M is scaled, which
// comes from sums of squares there and from Sigma's diagonal else; where the largest entry lies within rounding of a power
// of two they can differ by a factor of two, which moves only entries under 2^-26 of it (fp16 subnormals).
inline bool stats_makes_frags(const Dims& d) { return d.dtype == EA_BF16 && d.D <= 128; }
hipError_t launch_stats_frags(const Dims& d, const ScorePlan& sp, const void* q_win, int w, const float2* tab,
                              uint4* frags, float* post, hipStream_t st);
// mu == nullptr: zero means; sigma_shared: sigma holds one set of Hq heads for all sequences; clear /
// clear_words: words zeroed on the way (may be none)
hipError_t launch_prep_frags(const Dims& d, const ScorePlan& sp, const float* mu,
                             const float* sigma, uint4* frags, float* post, hipStream_t st, uint32_t* clear = nullptr,
                             size_t clear_words = 0, bool sigma_shared = false);

struct KeepOut { int32_t* idx; int64_t n_keep; };

// ea_score.hip
// tickets + unit * ticket_stride: the tile counters of the unit (ticket_word), zero at launch
hipError_t launch_score_mfma(const Dims& d, const ScorePlan& sp, const void* k, const void* v,
                             int64_t n, int64_t n_cap, const uint4* frags, const float* post,
                             float* logits, float* vnorm, float2* part, uint32_t* tickets,
                             int ticket_stride, hipStream_t st, const PageMap* pm = nullptr,
                             const float* kscale = nullptr, const float* vscale = nullptr, bool skip_v = false,
                             float* norms_out = nullptr);
// norms_out (register-fragment kernel, skip_v): sqrt(k^T M k) of every query head instead of the logits
// skip_v: V is neither read nor turned into norms (the caller weighs the pairs with norms of its own)
// kscale, vscale [units] (nullable): per-head scales of caches stored as e4m3 bytes (d.kv_fp8)
hipError_t launch_score_f32(const Dims& d, const void* k, const void* v, int64_t n, int64_t n_cap,
                            const float* mu, const float* sigma, double* logits, float* vnorm,
                            double2* part, int* nchunk_out, hipStream_t st);
// scores = (mean_g exp(l_g - lse_g) + eps) * vnorm; hist0 (nullable): first radix digit
// part: npart (max, sum exp) pairs per query head, each over a fixed block of keys; lse: scratch of
// one LT per query head (used when a head has too many partials to reduce inside pass B)
hipError_t launch_finalize(const Dims& d, int64_t n, const void* logits, int logits_f64,
                           const float* vnorm, const void* part, int npart, void* lse, float* scores,
                           uint32_t* hist0, hipStream_t st, const float* wnorm = nullptr, int lse_pass = 0,
                           const KeepOut* sel = nullptr);
// sel: the n_keep best pairs of every head are selected too, in the same launch (finish_in_one_launch; without wnorm; hist0:
// the histograms whose free words hold the status word)
// lse_pass: the partials do not exist yet; take them from the (fp32) logits, one per kLseBlock keys
// wnorm[i] = sqrt(max(2 d logits[i], 0)) for i < count
hipError_t launch_wnorm(const void* logits, int logits_f64, size_t count, int D, float* wnorm, hipStream_t st);

// ea_select.hip
// heads this short are selected by one workgroup per unit out of registers, in one launch (no global
// histograms: hist0 from the finalize pass is not needed then)
// (select + compact, one launch and three behind the clearing, us: 8 heads x 17000 30.3 and 34.5, x 20000 32.2 and 36.1,
// x 24000 35.7 and 39.1, x 32768 46.5 and 45.1; one x 20000 24.3 and 32; 48 x 20000 431 and 450)
constexpr int64_t kSelSmallMax = 24 * 1024;
inline bool select_in_one_launch(int64_t n) { return n <= kSelSmallMax; }
// Finalize and selection together, a workgroup per unit that keeps the scores in registers: a launch less, as long as what
// the finalize pass spreads over the chip is not too much for one CU (whole pass, us, two launches and one: 8 heads x 700
// 37.9 and 34.3, x 2500 44.2 and 41.7, x 5000 50.0 and 48.2, x 8192 55.8 and 56.5; 192 x 4608 319 and 314; 32 heads of G = 8 x
// 5000 103.3 and 102.0; fp32, 2 heads x 700 35.7 and 32.3, 4 heads of G = 7 x 3000 83.9 and 82.5, x 3900 95.0 and 96.2).
constexpr int64_t kFinishMax = 5 * 1024, kFinishMaxF32 = 4 * 1024;
inline bool finish_in_one_launch(const Dims& d, int64_t n) {
  return d.dtype == EA_BF16 ? n <= kFinishMax && n * d.G <= 40 * 1024 : n <= kFinishMaxF32 && n * d.G <= 21 * 1024;
}
hipError_t launch_finish_select(const Dims& d, int64_t n, const void* logits, int logits_f64, const float* vnorm, const void* part,
                                int npart, float* scores, const KeepOut& sel, uint32_t* hist, hipStream_t st);
hipError_t launch_select(const Dims& d, const float* scores, int64_t n, int64_t n_keep, int32_t* idx,
                         uint32_t* hist, uint32_t* blk, bool hist0_done, hipStream_t st);
hipError_t launch_zero(uint32_t* p, size_t count, hipStream_t st, uint32_t* extra = nullptr);

// ea_compact.hip
hipError_t launch_compact(const Dims& d, const void* k, const void* v, int64_t n, int64_t n_cap,
                          const int32_t* idx, int64_t n_keep, void* k_out, void* v_out,
                          uint32_t* flags, uint32_t* status, hipStream_t st,
                          const int32_t* lengths = nullptr, int64_t idx_stride = 0, const PageMap* pm = nullptr);
// pm != nullptr: k and v are block pools (in place only; n_cap unused)
// lengths != nullptr: unit u keeps lengths[u] <= n_keep rows, listed from idx + u * idx_stride

// ea_select.hip, head-adaptive budgets: ascending lists idx [units][n] and their lengths.  All of the scratch is zero at launch
// (hist0_done: but for the heads' first histograms, which are filled), but own, of one entry per unit, need not be
hipError_t launch_select_adaptive(const Dims& d, const float* scores, int64_t n, int64_t n_keep, int64_t floor, int32_t* idx,
                                  int32_t* lengths, uint32_t* hist, uint32_t* pool_hist, uint32_t* blk, uint2* own,
                                  bool hist0_done, hipStream_t st);

// order-free variant, in place: only the kept rows at or beyond n_keep move, into the evicted
// positions below it; perm (nullable) [units][n_keep] receives the source row of every position
hipError_t launch_compact_fill(const Dims& d, void* k, void* v, int64_t n, int64_t n_cap,
                               const int32_t* idx, int64_t n_keep, int32_t* perm, hipStream_t st,
                               const PageMap* pm = nullptr);

// ea_frontend.hip: q [B, Hq, w, d] fp32 = W_Q [Hq, d, dm] applied to hidden [B, w, dm] (dtype of d)
hipError_t launch_project(const Dims& d, const void* hidden, const void* wq, int w, int dm, float* q,
                          hipStream_t st);
// gram[g] = W_o^(g)^T W_o^(g) for w_o [Hq, dm, D] in the cache dtype
hipError_t launch_gram(const Dims& d, const void* w_o, int dm, float* gram, hipStream_t st);

// ea_baselines.hip: scorer = ea_scorer; scratch: units * kBaselineChunks * D floats
hipError_t launch_baseline(const Dims& d, int kind, const void* k, int64_t n, int64_t n_cap,
                           int64_t n_sink, float* scores, float* scratch, hipStream_t st);

int device_num_cu();

// hipFuncSetAttribute(MaxDynamicSharedMemorySize) once per (kernel, device) instead of on every
// launch: a static instance of this sits next to each launch of a kernel that needs more than
// 64 KiB of LDS.  Racing first calls at worst set the attribute twice.
struct LdsOptIn {
  size_t have[64] = {0};
  hipError_t ensure(const void* kern, size_t bytes) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
    if (dev >= 0 && have[dev] >= bytes) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess && dev >= 0) have[dev] = bytes;
    return e;
  }
};

}  // namespace ea

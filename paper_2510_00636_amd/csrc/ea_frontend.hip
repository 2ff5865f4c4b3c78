// Eq. 5 of the paper as printed starts from the hidden states: the queries are W_Q h (before the
// rotary embedding), so mean and covariance of the buffered hidden states, pushed through W_Q,
// are mean and covariance of the projected queries.  This file projects the buffer,
//     q[b][g][s][:] = W_Q[g] h[b][s][:]      (fp32 accumulation, fp32 result),
// and the statistics kernel then runs on q as un-rotated fp32 queries.  Forming the d_model x
// d_model covariance of the hidden states first, as the equation is written, would cost
// d_model / d times the arithmetic for the same result.
#include <hip/hip_runtime.h>

#include "ea_kernels.h"

namespace ea {

template <bool BF16>
__device__ __forceinline__ float load_elem(const void* p, size_t i) {
  if (BF16) return __uint_as_float((uint32_t)((const uint16_t*)p)[i] << 16);
  return ((const float*)p)[i];
}

// One workgroup = a 32 (samples) x 32 (channels) tile of one (sequence, query head); the d_model
// axis goes through LDS 32 at a time.  Thread (ty, tx) = (tid / 32, tid % 32) owns outputs
// (s0 + ty + 8 i, c0 + tx), i < 4.
template <bool BF16>
__global__ __launch_bounds__(256) void k_project(const void* __restrict__ hidden, const void* __restrict__ wq,
                                                 int w, int dm, int D, int Hq, float* __restrict__ q) {
  __shared__ float s_h[32][33], s_w[32][33];
  const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
  const int s0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
  const int b = blockIdx.z / Hq, g = blockIdx.z % Hq;
  const size_t hbase = (size_t)b * w * dm, wbase = (size_t)g * D * dm;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int m0 = 0; m0 < dm; m0 += 32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = ty + 8 * i, m = m0 + tx;
      const int s = min(s0 + row, w - 1);
      s_h[row][tx] = m < dm ? load_elem<BF16>(hidden, hbase + (size_t)s * dm + m) : 0.f;
      s_w[row][tx] = m < dm ? load_elem<BF16>(wq, wbase + (size_t)(c0 + row) * dm + m) : 0.f;
    }
    __syncthreads();
#pragma unroll 8
    for (int m = 0; m < 32; ++m) {
      const float wv = s_w[tx][m];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = fmaf(s_h[ty + 8 * i][m], wv, acc[i]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s = s0 + ty + 8 * i;
    if (s < w) q[(((size_t)b * Hq + g) * w + s) * D + c0 + tx] = acc[i];
  }
}

// The same projection on the matrix cores, for bf16 inputs whose rows are 16-byte aligned (d_model a
// multiple of 8): one workgroup = 16 MT samples x 32 channels with v_mfma_f32_16x16x32_bf16, blocks of 64 d_model entries
// at a time: lane (c, q) = (lane % 16, lane / 16) is an operand's 8 consecutive entries from 8 q on of its row c.  The NW
// wavefronts split the d_model axis into as many contiguous parts; the
// partial tiles meet in LDS and are added in wavefront order, so the result does not depend on timing.  bf16
// products are exact in fp32.
//
// What bounds it is the way of the rows from L2 into the workgroups.  A request that takes half of a line of 128 bytes costs
// as much as one for all of it, so a load takes eight rows' whole lines, and the operands come out of a patch of LDS that
// each wavefront has to itself.  Straight into the operand layout, four lanes on 64 bytes of a row, the loads came in at 20
// bytes per clock and CU: 128 x 4096 hidden states, 32 heads of 128 channels 27.8 -> 16 us; statistics and a short pass
// with them 69.2 -> 57.0, 512 x 4096 155 -> 99, 128 x 5120 and 40 heads 104 -> 70 (two us of each from the order of the
// workgroups).  The matrix W_Q alone takes 5.4 at the rate of a large read; more blocks in flight do not help.
typedef __bf16 pj_bf16x8 __attribute__((ext_vector_type(8)));
typedef float pj_floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t pj_u32x4 __attribute__((ext_vector_type(4)));

template <int MT, int NW>
__global__ __launch_bounds__(64 * NW) void k_project_mfma(const uint16_t* __restrict__ hidden,
                                                      const uint16_t* __restrict__ wq, int w, int dm, int D, int Hq,
                                                      float* __restrict__ q_out) {
  constexpr int ROWS = 16 * MT + 32, NL = ROWS / 8;       // of a block: samples, then channels; eight rows per load
  __shared__ union { pj_u32x4 patch[NW][ROWS * 8]; float acc[NW][16 * MT][32]; } s;
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tx = blockIdx.x, ty = blockIdx.y;
  if (gridDim.y % 8 == 0) {                                // the workgroups of the same channels on one die
    const int bid = blockIdx.y * gridDim.x + blockIdx.x;
    tx = bid / 8 % gridDim.x;
    ty = bid / (8 * gridDim.x) * 8 + bid % 8;
  }
  const int t0 = tx * 16 * MT, b = blockIdx.z;
  const int g = (ty * 32) / D, c0 = (ty * 32) % D;
  const int kq = (dm + 64 * NW - 1) / (64 * NW) * 64;     // entries per wavefront, a multiple of the block
  const int kbeg = min(dm, wave * kq), kend = min(dm, kbeg + kq);
  const int lrow = lane >> 3, lch = lane & 7;              // this lane's row and 16-byte chunk of a load
  const uint16_t* hb = hidden + (size_t)b * w * dm + lch * 8;
  const uint16_t* wb = wq + ((size_t)g * D + c0 + lrow) * dm + lch * 8;
  int arow[2 * MT];                                        // (at most 4096 samples of 2^20 entries; in entries / 8)
#pragma unroll
  for (int m = 0; m < 2 * MT; ++m) arow[m] = min(t0 + 8 * m + lrow, w - 1) * (dm / 8);
  pj_floatx4 acc[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[m][x] = pj_floatx4{0.f, 0.f, 0.f, 0.f};
  typedef pj_u32x4 Block[NL];
  auto row_at = [&](int i, int k0) __attribute__((always_inline)) {
    return i < 2 * MT ? hb + (size_t)arow[i < 2 * MT ? i : 0] * 8 + k0 : wb + (size_t)(8 * (i - 2 * MT)) * dm + k0;
  };
  auto fetch = [&](int k0, Block& f) __attribute__((always_inline)) {      // 64 entries, all inside the row
#pragma unroll
    for (int i = 0; i < NL; ++i) f[i] = *reinterpret_cast<const pj_u32x4*>(row_at(i, k0));
  };
  // into the wavefront's patch, the chunks of a row in an order of its own (row mod 8), so that neither the writes nor the
  // reads of the operands pile up in a bank
  pj_u32x4* patch = s.patch[wave];
  auto stage = [&](const Block& f) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NL; ++i) patch[(8 * i + lrow) * 8 + (lch ^ lrow)] = f[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      auto operand = [&](int row0) { return __builtin_bit_cast(pj_bf16x8, patch[(row0 + c) * 8 + ((4 * k + q) ^ (c & 7))]); };
      const pj_bf16x8 w0 = operand(16 * MT), w1 = operand(16 * MT + 16);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const pj_bf16x8 h = operand(16 * m);
        acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, w0, acc[m][0], 0, 0, 0);
        acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, w1, acc[m][1], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  const int full = (kend - kbeg) / 64;
  if (full > 0) {
    Block f0, f1;
    fetch(kbeg, f0);
    fetch(kbeg + 64 * min(1, full - 1), f1);
    for (int i = 0; i < full; i += 2) {                    // (past the last block: it once more, not used)
      stage(f0);
      fetch(kbeg + 64 * min(i + 2, full - 1), f0);
      multiply();
      if (i + 1 >= full) break;
      stage(f1);
      fetch(kbeg + 64 * min(i + 3, full - 1), f1);
      multiply();
    }
  }
  const int k0 = kbeg + 64 * full;
  if (k0 < kend) {                                         // d_model % 64 entries: a lane's eight lie inside the row or outside
    Block f;
    const pj_u32x4 zero4 = {0u, 0u, 0u, 0u};
    const bool in = k0 + 8 * lch < kend;
#pragma unroll
    for (int i = 0; i < NL; ++i) f[i] = in ? *reinterpret_cast<const pj_u32x4*>(row_at(i, k0)) : zero4;
    stage(f);
    multiply();
  }
  __syncthreads();
  // accumulator register v of lane (c, q) is the tile's entry (row 4 q + v, column c)
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v) s.acc[wave][16 * m + 4 * q + v][16 * x + c] = acc[m][x][v];
  __syncthreads();
  float* out = q_out + (((size_t)b * Hq + g) * w) * D + c0;
#pragma unroll
  for (int i = 0; i < 8 * MT / NW; ++i) {
    const int e = tid + 64 * NW * i, t = e >> 5, ch = e & 31;
    float sum = s.acc[0][t][ch];
#pragma unroll
    for (int p = 1; p < NW; ++p) sum += s.acc[p][t][ch];
    if (t0 + t < w) out[(size_t)(t0 + t) * D + ch] = sum;
  }
}

// Eq. 9 as printed weighs a pair by ||W_o v||.  With M_g = W_o^(g)^T W_o^(g) (d x d, from the d
// columns of W_o that query head g feeds) that norm is sqrt(v^T M_g v): a quadratic form of the
// same shape as Eq. 7's, so the score kernels evaluate it.  M_g depends on the weights only and is
// formed once per layer: one workgroup = a 32 x 32 tile of one head's M, the d_model axis through
// LDS 32 rows at a time, fp32 accumulation in row order.
template <bool BF16>
__global__ __launch_bounds__(256) void k_gram(const void* __restrict__ wo, int dm, int D, float* __restrict__ gram) {
  __shared__ float s_a[32][33], s_b[32][33];
  const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
  const int a0 = blockIdx.x * 32, b0 = blockIdx.y * 32, g = blockIdx.z;
  const size_t base = (size_t)g * dm * D;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int m0 = 0; m0 < dm; m0 += 32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + ty + 8 * i;
      s_a[ty + 8 * i][tx] = m < dm ? load_elem<BF16>(wo, base + (size_t)m * D + a0 + tx) : 0.f;
      s_b[ty + 8 * i][tx] = m < dm ? load_elem<BF16>(wo, base + (size_t)m * D + b0 + tx) : 0.f;
    }
    __syncthreads();
#pragma unroll 8
    for (int m = 0; m < 32; ++m) {
      const float bv = s_b[m][tx];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = fmaf(s_a[m][ty + 8 * i], bv, acc[i]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) gram[((size_t)g * D + a0 + ty + 8 * i) * D + b0 + tx] = acc[i];
}

hipError_t launch_gram(const Dims& d, const void* w_o, int dm, float* gram, hipStream_t st) {
  dim3 grid(d.D / 32, d.D / 32, d.Hq);
  if (d.dtype == EA_BF16)
    k_gram<true><<<grid, 256, 0, st>>>(w_o, dm, d.D, gram);
  else
    k_gram<false><<<grid, 256, 0, st>>>(w_o, dm, d.D, gram);
  return hipGetLastError();
}

hipError_t launch_project(const Dims& d, const void* hidden, const void* wq, int w, int dm, float* q,
                          hipStream_t st) {
  if (d.dtype == EA_BF16 && dm % 8 == 0 && ((uintptr_t)hidden % 16) == 0 && ((uintptr_t)wq % 16) == 0) {
    // The more samples a workgroup takes, the less often W_Q is read: 64 where that leaves two workgroups per CU, else 32 (us
    // of statistics and the short pass behind them, 64 and 32 samples: 128 x 4096 hidden states, 32 heads 57.9 and 57.0; 128 x
    // 5120, 40 heads 73.2 and 70.3; 200 x 4096, 32 heads 68.3 and 69.3; 512 x 4096 99 and 104.6), and fewer where the
    // workgroups would leave a quarter of the CUs without one (64 x 4096, 64 samples 55.0, 32 50.8).  (Rows of less than two
    // blocks gain nothing from the patch: 1024 samples x 72, 64 heads, 67 us straight into the operand layout and 73.)
    auto blocks = [&](int mt) { return (int64_t)((w + 16 * mt - 1) / (16 * mt)) * (d.Hq * d.D / 32) * d.B; };
    int mt = w > 32 ? 4 : w > 16 ? 2 : 1;
    if (mt == 4 && blocks(mt) < 2 * (int64_t)device_num_cu()) mt = 2;
    while (mt > 1 && blocks(mt) * 4 < 3 * (int64_t)device_num_cu()) mt /= 2;
    const dim3 gm((unsigned)((w + 16 * mt - 1) / (16 * mt)), (unsigned)(d.Hq * d.D / 32), (unsigned)d.B);
    const uint16_t* h = (const uint16_t*)hidden;
    const uint16_t* m = (const uint16_t*)wq;
#define EA_PROJECT(MM, NN) \
  if (mt == MM && nw == NN) k_project_mfma<MM, NN><<<gm, 64 * NN, 0, st>>>(h, m, w, dm, d.D, d.Hq, q)
    // four wavefronts over d_model where there are more workgroups than CUs or little to split (1024 workgroups x 5120 entries 100
    // and 108 us with eight of them, 256 x 2048 52.6 and 53.0; but 192 x 4096 59.3 and 58.2, 192 x 5120 50.6 and 49.4)
    const int nw = blocks(mt) > device_num_cu() || dm <= 2048 ? 4 : 8;
    EA_PROJECT(2, 8);
    EA_PROJECT(1, 8);
    EA_PROJECT(4, 4);
    EA_PROJECT(2, 4);
    EA_PROJECT(1, 4);
#undef EA_PROJECT
    return hipGetLastError();
  }
  dim3 grid((w + 31) / 32, d.D / 32, d.qheads());
  if (d.dtype == EA_BF16)
    k_project<true><<<grid, 256, 0, st>>>(hidden, wq, w, dm, d.D, d.Hq, q);
  else
    k_project<false><<<grid, 256, 0, st>>>(hidden, wq, w, dm, d.D, d.Hq, q);
  return hipGetLastError();
}

}  // namespace ea

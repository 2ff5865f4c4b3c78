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
// multiple of 8): one workgroup = 16 MT samples x 32 channels, its operands read straight from global memory in
// the layout v_mfma_f32_16x16x32_bf16 takes them: lane (c, q) = (lane % 16, lane / 16) holds 8 consecutive d_model
// entries of row c, so that four lanes read 64 contiguous bytes of a row and the two k-steps of a block of 64
// entries its whole 128-byte line.  The NW wavefronts split the d_model axis into as many contiguous parts; the
// partial tiles meet in LDS and are added in wavefront order, so the result does not depend on timing.  bf16
// products are exact in fp32.
//
// What bounds it is the way of the hidden states from L2 into the workgroups of every 32 channels.  With the 32x32x16
// form a lane read 64 contiguous bytes in four instructions, each of which touched 64 lines for 16 bytes of them, and
// every 32 samples read W_Q again: 128 x 4096 hidden states, 32 heads of 128 channels 36.5 -> 27.6 us (the matrix W_Q
// alone takes 5.4 at the rate of a large read).
typedef __bf16 pj_bf16x8 __attribute__((ext_vector_type(8)));
typedef float pj_floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t pj_u32x4 __attribute__((ext_vector_type(4)));

template <int MT, int NW>
__global__ __launch_bounds__(64 * NW) void k_project_mfma(const uint16_t* __restrict__ hidden,
                                                      const uint16_t* __restrict__ wq, int w, int dm, int D, int Hq,
                                                      float* __restrict__ q_out) {
  __shared__ float s_acc[NW][16 * MT][32];
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t0 = blockIdx.x * 16 * MT, b = blockIdx.z;
  const int g = (blockIdx.y * 32) / D, c0 = (blockIdx.y * 32) % D;
  const int kq = (dm + 64 * NW - 1) / (64 * NW) * 64;     // entries per wavefront, a multiple of the block
  const int kbeg = min(dm, wave * kq), kend = min(dm, kbeg + kq);
  const uint16_t* arow[MT];
  const uint16_t* brow[2];
#pragma unroll
  for (int m = 0; m < MT; ++m) arow[m] = hidden + ((size_t)b * w + min(t0 + 16 * m + c, w - 1)) * dm + q * 8;
#pragma unroll
  for (int x = 0; x < 2; ++x) brow[x] = wq + ((size_t)g * D + c0 + 16 * x + c) * dm + q * 8;
  pj_floatx4 acc[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[m][x] = pj_floatx4{0.f, 0.f, 0.f, 0.f};
  struct Block { pj_u32x4 a[2][MT], w[2][2]; };
  auto fetch = [&](int k0, Block& f) __attribute__((always_inline)) {      // 64 entries, all inside the row
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int m = 0; m < MT; ++m) f.a[s][m] = *reinterpret_cast<const pj_u32x4*>(arow[m] + k0 + 32 * s);
#pragma unroll
      for (int x = 0; x < 2; ++x) f.w[s][x] = *reinterpret_cast<const pj_u32x4*>(brow[x] + k0 + 32 * s);
    }
  };
  auto multiply = [&](const Block& f) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int x = 0; x < 2; ++x)
          acc[m][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(pj_bf16x8, f.a[s][m]),
                                                             __builtin_bit_cast(pj_bf16x8, f.w[s][x]), acc[m][x], 0, 0, 0);
  };
  const int full = (kend - kbeg) / 64;
  if (full > 0) {
    Block f0, f1;
    fetch(kbeg, f0);
    for (int i = 0; i < full; i += 2) {                    // (past the last block: it once more, not used)
      fetch(kbeg + 64 * min(i + 1, full - 1), f1);
      multiply(f0);
      fetch(kbeg + 64 * min(i + 2, full - 1), f0);
      if (i + 1 < full) multiply(f1);
    }
  }
  const int k0 = kbeg + 64 * full;
  if (k0 < kend) {                                         // d_model % 64 entries: a lane's eight lie inside the row or outside
    Block f;
    const pj_u32x4 zero4 = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bool in = k0 + 32 * s + 8 * q < kend;
#pragma unroll
      for (int m = 0; m < MT; ++m) f.a[s][m] = in ? *reinterpret_cast<const pj_u32x4*>(arow[m] + k0 + 32 * s) : zero4;
#pragma unroll
      for (int x = 0; x < 2; ++x) f.w[s][x] = in ? *reinterpret_cast<const pj_u32x4*>(brow[x] + k0 + 32 * s) : zero4;
    }
    multiply(f);
  }
  // accumulator register v of lane (c, q) is the tile's entry (row 4 q + v, column c)
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v) s_acc[wave][16 * m + 4 * q + v][16 * x + c] = acc[m][x][v];
  __syncthreads();
  float* out = q_out + (((size_t)b * Hq + g) * w) * D + c0;
#pragma unroll
  for (int i = 0; i < 8 * MT / NW; ++i) {
    const int e = tid + 64 * NW * i, t = e >> 5, ch = e & 31;
    float sum = s_acc[0][t][ch];
#pragma unroll
    for (int p = 1; p < NW; ++p) sum += s_acc[p][t][ch];
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
    // The more samples a workgroup takes, the less often W_Q is read: as many as leave workgroups for three quarters of the
    // CUs (with the statistics, us: 64 x 4096 and 32 heads of 128 channels, 64 samples 37.8, 32 29.7; 100 x 4104 and 24
    // heads 35.1 and 44.3).
    auto blocks = [&](int mt) { return (int64_t)((w + 16 * mt - 1) / (16 * mt)) * (d.Hq * d.D / 32) * d.B; };
    int mt = w > 32 ? 4 : w > 16 ? 2 : 1;
    while (mt > 1 && blocks(mt) * 4 < 3 * (int64_t)device_num_cu()) mt /= 2;
    const dim3 gm((unsigned)((w + 16 * mt - 1) / (16 * mt)), (unsigned)(d.Hq * d.D / 32), (unsigned)d.B);
    const uint16_t* h = (const uint16_t*)hidden;
    const uint16_t* m = (const uint16_t*)wq;
#define EA_PROJECT(MM, NN) \
  if (mt == MM && nw == NN) k_project_mfma<MM, NN><<<gm, 64 * NN, 0, st>>>(h, m, w, dm, d.D, d.Hq, q)
    // four wavefronts over d_model where there are more workgroups than CUs or little to split (320 workgroups x 5120 entries 76
    // and 72.5 us with the statistics, 256 x 4096 40.5 and 43.7)
    const int nw = blocks(mt) > device_num_cu() || dm <= 2048 ? 4 : 8;
    EA_PROJECT(4, 8);
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

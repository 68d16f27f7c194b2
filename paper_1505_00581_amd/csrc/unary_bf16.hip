// Split-precision unary table: U[i][n] = sqrt(max(|f_i|^2 + |g_n|^2 - 2 f_i . g_n, 0))
// with descriptors rounded to BF16 (Eq. 2 expanded; Section 3.3's look-up
// table).  The dot products run on MFMA (BF16 inputs, FP32 accumulation), the
// squared norms are taken in FP32 from the same BF16-rounded vectors, and the
// descriptor length is zero-padded to a multiple of 32 (162 -> 192).
#include "stm_internal.h"

namespace stm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bf16 bits, round to nearest even (inputs are finite).
__device__ __forceinline__ uint16_t bf16_bits(float x) {
  const uint32_t b = __float_as_uint(x);
  return static_cast<uint16_t>((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float bf16_value(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// out [np][dp] BF16 (zero rows n >= n_valid, zero columns d >= dim), norm2[n] =
// sum of squares of the rounded row in FP32, index order.  A wave takes 16 rows,
// 32 columns at a time through LDS (the next ones in flight): rows are read and
// written contiguously, then a lane sums each.  Bound by that chain of reads:
// 31,700 x 162 and 75 x 162 took 44 us each with one thread walking a row in
// memory, 18 with 64 rows a wave and nothing in flight, 9 now.
constexpr int kCastRows = 16, kCastCols = 32;
__global__ __launch_bounds__(64) void k_to_bf16(const float* __restrict__ x, int32_t n_valid, int32_t dim, int32_t np,
                                               int32_t dp, uint16_t* __restrict__ out, float* __restrict__ norm2) {
  __shared__ uint16_t tile[kCastRows][kCastCols + 2];  // 17 words a row: a lane's own row without bank conflicts
  const int lane = threadIdx.x, half = lane >> 5, col = lane & 31;
  const int32_t n0 = blockIdx.x * kCastRows;
  float v[kCastRows / 2];
  const auto fetch = [&](int32_t d) {
#pragma unroll
    for (int q = 0; q < kCastRows / 2; ++q) {
      const int32_t n = n0 + 2 * q + half;
      const bool in = n < n_valid && d < dim;
      const float r = x[in ? (long long)n * dim + d : 0];
      v[q] = in ? r : 0.f;
    }
  };
  float acc = 0.f;
  fetch(col);
  for (int32_t d0 = 0; d0 < dp; d0 += kCastCols) {  // dp is a multiple of 32
#pragma unroll
    for (int q = 0; q < kCastRows / 2; ++q) {
      const uint16_t h = bf16_bits(v[q]);
      const int32_t n = n0 + 2 * q + half;
      tile[2 * q + half][col] = h;
      if (n < np) out[(long long)n * dp + d0 + col] = h;
    }
    if (d0 + kCastCols < dp) fetch(d0 + kCastCols + col);
    __syncthreads();
    if (lane < kCastRows) {
#pragma unroll
      for (int c = 0; c < kCastCols; ++c) {
        const float w = bf16_value(tile[lane][c]);
        acc = fmaf(w, w, acc);
      }
    }
    __syncthreads();
  }
  if (lane < kCastRows && n0 + lane < np) norm2[n0 + lane] = acc;
}

// One wave computes a 16 (model rows) x 64 (scene points) block with four
// 16x16 MFMA tiles; K runs over dp in steps of 32.  Operand layout of
// v_mfma_f32_16x16x32_bf16: lane l holds row (l % 16) of A and column (l % 16)
// of B at k = 8 (l / 16) .. 8 (l / 16) + 7 of the step; the accumulator holds
// rows 4 (l / 16) + j, j = 0..3, of column l % 16.
constexpr int kWavesPerBlock = 4;

__global__ __launch_bounds__(kWavesPerBlock * 64) void k_unary_bf16(
    const uint16_t* __restrict__ fb, const float* __restrict__ fn, int32_t M,
    const uint16_t* __restrict__ gb, const float* __restrict__ gn, int32_t S, int32_t dp,
    float* __restrict__ U) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int row0 = blockIdx.y * 16;
  const int col0 = (blockIdx.x * kWavesPerBlock + wv) * 64;
  const int lr = lane & 15, kq = (lane >> 4) * 8;
  f32x4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* arow = fb + (long long)(row0 + lr) * dp + kq;
  for (int k0 = 0; k0 < dp; k0 += 32) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(arow + k0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(gb + (long long)(col0 + t * 16 + lr) * dp + kq + k0);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int col = col0 + t * 16 + lr;
    const float g2 = gn[col];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = row0 + (lane >> 4) * 4 + j;
      const float d2 = fn[row] + g2 - 2.f * acc[t][j];
      if (row < M && col < S) U[(long long)row * S + col] = __builtin_sqrtf(fmaxf(d2, 0.f));
    }
  }
}

}  // namespace

int32_t bf16_padded_dim(int32_t dim) { return (dim + 31) / 32 * 32; }

hipError_t launch_to_bf16(const float* x, int32_t n_valid, int32_t dim, int32_t np, uint16_t* out,
                          float* norm2, hipStream_t st) {
  hipLaunchKernelGGL(k_to_bf16, dim3((np + kCastRows - 1) / kCastRows), dim3(64), 0, st, x, n_valid, dim, np,
                     bf16_padded_dim(dim), out, norm2);
  return hipGetLastError();
}

hipError_t launch_unary_bf16(const uint16_t* fb, const float* fn, int32_t M, const uint16_t* gb,
                             const float* gn, int32_t S, int32_t dim, float* U, hipStream_t st) {
  const int32_t cols_per_block = kWavesPerBlock * 64;
  dim3 grid((S + cols_per_block - 1) / cols_per_block, (M + 15) / 16);
  hipLaunchKernelGGL(k_unary_bf16, grid, dim3(kWavesPerBlock * 64), 0, st, fb, fn, M, gb, gn, S,
                     bf16_padded_dim(dim), U);
  return hipGetLastError();
}

}  // namespace stm

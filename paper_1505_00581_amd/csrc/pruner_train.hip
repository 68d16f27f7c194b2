// FP32 training pass of the candidate pruner: forward, listwise loss and
// backward over G groups of 64 rows (the network and its inputs are stated in
// pruner.hip).  The contractions run on the FP32 matrix instructions, whose
// result is the fmaf chain over ascending k, so activations are those of a
// scalar loop bit for bit.
//
// Three properties of the inputs carry the layout:
//  * the 64 rows of a group share the model descriptor f_i, the first D inputs
//    of layer 1: its part of the chain is computed once per model point
//    (k_train_prefix) and is the rows' initial accumulator;
//  * for the same reason the model half of dW1 is a product over groups (the
//    group's column sum of dZ1 times f_i), not over rows;
//  * a group's rows are one workgroup: the loss needs no other rows, so
//    forward, loss and the activations' backward run in one launch with h1, h2
//    and dZ2 handed from layer to layer in LDS.
#include <math.h>

#include <algorithm>

#include "stm_internal.h"

namespace stm {
namespace {

constexpr int H = kPrunerHidden;
constexpr int kRows = 64;       // rows of a group
constexpr int kTile = 32;       // inputs staged at a time
constexpr int kTileLd = kTile + 4;
constexpr int kHidLd = H + 4;   // both strides are 4 mod 64 banks times an odd number: 16-byte reads do not conflict

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Column sums of one group, gsum [G][kGsum]: dZ1 [128], dZ2 [128], ds h2 [128], ds.
constexpr int kGsum = 3 * H + 4;

struct Theta {
  const float *W1, *b1, *W2, *b2, *w3, *b3;
};
__device__ __forceinline__ Theta theta_of(const float* th, int NI) {
  Theta p;
  p.W1 = th;
  p.b1 = p.W1 + (long long)H * NI;
  p.W2 = p.b1 + H;
  p.b2 = p.W2 + H * H;
  p.w3 = p.b2 + H;
  p.b3 = p.w3 + H;
  return p;
}

// Place of input k (0..31) in a staged row: even inputs, then odd ones.  The
// 32 x 32 x 2 instruction takes input 2 j + h from lane half h, so a lane's
// inputs of four consecutive instructions are one 16-byte read.
__device__ __forceinline__ int k_place(int k) { return (k & 1) * (kTile / 2) + (k >> 1); }

// Row of accumulator register j in a 32 x 32 tile (the column is lane % 32).
__device__ __forceinline__ int acc_row(int lane, int j) { return 8 * (j >> 2) + 4 * (lane >> 5) + (j & 3); }

// P[i][o] = sum over d < D of (D f_i[d]) W1[o][d], ascending: the model part
// of layer 1's chain, two model points per workgroup.
constexpr int kPrefixPoints = 2, kPrefixTile = 64;
__global__ __launch_bounds__(256) void k_train_prefix(PrunerTrain t) {
  __shared__ __align__(16) float ws[H][kPrefixTile + 4];
  __shared__ __align__(16) float fs[kPrefixPoints][kPrefixTile];
  const int tid = threadIdx.x, o = tid & (H - 1), half = tid >> 7;
  const int D = t.D, NI = 2 * D + 8, i0 = blockIdx.x * kPrefixPoints;
  const float scale = static_cast<float>(D);
  float acc = 0.f;
  for (int k0 = 0; k0 < D; k0 += kPrefixTile) {  // inputs past D count as 0: the chain keeps its value
    const int kk = tid & (kPrefixTile - 1), k = min(k0 + kk, D - 1);
    const bool in = k0 + kk < D;
    float w[H * kPrefixTile / 256];
#pragma unroll
    for (int j = 0; j < H * kPrefixTile / 256; ++j) w[j] = t.theta[(long long)(tid / kPrefixTile + 4 * j) * NI + k];
    const float f = t.mdesc[(long long)min(i0 + (tid >> 6) % kPrefixPoints, t.M - 1) * D + k];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < H * kPrefixTile / 256; ++j) ws[tid / kPrefixTile + 4 * j][kk] = in ? w[j] : 0.f;
    if (tid < kPrefixPoints * kPrefixTile) fs[tid / kPrefixTile][kk] = in ? scale * f : 0.f;
    __syncthreads();
#pragma unroll 4
    for (int q = 0; q < kPrefixTile; q += 4) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(&ws[o][q]), a = *reinterpret_cast<const f32x4*>(&fs[half][q]);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = fmaf(a[e], b[e], acc);
    }
  }
  if (i0 + half < t.M) t.prefix[(long long)(i0 + half) * H + o] = acc;
}

struct RowsShared {
  float a[kRows][kTileLd];  // staged inputs of layer 1
  float b[H][kTileLd];      // staged weights, one row per output unit
  float hid[kRows][kHidLd]; // h1, then h2, then dZ2
  float sum1[2][H], sum2[2][H], sumw[2][H];
  float sc[kRows], ds[kRows];
  int32_t node[kRows];
};

// One group per workgroup, four waves; wave (wr, wc) owns rows 32 wr .. and
// units 64 wc .. of every layer as two 32 x 32 tiles.  Bound by the matrix
// instructions (7.1 GFLOP at 1,024 groups and D = 162: 101 us, 70 TFLOP/s of
// FP32); scalar layers, loss and column sums in launches of their own took
// 750 us there.
__global__ __launch_bounds__(256, 2) void k_train_rows(PrunerTrain t) {
  __shared__ __align__(16) RowsShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wr = wv >> 1, wc = wv & 1, l32 = lane & 31, lh = lane >> 5;
  const int g = blockIdx.x, D = t.D, NI = 2 * D + 8;
  const long long r0 = (long long)g * kRows;
  const Theta P = theta_of(t.theta, NI);
  const float scale = static_cast<float>(D);
  if (tid < kRows) sh.node[tid] = t.node[r0 + tid];
  __syncthreads();

  f32x16 acc[2];
  // arow: this lane's row of the 32 staged inputs, of which the first 8 nq count
  const auto tile_gemm = [&](const float* arow, int nq) {
#pragma unroll
    for (int q = 0; q < kTile / 8; ++q) {
      if (q >= nq) break;
      const f32x4 a = *reinterpret_cast<const f32x4*>(arow + lh * (kTile / 2) + 4 * q);
      f32x4 b[2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
        b[u] = *reinterpret_cast<const f32x4*>(&sh.b[wc * 64 + u * 32 + l32][lh * (kTile / 2) + 4 * q]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[u][e], acc[u], 0, 0, 0);
    }
  };
  float wb[H * kTile / 256];  // the next weight tile in flight
  const auto store_b_rows = [&](bool in) {  // read as rows of the output units: input tid % 32 (0 unless `in`)
#pragma unroll
    for (int j = 0; j < H * kTile / 256; ++j) sh.b[(tid >> 5) + 8 * j][k_place(tid & 31)] = in ? wb[j] : 0.f;
  };
  const auto fetch_w2 = [&](int k0) {
#pragma unroll
    for (int j = 0; j < H * kTile / 256; ++j) wb[j] = P.W2[((tid >> 5) + 8 * j) * H + k0 + (tid & 31)];
  };
  const auto fetch_w2t = [&](int k0) {  // transposed: rows k of W2 are the inputs
#pragma unroll
    for (int j = 0; j < H * kTile / 256; ++j) wb[j] = P.W2[(k0 + (tid >> 7) + 2 * j) * H + (tid & 127)];
  };

  // ---- layer 1: the chain continues after the model part with [D g_n, phi]
  {
    const int i = t.groups[g].y;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float p = t.prefix[(long long)i * H + wc * 64 + u * 32 + l32];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[u][j] = sh.node[wr * 32 + acc_row(lane, j)] < 0 ? 0.f : p;
    }
    // tiles of the descriptor (the last one padded with zeros: the chain keeps
    // its value), then one of the 8 features; every read of a tile is
    // unconditional, so that all of them are in flight together
    constexpr int kReads = kRows * kTile / 256;
    float xa[kReads];
    const int kk = tid & 31, row0 = tid >> 5;
    uint32_t live = 0;  // bit j: row row0 + 8 j holds a candidate
#pragma unroll
    for (int j = 0; j < kReads; ++j) live |= sh.node[row0 + 8 * j] >= 0 ? 1u << j : 0u;
    const int nd = (D + kTile - 1) / kTile;
    const auto fetch = [&](int q) {
      const int k = q < nd ? min(q * kTile + kk, D - 1) : min(kk, 7);
      if (q < nd) {
#pragma unroll
        for (int j = 0; j < kReads; ++j) xa[j] = t.sdesc[(long long)max(sh.node[row0 + 8 * j], 0) * D + k];
      } else {
#pragma unroll
        for (int j = 0; j < kReads; ++j) xa[j] = t.phi[(r0 + row0 + 8 * j) * 8 + k];
      }
      const float* w = P.W1 + (long long)row0 * NI + (q < nd ? D : 2 * D) + k;
#pragma unroll
      for (int j = 0; j < H * kTile / 256; ++j) wb[j] = w[(long long)(8 * j) * NI];
    };
    fetch(0);
    for (int q = 0; q <= nd; ++q) {
      const int left = q < nd ? D - q * kTile : 8;  // inputs of this tile
      const float f = q < nd ? scale : 1.f;
#pragma unroll
      for (int j = 0; j < kReads; ++j)
        sh.a[row0 + 8 * j][k_place(kk)] = (live >> j & 1u) && kk < left ? f * xa[j] : 0.f;
      store_b_rows(kk < left);
      __syncthreads();
      if (q < nd) fetch(q + 1); else fetch_w2(0);
      tile_gemm(sh.a[wr * 32 + l32], (min(left, kTile) + 7) / 8);
      __syncthreads();
    }
  }
  uint32_t live1 = 0;  // bit 16 u + j: h1 of accumulator register j of tile u is positive
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int o = wc * 64 + u * 32 + l32;
    const float bias = P.b1[o];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int row = wr * 32 + acc_row(lane, j);
      const float h = fmaxf(acc[u][j] + bias, 0.f);
      if (h > 0.f) live1 |= 1u << (16 * u + j);
      sh.hid[row][(o & ~31) + k_place(o & 31)] = h;
      if (t.labels) t.h1[(r0 + row) * H + o] = h;
      acc[u][j] = 0.f;
    }
  }

  // ---- layer 2
  for (int k0 = 0; k0 < H; k0 += kTile) {
    store_b_rows(true);
    __syncthreads();
    if (k0 + kTile < H) fetch_w2(k0 + kTile); else fetch_w2t(0);
    tile_gemm(&sh.hid[wr * 32 + l32][k0], kTile / 8);
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int o = wc * 64 + u * 32 + l32;
    const float bias = P.b2[o];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      acc[u][j] = fmaxf(acc[u][j] + bias, 0.f);
      sh.hid[wr * 32 + acc_row(lane, j)][o] = acc[u][j];
    }
  }
  __syncthreads();

  // ---- scores (four threads per row), loss and its derivative (one wave)
  {
    const int row = tid >> 2, q = (tid & 3) * 32;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 32; k += 4) {
      const f32x4 h = *reinterpret_cast<const f32x4*>(&sh.hid[row][q + k]);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(h[e], P.w3[q + k + e], s);
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    if ((tid & 3) == 0) sh.sc[row] = s + P.b3[0];
  }
  __syncthreads();
  if (wv == 0) {
    const float s = sh.sc[lane];
    const int32_t n = sh.node[lane];
    const bool valid = n >= 0;
    if (t.scores) t.scores[r0 + lane] = valid ? s : -__builtin_inff();
    if (t.labels) {
      float mx = valid ? s : -__builtin_inff();
      for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      const float e = valid ? expf(s - mx) : 0.f;
      float z = e;
      for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off);
      // the label is a node id; its slot is the lane holding it (none: NaN loss, no gradient)
      const unsigned long long hit = __ballot(valid && n == t.labels[g]);
      const int lab = hit ? __ffsll(static_cast<long long>(hit)) - 1 : -1;
      const float sl = __shfl(s, lab < 0 ? 0 : lab);
      if (lane == 0) t.loss[g] = lab < 0 ? __builtin_nanf("") : -(sl - mx - logf(z));
      const float d = lab < 0 ? 0.f : ((valid ? e / z : 0.f) - (lane == lab ? 1.f : 0.f)) / static_cast<float>(t.G);
      sh.ds[lane] = d;
      float sum = d;
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
      if (lane == 0) t.gsum[(long long)g * kGsum + 3 * H] = sum;
    }
  }
  if (!t.labels) return;
  __syncthreads();

  // ---- dZ2 = ds w3 [h2 > 0], the column sums of dZ2 and ds h2
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int o = wc * 64 + u * 32 + l32;
    const float w3 = P.w3[o];
    float s2 = 0.f, sw = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int row = wr * 32 + acc_row(lane, j);
      const float d = sh.ds[row], h = acc[u][j];
      const float z = h > 0.f ? d * w3 : 0.f;
      sw = fmaf(d, h, sw);
      s2 += z;
      sh.hid[row][(o & ~31) + k_place(o & 31)] = z;
      t.dz2[(r0 + row) * H + o] = z;
      acc[u][j] = 0.f;
    }
    s2 += __shfl_xor(s2, 32);
    sw += __shfl_xor(sw, 32);
    if (lh == 0) {
      sh.sum2[wr][o] = s2;
      sh.sumw[wr][o] = sw;
    }
  }

  // ---- dZ1 = (dZ2 W2) [h1 > 0]
  for (int k0 = 0; k0 < H; k0 += kTile) {
#pragma unroll
    for (int j = 0; j < H * kTile / 256; ++j) sh.b[tid & 127][k_place((tid >> 7) + 2 * j)] = wb[j];
    __syncthreads();
    if (k0 + kTile < H) fetch_w2t(k0 + kTile);
    tile_gemm(&sh.hid[wr * 32 + l32][k0], kTile / 8);
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int o = wc * 64 + u * 32 + l32;
    float s1 = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float z = (live1 >> (16 * u + j)) & 1u ? acc[u][j] : 0.f;
      s1 += z;
      t.dz1[(r0 + wr * 32 + acc_row(lane, j)) * H + o] = z;
    }
    s1 += __shfl_xor(s1, 32);
    if (lh == 0) sh.sum1[wr][o] = s1;
  }
  __syncthreads();
  if (tid < H) {
    float* gs = t.gsum + (long long)g * kGsum;
    gs[tid] = sh.sum1[0][tid] + sh.sum1[1][tid];
    gs[H + tid] = sh.sum2[0][tid] + sh.sum2[1][tid];
    gs[2 * H + tid] = sh.sumw[0][tid] + sh.sumw[1][tid];
  }
}

// ---- weight gradients --------------------------------------------------------------
// out[o][c] = sum over rows of dZ[row][o] X[row][c], partial over chunks of
// rows.  Three products share the launch, each in tiles of 128 x 64: dW2 (dZ2,
// h1), the scene half of dW1 (dZ1, [D g_n, phi]) over the rows, and the model
// half of dW1 (the groups' sums of dZ1, D f_i) over the groups.  Bound by the
// latency of the gathered rows against 32 matrix instructions a tile (1,024
// groups, D = 162: 106 us, 51 TFLOP/s; 412 us as scalar products over all rows).
constexpr int kGradCols = 64, kGradRows = 32;
constexpr int kChunkGroups = 8;  // groups of the rows' largest chunk
constexpr int kZLd = H + 32, kXLd = kGradCols + 32;  // 32 mod 64 banks: the lane halves read different banks

struct GradPlan {
  int tiles2, tilesB, tilesA;  // column tiles of the three products
  int chunk;                   // rows (groups) of a chunk, a multiple of kRows
  int nch, ncha;               // chunks over the rows and over the groups
  float *part2, *partB, *partA;
};

struct GradShared {
  float z[kGradRows][kZLd];
  float x[kGradRows][kXLd];
};

// Column tile `tile` of product JOB (0: dW2, 1: scene half of dW1, 2: model
// half).  Every read of a tile is unconditional (indices clamped, values
// selected afterwards), so that all of them are in flight together.
template <int JOB>
__device__ __forceinline__ void wgrad_tile(GradShared& sh, const PrunerTrain& t, int chunk, int tile, float* part) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l32 = lane & 31, lh = lane >> 5, wo = (wv >> 1) * 64, wc = (wv & 1) * 32;
  const int D = t.D, ncol = JOB == 0 ? H : JOB == 1 ? D + 8 : D;
  const int c0 = tile * kGradCols;
  const long long n_rows = JOB == 2 ? t.G : (long long)t.G * kRows;
  const long long rbeg = (long long)blockIdx.y * chunk;
  const long long rend = rbeg + chunk < n_rows ? rbeg + chunk : n_rows;
  const float* Z = JOB == 0 ? t.dz2 : JOB == 1 ? t.dz1 : t.gsum;
  constexpr int zld = JOB == 2 ? kGsum : H;

  f32x16 acc[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[u][j] = 0.f;
  constexpr int kZReads = kGradRows * H / 1024, kXReads = kGradRows * kGradCols / 256;
  f32x4 zr[kZReads];
  float xr[kXReads];
  int32_t idx[kXReads];  // the next rows' scene nodes (model points), read a tile ahead of their descriptors
  uint32_t live = 0;     // bit j: xr[j] is of a candidate, not of an empty slot
  const int c = min(c0 + (tid & (kGradCols - 1)), ncol - 1);  // columns past the end are not stored
  const float scale = JOB == 2 || (JOB == 1 && c < D) ? static_cast<float>(D) : 1.f;
  const auto row_of = [&](long long rb, int j) { return min(rb + (tid >> 6) + 4 * j, rend - 1); };
  const auto fetch_index = [&](long long rb) {
    if constexpr (JOB != 0)
#pragma unroll
      for (int j = 0; j < kXReads; ++j) {
        const long long r = row_of(rb, j);
        idx[j] = JOB == 2 ? t.groups[r].y : t.node[r];
      }
  };
  // rows past the chunk read its last row; their dZ counts as 0
  const auto fetch = [&](long long rb) {
#pragma unroll
    for (int j = 0; j < kZReads; ++j) {
      const long long r = rb + (tid >> 5) + 8 * j;
      zr[j] = *reinterpret_cast<const f32x4*>(Z + min(r, rend - 1) * zld + (tid & 31) * 4);
    }
#pragma unroll
    for (int j = 0; j < kXReads; ++j) {
      const long long r = row_of(rb, j);
      if constexpr (JOB == 0) {
        xr[j] = t.h1[r * H + c];
      } else if constexpr (JOB == 2) {
        xr[j] = t.mdesc[(long long)idx[j] * D + c];
      } else {
        const float* gs = t.sdesc + (long long)max(idx[j], 0) * D + c;
        const float* ps = t.phi + r * 8 + (c - D);
        xr[j] = *(c < D ? gs : ps);
        live = idx[j] >= 0 ? live | (1u << j) : live & ~(1u << j);
      }
    }
  };
  fetch_index(rbeg);
  fetch(rbeg);
  if (rbeg + kGradRows < rend) fetch_index(rbeg + kGradRows);
  for (long long rb = rbeg; rb < rend; rb += kGradRows) {
#pragma unroll
    for (int j = 0; j < kZReads; ++j) {
      const int row = (tid >> 5) + 8 * j;  // (only the groups' chunks end inside a tile)
      const f32x4 z = JOB == 2 && rb + row >= rend ? f32x4{0.f, 0.f, 0.f, 0.f} : zr[j];
      *reinterpret_cast<f32x4*>(&sh.z[row][(tid & 31) * 4]) = z;
    }
#pragma unroll
    for (int j = 0; j < kXReads; ++j)  // an empty slot's inputs count as 0
      sh.x[(tid >> 6) + 4 * j][tid & (kGradCols - 1)] = JOB == 1 && !(live >> j & 1u) ? 0.f : scale * xr[j];
    __syncthreads();
    if (rb + kGradRows < rend) fetch(rb + kGradRows);
    if (rb + 2 * kGradRows < rend) fetch_index(rb + 2 * kGradRows);
#pragma unroll
    for (int k = 0; k < kGradRows; k += 2) {
      const float x = sh.x[k + lh][wc + l32];
#pragma unroll
      for (int u = 0; u < 2; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(sh.z[k + lh][wo + u * 32 + l32], x, acc[u], 0, 0, 0);
    }
    __syncthreads();
  }
  float* out = part + (long long)blockIdx.y * H * ncol;
  const int co = c0 + wc + l32;
  if (co < ncol)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < 16; ++j) out[(long long)(wo + u * 32 + acc_row(lane, j)) * ncol + co] = acc[u][j];
}

__global__ __launch_bounds__(256) void k_train_wgrad(PrunerTrain t, GradPlan p) {
  __shared__ __align__(16) GradShared sh;
  const int tile = blockIdx.x;
  if (tile < p.tiles2) {
    wgrad_tile<0>(sh, t, p.chunk, tile, p.part2);
  } else if (tile < p.tiles2 + p.tilesB) {
    wgrad_tile<1>(sh, t, p.chunk, tile - p.tiles2, p.partB);
  } else if ((int)blockIdx.y < p.ncha) {
    wgrad_tile<2>(sh, t, p.chunk, tile - p.tiles2 - p.tilesB, p.partA);
  }
}

// The packed gradient: blocks below `dense` sum the weight partials over their
// chunks, one element per thread; the rest sum the groups' column sums (biases
// and w3), 8 columns by 32 strided parts per block.
__global__ __launch_bounds__(256) void k_train_reduce(PrunerTrain t, GradPlan p, int dense) {
  const int D = t.D, NI = 2 * D + 8;
  const long long n1 = (long long)H * NI;
  float* gb1 = t.grad + n1;
  float* gW2 = gb1 + H;
  float* gb2 = gW2 + H * H;
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < dense) {
    const long long e = (long long)blockIdx.x * 256 + tid;
    const float* src;
    long long stride;
    int n;
    float* dst;
    if (e < n1) {
      const int o = static_cast<int>(e / NI), c = static_cast<int>(e % NI);
      src = c < D ? p.partA + (long long)o * D + c : p.partB + (long long)o * (D + 8) + (c - D);
      stride = (long long)H * (c < D ? D : D + 8);
      n = c < D ? p.ncha : p.nch;
      dst = t.grad + e;
    } else if (e < n1 + H * H) {
      src = p.part2 + (e - n1);
      stride = H * H;
      n = p.nch;
      dst = gW2 + (e - n1);
    } else {
      return;
    }
    float acc[8] = {};
    int q = 0;
    for (; q + 8 <= n; q += 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[u] += src[(q + u) * stride];
    for (; q < n; ++q) acc[0] += src[q * stride];
    *dst = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    return;
  }
  __shared__ float part[32][8];
  const int col = (blockIdx.x - dense) * 8 + (tid & 7), seg = tid >> 3;
  float s = 0.f;
  if (col <= 3 * H)
#pragma unroll 8
    for (int g = seg; g < t.G; g += 32) s += t.gsum[(long long)g * kGsum + col];
  part[seg][tid & 7] = s;
  __syncthreads();
  if (tid < 8 && col <= 3 * H) {
    float v = 0.f;
    for (int q = 0; q < 32; ++q) v += part[q][tid];
    float* dst = col < H ? gb1 + col : gb2 + (col - H);  // b2, w3 and b3 follow each other
    *dst = v;
  }
}

inline int ceil_div(long long a, long long b) { return static_cast<int>((a + b - 1) / b); }

// Chunks of 64 ceil(G / 128) rows, about five column tiles times 128 chunks of
// workgroups, but of at most 512 rows: a longer chain of FP32 additions would only
// cost accuracy (65,536 equal groups: 0.33 of the rounding bound of these sums,
// 2.2 with chunks of 32,768 rows), and the shorter one costs no more than 2% (8,192
// groups, D = 162: 1.80 ms against 1.76).  Above 524,280 groups the grid's limit
// of chunks makes them longer again.
GradPlan grad_plan(int G, int D, float* part) {
  GradPlan p;
  p.tiles2 = H / kGradCols;
  p.tilesB = ceil_div(D + 8, kGradCols);
  p.tilesA = ceil_div(D, kGradCols);
  p.chunk = kRows * std::max(std::min(ceil_div(G, 128), kChunkGroups), ceil_div(G, 65535));
  p.nch = ceil_div((long long)G * kRows, p.chunk);
  p.ncha = ceil_div(G, p.chunk);
  p.part2 = part;
  p.partB = p.part2 + (long long)p.nch * H * H;
  p.partA = p.partB + (long long)p.nch * H * (D + 8);
  return p;
}

}  // namespace

long long pruner_part_floats(int G, int D) {
  const GradPlan p = grad_plan(G, D, nullptr);
  return (long long)H * ((long long)p.nch * (H + D + 8) + (long long)p.ncha * D);
}

long long pruner_gsum_floats(int G) { return (long long)G * kGsum; }

hipError_t launch_pruner_train(const PrunerTrain& t, hipStream_t st) {
  hipLaunchKernelGGL(k_train_prefix, dim3(ceil_div(t.M, kPrefixPoints)), dim3(256), 0, st, t);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_train_rows, dim3(t.G), dim3(256), 0, st, t);
  if ((e = hipGetLastError()) != hipSuccess || !t.labels) return e;
  const GradPlan p = grad_plan(t.G, t.D, t.part);
  hipLaunchKernelGGL(k_train_wgrad, dim3(p.tiles2 + p.tilesB + p.tilesA, p.nch), dim3(256), 0, st, t, p);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int dense = ceil_div((long long)H * (2 * t.D + 8 + H), 256);
  hipLaunchKernelGGL(k_train_reduce, dim3(dense + ceil_div(3 * H + 1, 8)), dim3(256), 0, st, t, p, dense);
  return hipGetLastError();
}

}  // namespace stm

// Learned candidate pruner: features, the Adam step and the BF16 inference
// kernel with top-k selection (the FP32 training pass is pruner_train.hip).  Not part of the paper: it shortens the candidate lists the
// exact recursion (Section 2.2) runs on; the exact recursion stays the
// fallback and the reference for the energy gap.
//
// One group = the candidates of one model point i at one offset tau; a group
// occupies 64 rows (one per candidate slot; slots past the list are invalid).
// Row input x = [D f_i (D), D g_n (D), phi (8)] (descriptors are L1-normalised;
// the factor D brings their entries to order 1) with phi:
//   0  (t'_n - (tau + t_i - t_0)) / 4
//   1,2 ((p'_n - p'_{q_a}) - (p_i - p_a)) / 64,  3,4 the same for neighbour b
//   5  log((|p'_n - p'_{q_a}| + 1) / (|p_i - p_a| + 1))
//   6  U(i, n) - min over the group's candidates of U(i, .)
//   7  i / (M - 1)
// with a = i - 1, b = i + 1 (the one neighbour twice at the chain ends) and q_j
// the candidate of neighbour j with the smallest U (lowest index on ties).
// Network: h1 = relu(W1 x + b1), h2 = relu(W2 h1 + b2), s = w3 . h2 + b3, 128
// hidden units; parameters packed as [W1 (128 x NI), b1, W2 (128 x 128), b2,
// w3, b3], NI = 2 D + 8.
#include <math.h>

#include "dp_math.h"
#include "stm_internal.h"

namespace stm {
namespace {

constexpr int H = kPrunerHidden;

// ---- features --------------------------------------------------------------------

__device__ __forceinline__ int wave_argmin_node(const CandRange& c, const float* __restrict__ Urow, int lane) {
  const int k = c.k1 + c.k2;
  if (k <= 0) return -1;
  const float v = lane < k ? Urow[cand_node(c, lane)] : __builtin_inff();
  const float best = wave_min(v);
  return cand_node(c, __ffsll(static_cast<long long>(__ballot(v == best))) - 1);
}

// Candidate node and features of lane `lane` of group (tau, i); node -1 past
// the list.  Returns the neighbours' chosen candidates in qa, qb.
__device__ void group_features(const ModelView& m, const SceneView& s, const float* __restrict__ U,
                               long long us, const SearchParams& sp, int tau, int i, int lane, int& node,
                               float phi[8], int& qa, int& qb) {
  const int M = m.M, t0 = m.t[0];
  const int a = i >= 1 ? i - 1 : i + 1;
  const int b = i <= M - 2 ? i + 1 : i - 1;
  const CandRange ci = point_candidates(s.fstart, s.F, tau + m.t[i] - t0, sp);
  const CandRange ca = point_candidates(s.fstart, s.F, tau + m.t[a] - t0, sp);
  const CandRange cb = point_candidates(s.fstart, s.F, tau + m.t[b] - t0, sp);
  qa = wave_argmin_node(ca, U + (long long)a * us, lane);
  qb = wave_argmin_node(cb, U + (long long)b * us, lane);
  const int k = ci.k1 + ci.k2;
  node = lane < k ? cand_node(ci, lane) : -1;
  const int best = wave_argmin_node(ci, U + (long long)i * us, lane);
#pragma unroll
  for (int f = 0; f < 8; ++f) phi[f] = 0.f;
  if (node < 0) return;
  const float2 pn = s.xy[node], pi = m.xy[i], pa = m.xy[a], pb = m.xy[b];
  phi[0] = static_cast<float>(s.t[node] - (tau + m.t[i] - t0)) * 0.25f;
  if (qa >= 0) {
    const float2 q = s.xy[qa];
    phi[1] = ((pn.x - q.x) - (pi.x - pa.x)) * (1.f / 64.f);
    phi[2] = ((pn.y - q.y) - (pi.y - pa.y)) * (1.f / 64.f);
    phi[5] = logf((sqrtf((pn.x - q.x) * (pn.x - q.x) + (pn.y - q.y) * (pn.y - q.y)) + 1.f) /
                  (sqrtf((pi.x - pa.x) * (pi.x - pa.x) + (pi.y - pa.y) * (pi.y - pa.y)) + 1.f));
  }
  if (qb >= 0) {
    const float2 q = s.xy[qb];
    phi[3] = ((pn.x - q.x) - (pi.x - pb.x)) * (1.f / 64.f);
    phi[4] = ((pn.y - q.y) - (pi.y - pb.y)) * (1.f / 64.f);
  }
  phi[6] = U[(long long)i * us + node] - U[(long long)i * us + best];
  phi[7] = static_cast<float>(i) / static_cast<float>(M - 1);
}

// One 64-lane block per group: rows node [G*64], phi [G*64][8], q [G][2].
// Groups are groups[g] = (tau, i), or (tau0 + g / M, g % M) when groups is
// null; q may be null.
__global__ __launch_bounds__(64) void k_group_rows(ModelView m, SceneView s, const float* __restrict__ U,
                                                  long long us, SearchParams sp, const int2* __restrict__ groups,
                                                  int tau0, int32_t* __restrict__ node, float* __restrict__ phi,
                                                  int32_t* __restrict__ q) {
  const long long g = blockIdx.x;
  const int lane = threadIdx.x;
  const int2 gi = groups ? groups[g] : make_int2(tau0 + static_cast<int>(g / m.M), static_cast<int>(g % m.M));
  int n, qa, qb;
  float f[8];
  group_features(m, s, U, us, sp, gi.x, gi.y, lane, n, f, qa, qb);
  const long long r = g * 64 + lane;
  node[r] = n;
  float4* ph = reinterpret_cast<float4*>(phi + r * 8);
  ph[0] = make_float4(f[0], f[1], f[2], f[3]);
  ph[1] = make_float4(f[4], f[5], f[6], f[7]);
  if (q && lane == 0) {
    q[2 * g] = qa;
    q[2 * g + 1] = qb;
  }
}

// Adam (Kingma and Ba) on the packed parameters; c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ theta, const float* __restrict__ g,
                                             float* __restrict__ m, float* __restrict__ v, long long n, float lr,
                                             float beta1, float beta2, float eps, float c1, float c2) {
  const long long j = (long long)blockIdx.x * 256 + threadIdx.x;
  if (j >= n) return;
  const float gj = g[j];
  const float mj = beta1 * m[j] + (1.f - beta1) * gj;
  const float vj = beta2 * v[j] + (1.f - beta2) * gj * gj;
  m[j] = mj;
  v[j] = vj;
  theta[j] -= lr * (mj / c1) / (sqrtf(vj / c2) + eps);
}


// ---- BF16 inference ------------------------------------------------------------------

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float x) {
  const uint32_t b = __float_as_uint(x);
  return static_cast<uint16_t>((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

// out [rows][dp] BF16 of W[o * ld + off + d] (d < D), zero for D <= d < dp.
__global__ void k_cast_rows_bf16(const float* __restrict__ W, int rows, int ld, int off, int D, int dp,
                                 uint16_t* __restrict__ out) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)rows * dp) return;
  const int o = static_cast<int>(e / dp), d = static_cast<int>(e % dp);
  out[e] = d < D ? to_bf16(W[(long long)o * ld + off + d]) : 0;
}

// P[n][o] = scale * sum_d X[n][d] Wp[o][d] + bias[o] for o < 128 (bias
// nullable): BF16 inputs on MFMA, FP32 accumulation and output.
// Xb [np][dp] zero-padded to a multiple of 16 rows; one 4-wave block per 16
// rows, each wave 32 output columns (two 16x16 tiles).
__global__ __launch_bounds__(256) void k_project_bf16(const uint16_t* __restrict__ Xb, int n, int dp,
                                                     const uint16_t* __restrict__ Wb, float scale,
                                                     const float* __restrict__ bias, float* __restrict__ P) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int row0 = blockIdx.x * 16, lr = lane & 15, kq = (lane >> 4) * 8;
  f32x4_t acc[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
  for (int k0 = 0; k0 < dp; k0 += 32) {
    const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(Xb + (long long)(row0 + lr) * dp + k0 + kq);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int col = wv * 32 + t * 16 + lr;
      const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(Wb + (long long)col * dp + k0 + kq);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = row0 + (lane >> 4) * 4 + j;
      if (row < n) {
        const int o = wv * 32 + t * 16 + lr;
        P[(long long)row * H + o] = scale * acc[t][j] + (bias ? bias[o] : 0.f);
      }
    }
}

// Inference: one wave per group, no block barriers after the set-up.  Bound by
// instruction issue beside the matrix cores (173 us of them at 104,000 groups of
// 64); two candidate tiles at a time share the reads of W2: 507 us, 562 with one.
//
// Layer 1 runs transposed, Z1^T [hidden k][candidate c], per 16 x 16 tile
// (kt, ct): the accumulator starts at A'_i[k] + B_n[k] (A' = W1a (D f) + b1,
// B = W1b (D g), both from the BF16 projections) and takes W1c phi on
// v_mfma_f32_16x16x4_f32 (K = 8 as two steps, FP32).  Its accumulator layout
// (lane l: k = 16 kt + 4 (l / 16) + j, c = 16 ct + l % 16) is used directly as
// the B operand of layer 2 on v_mfma_f32_16x16x32_bf16: the 32-wide K block p
// takes tiles kt = 2p and 2p + 1, so lane l supplies hidden units
// 32p + 16h + 4 (l / 16) + j (h, j in {0,1} x {0..3}); W2 sits in LDS permuted
// to the same order, so no data moves between the layers.
constexpr int kInferWaves = 8;
constexpr int kW2Row = H + 8;  // bf16 per permuted W2 row (padding against bank conflicts)

struct alignas(16) InferShared {
  uint16_t w2p[H * kW2Row];   // W2 rows o, K order of the MFMA operand
  float b2[H], w3[H];
  float phi[kInferWaves][64][9];  // per wave: features of the 64 slots (+ pad)
  int32_t node[kInferWaves][64];
  unsigned long long key[kInferWaves][64];  // per wave: selection keys of the 64 slots
};

// Selection key of a slot: smaller is kept first.  Frame distance (0 under the
// score rule), then the score descending, then the slot; unique per slot.
__device__ __forceinline__ unsigned long long select_key(int df, float sc, int slot) {
  unsigned int u = __float_as_uint(sc + 0.f);  // -0 counts as +0
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // order-preserving map of floats to unsigned
  return (static_cast<unsigned long long>(df) << 38) | (static_cast<unsigned long long>(~u) << 6) |
         static_cast<unsigned long long>(slot);
}

// Position of hidden unit u inside a permuted W2 row.
__device__ __forceinline__ int w2_pos(int u) {
  const int p = u >> 5, r = u & 31, h = r >> 4, g = (r & 15) >> 2, j = r & 3;
  return ((p * 4 + g) * 8) + h * 4 + j;
}

__global__ __launch_bounds__(kInferWaves * 64) __attribute__((amdgpu_waves_per_eu(4))) void k_pruner_infer(
    ModelView m, SceneView s, const int32_t* __restrict__ gnode, const float* __restrict__ gphi,
    const int2* __restrict__ groups, long long n_groups, int tau0, const float* __restrict__ theta, int D,
    const float* __restrict__ A, const float* __restrict__ B, int topk, int rule, int32_t* __restrict__ cand,
    int32_t* __restrict__ count, float* __restrict__ scores) {
  __shared__ InferShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int NI = 2 * D + 8;
  const float* W1 = theta;
  const float* b1 = W1 + (long long)H * NI;
  const float* W2 = b1 + H;
  const float* b2 = W2 + H * H;
  const float* w3 = b2 + H;
  const float b3 = w3[H];
  for (int e = tid; e < H * H; e += kInferWaves * 64) {
    const int o = e >> 7, u = e & 127;
    sh.w2p[o * kW2Row + w2_pos(u)] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(W2[e]));
  }
  for (int e = tid; e < H; e += kInferWaves * 64) {
    sh.b2[e] = b2[e];
    sh.w3[e] = w3[e];
  }
  // layer-1 A operands (W1 phi columns): lane l holds W1c[16 kt + l % 16][l / 16 + 4 h]
  float w1c[8][2];
  const int lr = lane & 15, lq = lane >> 4;
#pragma unroll
  for (int kt = 0; kt < 8; ++kt)
#pragma unroll
    for (int h = 0; h < 2; ++h) w1c[kt][h] = W1[(long long)(16 * kt + lr) * NI + 2 * D + lq + 4 * h];
  __syncthreads();

  float(*phi)[9] = sh.phi[wv];
  int32_t* node = sh.node[wv];
  const long long stride = (long long)gridDim.x * kInferWaves;
  for (long long g = (long long)blockIdx.x * kInferWaves + wv; g < n_groups; g += stride) {
    const int2 gi = groups ? groups[g] : make_int2(tau0 + static_cast<int>(g / m.M), static_cast<int>(g % m.M));
    const int n = gnode[g * 64 + lane];
    {
      const float4* gp = reinterpret_cast<const float4*>(gphi + (g * 64 + lane) * 8);
      const float4 f0 = gp[0], f1 = gp[1];
      node[lane] = n;
      phi[lane][0] = f0.x; phi[lane][1] = f0.y; phi[lane][2] = f0.z; phi[lane][3] = f0.w;
      phi[lane][4] = f1.x; phi[lane][5] = f1.y; phi[lane][6] = f1.z; phi[lane][7] = f1.w;
    }
    // the wave's LDS writes above are read by other lanes of the same wave below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // A'_i rows for this lane's hidden units: k = 16 kt + 4 lq + j
    float4 arow[8];
#pragma unroll
    for (int kt = 0; kt < 8; ++kt) arow[kt] = *reinterpret_cast<const float4*>(A + (long long)gi.y * H + 16 * kt + 4 * lq);
    float sc = -__builtin_inff();
#pragma unroll 1
    for (int c0 = 0; c0 < 4; c0 += 2) {  // two candidate tiles at a time share the reads of W2
      bf16x8_t hb[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int c = 16 * (c0 + t) + lr;  // this lane's candidate in the tile
        const int nc = node[c];
        const float p0 = phi[c][lq], p1 = phi[c][lq + 4];
        const float* brow = B + (long long)(nc < 0 ? 0 : nc) * H + 4 * lq;
#pragma unroll
        for (int kt = 0; kt < 8; ++kt) {
          const float4 bv = *reinterpret_cast<const float4*>(brow + 16 * kt);
          f32x4_t z = {arow[kt].x + bv.x, arow[kt].y + bv.y, arow[kt].z + bv.z, arow[kt].w + bv.w};
          z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1c[kt][0], p0, z, 0, 0, 0);
          z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1c[kt][1], p1, z, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            // v_cvt_pk_bf16_f32, nearest even; an empty slot's column is dropped below
            hb[t][kt >> 1][(kt & 1) * 4 + j] = static_cast<__bf16>(fmaxf(z[j], 0.f));
          }
        }
      }
      float part[2] = {0.f, 0.f};
#pragma unroll 2
      for (int ot = 0; ot < 8; ++ot) {
        f32x4_t acc[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
        const uint16_t* wrow = sh.w2p + (16 * ot + lr) * kW2Row + lq * 8;
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
          const bf16x8_t wa = *reinterpret_cast<const bf16x8_t*>(wrow + pb * 32);
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, hb[t][pb], acc[t], 0, 0, 0);
        }
        // rows of acc: output units o = 16 ot + 4 lq + j, column: candidate c
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int o = 16 * ot + 4 * lq + j;
          const float b2o = sh.b2[o], w3o = sh.w3[o];
#pragma unroll
          for (int t = 0; t < 2; ++t) part[t] = fmaf(fmaxf(acc[t][j] + b2o, 0.f), w3o, part[t]);
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        part[t] += __shfl_xor(part[t], 16);
        part[t] += __shfl_xor(part[t], 32);
        if (c0 + t == lq) sc = part[t] + b3;  // lane l = 16 ct + l % 16 owns candidate l
      }
    }
    if (n < 0) sc = -__builtin_inff();
    if (scores) scores[g * 64 + lane] = sc;
    // rank: candidates ahead in the selection order.  Score rule: a higher
    // score, or an equal score and a lower slot.  Frames-first rule: a frame
    // nearer the shifted model frame, then the score rule inside a frame.
    // Time-nearest rule: a nearer frame, then the lower slot (the score is
    // not consulted).  Empty slots carry -inf and the largest frame distance:
    // ranked last.
    const int df = n < 0 ? (1 << 25) : abs(s.t[n] - (gi.x + m.t[gi.y] - m.t[0]));
    const unsigned long long key = select_key(rule ? df : (n < 0 ? 1 : 0), rule == 2 ? 0.f : sc, lane);
    sh.key[wv][lane] = key;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int rank = 0;
    const ulonglong2* kk = reinterpret_cast<const ulonglong2*>(sh.key[wv]);
#pragma unroll 8
    for (int j = 0; j < 32; ++j) {
      const ulonglong2 o = kk[j];  // the same address in every lane: a broadcast read
      rank += (o.x < key) + (o.y < key);
    }
    const bool keep = n >= 0 && rank < topk;
    const unsigned long long mask = __ballot(keep);
    const int pos = __popcll(mask & ((1ull << lane) - 1ull));
    if (keep) cand[g * topk + pos] = n;
    if (lane == 0) count[g] = __popcll(mask);
    // every lane has read this group's LDS rows before the next group rewrites them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Rows of the exact re-solve of offsets taus[r] back into the outputs of the
// offset range starting at tau0; fell_back[tau - tau0] = 1.
__global__ __launch_bounds__(64) void k_scatter_fallback(const int32_t* __restrict__ taus, int tau0, int M,
                                                        const float* __restrict__ e32, const double* __restrict__ e64,
                                                        const double* __restrict__ eu, const int32_t* __restrict__ as,
                                                        float* __restrict__ o32, double* __restrict__ o64,
                                                        double* __restrict__ ou, int32_t* __restrict__ oas,
                                                        int32_t* __restrict__ fell) {
  const int r = blockIdx.x, lane = threadIdx.x;
  const long long d = taus[r] - tau0;
  for (int i = lane; i < M; i += 64) oas[d * M + i] = as[(long long)r * M + i];
  if (lane == 0) {
    o32[d] = e32[r];
    if (o64) o64[d] = e64[r];
    if (ou) ou[d] = eu[r];
    if (fell) fell[d] = 1;
  }
}

// Caller-given candidate lists: bad[0] |= 1 for a count outside [0, kc], 2 for a
// node outside [0, S), 4 for a list not strictly ascending; bad[1] += 2 for a list
// that holds the nodes of the list before it (of the same offset), -5 for one that
// does not, over the lists of at most 512 workgroups spread over the launch (one
// addition a wave: over a sixteenth of the workgroups they took 50 us below).  One pair's lists of M points,
// or (pairs given) those of pair blockIdx.y.  Bound by reading the lists: a wave
// takes kListRows lists at a time, one entry per lane (kc <= 64), so its reads
// are contiguous and all in flight together.  Against one thread per list and
// one launch per pair, the lists of 50 x 678 offsets x 30 points x 60 nodes take
// 60 us instead of 750.
constexpr int kListRows = 8;
__global__ __launch_bounds__(256) void k_check_lists(const PairDev* __restrict__ pairs,
                                                    const int32_t* __restrict__ cand,
                                                    const int32_t* __restrict__ count, long long rows, int M, int kc,
                                                    int S, int32_t* __restrict__ bad) {
  if (pairs) {
    const PairDev& p = pairs[blockIdx.y];
    cand = p.cand;
    count = p.ccount;
    M = p.m.M;
    rows = (long long)p.n_tau * M;
    S = p.s.S;
  }
  const int lane = threadIdx.x & 63;
  const long long r0 = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * kListRows;
  if (r0 >= rows) return;
  int32_t n[kListRows], v[kListRows];
#pragma unroll
  for (int q = 0; q < kListRows; ++q) {
    const long long r = r0 + q < rows ? r0 + q : rows - 1;
    n[q] = count[r];
    v[q] = cand[r * kc + (lane < kc ? lane : 0)];
  }
  int b = 0;
#pragma unroll
  for (int q = 0; q < kListRows; ++q) {
    const int32_t before = __shfl_up(v[q], 1);
    if (n[q] < 0 || n[q] > kc) {
      b |= 1;
    } else if (lane < n[q]) {
      if (v[q] < 0 || v[q] >= S) b |= 2;
      else if (lane > 0 && v[q] <= before) b |= 4;
    }
  }
  if (b) atomicOr(bad, b);
  const uint32_t every = max(1u, gridDim.x * gridDim.y / 256);
  if ((blockIdx.y * gridDim.x + blockIdx.x) % every == 0) {
    int vote = 0, j = static_cast<int>(r0 % M);  // point of row r0 + q
#pragma unroll
    for (int q = 1; q < kListRows; ++q) {
      j = j + 1 < M ? j + 1 : 0;
      if (r0 + q >= rows || j == 0) continue;
      const bool same = n[q] == n[q - 1] && __all(lane >= n[q] || v[q] == v[q - 1]);
      vote += same ? 2 : -5;
    }
    if (lane == 0 && vote != 0) atomicAdd(bad + 1, vote);
  }
}

inline int blocks(long long n, int per) { return static_cast<int>((n + per - 1) / per); }

}  // namespace

hipError_t launch_group_rows(const ModelView& m, const SceneView& s, const float* U, long long us,
                             const SearchParams& sp, const int2* groups, int tau0, long long G, int32_t* node,
                             float* phi, int32_t* q, hipStream_t st) {
  if (G <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_group_rows, dim3(static_cast<unsigned>(G)), dim3(64), 0, st, m, s, U, us, sp, groups, tau0,
                     node, phi, q);
  return hipGetLastError();
}

hipError_t launch_adam(float* theta, const float* g, float* m, float* v, long long n, float lr, float beta1,
                       float beta2, float eps, float c1, float c2, hipStream_t st) {
  hipLaunchKernelGGL(k_adam, dim3(blocks(n, 256)), dim3(256), 0, st, theta, g, m, v, n, lr, beta1, beta2, eps, c1,
                     c2);
  return hipGetLastError();
}

hipError_t launch_cast_rows_bf16(const float* W, int rows, int ld, int off, int D, int dp, uint16_t* out,
                                 hipStream_t st) {
  hipLaunchKernelGGL(k_cast_rows_bf16, dim3(blocks((long long)rows * dp, 256)), dim3(256), 0, st, W, rows, ld, off,
                     D, dp, out);
  return hipGetLastError();
}

hipError_t launch_project_bf16(const uint16_t* Xb, int n, int dp, const uint16_t* Wb, float scale,
                               const float* bias, float* P, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_project_bf16, dim3(blocks(n, 16)), dim3(256), 0, st, Xb, n, dp, Wb, scale, bias, P);
  return hipGetLastError();
}

hipError_t launch_pruner_infer(const PrunerInfer& q, hipStream_t st) {
  if (q.n_groups <= 0) return hipSuccess;
  int n_cu = 256, dev = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  const long long want = (q.n_groups + kInferWaves - 1) / kInferWaves;
  const long long grid = want < (long long)n_cu * 2 ? want : (long long)n_cu * 2;
  hipError_t e = launch_group_rows(q.m, q.s, q.U, q.us, q.sp, q.groups, q.tau0, q.n_groups, q.node, q.phi, nullptr,
                                  st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pruner_infer, dim3(static_cast<unsigned>(grid)), dim3(kInferWaves * 64), 0, st, q.m, q.s,
                     q.node, q.phi, q.groups, q.n_groups, q.tau0, q.theta, q.D, q.A, q.B, q.topk, q.rule, q.cand,
                     q.count, q.scores);
  return hipGetLastError();
}

hipError_t launch_scatter_fallback(const int32_t* taus, int n, int tau0, int M, const float* e32, const double* e64,
                                  const double* eu, const int32_t* as, float* o32, double* o64, double* ou,
                                  int32_t* oas, int32_t* fell, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_fallback, dim3(n), dim3(64), 0, st, taus, tau0, M, e32, e64, eu, as, o32, o64, ou,
                     oas, fell);
  return hipGetLastError();
}

hipError_t launch_check_lists(const int32_t* cand, const int32_t* count, long long rows, int M, int kc, int S,
                              int32_t* bad, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_check_lists, dim3(blocks(rows, 4 * kListRows)), dim3(256), 0, st, nullptr, cand, count, rows, M,
                     kc, S, bad);
  return hipGetLastError();
}

hipError_t launch_check_pair_lists(const PairDev* pairs, int n_pairs, long long rows_max, int kc, int32_t* bad,
                                   hipStream_t st) {
  for (int p = 0; rows_max > 0 && p < n_pairs; p += 65535) {  // the grid's limit in y
    const int n = n_pairs - p < 65535 ? n_pairs - p : 65535;
    hipLaunchKernelGGL(k_check_lists, dim3(blocks(rows_max, 4 * kListRows), n), dim3(256), 0, st, pairs + p, nullptr,
                       nullptr, 0ll, 0, kc, 0, bad);
  }
  return hipGetLastError();
}

}  // namespace stm

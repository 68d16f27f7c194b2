// Preparation kernels of the matching path: input validation, the scene
// frame index, candidate lists, the unary table and work counts.
#include <math.h>

#include "stm_internal.h"

namespace stm {
namespace {

constexpr int kBlock = 256;

inline int grid_for(long long n, int block, int cap = 65535 * 4) {
  long long g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return static_cast<int>(g);
}

// ---- validation -------------------------------------------------------------
// bit 0: model frames not strictly increasing; bit 1: scene frames decreasing;
// bit 2: scene frame outside [0, F); bit 3: non-finite model data; bit 4:
// non-finite scene data.
__global__ void k_validate(ModelView m, SceneView s, int32_t* out) {
  const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long stride = (long long)gridDim.x * blockDim.x;
  int32_t bits = 0;
  for (long long i = tid; i < m.M; i += stride) {
    if (i > 0 && m.t[i] <= m.t[i - 1]) bits |= 1;
    const float2 p = m.xy[i];
    if (!isfinite(p.x) || !isfinite(p.y)) bits |= 8;
  }
  for (long long i = tid; i < (long long)m.M * s.dim; i += stride)
    if (!isfinite(m.desc[i])) bits |= 8;
  for (long long i = tid; i < s.S; i += stride) {
    const int32_t ti = s.t[i];
    if (i > 0 && ti < s.t[i - 1]) bits |= 2;
    if (ti < 0 || ti >= s.F) bits |= 4;
    const float2 p = s.xy[i];
    if (!isfinite(p.x) || !isfinite(p.y)) bits |= 16;
  }
  for (long long i = tid; i < (long long)s.S * s.dim; i += stride)
    if (!isfinite(s.desc[i])) bits |= 16;
  if (bits) atomicOr(out, bits);
  if (tid == 0) out[1] = m.t[m.M - 1] - m.t[0];
}

// ---- frame index: fstart[f] = first node with frame >= f, f in [0, F] -------
__global__ void k_fstart(const int32_t* __restrict__ t, int32_t S, int32_t F,
                         int32_t* __restrict__ fstart) {
  const int32_t f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f > F) return;
  int32_t lo = 0, hi = S;
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (t[mid] < f) lo = mid + 1; else hi = mid;
  }
  fstart[f] = lo;
}

// ---- candidate lists (one 64-lane block per offset) ----------------------------
__global__ void k_candidates(ModelView m, SceneView s, SearchParams sp, int32_t tau0,
                             int32_t* __restrict__ cand, int32_t* __restrict__ count) {
  const int32_t tl = blockIdx.x, lane = threadIdx.x;
  const int32_t tau = tau0 + tl;
  for (int32_t i = 0; i < m.M; ++i) {
    const CandRange c = point_candidates(s.fstart, s.F, tau + m.t[i] - m.t[0], sp);
    const int32_t k = c.k1 + c.k2;
    int32_t* row = cand + ((long long)tl * m.M + i) * sp.K;
    for (int32_t a = lane; a < sp.K; a += 64) row[a] = a < k ? cand_node(c, a) : -1;
    if (lane == 0) count[(long long)tl * m.M + i] = k;
  }
}

// ---- unary table U[i][n] = ||f_i - g_n|| in FP32 (Eq. 2) -----------------------
// A workgroup computes 16 R model rows by 16 N scene points, thread (tr, tn) the
// R x N distances of rows tr + 16 j and points tn + 16 j, so that a staged value
// is read once per R or N distances and a thread reads its values four
// dimensions at a time.  Each distance is accumulated over the dimensions in
// ascending order.  Tiles of KT dimensions go through LDS, read a tile ahead.
// Bound by the two VALU instructions per dimension (75 x 31.7k at 162: 31 us
// against 19.5 of issue; with one point per thread and a row value read per
// distance, bound by LDS, 63 us) or, for a table of a few tiles, by their
// latency (20 x 460: 5.5 us, 36 before).
constexpr int kUnaryMaxDim = 256;
constexpr int kUnaryFewBlocks = 128;

template <int R, int N, int KT>
__global__ __launch_bounds__(kBlock) void k_unary_f32(ModelView m, SceneView s, float* __restrict__ U) {
  constexpr int kLd = KT + 4;  // a multiple of 4, odd after division by 4: 16-byte reads of 16 rows hit distinct banks
  constexpr int kRowsPerPass = kBlock / KT;
  constexpr int kRows = 16 * R, kPts = 16 * N;
  constexpr int kRowReads = kRows / kRowsPerPass, kPtReads = kPts / kRowsPerPass;
  __shared__ __align__(16) float fs[kRows][kLd];
  __shared__ __align__(16) float gs[kPts][kLd];
  const int32_t dim = s.dim, tid = threadIdx.x;
  const int32_t i0 = blockIdx.y * kRows, n0 = blockIdx.x * kPts;
  const int32_t tr = tid >> 4, tn = tid & 15;
  const int32_t kk = tid % KT, kr = tid / KT;
  float fr[kRowReads], gr[kPtReads];
  // rows and points past the end read the last one (their results are not
  // stored), dimensions past the end count as 0
  const auto fetch = [&](int32_t d0) {
    const bool dok = d0 + kk < dim;
    const int32_t d = dok ? d0 + kk : 0;
#pragma unroll
    for (int j = 0; j < kRowReads; ++j) {
      const float v = m.desc[(long long)min(i0 + kr + kRowsPerPass * j, m.M - 1) * dim + d];
      fr[j] = dok ? v : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kPtReads; ++j) {
      const float v = s.desc[(long long)min(n0 + kr + kRowsPerPass * j, s.S - 1) * dim + d];
      gr[j] = dok ? v : 0.f;
    }
  };
  float acc[R][N];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < N; ++c) acc[r][c] = 0.f;
  fetch(0);
  for (int32_t d0 = 0; d0 < dim; d0 += KT) {
    __syncthreads();  // the previous tile is consumed
#pragma unroll
    for (int j = 0; j < kRowReads; ++j) fs[kr + kRowsPerPass * j][kk] = fr[j];
#pragma unroll
    for (int j = 0; j < kPtReads; ++j) gs[kr + kRowsPerPass * j][kk] = gr[j];
    __syncthreads();
    if (d0 + KT < dim) fetch(d0 + KT);
#pragma unroll 2
    for (int k = 0; k < KT; k += 4) {
      float4 f[R], g[N];
#pragma unroll
      for (int r = 0; r < R; ++r) f[r] = *reinterpret_cast<const float4*>(&fs[tr + 16 * r][k]);
#pragma unroll
      for (int c = 0; c < N; ++c) g[c] = *reinterpret_cast<const float4*>(&gs[tn + 16 * c][k]);
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const float a0 = f[r].x - g[c].x, a1 = f[r].y - g[c].y, a2 = f[r].z - g[c].z, a3 = f[r].w - g[c].w;
          acc[r][c] = fmaf(a3, a3, fmaf(a2, a2, fmaf(a1, a1, fmaf(a0, a0, acc[r][c]))));
        }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int32_t i = i0 + tr + 16 * r, n = n0 + tn + 16 * c;
      if (i < m.M && n < s.S) U[(long long)i * s.S + n] = sqrtf(acc[r][c]);
    }
}

// ---- model angles of the triangle ending at point i (FP64, then rounded) ------
// theta[i] = (angle at i-1 of (i, i-1, i-2), angle at i of (i-1, i, i-2)),
// oriented, 0 for a zero-length side (Eq. 6).
__device__ __forceinline__ void model_angle(const float2* __restrict__ xy, int32_t i, float2* __restrict__ theta) {
  if (i < 2) { theta[i] = make_float2(0.f, 0.f); return; }
  const float2 pi = xy[i], pj = xy[i - 1], pk = xy[i - 2];
  const double mid = ang64(pi.x, pi.y, pj.x, pj.y, pk.x, pk.y);
  const double end = ang64(pj.x, pj.y, pi.x, pi.y, pk.x, pk.y);
  theta[i] = make_float2(static_cast<float>(mid), static_cast<float>(end));
}

__global__ void k_model_angles(ModelView m, float2* __restrict__ theta) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m.M) model_angle(m.xy, i, theta);
}

// Several models in one launch (model blockIdx.y): each is a few microseconds
// of latency, so fifty launches took 97 us and one takes 3.
constexpr int kAngleModels = 64;  // models per launch, passed as kernel arguments
struct AngleModels {
  const float2* xy[kAngleModels];
  long long row[kAngleModels];
  int32_t M[kAngleModels];
};
__global__ void k_models_angles(AngleModels m, float2* __restrict__ theta) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x, q = blockIdx.y;
  if (i < m.M[q]) model_angle(m.xy[q], i, theta + m.row[q]);
}

// ---- work counts (one 64-lane block per offset) --------------------------------
__global__ void k_count(ModelView m, SceneView s, SearchParams sp, int32_t tau0,
                        unsigned long long* __restrict__ counts) {
  __shared__ int32_t tt[3][64];
  __shared__ int32_t nn[3][64];  // node ids (node-order causality)
  __shared__ int32_t kk[3];
  const int32_t tau = tau0 + blockIdx.x, lane = threadIdx.x;
  unsigned long long dc = 0, fc = 0, dr = 0, fr = 0;
  for (int32_t i = 0; i < m.M; ++i) {
    const CandRange c = point_candidates(s.fstart, s.F, tau + m.t[i] - m.t[0], sp);
    const int32_t k = c.k1 + c.k2;
    __syncthreads();
    if (lane < k) {
      tt[i % 3][lane] = s.t[cand_node(c, lane)];
      nn[i % 3][lane] = cand_node(c, lane);
    }
    if (lane == 0) kk[i % 3] = k;
    __syncthreads();
    if (i >= 1) {
      const int32_t kp = kk[(i - 1) % 3], kc = kk[i % 3];
      const int32_t T = pair_limit(sp), TS = span_limit(sp);
      // lane = candidate r of point i-1
      if (lane < kp) {
        const int32_t tr = tt[(i - 1) % 3][lane], nr = nn[(i - 1) % 3][lane];
        const int32_t* tcur = tt[i % 3];
        const int32_t* ncur = nn[i % 3];
        int32_t na = 0;
        for (int32_t a = 0; a < kc; ++a) na += consecutive_ok(sp, T, nr, tr, ncur[a], tcur[a]);
        dc += kc;
        fc += na;
        if (i >= 2) {
          const int32_t kq = kk[(i - 2) % 3];
          const int32_t* tprev = tt[(i - 2) % 3];
          const int32_t* nprev = nn[(i - 2) % 3];
          dr += (unsigned long long)kq * kc;
          if (TS <= 0) {
            int32_t nk = 0;
            for (int32_t q = 0; q < kq; ++q) nk += consecutive_ok(sp, T, nprev[q], tprev[q], nr, tr);
            fr += (unsigned long long)nk * na;
          } else {
            // span reading: for each admissible predecessor, the admissible
            // columns less than TS frames after it (frames ascend, so the
            // bound only moves forward)
            int32_t a = 0, n_below = 0;
            for (int32_t q = 0; q < kq; ++q) {
              if (!admissible(tprev[q], tr, T)) continue;
              for (; a < kc && tcur[a] - tprev[q] < TS; ++a) n_below += admissible(tr, tcur[a], T);
              fr += n_below;
            }
          }
        }
      }
    }
  }
  // wave reductions, then one atomic per counter
  for (int off = 32; off > 0; off >>= 1) {
    dc += __shfl_xor(dc, off);
    fc += __shfl_xor(fc, off);
    dr += __shfl_xor(dr, off);
    fr += __shfl_xor(fr, off);
  }
  if (lane == 0) {
    atomicAdd(counts + 0, dc);
    atomicAdd(counts + 1, fc);
    atomicAdd(counts + 2, dr);
    atomicAdd(counts + 3, fr);
  }
}

}  // namespace

hipError_t launch_validate(const ModelView& m, const SceneView& s, int32_t* out, hipStream_t st) {
  const long long n = (long long)(m.M > s.S ? m.M : s.S) * (s.dim > 1 ? s.dim : 1);
  hipLaunchKernelGGL(k_validate, dim3(grid_for(n, kBlock, 4096)), dim3(kBlock), 0, st, m, s, out);
  return hipGetLastError();
}

hipError_t launch_fstart(const int32_t* t, int32_t S, int32_t F, int32_t* fstart, hipStream_t st) {
  hipLaunchKernelGGL(k_fstart, dim3(grid_for((long long)F + 1, kBlock)), dim3(kBlock), 0, st, t, S, F,
                     fstart);
  return hipGetLastError();
}

hipError_t launch_candidates(const ModelView& m, const SceneView& s, const SearchParams& sp,
                             int32_t tau0, int32_t n_tau, int32_t* cand, int32_t* count,
                             hipStream_t st) {
  if (n_tau <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_candidates, dim3(n_tau), dim3(64), 0, st, m, s, sp, tau0, cand, count);
  return hipGetLastError();
}

hipError_t launch_unary_f32(const ModelView& m, const SceneView& s, float* U, hipStream_t st) {
  if (s.dim > kUnaryMaxDim) return hipErrorInvalidValue;
  // Few tiles (a short scene, a block of one): 16 x 16 distances per workgroup
  // and 64 dimensions at a time, since the chain of tiles bounds it, not the
  // arithmetic.  us small / large by tiles of the large kind, 75 rows at 162
  // dimensions: 63 9.5 / 23.2, 125 14.1 / 23.8, 188 19.4 / 24.6, 250 24.5 / 25.6,
  // 500 45.5 / 31.6; at 16 dimensions 125 6.2 / 7.0, 188 8.2 / 7.4.  Otherwise the fewest row tiles times (R + 1): the arithmetic
  // of a tile grows with R, its reads of the scene do not.
  const auto blocks = [&](int rows, int pts) { return (long long)((m.M + rows - 1) / rows) * ((s.S + pts - 1) / pts); };
  int best = 5;
  const auto cost = [&](int r) { return (long long)((m.M + 16 * r - 1) / (16 * r)) * (r + 1); };
  for (int r = 4; r >= 1; --r)
    if (cost(r) < cost(best)) best = r;
#define STM_UNARY(R, N, KT)                                                                                  \
  hipLaunchKernelGGL((k_unary_f32<R, N, KT>), dim3((s.S + 16 * N - 1) / (16 * N), (m.M + 16 * R - 1) / (16 * R)), \
                     dim3(kBlock), 0, st, m, s, U)
  if (blocks(16 * best, 64) < kUnaryFewBlocks) STM_UNARY(1, 1, 64);
  else if (best == 5) STM_UNARY(5, 4, 32);
  else if (best == 4) STM_UNARY(4, 4, 32);
  else if (best == 3) STM_UNARY(3, 4, 32);
  else if (best == 2) STM_UNARY(2, 4, 32);
  else STM_UNARY(1, 4, 32);
#undef STM_UNARY
  return hipGetLastError();
}

hipError_t launch_model_angles(const ModelView& m, float2* theta, hipStream_t st) {
  hipLaunchKernelGGL(k_model_angles, dim3((m.M + 63) / 64), dim3(64), 0, st, m, theta);
  return hipGetLastError();
}

hipError_t launch_models_angles(const ModelView* m, const long long* row, int n, float2* theta, hipStream_t st) {
  for (int q0 = 0; q0 < n; q0 += kAngleModels) {
    AngleModels a{};
    const int k = n - q0 < kAngleModels ? n - q0 : kAngleModels;
    int32_t m_max = 1;
    for (int q = 0; q < k; ++q) {
      a.xy[q] = m[q0 + q].xy;
      a.row[q] = row[q0 + q];
      a.M[q] = m[q0 + q].M;
      m_max = a.M[q] > m_max ? a.M[q] : m_max;
    }
    hipLaunchKernelGGL(k_models_angles, dim3((m_max + 63) / 64, k), dim3(64), 0, st, a, theta);
  }
  return hipGetLastError();
}

hipError_t launch_count(const ModelView& m, const SceneView& s, const SearchParams& sp,
                        int32_t tau0, int32_t n_tau, unsigned long long* counts, hipStream_t st) {
  if (n_tau <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_count, dim3(n_tau), dim3(64), 0, st, m, s, sp, tau0, counts);
  return hipGetLastError();
}

}  // namespace stm

// The paper's own matching problem (Section 2.2): one trellis per (model,
// scene block) in which every model point may take any node of the block,
// pruned only by causality and closeness (Eq. 7, 8), whose consequences are
// the loop bounds of Section 3.4: with the block's nodes sorted by frame, the
// successors of a node (frames in (t, t + T)) and its predecessors (frames in
// (t - T, t)) are contiguous node ranges.
//
// Band layout.  A cell is a pair (r, c) of consecutive assignments with c a
// successor of r; the cells are numbered row after row (rowoff[r] + c -
// s_lo[r]), which is the layout of every step's value table V_i and of the
// cells' own directions A(r, c) = -phi(r -> c).  The (a_{i-2}, a_i) directions
// C(k, c) are needed for pairs two admissible steps apart (2 <= t_c - t_k <=
// 2T - 2), numbered row after row by k (qoff[k] + c - q_lo[k]); under the span
// reading of closeness a pair T or more frames apart holds +inf, which takes
// its terms out of every minimum.  The band and both direction tables depend
// on the scene block only and are built once.
//
// One launch per step i computes V_i from V_{i-1} for every model.  Wide bands
// and launches of few workgroups run k_trellis_wide.
// Otherwise a workgroup takes one tile, a rectangle of rows [r0, r1) by columns [c0, c1)
// holding at most 1024 cells (narrow bands: up to 64 consecutive rows whose
// successors span at most 128 nodes; wide bands: 32 rows by a 32-column
// window, so that a staged predecessor serves 32 rows and 32 columns), or at
// most 256 (8 rows by 32 columns) when 1024-cell tiles would give a launch few
// workgroups, thread t taking cells t, t + 256, ...  The predecessors of the
// tile's rows, a contiguous node range, are staged 20 or 24 at a time in LDS: the
// previous values with their directions va[k][r] (+inf where k is no
// predecessor of r) and the directions C[k][c] of the window's columns.  A
// wave runs over the union of its lanes' predecessor ranges; a lane outside
// its own range reads +inf, so the union changes no minimum.
//
// The last step's first row-major minimum is the optimum; backtracking
// recomputes each step's terms of the optimal cell over its predecessors with
// the same arithmetic (dp_math.h) and keeps the lowest node on ties.
#include <math.h>

#include "dp_math.h"
#include "stm_internal.h"

namespace stm {
namespace {

constexpr int kThreads = 256;                    // threads of a step workgroup
// Predecessors staged in LDS at a time and the occupancy target of a staged step
// launch: launches of many workgroups (several per CU) take 20 at a time at six
// waves per SIMD (80 registers), smaller ones 24 at five (50 models, rows of 376
// cells: 40.2 ms against 42.6 with 24 and 47.5 with 32 at four waves).
constexpr int kChunkWide = 20, kWavesWide = 6;    // launches of >= kManyTiles workgroups
constexpr int kChunkSmall = 24, kWavesSmall = 5;
constexpr int kManyTiles = 1024;

// First index of the ascending a[0..n) whose value is >= x (n if none).
__device__ __forceinline__ int32_t lower_bound64(const int32_t* __restrict__ a, int32_t n, long long x) {
  int32_t lo = 0, hi = n;
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if ((long long)a[mid] < x) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// A cell's value at step 1, l1 U_0(r) + l1 U_1(c) + l2 |dt_model - dt_scene|, and
// at a later step, l1 U_i(c) + q_w |dt_model - dt_scene| + the minimum over the
// predecessors; the roundings are spelled out so that every kernel that forms a
// value gives the same bits.
__device__ __forceinline__ float first_value(const TrellisRun& a, float u0, float u1, int32_t dtm, int32_t dts) {
  return fmaf(a.lambda2, fabsf(static_cast<float>(dtm - dts)), fmaf(a.lambda1, u1, __fmul_rn(a.lambda1, u0)));
}
__device__ __forceinline__ float step_value(float cu, float qw, int32_t dtm, int32_t dts, float best) {
  return fmaf(qw, fabsf(static_cast<float>(dtm - dts)), cu) + best;
}

// ---- the band of a scene block -------------------------------------------------
__global__ __launch_bounds__(256) void k_trellis_band(const int32_t* __restrict__ t, int32_t n, SearchParams sp,
                                                      TrellisBand b) {
  const int32_t r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n) return;
  const long long tr = t[r];
  const int32_t T = pair_limit(sp);
  const int32_t slo = lower_bound64(t, n, tr + 1);
  const int32_t shi = T > 0 ? lower_bound64(t, n, tr + T) : n;
  const int32_t qlo = lower_bound64(t, n, tr + 2);
  const int32_t qhi = T > 0 ? lower_bound64(t, n, tr + 2LL * T - 1) : n;
  b.s_lo[r] = slo;
  b.s_hi[r] = shi > slo ? shi : slo;
  b.p_hi[r] = lower_bound64(t, n, tr);
  b.p_lo[r] = T > 0 ? lower_bound64(t, n, tr - T + 1) : 0;
  b.q_lo[r] = qlo;
  b.q_hi[r] = qhi > qlo ? qhi : qlo;
  b.rowoff[r + 1] = shi > slo ? shi - slo : 0;  // widths; the scan makes offsets
  b.qoff[r + 1] = qhi > qlo ? qhi - qlo : 0;
  if (r == 0) {
    b.rowoff[0] = 0;
    b.qoff[0] = 0;
  }
}

// In-place inclusive scan of a[1..n] (a[0] = 0), one workgroup of 1024 threads.
__global__ __launch_bounds__(1024) void k_scan64(long long* __restrict__ a, int32_t n) {
  __shared__ long long wsum[16];
  __shared__ long long carry;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) carry = 0;
  __syncthreads();
  for (int32_t base = 1; base <= n; base += 1024) {
    const int32_t j = base + tid;
    long long v = j <= n ? a[j] : 0;
    for (int off = 1; off < 64; off <<= 1) {
      const long long u = __shfl_up(v, off);
      if (lane >= off) v += u;
    }
    if (lane == 63) wsum[wv] = v;
    __syncthreads();
    long long pre = carry;
    for (int q = 0; q < wv; ++q) pre += wsum[q];
    if (j <= n) a[j] = v + pre;
    __syncthreads();
    if (tid == 1023) carry = pre + v;
    __syncthreads();
  }
}

// Bases of the rows in the value and direction tables: cell (k, r) is base[2 k]
// + r, pair (k, c) is base[2 k + 1] + c.
__global__ __launch_bounds__(256) void k_trellis_bases(TrellisBand b, int32_t n) {
  const int32_t k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  b.base[2LL * k] = b.rowoff[k] - b.s_lo[k];
  b.base[2LL * k + 1] = b.qoff[k] - b.q_lo[k];
}

// Directions of the block: A (blockIdx.y = 0) over the cells of row r =
// blockIdx.x, C (blockIdx.y = 1) over the two-step pairs of row k = blockIdx.x.
// Coincident points give NaN and raise *flag; span-excluded C pairs are +inf.
__global__ __launch_bounds__(64) void k_trellis_dirs(TrellisBand b, const float2* __restrict__ xy,
                                                    const int32_t* __restrict__ t, int32_t span_lim,
                                                    int32_t* __restrict__ flag) {
  const int32_t r = blockIdx.x;
  const float2 pr = xy[r];
  int32_t same = 0;
  if (blockIdx.y == 0) {
    const int32_t lo = b.s_lo[r], hi = b.s_hi[r];
    float* out = b.A + b.rowoff[r] - lo;
    for (int32_t c = lo + threadIdx.x; c < hi; c += 64) {
      const float2 pc = xy[c];
      same |= pc.x == pr.x && pc.y == pr.y;
      out[c] = neg_dir<true>(pr, pc);
    }
  } else {
    const int32_t lo = b.q_lo[r], hi = b.q_hi[r];
    float* out = b.C + b.qoff[r] - lo;
    const int32_t tk = t[r];
    for (int32_t c = lo + threadIdx.x; c < hi; c += 64) {
      if (!span_ok(tk, t[c], span_lim)) {
        out[c] = __builtin_inff();
        continue;
      }
      const float2 pc = xy[c];
      same |= pc.x == pr.x && pc.y == pr.y;
      out[c] = neg_dir<true>(pr, pc);
    }
  }
  if (same) atomicOr(flag, 1);
}

// ---- the steps --------------------------------------------------------------------
// V_1(r, c) = l1 U_0(r) + l1 U_1(c) + l2 Delta(1, 0), row r = blockIdx.x of
// model blockIdx.y.
__global__ __launch_bounds__(64) void k_trellis_first(TrellisRun a) {
  const int32_t r = blockIdx.x;
  const TrellisModel md = a.models[blockIdx.y];
  const int32_t lo = a.band.s_lo[r], hi = a.band.s_hi[r];
  if (lo >= hi) return;
  const float* U0 = md.U;
  const float* U1 = md.U + a.n;
  const int32_t dtm = md.m.t[1] - md.m.t[0];
  const int32_t tr = a.t[r];
  float* out = md.V + a.band.rowoff[r] - lo;
  for (int32_t c = lo + threadIdx.x; c < hi; c += 64) out[c] = first_value(a, U0[r], U1[c], dtm, a.t[c] - tr);
}

template <int KC>
struct StepShared {
  float2 va[KC][kTrellisTileRows];  // (V_{i-1}(k, r), A(k, r)); +inf where k is no predecessor of r
  float ct[KC][kTrellisTileCols];   // C(k, c)
  int32_t plo[kTrellisTileRows], phi[kTrellisTileRows], slo[kTrellisTileRows], tr[kTrellisTileRows];
  int32_t cstart[kTrellisTileRows + 1];  // first tile cell of each row
  int16_t crow[kTrellisTileCells];       // row of each tile cell
  float cu[kTrellisTileCols];            // l1 U_i(c)
  int32_t tc[kTrellisTileCols];
};

// V_i for the tile blockIdx.x of model blockIdx.y (skipped when i >= M); tiles
// of at most SLOTS * 256 cells, SLOTS cells per thread.
template <bool DEGEN, int KC, int WAVES, int SLOTS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(WAVES)))
void k_trellis_step(TrellisRun a, int32_t i) {
  constexpr int kChunk = KC;
  constexpr int kSlots = SLOTS;  // cells per thread
  __shared__ StepShared<KC> sh;
  const TrellisModel md = a.models[blockIdx.y];
  const int32_t M = md.m.M;
  if (i >= M) return;
  const TrellisTile tl = a.tiles[blockIdx.x];
  const int32_t R = tl.r1 - tl.r0, CW = tl.c1 - tl.c0;
  const int tid = threadIdx.x, lane = tid & 63;
  const float INF = __builtin_inff();
  const TrellisBand& b = a.band;
  const float* Ui = md.U + (long long)i * a.n;
  const float* Vp = md.V + (long long)(i - 2) * a.Q;  // V_{i-1}
  float* Vi = md.V + (long long)(i - 1) * a.Q;

  // rows: predecessor and successor ranges, cell counts inside the window
  int32_t cnt = 0;
  if (tid < R) {
    const int32_t r = tl.r0 + tid;
    sh.plo[tid] = b.p_lo[r];
    sh.phi[tid] = b.p_hi[r];
    const int32_t lo = max(b.s_lo[r], tl.c0), hi = min(b.s_hi[r], tl.c1);
    sh.slo[tid] = lo;
    sh.tr[tid] = a.t[r];
    cnt = hi > lo ? hi - lo : 0;
  }
  if (tid < CW) {
    const int32_t c = tl.c0 + tid;
    sh.cu[tid] = __fmul_rn(a.lambda1, Ui[c]);
    sh.tc[tid] = a.t[c];
  }
  if (tid < 64) {  // R <= 64: one wave scans the counts
    int32_t incl = cnt;
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t u = __shfl_up(incl, off);
      if (lane >= off) incl += u;
    }
    if (tid < R) sh.cstart[tid] = incl - cnt;
    if (tid == 63) sh.cstart[R] = incl;  // = tl.ncell
    if (tid < R)
      for (int32_t q = incl - cnt; q < incl; ++q) sh.crow[q] = static_cast<int16_t>(tid);
  }
  __syncthreads();

  const float2 th = md.theta[i];
  const int32_t dtm = md.m.t[i] - md.m.t[i - 1];
  const float qw = a.lambda2 * (i <= M - 2 ? 2.f : 1.f);
  const float w = a.w;
  const int32_t ncell = tl.ncell;
  int rr[kSlots], cc[kSlots];
  float bm[kSlots], be[kSlots], best[kSlots];
  bool same[kSlots];
  int32_t wlo[kSlots], whi[kSlots];  // wave-uniform predecessor union of each slot
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const int32_t cid = tid + kThreads * j;
    const bool valid = cid < ncell;
    const int32_t q = valid ? cid : 0;
    const int row = sh.crow[q];
    const int32_t c = sh.slo[row] + (q - sh.cstart[row]);
    rr[j] = row;
    cc[j] = c - tl.c0;
    best[j] = INF;
    const int32_t r = tl.r0 + row;
    const float arc = b.A[b.rowoff[r] + (c - b.s_lo[r])];
    cell_brackets(th, -arc, bm[j], be[j]);
    const float2 xr = a.xy[r], xc = a.xy[c];
    same[j] = xr.x == xc.x && xr.y == xc.y;
    int32_t lo = valid ? sh.plo[row] : 0x7fffffff, hi = valid ? sh.phi[row] : -1;
    for (int off = 32; off > 0; off >>= 1) {
      lo = min(lo, __shfl_xor(lo, off));
      hi = max(hi, __shfl_xor(hi, off));
    }
    if (hi <= lo) lo = hi = 0;  // no valid lane, or no predecessors: an empty range
    wlo[j] = __builtin_amdgcn_readfirstlane(lo);
    whi[j] = __builtin_amdgcn_readfirstlane(hi);
  }

  // staging: one wave per predecessor row of a table at a time, so that the
  // predecessor k and its band offsets are wave-uniform (scalar loads) and a
  // lane takes one row (va) or one of 64 columns (ct) of the tile
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cgroups = (CW + 63) >> 6;  // 64-column groups of the window: 1 or 2
  for (int32_t k0 = tl.k0; k0 < tl.k1; k0 += kChunk) {
    const int32_t nk = min(kChunk, tl.k1 - k0);
    // rows kk = wv, wv + 4, ... of the chunk: every read of a table (of both
    // tables with one cell per thread, whose registers allow it) is issued
    // before the first store (fixed trip counts, unrolled; a lane without a
    // value reads index 0 and stores the default), so that a chunk waits for
    // one or two rounds of reads instead of one per row
    constexpr int kWaves = kThreads / 64;
    constexpr int kPerWave = kChunk / kWaves;
    static_assert(kChunk % kWaves == 0, "staged rows split evenly over the waves");
    float2 sv[kPerWave];
    bool okv[kPerWave];
#pragma unroll
    for (int s = 0; s < kPerWave; ++s) {
      const int kk = wv + kWaves * s;
      const int32_t k = kk < nk ? k0 + kk : tl.k1 - 1;  // wave-uniform, inside the band
      okv[s] = kk < nk && lane < R && k >= sh.plo[lane] && k < sh.phi[lane];
      const long long off = okv[s] ? b.rowoff[k] + (tl.r0 + lane - b.s_lo[k]) : 0;
      sv[s] = make_float2(Vp[off], b.A[off]);
    }
    const auto store_va = [&]() {
#pragma unroll
      for (int s = 0; s < kPerWave; ++s)
        if (lane < R) sh.va[wv + kWaves * s][lane] = okv[s] ? sv[s] : make_float2(INF, 0.f);
    };
    if constexpr (SLOTS > 1) store_va();
    float sc[kPerWave][2];
    bool okc[kPerWave][2];
#pragma unroll
    for (int s = 0; s < kPerWave; ++s) {
      const int kk = wv + kWaves * s;
      const int32_t k = kk < nk ? k0 + kk : tl.k1 - 1;
      const int32_t qlo = b.q_lo[k], qhi = b.q_hi[k];
      const long long qo = b.qoff[k];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int32_t c = tl.c0 + g * 64 + lane;
        okc[s][g] = kk < nk && g < cgroups && c < tl.c1 && c >= qlo && c < qhi;
        sc[s][g] = b.C[okc[s][g] ? qo + (c - qlo) : 0];
      }
    }
    if constexpr (SLOTS == 1) store_va();
#pragma unroll
    for (int s = 0; s < kPerWave; ++s)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int col = g * 64 + lane;
        if (g < cgroups && col < CW) sh.ct[wv + kWaves * s][col] = okc[s][g] ? sc[s][g] : 0.f;
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      // bounds relative to the chunk, in [0, nk] (an empty range gives hi <= lo)
      const int32_t lo = max(wlo[j], k0) - k0, hi = min(whi[j], k0 + nk) - k0;
      const float2* vcol = &sh.va[0][rr[j]];
      const float* ccol = &sh.ct[0][cc[j]];
      float bj = best[j];
      int32_t kk = lo;
      for (; kk + 7 < hi; kk += 8) {
        const float2 v0 = vcol[kk * kTrellisTileRows], v1 = vcol[(kk + 1) * kTrellisTileRows];
        const float2 v2 = vcol[(kk + 2) * kTrellisTileRows], v3 = vcol[(kk + 3) * kTrellisTileRows];
        const float t0 = relax<DEGEN>(v0.x, v0.y, ccol[kk * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t1 = relax<DEGEN>(v1.x, v1.y, ccol[(kk + 1) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t2 = relax<DEGEN>(v2.x, v2.y, ccol[(kk + 2) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t3 = relax<DEGEN>(v3.x, v3.y, ccol[(kk + 3) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        bj = fminf(fminf(bj, fminf(fminf(t0, t1), t2)), t3);
        const float2 v4 = vcol[(kk + 4) * kTrellisTileRows], v5 = vcol[(kk + 5) * kTrellisTileRows];
        const float2 v6 = vcol[(kk + 6) * kTrellisTileRows], v7 = vcol[(kk + 7) * kTrellisTileRows];
        const float t4 = relax<DEGEN>(v4.x, v4.y, ccol[(kk + 4) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t5 = relax<DEGEN>(v5.x, v5.y, ccol[(kk + 5) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t6 = relax<DEGEN>(v6.x, v6.y, ccol[(kk + 6) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t7 = relax<DEGEN>(v7.x, v7.y, ccol[(kk + 7) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        bj = fminf(fminf(bj, fminf(fminf(t4, t5), t6)), t7);
      }
      if (kk + 3 < hi) {
        const float2 v0 = vcol[kk * kTrellisTileRows], v1 = vcol[(kk + 1) * kTrellisTileRows];
        const float2 v2 = vcol[(kk + 2) * kTrellisTileRows], v3 = vcol[(kk + 3) * kTrellisTileRows];
        const float t0 = relax<DEGEN>(v0.x, v0.y, ccol[kk * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t1 = relax<DEGEN>(v1.x, v1.y, ccol[(kk + 1) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t2 = relax<DEGEN>(v2.x, v2.y, ccol[(kk + 2) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        const float t3 = relax<DEGEN>(v3.x, v3.y, ccol[(kk + 3) * kTrellisTileCols], bm[j], be[j], th, same[j], w);
        bj = fminf(fminf(bj, fminf(fminf(t0, t1), t2)), t3);
        kk += 4;
      }
      for (; kk < hi; ++kk) {
        const float2 v0 = vcol[kk * kTrellisTileRows];
        bj = fminf(bj, relax<DEGEN>(v0.x, v0.y, ccol[kk * kTrellisTileCols], bm[j], be[j], th, same[j], w));
      }
      best[j] = bj;
    }
    __syncthreads();
  }

#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const int32_t cid = tid + kThreads * j;
    if (cid < ncell) {
      const int32_t r = tl.r0 + rr[j], c = tl.c0 + cc[j];
      Vi[b.rowoff[r] + (c - b.s_lo[r])] = step_value(sh.cu[cc[j]], qw, dtm, sh.tc[cc[j]] - sh.tr[rr[j]], best[j]);
    }
  }
}

// ---- wide bands ---------------------------------------------------------------------
// Where a step has many cells per row (no closeness limit, or many points per
// frame), and in launches of few workgroups, a workgroup takes R rows by 64
// columns, lane = column, and its NW waves split the predecessors.  V_{i-1}(k, r)
// and A(k, r) of a predecessor k are wave-uniform: a wave reads those of 64
// predecessors at once and holds them in LDS rows of its own, read back as
// broadcasts; a lane reads one C(k, c) for its R cells.  No barrier but the one
// before the waves' minima meet.  8 rows by 4 waves is bound by the VALU (50 models on
// the whole video without a closeness limit 34.1 ms, one wave instruction per CU
// and cycle (13.7 lane-instructions a relaxation, 10 of them the term's); 36.2
// staged), 4 rows by 8 waves by latency (one model there 1.27 ms; 4.06 staged).
// As scalar loads instead, V and A gave 33.9 and 1.17 ms, but the predecessors of
// only some rows then need a loop of their own, whose chain of scalar loads took
// up to 2.3 ms.  Eight C values ahead instead of four: 35.4 and 1.31 ms.
template <bool DEGEN, int R, int NW>
__global__ __launch_bounds__(NW * 64) void k_trellis_wide(TrellisRun a, int32_t i) {
  // per wave: V and A of 64 predecessors of the R rows; at the end, behind a barrier,
  // the minima of all waves
  __shared__ __align__(16) float stage[NW][64][2 * R];
  const TrellisModel md = a.models[blockIdx.y];
  const int32_t M = md.m.M;
  if (i >= M) return;
  const TrellisTile tl = a.tiles[blockIdx.x];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TrellisBand& b = a.band;
  const float* Vp = md.V + (long long)(i - 2) * a.Q;  // V_{i-1}
  const int32_t c = min(tl.c0 + lane, tl.c1 - 1);
  const float2 th = md.theta[i];
  const float w = a.w;
  const float2 xc = a.xy[c];
  float bm[R], be[R], best[R];
  bool same[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int32_t r = min(tl.r0 + j, tl.r1 - 1);
    // a lane whose column is no successor of r reads another cell's direction
    const long long q = ro(b.base + 2LL * r) + c;
    cell_brackets(th, -b.A[min(max(q, 0LL), a.Q - 1)], bm[j], be[j]);
    const float2 xr = ro(a.xy + r);
    same[j] = xr.x == xc.x && xr.y == xc.y;
    best[j] = __builtin_inff();
  }
  // this wave's predecessors [kb, ke): 64 at a time, lane l reads V and A of
  // predecessor l for the R rows (a chunk ahead of their use; +inf where l is no
  // predecessor of the row, which changes no minimum) and the wave stages them in
  // its own LDS rows; C is read four predecessors ahead
  const int32_t seg = (tl.k1 - tl.k0 + NW - 1) / NW;
  const int32_t kb = min(tl.k0 + wv * seg, tl.k1), ke = min(kb + seg, tl.k1);
  constexpr int kAhead = 4;
  int32_t rj[R], plo[R], phi[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    rj[j] = min(tl.r0 + j, tl.r1 - 1);
    plo[j] = ro(b.p_lo + rj[j]);
    phi[j] = min(ro(b.p_hi + rj[j]), ke);
  }
  float rv[R], ra[R];
  longlong2 bases, bases_next;  // this lane's predecessor's bases in the value and C tables
  const auto fetch_bases = [&](int32_t k0) {
    const int32_t k = min(k0 + lane, ke - 1);
    bases_next.x = b.base[2LL * k];
    bases_next.y = b.base[2LL * k + 1];
  };
  const auto fetch = [&](int32_t k0) {
    bases = bases_next;
    const int32_t k = k0 + lane;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const bool in = k >= plo[j] && k < phi[j];
      const long long q = in ? bases.x + rj[j] : 0;
      const float v = Vp[q];
      ra[j] = b.A[q];
      rv[j] = in ? v : __builtin_inff();
    }
    fetch_bases(k0 + 64);
  };
  if (kb < ke) {
    fetch_bases(kb);
    fetch(kb);
    for (int32_t k0 = kb; k0 < ke; k0 += 64) {
      const int32_t n = min(64, ke - k0);
      float* row = stage[wv][lane];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        row[j] = rv[j];
        row[R + j] = ra[j];
      }
      // C of predecessor k0 + kk: a wave-uniform base, kept as an offset from the
      // first.  Pairs outside the band (of cells or predecessors that do not count)
      // read its neighbours, or the margin of n floats on either side of the table.
      const long long c_first = __shfl(bases.y, 0);
      const int32_t c_rel = static_cast<int32_t>(bases.y - c_first);
      const float* cp = b.C + c_first + c;
      const auto c_at = [&](int32_t kk) { return cp[__builtin_amdgcn_readlane(c_rel, min(kk, n - 1))]; };
      float cn[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) cn[u] = c_at(u);
      if (k0 + 64 < ke) fetch(k0 + 64);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      for (int32_t g = 0; g < n; g += kAhead) {
        float cc[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) cc[u] = cn[u];
        if (g + kAhead < n)
#pragma unroll
          for (int u = 0; u < kAhead; ++u) cn[u] = c_at(g + kAhead + u);
#pragma unroll
        for (int u = 0; u < kAhead; u += 2) {
          const float* s0 = stage[wv][g + u];
          const float* s1 = stage[wv][g + u + 1];
#pragma unroll
          for (int j = 0; j < R; ++j)
            best[j] = fminf(fminf(best[j], relax<DEGEN>(s0[j], s0[R + j], cc[u], bm[j], be[j], th, same[j], w)),
                            relax<DEGEN>(s1[j], s1[R + j], cc[u + 1], bm[j], be[j], th, same[j], w));
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
  float* part = &stage[0][0][0];  // [NW][R][64]
  static_assert(sizeof(stage) >= sizeof(float) * NW * R * 64, "minima in the staging rows");
  __syncthreads();
#pragma unroll
  for (int j = 0; j < R; ++j) part[(wv * R + j) * 64 + lane] = best[j];
  __syncthreads();
  float* Vi = md.V + (long long)(i - 1) * a.Q;
  const int32_t dtm = md.m.t[i] - md.m.t[i - 1];
  const float qw = a.lambda2 * (i <= M - 2 ? 2.f : 1.f);
  const float cu = __fmul_rn(a.lambda1, md.U[(long long)i * a.n + c]);
  for (int j = wv; j < tl.r1 - tl.r0; j += NW) {
    const int32_t r = tl.r0 + j, lo = b.s_lo[r], hi = b.s_hi[r];
    float m = part[j * 64 + lane];
#pragma unroll
    for (int q = 1; q < NW; ++q) m = fminf(m, part[(q * R + j) * 64 + lane]);
    if (tl.c0 + lane < tl.c1 && c >= lo && c < hi)
      Vi[b.rowoff[r] + (c - lo)] = step_value(cu, qw, dtm, a.t[c] - a.t[r], m);
  }
}

// ---- small bands: every step in one launch ------------------------------------------
// When the band's cells and two-step pairs fit one workgroup's LDS (the whole
// video at T = 10: 7.5k cells, 14k pairs), one launch runs steps 1..M-1 with
// V_{i-1}, A and C in LDS and a workgroup barrier between steps, instead of a
// launch per step whose dependent global reads make up most of its time.
//
// A model is split into parts by the second node c of a cell: a part owns columns
// [c0, c1) and, since V_i(r, c) needs V_{i-1}(k, r) of its predecessors r only,
// computes at step i the columns [lim_i, c1) with lim_{M-1} = c0 and lim_{i-1} the
// first predecessor of lim_i.  The columns before c0 are computed by several
// parts, but no part waits for another: the launch needs no barrier across
// workgroups and a few models fill the chip.  In LDS the cells lie by column, so
// that the columns of a part are one slice and the predecessors of a node are
// adjacent: a term is two LDS reads at running addresses and its arithmetic.  The
// threads take the cells by row, as the value tables hold them: the lanes of one
// row read the same V and A (by column, the reads met in a quarter of the banks:
// 198 us).  Bound by the LDS latency of the short predecessor loops (the whole
// video at T = 10, 50 models in 5 parts: 172 us for 28 steps of at most 2.9k cells
// a part, against 336 with one part a model and an offset table read per term).
constexpr int kFusedThreads = 1024;
constexpr int kFusedSlots = 8;                                   // cells per thread
constexpr int kFusedLds = 160 * 1024 - 512;                      // bytes of the LDS pool

constexpr long long fused_bytes(long long Q, long long QC, long long m_max) { return 8 * Q + 4 * QC + 16 * (m_max + 1); }

// A barrier for data exchanged through LDS only: __syncthreads() would also wait
// for the value tables' stores, which no wave of the launch reads.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <bool DEGEN>
__global__ __launch_bounds__(kFusedThreads) void k_trellis_fused(TrellisRun a) {
  __shared__ __align__(16) unsigned char pool[kFusedLds];
  const TrellisModel md = a.models[blockIdx.y];
  const int32_t M = md.m.M;
  const TrellisBand& b = a.band;
  const TrellisColumns& cb = a.cols;
  const int2 own = cb.own[blockIdx.x];
  const int32_t* lim = cb.lim + (long long)blockIdx.x * cb.lim_stride;  // lim[d] = lim_{M-1-d}
  const int32_t cmin = lim[M - 2], c1 = own.y, rmin = b.p_lo[cmin];
  const int32_t q0 = cb.pb[cmin], x0 = cb.qb[cmin];
  const int32_t n_cells = cb.pb[c1] - q0, n_pairs = cb.qb[c1] - x0;
  // the part's rows, whole: cells [row0, row0 + n_row) of the band, some of them outside the part's columns
  const int32_t row0 = static_cast<int32_t>(b.rowoff[rmin]), n_row = static_cast<int32_t>(b.rowoff[c1]) - row0;
  const int tid = threadIdx.x;
  const float INF = __builtin_inff();
  float2* VA = reinterpret_cast<float2*>(pool);           // (V_{i-1}, A) of the part's cells, by column
  float* C = reinterpret_cast<float*>(VA + n_cells);      // C of its two-step pairs, by column
  // of every step: the model angles, frame gap and first live column
  struct Step {
    float2 th;
    int32_t dtm, live;
  };
  Step* steps = reinterpret_cast<Step*>(pool + kFusedLds) - M;
  for (int32_t i = tid; i < M; i += kFusedThreads)
    steps[i] = i < 2 ? Step{make_float2(0.f, 0.f), 0, 0}
                     : Step{md.theta[i], md.m.t[i] - md.m.t[i - 1], lim[M - 1 - i]};
  for (int32_t q = tid; q < n_cells; q += kFusedThreads) VA[q].y = cb.At[q0 + q];
  for (int32_t q = tid; q < n_pairs; q += kFusedThreads) C[q] = cb.Ct[x0 + q];

  // the thread's cells and step 1: V_1(r, c) = l1 (U_0(r) + U_1(c)) + l2 |dt|.
  // Packed in 16 bits each (at most 8192 cells and 40.8k pairs): the places of
  // the first predecessor's cell (k, r) in VA and pair (k, c) in C, the cell's own
  // place in VA, the number of predecessors.  Cells outside the part's columns
  // have column -1.
  uint32_t at[kFusedSlots], me[kFusedSlots];
  int32_t cc[kFusedSlots], dt[kFusedSlots];
  float arc[kFusedSlots], nv[kFusedSlots];
  uint32_t same = 0;  // bit j: the points of cell j coincide
  const int32_t dtm1 = md.m.t[1] - md.m.t[0];
#pragma unroll
  for (int j = 0; j < kFusedSlots; ++j) {
    const int32_t x = tid + kFusedThreads * j;
    at[j] = me[j] = 0;
    cc[j] = -1;
    dt[j] = 0;
    arc[j] = nv[j] = 0.f;
    if (x < n_row) {
      const int32_t r = cb.row[row0 + x], c = b.s_lo[r] + (row0 + x - static_cast<int32_t>(b.rowoff[r]));
      if (c >= cmin && c < c1) {
        // (a row before cmin has its predecessors outside the part: its cells are needed at step 1 only)
        const int32_t k = b.p_lo[r], n_pred = r >= cmin ? b.p_hi[r] - k : 0;
        if (n_pred > 0)
          at[j] = static_cast<uint32_t>(cb.pb[r] - q0) | static_cast<uint32_t>(cb.qb[c] - x0 + (k - cb.qp_lo[c])) << 16;
        me[j] = static_cast<uint32_t>(cb.pb[c] - q0 + (r - b.p_lo[c])) | static_cast<uint32_t>(n_pred) << 16;
        cc[j] = c;
        dt[j] = a.t[c] - a.t[r];
        arc[j] = b.A[row0 + x];
        if (DEGEN) {
          const float2 xr = a.xy[r], xc = a.xy[c];
          if (xr.x == xc.x && xr.y == xc.y) same |= 1u << j;
        }
        const float v = first_value(a, md.U[r], md.U[a.n + c], dtm1, dt[j]);
        VA[me[j] & 0xffffu].x = v;
        if (c >= own.x) md.V[row0 + x] = v;
      }
    }
  }
  float u[kFusedSlots];  // U of the cells' columns, read a step ahead
  const auto read_u = [&](int32_t i) {
    const float* Ui = md.U + (long long)i * a.n;
#pragma unroll
    for (int j = 0; j < kFusedSlots; ++j)
      if (cc[j] >= 0) u[j] = Ui[cc[j]];
  };
  if (M > 2) read_u(2);
  lds_barrier();

  for (int32_t i = 2; i < M; ++i) {
    const Step st = steps[i];
    const float2 th = st.th;
    const int32_t dtm = st.dtm, live = st.live;  // columns from `live` on are needed
    const float qw = a.lambda2 * (i <= M - 2 ? 2.f : 1.f);
    float* Vi = md.V + (long long)(i - 1) * a.Q + row0;
#pragma unroll
    for (int j = 0; j < kFusedSlots; ++j) {
      if (cc[j] >= live) {
        const float cu = __fmul_rn(a.lambda1, u[j]);
        float bm, be;
        cell_brackets(th, -arc[j], bm, be);
        const float2* va = VA + (at[j] & 0xffffu);
        const float* cx = C + (at[j] >> 16);
        const bool sm = same >> j & 1u;
        float best = INF;
        const int32_t n_pred = me[j] >> 16;
        int32_t k = 0;
        for (; k + 1 < n_pred; k += 2) {
          const float2 v0 = va[k], v1 = va[k + 1];
          const float t0 = relax<DEGEN>(v0.x, v0.y, cx[k], bm, be, th, sm, a.w);
          const float t1 = relax<DEGEN>(v1.x, v1.y, cx[k + 1], bm, be, th, sm, a.w);
          best = fminf(fminf(best, t0), t1);
        }
        if (k < n_pred) {
          const float2 v0 = va[k];
          best = fminf(best, relax<DEGEN>(v0.x, v0.y, cx[k], bm, be, th, sm, a.w));
        }
        nv[j] = step_value(cu, qw, dtm, dt[j], best);
      }
    }
    if (i + 1 < M) read_u(i + 1);
    lds_barrier();  // every read of V_{i-1} done
#pragma unroll
    for (int j = 0; j < kFusedSlots; ++j)
      if (cc[j] >= live) {
        VA[me[j] & 0xffffu].x = nv[j];
        if (cc[j] >= own.x) Vi[tid + kFusedThreads * j] = nv[j];
      }
    lds_barrier();
  }
}

// The direction tables by column: cell (k, c) and pair (k, c) of column c =
// blockIdx.x, k ascending.
__global__ __launch_bounds__(64) void k_trellis_columns(TrellisBand b, TrellisColumns cb) {
  const int32_t c = blockIdx.x;
  for (int32_t q = cb.pb[c] + threadIdx.x; q < cb.pb[c + 1]; q += 64) {
    const int32_t k = b.p_lo[c] + (q - cb.pb[c]);
    cb.At[q] = b.A[b.base[2LL * k] + c];
  }
  for (int32_t q = cb.qb[c] + threadIdx.x; q < cb.qb[c + 1]; q += 64) {
    const int32_t k = cb.qp_lo[c] + (q - cb.qb[c]);
    cb.Ct[q] = b.C[b.base[2LL * k + 1] + c];
  }
}

// ---- optimum and backtracking, one workgroup per model ---------------------------
// Backtracking is a chain of dependent reads, one per step: the nodes' ranges and
// bases are held in LDS (up to kFinalNodes nodes), a cell's own direction comes
// from the lane that chose it, and only the predecessors' values and directions
// are read from memory.  One wave walks bands of at most 64 predecessors per
// node; wider ones are split over the workgroup's waves (one model on the whole
// video without a closeness limit: 378 -> 108 us; 50 models at T = 10: 53 -> 31).
constexpr int kFinalThreads = 1024;
constexpr int kFinalNodes = 4096;

template <bool DEGEN>
__global__ __launch_bounds__(kFinalThreads) void k_trellis_final(TrellisRun a) {
  constexpr int kWaves = kFinalThreads / 64;
  __shared__ int4 nodes[kFinalNodes];  // value base, direction base, predecessors [z, w) of a node
  __shared__ float red_v[2][kWaves], red_a[2][kWaves];
  __shared__ long long red_i[kWaves];
  __shared__ int32_t red_k[2][kWaves];
  __shared__ int32_t row_sh;
  const int32_t q = blockIdx.x;
  const TrellisModel md = a.models[q];
  const int32_t M = md.m.M;
  const TrellisBand& b = a.band;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float INF = __builtin_inff();
  const bool in_lds = a.n <= kFinalNodes;  // (then bases fit 32 bits: at most n^2 / 2 cells)
  int wide = 0;
  for (int32_t k = tid; k < a.n; k += kFinalThreads) {
    const int32_t lo = b.p_lo[k], hi = b.p_hi[k];
    wide |= hi - lo > 64;
    if (in_lds) nodes[k] = make_int4(static_cast<int32_t>(b.base[2LL * k]), static_cast<int32_t>(b.base[2LL * k + 1]), lo, hi);
  }
  // the first row-major minimum of V_{M-1}
  const float* VM = md.V + (long long)(M - 2) * a.Q;
  float bv = INF;
  long long bi = 0x7fffffffffffffffLL;
#pragma unroll 8
  for (long long x = tid; x < a.Q; x += kFinalThreads) {
    const float v = VM[x];
    if (v < bv) { bv = v; bi = x; }  // x ascends: the first minimum of this thread
  }
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(bv, off);
    const long long oi = __shfl_xor(bi, off);
    if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (lane == 0) { red_v[0][wv] = bv; red_i[wv] = bi; }
  wide = __syncthreads_or(wide);
  for (int w2 = 0; w2 < kWaves; ++w2)
    if (red_v[0][w2] < bv || (red_v[0][w2] == bv && red_i[w2] < bi)) { bv = red_v[0][w2]; bi = red_i[w2]; }
  if (tid == 0) a.e32[q] = bv;
  int32_t* out = a.assign + md.assign0;
  if (!(bv < INF)) {
    for (int i = tid; i < M; i += kFinalThreads) out[i] = -1;
    return;
  }
  // the optimal final cell: the row whose cells hold the index
  for (int32_t k = tid; k < a.n; k += kFinalThreads)
    if (b.rowoff[k] <= bi && bi < b.rowoff[k + 1]) row_sh = k;
  __syncthreads();
  if (!wide && wv != 0) return;
  int32_t r = row_sh, c = b.s_lo[r] + static_cast<int32_t>(bi - b.rowoff[r]);
  float arc = b.A[bi];  // the direction of cell (r, c)
  if (tid == 0) {
    out[M - 1] = a.node0 + c;
    out[M - 2] = a.node0 + r;
  }
  const auto node = [&](int32_t k, long long& vb, long long& cb, int32_t& lo, int32_t& hi) {
    if (in_lds) {
      const int4 x = nodes[k];
      vb = x.x;
      cb = x.y;
      lo = x.z;
      hi = x.w;
    } else {
      vb = b.base[2LL * k];
      cb = b.base[2LL * k + 1];
      lo = b.p_lo[k];
      hi = b.p_hi[k];
    }
  };
  const int32_t TS = a.span_lim;
  float2 th = md.theta[M - 1];
  for (int32_t i = M - 1; i >= 2; --i) {
    const float2 th_next = md.theta[i - 1];
    const float* Vp = md.V + (long long)(i - 2) * a.Q;  // V_{i-1}
    float bm, be;
    cell_brackets(th, -arc, bm, be);
    bool same = false;
    if (DEGEN) {
      const float2 xr = a.xy[r], xc = a.xy[c];
      same = xr.x == xc.x && xr.y == xc.y;
    }
    const int32_t tcv = TS > 0 ? a.t[c] : 0;
    long long rvb, rcb;
    int32_t lo, hi;
    node(r, rvb, rcb, lo, hi);
    float tot = INF, ta = 0.f;  // this lane's minimum and the direction of its cell (k, r)
    int32_t bk = 0x7fffffff;
    for (int32_t k = lo + (wide ? tid : lane); k < hi; k += wide ? kFinalThreads : 64) {
      if (!span_ok(TS > 0 ? a.t[k] : 0, tcv, TS)) continue;
      long long vb, cb;
      int32_t l2, h2;
      node(k, vb, cb, l2, h2);
      const float av = b.A[vb + r];
      const float v = relax<DEGEN>(Vp[vb + r], av, b.C[cb + c], bm, be, th, same, a.w);
      if (v < tot) { tot = v; bk = k; ta = av; }  // k ascends: the lowest k of this lane's minimum
    }
    const auto meet = [&](float ov, int32_t ok, float oa) {
      if (ov < tot || (ov == tot && ok < bk)) { tot = ov; bk = ok; ta = oa; }
    };
    if (!wide) {  // one predecessor a lane, k ascending: the first lane of the minimum
      const float m = wave_min(tot);
      const int first = __ffsll(static_cast<long long>(__ballot(tot == m))) - 1;
      bk = __builtin_amdgcn_readlane(bk, first);
      ta = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ta), first));
    } else {
      for (int off = 32; off > 0; off >>= 1) meet(__shfl_xor(tot, off), __shfl_xor(bk, off), __shfl_xor(ta, off));
      const int s = i & 1;  // the buffers alternate: one barrier a step
      if (lane == 0) {
        red_v[s][wv] = tot;
        red_k[s][wv] = bk;
        red_a[s][wv] = ta;
      }
      __syncthreads();
      for (int w2 = 0; w2 < kWaves; ++w2) meet(red_v[s][w2], red_k[s][w2], red_a[s][w2]);
    }
    if (bk == 0x7fffffff) {  // no predecessor: cannot happen on a finite optimum
      for (int j = lane; j < M && wv == 0; j += 64) out[j] = -1;
      return;
    }
    if (tid == 0) out[i - 2] = a.node0 + bk;
    c = r;
    r = bk;
    arc = ta;
    th = th_next;
  }
}

}  // namespace

hipError_t launch_trellis_band(const int32_t* t, int32_t n, const SearchParams& sp, const TrellisBand& b,
                               hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_trellis_band, dim3((n + 255) / 256), dim3(256), 0, st, t, n, sp, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scan64, dim3(1), dim3(1024), 0, st, b.rowoff, n);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_scan64, dim3(1), dim3(1024), 0, st, b.qoff, n);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_trellis_bases, dim3((n + 255) / 256), dim3(256), 0, st, b, n);
  return hipGetLastError();
}

hipError_t launch_trellis_dirs(const TrellisBand& b, int32_t n, const float2* xy, const int32_t* t, int32_t span_lim,
                               int32_t* flag, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_trellis_dirs, dim3(n, 2), dim3(64), 0, st, b, xy, t, span_lim, flag);
  return hipGetLastError();
}

bool trellis_fits_fused(long long Q, long long QC, int32_t m_max) {
  return Q > 0 && Q <= (long long)kFusedThreads * kFusedSlots && fused_bytes(Q, QC, m_max) <= kFusedLds;
}

hipError_t launch_trellis_columns(const TrellisBand& b, const TrellisColumns& c, int32_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_trellis_columns, dim3(n), dim3(64), 0, st, b, c);
  return hipGetLastError();
}

namespace {

template <bool DEGEN>
void launch_step(const TrellisRun& a, int32_t n_tiles, TrellisTiling tiling, int32_t i, hipStream_t st) {
  const dim3 grid(n_tiles, a.n_models);
  // (1024-cell tiles are cut only for launches of many workgroups)
  const bool many = (long long)n_tiles * a.n_models >= kManyTiles;
  constexpr int kS = kTrellisSmallTileCells / kThreads, kL = kTrellisTileCells / kThreads;
  if (tiling == TrellisTiling::kWide8)
    hipLaunchKernelGGL((k_trellis_wide<DEGEN, 8, 4>), grid, dim3(4 * 64), 0, st, a, i);
  else if (tiling == TrellisTiling::kWide4)
    hipLaunchKernelGGL((k_trellis_wide<DEGEN, 4, 8>), grid, dim3(8 * 64), 0, st, a, i);
  else if (tiling == TrellisTiling::kCells1024)
    hipLaunchKernelGGL((k_trellis_step<DEGEN, kChunkWide, kWavesWide, kL>), grid, dim3(kThreads), 0, st, a, i);
  else if (many)
    hipLaunchKernelGGL((k_trellis_step<DEGEN, kChunkWide, kWavesWide, kS>), grid, dim3(kThreads), 0, st, a, i);
  else
    hipLaunchKernelGGL((k_trellis_step<DEGEN, kChunkSmall, kWavesSmall, kS>), grid, dim3(kThreads), 0, st, a, i);
}

}  // namespace

hipError_t launch_trellis_run(const TrellisRun& a, int32_t n_tiles, TrellisTiling tiling, int32_t m_max, bool degen,
                              bool fused, hipStream_t st) {
  if (a.n_models <= 0) return hipSuccess;
  hipError_t e;
  if (fused) {
    if (a.cols.parts < 1) return hipErrorInvalidValue;
    const dim3 grid(a.cols.parts, a.n_models);
    if (degen)
      hipLaunchKernelGGL(k_trellis_fused<true>, grid, dim3(kFusedThreads), 0, st, a);
    else
      hipLaunchKernelGGL(k_trellis_fused<false>, grid, dim3(kFusedThreads), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else if (a.Q > 0) {
    hipLaunchKernelGGL(k_trellis_first, dim3(a.n, a.n_models), dim3(64), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int32_t i = 2; i < m_max && n_tiles > 0; ++i) {
      if (degen) launch_step<true>(a, n_tiles, tiling, i, st);
      else launch_step<false>(a, n_tiles, tiling, i, st);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  const dim3 one(a.n_models), threads(kFinalThreads);
  if (degen)
    hipLaunchKernelGGL(k_trellis_final<true>, one, threads, 0, st, a);
  else
    hipLaunchKernelGGL(k_trellis_final<false>, one, threads, 0, st, a);
  return hipGetLastError();
}

}  // namespace stm

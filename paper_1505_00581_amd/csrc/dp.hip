// The exact min-sum recursion of the matching (Section 2.2), one workgroup per
// (model, scene, offset) matching, with the triplet cost fused into the
// minimisation; backtracking and the FP64 re-score of the result.
//
// The forward pass keeps only running minima: each step's cell values are
// written to device memory, and backtracking (Eq. 12) recomputes, along the
// optimal path only, the minimising predecessor of each step with the same
// arithmetic as the forward pass, so ties resolve to the lowest index.
//
// Forward form of Eq. 10-13.  With a_i the candidate index of model point i:
//   V_1(a_0, a_1) = l1 U_0 + l1 U_1 + Q_1(a_0, a_1)
//   V_i(a_{i-1}, a_i) = l1 U_i(a_i) + Q_i(a_{i-1}, a_i)
//       + min_{a_{i-2}} [ V_{i-1}(a_{i-2}, a_{i-1}) + l2 l3 D^g_i(a_{i-2}, a_{i-1}, a_i) ]
// where Q_i = l2 c_i Delta(i, i-1), +inf unless the pair is admissible (Eq. 7,
// 8), and c_i counts the triangles holding the pair (i, i-1) (2 inside the
// chain, 1 at its ends), so every D^t term of Eq. 4 is charged exactly once.
// The optimum is min V_{M-1}; the argmin a_{i-2} of each step on the optimal
// path is found again during backtracking.
//
// D^g from pairwise directions.  With phi(p -> q) the direction of q - p, the
// oriented angle at b of (a, b, c) is phi(b -> c) - phi(b -> a) mod 2 pi, and
// reversing a direction adds pi.  Hence, for the triangle (i, i-1, i-2) with
// model angles th_mid (at i-1) and th_end (at i):
//   delta_mid = wrap( -phi(z_{i-2} -> z_{i-1}) + [th_mid - pi + phi(z_{i-1} -> z_i)] )
//   delta_end = wrap( -phi(z_{i-2} -> z_i)     + [th_end + phi(z_{i-1} -> z_i)] )
// The first addend depends on (a_{i-2}, a_{i-1}) resp. (a_{i-2}, a_i) and is a
// table of K x K directions; the bracket depends only on the cell (a_{i-1},
// a_i).  So atan2 runs K^2 times per step and the K^3 relaxations need only
// adds, |wrap| via pi - |pi - |x|| (valid for |x| <= 2 pi), a square root,
// fused multiply-adds and a compare.
//
// Layout.  Candidates are sorted by frame, so the rows a_{i-1} of one frame
// share one contiguous range of admissible columns a_i and one contiguous
// range of admissible predecessors a_{i-2} (the paper's loop bounds of
// Section 3.4).  Each step builds a schedule of 64-cell chunks over the
// admissible cells only, frame group by frame group; a lane takes one cell of
// a chunk, the waves take chunks round-robin, and every lane of a chunk shares
// the predecessor loop bounds.  For explicit lists on sparse scenes (about
// one point per frame, lists spanning many frames) a group has only a few
// cells, so the packed variant numbers all cells of a step across the chunks
// and gives lane l of packed chunk p cell 64 p + l, each lane with its own
// predecessor range; the minima, and so every result, are the same.  Per step
// the LDS holds the previous V cells with their directions and the (a_{i-2},
// a_i) direction table; the new cells stay in registers until every wave has
// finished reading, then replace the old ones (list variant: go to a second buffer).
// Only admissible cells are ever read back.
//
// Degenerate triangles.  A zero-length side gives a scene angle of 0 in the
// definition, which the direction form does not reproduce.  The fast variant
// detects coincident points on pairs that can be admissible and flags the
// matching; the flagged matchings are recomputed by the variant that marks
// coincident directions as NaN and substitutes the model angle.
//
// Dummy assignments (Eq. 2).  With dummies every point also has the state
// epsilon at unary cost W^d; a Delta term needs both of its points matched,
// D^g all three, and the constraints bind matched consecutive points only.
// So a triangle holding epsilon adds no D^g, and the cells with epsilon follow
// from the step before without the K^3 loop:
//   V_i(r, c)     = l1 U_i(c) + Q_i(r, c) + min(V_{i-1}(eps, r), min_k [...])
//   V_i(r, eps)   = l1 W^d + min(V_{i-1}(eps, r), min_{k admissible} V_{i-1}(k, r))
//   V_i(eps, c)   = l1 U_i(c) + m_{i-1},   V_i(eps, eps) = l1 W^d + m_{i-1}
// with m_{i-1} = min(V_{i-1}(eps, eps), min_k V_{i-1}(k, eps)).  Each step keeps
// these as two K-vectors and a scalar beside the K x K cells; epsilon is index
// 64 in the final argmin and in backtracking (after every candidate, so ties
// go to candidates) and index K in the value tables, whose rows then have
// K + 1 entries.
//
// Alternative readings.  Unsigned angles (a template variant): the terms
// compare magnitudes, the scene's angles at z_{i-1} and z_i being wrap(pi +
// anew - A) and wrap(anew - C) of the same stored directions (dp_math.h).
// Node-order causality (a run-time switch of the schedule): consecutive points
// take increasing node ids, so within a frame every row has its own columns
// (the nodes above it) and its own predecessors (the nodes below it); every row
// is then a group of its own, its ranges counted from the windowed lists' node
// ranges, and the chunk loop is unchanged.
#include <math.h>

#include "dp_math.h"
#include "stm_internal.h"

namespace stm {
namespace {

constexpr int kMaxList = 64;  // longest candidate list = wavefront lanes
constexpr int kEps = kMaxList;  // index of the dummy state epsilon
constexpr int32_t kDummyNode = -2;  // epsilon in assignments

// A chunk of the cells of one step: the admissible cells (a_{i-1}, a_i) of the
// rows r0.. r0+nr-1 of one frame group, flattened row-major over their common
// column range [clo, clo + nc); the chunk covers flat cells [e0, e0 + 64).  All
// rows of the group share the predecessor range [lo, hi).
struct Chunk {
  int r0, clo, nc, e0, lo, hi, ncell;
};

__device__ __forceinline__ uint2 pack_chunk(int r0, int clo, int nc, int e0, int lo, int hi, int ncell) {
  return make_uint2(static_cast<uint32_t>(r0) | (static_cast<uint32_t>(clo) << 6) |
                        (static_cast<uint32_t>(nc) << 12) | (static_cast<uint32_t>(e0) << 19),
                    static_cast<uint32_t>(lo) | (static_cast<uint32_t>(hi) << 7) |
                        (static_cast<uint32_t>(ncell) << 14));
}

// Decodes a descriptor read from LDS; the fields are wave-uniform, so they are
// moved to scalar registers and the loops over them stay scalar.
__device__ __forceinline__ Chunk unpack_chunk(uint2 d) {
  const uint32_t x = __builtin_amdgcn_readfirstlane(d.x), y = __builtin_amdgcn_readfirstlane(d.y);
  Chunk c;
  c.r0 = x & 63;
  c.clo = (x >> 6) & 63;
  c.nc = (x >> 12) & 127;
  c.e0 = x >> 19;
  c.lo = y & 127;
  c.hi = (y >> 7) & 127;
  c.ncell = y >> 14;
  return c;
}

// Number of entries < x in the ascending list a[0..n).
// Lists hold at most 64 entries, so seven probes at fixed strides suffice; the
// probes do not branch on the data, and independent searches interleave their
// reads.
__device__ __forceinline__ int count_lt(const int32_t* a, int n, int x) {
  if (n <= 0) return 0;
  int pos = 0;
#pragma unroll
  for (int step = 64; step > 0; step >>= 1) {
    const int probe = pos + step;
    const int32_t v = a[(probe <= n ? probe : n) - 1];
    if (probe <= n && v < x) pos = probe;
  }
  return pos;
}

__device__ __forceinline__ float lane_value(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// A cell's value at step 1, (l1 U_0(r) + l1 U_1(c)) + l2 |dt_model - dt_scene|, and
// at a later step, l1 U_i(c) + q_w |dt_model - dt_scene| + the minimum over the
// predecessors.  The roundings are spelled out: left to the compiler, a product
// formed outside the block of its sum (dp_forward_few) is rounded by itself, and
// the layouts differ in the last bit.
__device__ __forceinline__ float first_cell(float cr, float cc, float l2, int dtm, int dts) {
  return fmaf(l2, fabsf(static_cast<float>(dtm - dts)), cr + cc);
}
__device__ __forceinline__ float later_cell(float cu, float qw, int dtm, int dts, float best) {
  return fmaf(qw, fabsf(static_cast<float>(dtm - dts)), cu) + best;
}

// Cell of lane `lane` in chunk c: row r and column a; false past the last cell.
__device__ __forceinline__ bool chunk_cell(const Chunk& c, int lane, int& r, int& a) {
  const int e = c.e0 + lane;
  // e < 4096 and nc <= 64: (e + 1/2) / nc stays >= 1/128 away from an integer,
  // far above the float rounding, so the truncation is the exact quotient.
  const int q = static_cast<int>((static_cast<float>(e) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(c.nc)));
  r = c.r0 + q;
  a = c.clo + (e - q * c.nc);
  return e < c.ncell;
}

// Builds the chunk schedule of one step, run by one wave (lane = row).  Rows
// are the candidates of point i-1 (frames trow, ascending), columns those of
// point i (tcol), predecessors those of point i-2 (tprev, or none for the
// first pair).  The rows of one frame f share the admissible columns (frames in
// (f, f + T)) and predecessors (frames in (f - T, f)).  Each group gives
// ceil(rows * columns / 64) <= rows chunks, so a step has at most K chunks.
// With pstart (packed variant): pstart[j] = number of the first cell of chunk
// j when the step's cells are numbered chunk after chunk, pstart[n] = the
// step's cell count, also stored in *ptot.
__device__ void build_schedule(const int32_t* trow, int nrow, const int32_t* tcol, int ncol,
                               const int32_t* tprev, int nprev, int T, uint2* out, int32_t* nout,
                               int lane, int16_t* pstart, int32_t* ptot, const CandRange* ring, int sr, int sc,
                               int sp) {
  const int f = lane < nrow ? trow[lane] : 0;
  // node-order causality (ring: the windowed node ranges of the candidate
  // ring in LDS, sr, sc, sp: the rows', columns' and predecessors' slots;
  // null for frame order): every row is a group of its own, its columns the
  // nodes above its own within T frames, its predecessors the nodes below it
  // within T frames
  const bool node = ring != nullptr;
  const bool start = lane < nrow && (node || lane == 0 || trow[lane - 1] != f);
  const unsigned long long starts = __ballot(start);
  int nchunk = 0, nr = 0, nc = 0, clo = 0, chi = 0, lo = 0, hi = 0;
  if (node) {
    if (start) {
      const int nd = cand_node(ring[sr], lane);
      clo = range_count_le(ring[sc], nd);
      chi = T > 0 ? count_lt(tcol, ncol, f > 0x7fffffff - T ? 0x7fffffff : f + T) : ncol;
      if (tprev) {
        hi = range_count_lt(ring[sp], nd);
        lo = T > 0 ? count_lt(tprev, nprev, f - T + 1) : 0;
      }
    }
  } else if (__popcll(starts) <= 16) {
    // few frame groups: each lane holds one column and one predecessor frame,
    // and every count is a ballot, one group after the other
    const int32_t tc = lane < ncol ? tcol[lane] : 0x7fffffff;  // frames are < 0x7fffffff
    const int32_t tp = tprev && lane < nprev ? tprev[lane] : 0x7fffffff;
    unsigned long long rem = starts;
    while (rem) {
      const int g = __ffsll(static_cast<long long>(rem)) - 1;
      rem &= rem - 1;
      const int fg = __builtin_amdgcn_readlane(f, g);
      const int c0 = __popcll(__ballot(tc < fg + 1));
      const int c1 = T > 0 ? __popcll(__ballot(tc < (fg > 0x7fffffff - T ? 0x7fffffff : fg + T))) : ncol;
      const int p1 = __popcll(__ballot(tp < fg));
      const int p0 = T > 0 ? __popcll(__ballot(tp < fg - T + 1)) : 0;
      if (lane == g) {
        clo = c0;
        chi = c1;
        hi = p1;
        lo = p0;
      }
    }
  } else if (start) {
    // many groups (sparse scenes): binary searches, one group per lane
    clo = count_lt(tcol, ncol, f + 1);
    chi = T > 0 ? count_lt(tcol, ncol, f > 0x7fffffff - T ? 0x7fffffff : f + T) : ncol;
    if (tprev) {
      hi = count_lt(tprev, nprev, f);
      lo = T > 0 ? count_lt(tprev, nprev, f - T + 1) : 0;
    }
  }
  if (start) {
    const unsigned long long later = starts & ~((2ull << lane) - 1ull);
    const int next = later ? __ffsll(static_cast<long long>(later)) - 1 : nrow;
    nr = next - lane;
    nc = chi > clo ? chi - clo : 0;
    nchunk = (nr * nc + 63) >> 6;
  }
  int incl = nchunk;
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off);
    if (lane >= off) incl += v;
  }
  if (start)
    for (int c = 0; c < nchunk; ++c) out[incl - nchunk + c] = pack_chunk(lane, clo, nc, c * 64, lo, hi, nr * nc);
  const int total = __shfl(incl, 63);
  if (lane == 0) *nout = total;
  if (pstart) {
    int cells = nr * nc;  // inclusive scan of the groups' cell counts
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(cells, off);
      if (lane >= off) cells += v;
    }
    if (start)
      for (int c = 0; c < nchunk; ++c) pstart[incl - nchunk + c] = static_cast<int16_t>(cells - nr * nc + c * 64);
    const int ncells = __shfl(cells, 63);
    if (lane == 0) {
      pstart[total] = static_cast<int16_t>(ncells);
      *ptot = ncells;
    }
  }
}

// Cell 64 p + lane of a packed schedule: its chunk j (the last with pstart[j]
// <= the number), row r, column a and predecessor range [lo, hi).  A number
// past the step's cells decodes cell 0 (in-range reads) and returns false.
__device__ __forceinline__ bool packed_cell(const uint2* sched, const int16_t* pstart, int n_chunks, int n_cells,
                                            int num, int& r, int& a, int& lo, int& hi) {
  const bool valid = num < n_cells;
  const int e_all = valid ? num : 0;
  int j = 0, j1 = n_chunks;  // pstart[j] <= e_all < pstart[j1]
  while (j1 - j > 1) {
    const int mid = (j + j1) >> 1;
    if (pstart[mid] <= e_all) j = mid; else j1 = mid;
  }
  const uint2 d = sched[j];
  const int r0 = d.x & 63, clo = (d.x >> 6) & 63, nc = (d.x >> 12) & 127, e0 = d.x >> 19;
  lo = d.y & 127;
  hi = (d.y >> 7) & 127;
  const int e = e0 + (e_all - pstart[j]);
  const int q = static_cast<int>((static_cast<float>(e) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(nc)));
  r = r0 + q;
  a = clo + (e - q * nc);
  return valid;
}

// Per-step vectors of the dummy state, double-buffered by step parity:
// de[b][c] = V(eps, c), df[b][r] = V(r, eps), dg[b] = V(eps, eps).
template <int KL, bool DUMMY>
struct DummyShared {};
template <int KL>
struct DummyShared<KL, true> {
  float de[2][KL];
  float df[2][KL];
  float dg[2];
};

// The cells of the previous step, [a_{i-2}][a_{i-1}]: (V_{i-1}, -phi(z_{i-2} ->
// z_{i-1})).  The list variant keeps two buffers of values apart from the
// directions, so that a step that keeps the directions of the one before needs no
// barrier between reading and publishing; where every step is built anew the third
// read per term costs more (windowed lists of 64 at one point per frame, 3000
// offsets x 75 points: 9.13 ms, 8.80 with values and directions side by side), so
// the variant is taken for explicit lists of which more than five of seven repeat
// the one before them: 20 models x 678 blocks of 60 nodes whose lists change every
// 3 points 6.19 ms (5.63 without it), every 4 points 5.36 (5.63), never 2.73 (5.65).
template <int KL, bool LISTS>
struct CellShared {
  float2 va[KL * KL];
};
template <int KL>
struct CellShared<KL, true> {
  float v[2][KL * KL];
  float dir[KL * KL];
  int32_t same[8];  // list j (at j & 7) holds the nodes of list j - 1
};
// Packed schedules: the first cell number of every chunk and the step's cell count.
template <int KL, bool PACKED>
struct PackedShared {};
template <int KL>
struct PackedShared<KL, true> {
  int16_t pstart[2][KL + 1];
  int32_t ptot[2];
};

template <int NW, int KL, bool DUMMY = false, bool PACKED = false, bool LISTS = false>
struct DPShared : DummyShared<KL, DUMMY>, CellShared<KL, LISTS>, PackedShared<KL, PACKED> {
  float ct[KL * KL];    // [a_{i-2}][a_i]: -phi(z_{i-2} -> z_i)
  float2 cxy[4][KL];    // candidate ring: coordinates,
  int32_t ctt[4][KL];   //   frames,
  float cu[4][KL];      //   l1 * U
  uint2 sched[2][KL];   // chunk schedules of the current and the previous step
  int32_t nch[2];
  int32_t ck[4];        //   list lengths
  CandRange crange[4];  //   the windowed lists' node ranges (node-order causality)
  int32_t flag;         // coincident points seen (fast variant)
  float red_v[NW];
  int32_t red_i[NW];
  float res_v;
  int32_t res_i;
};

// One matching: a model against a scene at offset tau.
struct MatchView {
  ModelView m;
  SceneView s;
  SearchParams sp;
  const float* U;       // unary table: row j = model point j, row stride us
  long long us;
  const float2* theta;  // model angles of the triangle ending at each point
  float lambda1, lambda2, w;
  float cw;             // l1 * W^d, the unary cost of the dummy
  int vs;               // value-table row length: K, or K + 1 with dummies
  int tau;
  // explicit candidate lists of this matching (null: the windowed rule):
  // point j's nodes are cand[j * cstride + a], a < ccount[j], ascending
  const int32_t* cand;
  const int32_t* ccount;
  int cstride;
};

// Candidate list of point j of a matching: explicit, or the windowed rule.
struct Cands {
  CandRange r;
  const int32_t* list;
  int n;
  __device__ __forceinline__ int count() const { return list ? n : r.k1 + r.k2; }
  __device__ __forceinline__ int node(int a) const { return list ? ro(list + a) : cand_node(r, a); }
};

template <bool LISTS = false>
__device__ __forceinline__ Cands cands_of(const MatchView& a, int j) {
  Cands c;
  if (LISTS || a.cand) {
    c.list = a.cand + (long long)j * a.cstride;
    c.n = ro(a.ccount + j);
    c.r = CandRange{0, 0, 0, 0};
  } else {
    c.list = nullptr;
    c.n = 0;
    c.r = point_candidates(a.s.fstart, a.s.F, a.tau + ro(a.m.t + j) - ro(a.m.t), a.sp);
  }
  return c;
}

// Value table of step i (cells V_i(a_{i-1}, a_i), i = 1..M-2) inside the
// matching's scratch vt [M-2][vs][vs], stored by column: V_i(r, c) at c * vs +
// r, so that backtracking reads the values of one column (every predecessor of
// the chosen cell) contiguously (with dummies, index K holds the epsilon state
// on either side).  By row the stores touch fewer lines, but they are hidden:
// the recursion's launch takes the same 5.50 ms at 1387 offsets x 75 points, K =
// 64, and the backtracking 157 us instead of 121.
__device__ __forceinline__ float* vtable(float* vt, const MatchView& a, int i) {
  return vt + (long long)(i - 1) * a.vs * a.vs;
}
__device__ __forceinline__ const float* vtable(const float* vt, const MatchView& a, int i) {
  return vt + (long long)(i - 1) * a.vs * a.vs;
}

struct DPResult {
  float v;   // optimum (+inf if infeasible)
  int idx;   // r * KL + c of the first minimising final pair (a_{M-2}, a_{M-1});
             // with dummies r * (KL + 1) + c, epsilon = KL
  int flag;  // coincident points seen (fast variant)
};

// Forward pass of one matching by the whole workgroup (NW waves): writes the
// value tables of steps 1..M-2 to vtm and returns the optimum to every thread.
template <int NW, bool DEGEN, int KL, bool DUMMY = false, bool PACKED = false, bool UNS = false, bool LISTS = false>
__device__ __forceinline__ DPResult dp_forward(DPShared<NW, KL, DUMMY, PACKED, LISTS>& sh, const MatchView& a, float* vtm) {
  static_assert(KL == 16 || KL == 64, "list capacity");
  static_assert(!DUMMY || KL == kMaxList, "dummies use the 64-slot layout");
  static_assert(!PACKED || (KL == kMaxList && !DUMMY), "packed schedules: 64-slot layout, no dummies");
  static_assert(!LISTS || PACKED, "list variant: packed schedules");
  constexpr bool RUNS = LISTS && !DEGEN;  // steps whose lists do not change keep their tables
  constexpr int RPW = KL / NW;  // chunk slots per wave (a step has <= KL chunks)
  const int tau = a.tau;
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int M = a.m.M;
  const int T = pair_limit(a.sp);   // consecutive points
  const int TS = span_limit(a.sp);  // first and last points of a triangle (span reading)
  const int Kc = a.sp.K;
  const int VS = a.vs;
  const int tm0 = ro(a.m.t);
  const float INF = __builtin_inff();
  constexpr int kBuilder = NW - 1;  // wave that builds the schedules

  // chunk slots of schedule b, and the cell of this lane in slot ch (packed
  // schedules: cell number 64 ch + lane; lo/hi only set there)
  auto n_slots = [&](int b) {
    if constexpr (PACKED) return (sh.ptot[b] + 63) >> 6;
    else return sh.nch[b];
  };
  auto slot_cell = [&](int b, int ch, int& r, int& col) {
    if constexpr (PACKED) {
      int lo, hi;
      return packed_cell(sh.sched[b], sh.pstart[b], sh.nch[b], sh.ptot[b], ch * 64 + lane, r, col, lo, hi);
    } else {
      return chunk_cell(unpack_chunk(sh.sched[b][ch]), lane, r, col);
    }
  };
  // the same, with an in-range cell for lanes past the last one (their reads)
  auto slot_cell_safe = [&](int b, int ch, int& r, int& col) {
    if constexpr (PACKED) {
      return slot_cell(b, ch, r, col);
    } else {
      const Chunk c = unpack_chunk(sh.sched[b][ch]);
      const bool valid = chunk_cell(c, lane, r, col);
      if (!valid) { r = c.r0; col = c.clo; }  // in-range reads; results unused
      return valid;
    }
  };
  // lists i, i - 1, i - 2 each hold the nodes of the list before them
  auto same_lists = [&](int i) {
    if constexpr (RUNS) {
      const int32_t s = sh.same[i & 7] & sh.same[(i - 1) & 7] & sh.same[(i - 2) & 7];
      return __builtin_amdgcn_readfirstlane(s) != 0;
    } else {
      return false;
    }
  };
  // sr, sc, sp: ring slots of the rows', columns' and predecessors' lists
  auto schedule = [&](int sr, int sc, int spv, int b) {
    const int32_t* trow = sh.ctt[sr];
    const int32_t* tcol = sh.ctt[sc];
    const int32_t* tprev = spv >= 0 ? sh.ctt[spv] : nullptr;
    const int nrow = sh.ck[sr], ncol = sh.ck[sc], nprev = spv >= 0 ? sh.ck[spv] : 0;
    const CandRange* ring = a.sp.node ? sh.crange : nullptr;
    if constexpr (PACKED)
      build_schedule(trow, nrow, tcol, ncol, tprev, nprev, T, sh.sched[b], &sh.nch[b], lane, sh.pstart[b],
                     &sh.ptot[b], ring, sr, sc, spv);
    else
      build_schedule(trow, nrow, tcol, ncol, tprev, nprev, T, sh.sched[b], &sh.nch[b], lane, nullptr, nullptr,
                     ring, sr, sc, spv);
  };

  // The candidates of list j, read by wave 0 in three parts, each a step before
  // the next, so that their latencies overlap the recursions between: fetch_list
  // issues the reads of the list (its frame boundaries, or its nodes),
  // fetch_values those of its nodes' position, frame and unary cost, and
  // commit_slot stores them into ring slot j & 3.
  struct ListRegs {
    Cands c;
    int32_t node;  // explicit lists: this lane's entry
  };
  struct SlotRegs {
    Cands c;
    float2 xy;
    int32_t t;
    float u;
    int32_t node = -1;  // packed: this lane's node, -1 past the list
    bool same = false;  // packed: the list holds the nodes of the list before
  };
  int32_t count_l = 0;  // list variant: the lengths of 64 lists, one per lane
  auto fetch_list = [&](int j) {
    ListRegs l;
    if (wv == 0) {
      if (LISTS) {
        if ((j & 63) == 0) count_l = a.ccount[min(j + lane, M - 1)];
        l.c.list = a.cand + (long long)j * a.cstride;
        l.c.n = __builtin_amdgcn_readlane(count_l, j & 63);
        l.c.r = CandRange{0, 0, 0, 0};
      } else {
        l.c = cands_of(a, j);
      }
      if (l.c.list) l.node = ro(l.c.list + (lane < a.cstride ? lane : 0));
    }
    return l;
  };
  // f: the previous list's values, kept where the lists hold the same nodes
  auto fetch_values = [&](int j, const ListRegs& l, SlotRegs& f) {
    if (wv == 0) {
      f.c = l.c;
      const int n = f.c.list ? l.node : cand_node(f.c.r, lane);
      const bool in = lane < f.c.count();
      if constexpr (RUNS) {
        const int nd = in ? n : -1;
        f.same = j > 0 && __all(nd == f.node);
        f.node = nd;
        if (lane == 0) sh.same[j & 7] = f.same;
      }
      if (in) {
        if (!f.same) {
          f.xy = ro(a.s.xy + n);
          f.t = ro(a.s.t + n);
        }
        f.u = ro(a.U + (long long)j * a.us + n);
      }
    }
  };
  // unary: the slot holds the list's other data already
  auto commit_slot = [&](int j, const SlotRegs& f, bool unary = false) {
    if (wv == 0) {
      const int k = f.c.count();
      const int sl = j & 3;
      if (lane < k) sh.cu[sl][lane] = a.lambda1 * f.u;
      if (unary) return;
      if (lane < k) {
        sh.cxy[sl][lane] = f.xy;
        sh.ctt[sl][lane] = f.t;
      }
      if (lane == 0) {
        sh.ck[sl] = k;
        sh.crange[sl] = f.c.r;
      }
    }
  };

  ListRegs list_next;  // list i + 2 in flight during step i - 1's recursion and step i's phase 1
  SlotRegs next;       // list i + 1's values, likewise
  if (threadIdx.x == 0) sh.flag = 0;
  {
    const ListRegs l0 = fetch_list(0), l1 = fetch_list(1), l2 = fetch_list(2);
    SlotRegs f0, f1, f2;
    fetch_values(0, l0, f0);
    f1 = f0;
    fetch_values(1, l1, f1);
    f2 = f1;
    fetch_values(2, l2, f2);
    next = f2;
    commit_slot(0, f0);
    commit_slot(1, f1);
    commit_slot(2, f2);
  }
  __syncthreads();
  if (wv == kBuilder) schedule(0, 1, -1, 1);
  __syncthreads();
  if (3 < M) fetch_values(3, fetch_list(3), next);
  if (4 < M) list_next = fetch_list(4);

  float vr[RPW], ar[RPW];
  // LDS index (row * KL + column) of each slot's cell, negative: none; packed:
  // in the low 12 bits, then the first predecessor and the count (7 bits each)
  int pi[RPW];
  constexpr int kCell = PACKED ? 0xfff : -1;
  // packed: largest count of the slot's lanes, and kFew if a lane has fewer than
  // four predecessors
  constexpr int kFew = 1 << 8;
  int longest[PACKED ? RPW : 1];
  int b_prev = 1;             // schedule buffer of the previous step
#pragma unroll
  for (int s = 0; s < RPW; ++s) { vr[s] = INF; ar[s] = 0.f; pi[s] = -1; }

  // ---- the first pair (points 0, 1) ------------------------------------------
  {
    const int dtm = ro(a.m.t + 1) - ro(a.m.t);
    const int nch = n_slots(1);
    float* vt = vtable(vtm, a, 1);
#pragma unroll
    for (int s = 0; s < RPW; ++s) {
      const int ch = wv + NW * s;
      if (ch < nch) {
        int r, col;
        const bool valid = slot_cell_safe(1, ch, r, col);
        const int tr = sh.ctt[0][r], tp = sh.ctt[1][col];
        const float2 xr = sh.cxy[0][r], xa = sh.cxy[1][col];
        const bool same = xa.x == xr.x && xa.y == xr.y;
        if (!DEGEN && same && valid) sh.flag = 1;
        vr[s] = first_cell(sh.cu[0][r], sh.cu[1][col], a.lambda2, dtm, tp - tr);
        ar[s] = neg_dir<DEGEN>(xr, xa);
        if (valid) vt[col * VS + r] = vr[s];
        pi[s] = valid ? r * KL + col : -1;
        if constexpr (LISTS) {
          if (valid) sh.v[1][pi[s]] = vr[s];
        }
      }
    }
    if constexpr (DUMMY) {
      if (wv == 0) {
        const float cw = a.cw;
        if (lane < sh.ck[1]) {
          const float e = cw + sh.cu[1][lane];
          sh.de[1][lane] = e;
          vt[lane * VS + Kc] = e;
        }
        if (lane < sh.ck[0]) {
          const float f = sh.cu[0][lane] + cw;
          sh.df[1][lane] = f;
          vt[Kc * VS + lane] = f;
        }
        if (lane == 0) {
          sh.dg[1] = cw + cw;
          vt[Kc * VS + Kc] = cw + cw;
        }
      }
    }
  }

  // Angles and frames of the model points, one point per lane and 64 points at
  // a time, read by readlane (kLanes: where a step is short a scalar read of its
  // point is waited for, 0.9 of 4.6 ms over blocks of 60 nodes without their
  // terms; where the terms fill the step it is hidden).
  constexpr bool kLanes = PACKED || KL < kMaxList;
  float2 th_l = make_float2(0.f, 0.f);
  int32_t tm_l = 0, tm_prev = 0;
  auto load_points = [&](int i0) {
    const int j = min(i0 + lane, M - 1);
    th_l = a.theta[j];
    tm_l = a.m.t[j];
  };
  if constexpr (kLanes) {
    load_points(0);
    tm_prev = __builtin_amdgcn_readlane(tm_l, 1);
  }
  // the angles of point i and its frames since point i - 1
  auto point = [&](int i, float2& th, int& dtm) {
    if constexpr (kLanes) {
      if ((i & 63) == 0) load_points(i);
      th.x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(th_l.x), i & 63));
      th.y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(th_l.y), i & 63));
      const int tm = __builtin_amdgcn_readlane(tm_l, i & 63);
      dtm = tm - tm_prev;
      tm_prev = tm;
    } else {
      th = ro(a.theta + i);
      dtm = ro(a.m.t + i) - ro(a.m.t + (i - 1));
    }
  };

  // Packed cells: the minimum over a lane's predecessors [lo, lo + len) of its
  // cell (row r, column col).  The wave runs to its longest range: four
  // predecessors per trip, the last trip moved back onto the end of the lane's
  // range (a repeated predecessor changes no minimum), one or two left over one
  // at a time; lanes with fewer than four take theirs one by one instead.
  auto packed_min = [&](int vb, int r, int col, int lo, int len, int longest, float bm, float be, float2 th,
                        bool same) {
    float best = INF;
    if constexpr (PACKED) {
      const float* ccol = sh.ct + col;
      const float w = a.w;
      const auto term = [&](int o) {  // the predecessor at offset o = k KL
        float2 c;
        if constexpr (LISTS) c = make_float2(sh.v[vb][o + r], sh.dir[o + r]);
        else c = sh.va[o + r];
        return relax<DEGEN, UNS>(c.x, c.y, ccol[o], bm, be, th, same, w);
      };
      const int n = longest & (kFew - 1);
      const int end = max(lo + len - 1, 0);  // the lane's last predecessor
      const int k1 = max(end - 3, 0), k0 = min(lo, k1);
      int j = 0;
      for (; j + 2 < n; j += 4) {
        const int o = min(k0 + j, k1) * KL;
        const float t0 = term(o), t1 = term(o + KL), t2 = term(o + 2 * KL), t3 = term(o + 3 * KL);
        best = fminf(fminf(best, fminf(fminf(t0, t1), t2)), t3);
      }
      for (; j < n; ++j) best = fminf(best, term(min(lo + j, end) * KL));
      if (longest & kFew) {
        float few = INF;
        for (j = 0; j < min(n, 3); ++j) few = fminf(few, term(min(lo + j, end) * KL));
        best = len < 4 ? (len > 0 ? few : INF) : best;
      }
    }
    return best;
  };

  // A run of steps whose lists all hold the same nodes (a block searched whole):
  // schedule, cells, ranges and directions stay those of step i - 1, the lists
  // change their unary costs only, and one barrier a step is enough.  NS: chunk
  // slots per wave (steps of more than 2 NW chunks are bound by their terms and
  // take the loop below).  Returns the first step past the run.  Bound by
  // instruction issue and the barrier (nine chunks on eight waves at T = 10).
  // 50 models x 678 blocks of 60 nodes, 30 points: 6.0 ms with the tables kept,
  // 13.9 with every step built anew; spreading the ninth chunk over all waves
  // cost as much as it evened out.
  auto same_steps = [&](int i, int nch, auto ns) {
    constexpr int NS = decltype(ns)::value;
    if constexpr (RUNS) {
      int dt[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s)
        dt[s] = sh.ctt[i & 3][pi[s] & (KL - 1)] - sh.ctt[(i - 1) & 3][(pi[s] >> 6) & (KL - 1)];
      for (;;) {
        if (i + 1 < M) commit_slot(i + 1, next, next.same);
        if (i + 2 < M) fetch_values(i + 2, list_next, next);
        if (i + 3 < M) list_next = fetch_list(i + 3);
        const bool again = i + 1 < M && __builtin_amdgcn_readfirstlane(sh.same[(i + 1) & 7]) != 0;
        float2 th;
        int dtm;
        point(i, th, dtm);
        const float qw = a.lambda2 * (i <= M - 2 ? 2.f : 1.f);
        float* vt = i <= M - 2 ? vtable(vtm, a, i) : nullptr;
        const int vb = (i & 1) ^ 1;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          if (wv + NW * s < nch) {
            const int r = (pi[s] >> 6) & (KL - 1), col = pi[s] & (KL - 1);
            float bm, be;
            cell_consts<UNS>(th, ar[s], bm, be);
            const float best = packed_min(vb, r, col, (pi[s] >> 12) & 127, (pi[s] >> 19) & 127, longest[s], bm, be,
                                          th, false);
            const float v = later_cell(sh.cu[i & 3][col], qw, dtm, dt[s], best);
            if (pi[s] >= 0) {
              sh.v[vb ^ 1][pi[s] & kCell] = v;
              if (vt) vt[col * VS + r] = v;
            }
          }
        }
        __syncthreads();
        ++i;
        if (!again) break;
      }
    }
    return i;
  };

  // ---- points 2 .. M-1 -----------------------------------------------------------
  for (int i = 2; i < M; ++i) {
    if constexpr (RUNS) {
      if (i >= 3 && same_lists(i)) {
        const int n = n_slots(b_prev);
        if (n <= 2 * NW) {
          i = n <= NW ? same_steps(i, n, std::integral_constant<int, 1>{})
                      : same_steps(i, n, std::integral_constant<int, 2>{});
          if (i >= M) break;
        }
      }
    }
    const int s2 = (i - 2) & 3, s1 = (i - 1) & 3, s0 = i & 3;
    const int Kq = sh.ck[s2], Kp = sh.ck[s1], Kn = sh.ck[s0];
    // Consecutive points with one and the same list (a block searched whole):
    // schedule, cells and directions are those of the previous step.
    const bool reuse = RUNS && i >= 3 && same_lists(i);
    const int prv = PACKED ? b_prev : (i & 1) ^ 1, cur = reuse ? prv : prv ^ 1;
    b_prev = cur;

    // Phase 1: publish the previous step's cells, build this step's schedule and
    // (a_{i-2}, a_i) direction table, prefetch the next candidate list.
    if (!reuse) {
      const int nprev = n_slots(prv);
#pragma unroll
      for (int s = 0; s < RPW; ++s) {
        const int ch = wv + NW * s;
        if (ch < nprev && pi[s] >= 0) {
          if constexpr (LISTS) sh.dir[pi[s] & kCell] = ar[s];
          else sh.va[pi[s] & kCell] = make_float2(vr[s], ar[s]);
        }
      }
    }
    if (wv == kBuilder && !reuse) schedule(s1, s0, s2, cur);
    if (!reuse) {
      // the (a_{i-2}, a_i) direction of row k, column c; a pair is used only
      // if some z_{i-1} fits strictly between its frames and within T of
      // both: 2 <= t_i - t_{i-2} <= 2T - 2 (node order: between its nodes,
      // so the frames may be equal).  Under the span reading a pair whose
      // frames are TS or more apart gets +inf, which takes its terms out of
      // every minimum.
      const int gap_min = a.sp.node ? 0 : 2;
      const auto direction = [&](int k, int c, int tc, float2 pc) {
        const int gap = tc - sh.ctt[s2][k];
        if (gap >= gap_min && (T <= 0 || gap <= 2 * T - 2)) {
          if (TS > 0 && gap >= TS) {
            sh.ct[k * KL + c] = INF;
            return;
          }
          const float2 pk = sh.cxy[s2][k];
          if (!DEGEN && pk.x == pc.x && pk.y == pc.y) sh.flag = 1;
          sh.ct[k * KL + c] = neg_dir<DEGEN>(pk, pc);
        }
      };
      if (KL == kMaxList && !PACKED && Kn <= 48) {
        // short lists (density caps): the Kq x Kn pairs spread over the
        // threads (with 8 or more waves, all but the builder's, which has the
        // schedule to build: 2% faster than sharing the table with it);
        // p < 4096 and Kn <= 64 keep (p + 1/2) / Kn at least 1/128 from an
        // integer, so the truncated float quotient is exact
        const float rn = __builtin_amdgcn_rcpf(static_cast<float>(Kn));
        const int stride = NW >= 8 ? (NW - 1) * 64 : NW * 64;
        for (int p = (NW >= 8 && wv == kBuilder) ? Kq * Kn : threadIdx.x; p < Kq * Kn; p += stride) {
          const int k = static_cast<int>((static_cast<float>(p) + 0.5f) * rn);
          const int c = p - k * Kn;
          direction(k, c, sh.ctt[s0][c], sh.cxy[s0][c]);
        }
      } else if (KL == kMaxList && NW >= 8) {
        // each wave but the schedule's builder keeps one column c per lane and
        // walks the rows k
        if (wv != kBuilder && lane < Kn) {
          const int tc = sh.ctt[s0][lane];
          const float2 pc = sh.cxy[s0][lane];
          for (int k = wv; k < Kq; k += NW - 1) direction(k, lane, tc, pc);
        }
      } else {
        // each thread keeps one column c and walks the rows k
        constexpr int kRowsPerPass = NW * 64 / KL;
        const int c = threadIdx.x & (KL - 1);
        if (c < Kn) {
          const int tc = sh.ctt[s0][c];
          const float2 pc = sh.cxy[s0][c];
          for (int k = threadIdx.x / KL; k < Kq; k += kRowsPerPass) direction(k, c, tc, pc);
        }
      }
    }
    if (i + 1 < M) commit_slot(i + 1, next);
    if (!reuse) __syncthreads();
    if (i + 2 < M) fetch_values(i + 2, list_next, next);
    if (i + 3 < M) list_next = fetch_list(i + 3);

    // Phase 2: the minima over a_{i-2} of every admissible cell, chunk by chunk.
    float2 th;
    int dtm;
    point(i, th, dtm);
    const float qw = a.lambda2 * (i <= M - 2 ? 2.f : 1.f);
    float* vt = i <= M - 2 ? vtable(vtm, a, i) : nullptr;
    const float w = a.w;
    const int nch = n_slots(cur);
    const int vb = (i & 1) ^ 1;  // list variant: buffer of V_{i-1}
#pragma unroll
    for (int s = 0; s < RPW; ++s) {
      const int ch = wv + NW * s;
      float vnew = INF, anew = 0.f;
      if constexpr (PACKED) {
        if (ch < nch) {
          // lane-own cell and predecessor range; the wave runs to the longest
          // range, a lane past its own repeats its last predecessor (which
          // changes no minimum)
          bool same = false;
          if (!reuse) {
            int r, col, lo, hi;
            const bool valid = packed_cell(sh.sched[cur], sh.pstart[cur], sh.nch[cur], sh.ptot[cur], ch * 64 + lane,
                                           r, col, lo, hi);
            const float2 xr = sh.cxy[s1][r], xa = sh.cxy[s0][col];
            same = xa.x == xr.x && xa.y == xr.y;
            if (!DEGEN && same && valid) sh.flag = 1;
            ar[s] = neg_dir<DEGEN>(xr, xa);
            const int n = hi - lo;
            pi[s] = (r * KL + col) | lo << 12 | n << 19 | (valid ? 0 : 1 << 31);
            int n_max = n;
            for (int off = 32; off > 0; off >>= 1) n_max = max(n_max, __shfl_xor(n_max, off));
            longest[s] = __builtin_amdgcn_readfirstlane(n_max) | (__any(n < 4) ? kFew : 0);
          }
          const int r = (pi[s] >> 6) & (KL - 1), col = pi[s] & (KL - 1);
          const int lo = (pi[s] >> 12) & 127, len = (pi[s] >> 19) & 127;
          const int tr = sh.ctt[s1][r], tp = sh.ctt[s0][col];
          anew = ar[s];
          float bm, be;
          cell_consts<UNS>(th, anew, bm, be);
          const float best = packed_min(vb, r, col, lo, len, longest[s], bm, be, th, same);
          vnew = later_cell(sh.cu[s0][col], qw, dtm, tp - tr, best);
          if (pi[s] >= 0) {
            if constexpr (LISTS) sh.v[vb ^ 1][pi[s] & kCell] = vnew;
            if (vt) vt[col * VS + r] = vnew;
          }
          vr[s] = vnew;
        }
      } else {
        if (ch < nch) {
          const Chunk c = unpack_chunk(sh.sched[cur][ch]);
          int r, col;
          const bool valid = chunk_cell(c, lane, r, col);
          if (!valid) { r = c.r0; col = c.clo; }  // in-range reads; results unused
          const int tr = sh.ctt[s1][r], tp = sh.ctt[s0][col];
          const float2 xr = sh.cxy[s1][r], xa = sh.cxy[s0][col];
          const bool same = xa.x == xr.x && xa.y == xr.y;
          if (!DEGEN && same && valid) sh.flag = 1;
          anew = neg_dir<DEGEN>(xr, xa);
          float bm, be;
          cell_consts<UNS>(th, anew, bm, be);
          const float2* vcol = sh.va + r;
          const float* ccol = sh.ct + col;
          float best = INF;
          if constexpr (DUMMY) best = sh.de[prv][r];  // predecessor epsilon: no D^g
          // eight predecessors per trip (one address step per table; the wide
          // layouts only, where few chunk slots leave registers for it), then
          // four, then one at a time
          int k = c.lo;
          constexpr bool kEight = NW >= 8 && KL == kMaxList;
          for (; kEight && k + 7 < c.hi; k += 8) {
            const float2 v0 = vcol[k * KL], v1 = vcol[(k + 1) * KL];
            const float2 v2 = vcol[(k + 2) * KL], v3 = vcol[(k + 3) * KL];
            const float t0 = relax<DEGEN, UNS>(v0.x, v0.y, ccol[k * KL], bm, be, th, same, w);
            const float t1 = relax<DEGEN, UNS>(v1.x, v1.y, ccol[(k + 1) * KL], bm, be, th, same, w);
            const float t2 = relax<DEGEN, UNS>(v2.x, v2.y, ccol[(k + 2) * KL], bm, be, th, same, w);
            const float t3 = relax<DEGEN, UNS>(v3.x, v3.y, ccol[(k + 3) * KL], bm, be, th, same, w);
            best = fminf(fminf(best, fminf(fminf(t0, t1), t2)), t3);
            const float2 v4 = vcol[(k + 4) * KL], v5 = vcol[(k + 5) * KL];
            const float2 v6 = vcol[(k + 6) * KL], v7 = vcol[(k + 7) * KL];
            const float t4 = relax<DEGEN, UNS>(v4.x, v4.y, ccol[(k + 4) * KL], bm, be, th, same, w);
            const float t5 = relax<DEGEN, UNS>(v5.x, v5.y, ccol[(k + 5) * KL], bm, be, th, same, w);
            const float t6 = relax<DEGEN, UNS>(v6.x, v6.y, ccol[(k + 6) * KL], bm, be, th, same, w);
            const float t7 = relax<DEGEN, UNS>(v7.x, v7.y, ccol[(k + 7) * KL], bm, be, th, same, w);
            best = fminf(fminf(best, fminf(fminf(t4, t5), t6)), t7);
          }
          if (k + 3 < c.hi) {
            const float2 v0 = vcol[k * KL], v1 = vcol[(k + 1) * KL];
            const float2 v2 = vcol[(k + 2) * KL], v3 = vcol[(k + 3) * KL];
            const float t0 = relax<DEGEN, UNS>(v0.x, v0.y, ccol[k * KL], bm, be, th, same, w);
            const float t1 = relax<DEGEN, UNS>(v1.x, v1.y, ccol[(k + 1) * KL], bm, be, th, same, w);
            const float t2 = relax<DEGEN, UNS>(v2.x, v2.y, ccol[(k + 2) * KL], bm, be, th, same, w);
            const float t3 = relax<DEGEN, UNS>(v3.x, v3.y, ccol[(k + 3) * KL], bm, be, th, same, w);
            best = fminf(fminf(best, fminf(fminf(t0, t1), t2)), t3);
            k += 4;
          }
          for (; k < c.hi; ++k) {
            const float2 v0 = vcol[k * KL];
            best = fminf(best, relax<DEGEN, UNS>(v0.x, v0.y, ccol[k * KL], bm, be, th, same, w));
          }
          vnew = later_cell(sh.cu[s0][col], qw, dtm, tp - tr, best);
          if (valid && vt) vt[col * VS + r] = vnew;
          pi[s] = valid ? r * KL + col : -1;
          vr[s] = vnew;
          ar[s] = anew;
        }
      }
      // a slot past the step's chunk count keeps stale registers: every reader
      // (publication, the final minimum) checks the slot against that count
    }
    if constexpr (DUMMY) {
      // the epsilon cells of step i, from step i-1's cells and epsilon cells
      const float cw = a.cw;
      // V_i(r, eps): over the admissible predecessors of row r, no D^g; eight
      // lanes per row split its predecessors, the rows spread over the waves
      for (int r0 = wv * 8; r0 < Kp; r0 += NW * 8) {
        const int r = r0 + (lane >> 3), sub = lane & 7;
        float m = INF;
        if (r < Kp) {
          const int f = sh.ctt[s1][r];
          const int hi = count_lt(sh.ctt[s2], Kq, f);
          const int lo = T > 0 ? count_lt(sh.ctt[s2], Kq, f - T + 1) : 0;
          for (int k = lo + sub; k < hi; k += 8) m = fminf(m, sh.va[k * KL + r].x);
        }
        m = fminf(m, __shfl_xor(m, 1));
        m = fminf(m, __shfl_xor(m, 2));
        m = fminf(m, __shfl_xor(m, 4));
        if (r < Kp && sub == 0) {
          const float v = cw + fminf(sh.de[prv][r], m);
          sh.df[cur][r] = v;
          if (vt) vt[Kc * VS + r] = v;
        }
      }
      if (wv == kBuilder) {
        float m = lane < Kq ? sh.df[prv][lane] : INF;
        for (int off = 32; off > 0; off >>= 1) m = fminf(m, __shfl_xor(m, off));
        m = fminf(m, sh.dg[prv]);
        if (lane < Kn) {
          const float v = sh.cu[s0][lane] + m;
          sh.de[cur][lane] = v;
          if (vt) vt[lane * VS + Kc] = v;
        }
        if (lane == 0) {
          sh.dg[cur] = cw + m;
          if (vt) vt[Kc * VS + Kc] = cw + m;
        }
      }
    }
    __syncthreads();
  }

  // ---- optimum: first row-major minimum of V_{M-1}(a_{M-2}, a_{M-1}) ------------
  {
    constexpr int RS = KL + (DUMMY ? 1 : 0);  // row stride of the result index
    const int last = PACKED ? b_prev : (M - 1) & 1;
    const int nch = n_slots(last);
    float bv = INF;
    int bi = 0x7fffffff;
#pragma unroll
    for (int s = 0; s < RPW; ++s) {
      const int ch = wv + NW * s;
      if constexpr (PACKED) {
        if (ch < nch && pi[s] >= 0) {
          const int idx = pi[s] & kCell;
          float v = vr[s];
          if constexpr (LISTS) v = sh.v[(M - 1) & 1][idx];
          if (v < bv || (v == bv && idx < bi)) { bv = v; bi = idx; }
        }
      } else if (ch < nch) {
        int r, col;
        if (slot_cell(last, ch, r, col)) {
          const int idx = r * RS + col;
          if (vr[s] < bv || (vr[s] == bv && idx < bi)) { bv = vr[s]; bi = idx; }
        }
      }
    }
    if constexpr (DUMMY) {
      if (wv == 0) {
        auto take = [&](float v, int idx) {
          if (v < bv || (v == bv && idx < bi)) { bv = v; bi = idx; }
        };
        if (lane < sh.ck[(M - 2) & 3]) take(sh.df[last][lane], lane * RS + kEps);
        if (lane < sh.ck[(M - 1) & 3]) take(sh.de[last][lane], kEps * RS + lane);
        if (lane == 0) take(sh.dg[last], kEps * RS + kEps);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      const float ov = __shfl_xor(bv, off);
      const int oi = __shfl_xor(bi, off);
      if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (lane == 0) { sh.red_v[wv] = bv; sh.red_i[wv] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int q = 1; q < NW; ++q) {
        const float ov = sh.red_v[q];
        const int oi = sh.red_i[q];
        if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
      sh.res_v = bv;
      sh.res_i = bi == 0x7fffffff ? 0 : bi;
    }
    __syncthreads();
  }
  DPResult res;
  res.v = sh.res_v;
  res.idx = sh.res_i;
  res.flag = DEGEN ? 0 : sh.flag;
  return res;
}

// ---- forward pass of short lists ---------------------------------------------------
// The same recursion for short lists (KL = 16 or 32, plain reading), where the
// chain of steps of one matching bounds the launch: one barrier a step instead
// of two.  NW waves work on step i, writing its cells to
// a second buffer, then build the (a_{i-1}, a_{i+1}) directions of step i + 1;
// one more wave builds the schedule of step i + 1 and brings in list i + 2
// meanwhile (at step i the ring of four holds lists i - 1 .. i + 1 in use).  Every
// term, minimum and sum is the one dp_forward takes.  The second buffers cost 64-slot
// lists a workgroup per CU, so those stay with dp_forward.  20 points, lists of
// 16, 70 matchings: 53 us, 79 with four waves and two barriers, 146 with one
// wave.
template <int NW, int KL>
struct FewShared {
  float2 va[2][KL * KL];  // V_i and directions of step i's cells, by parity of i
  float ct[2][KL * KL];
  float2 cxy[4][KL];
  int32_t ctt[4][KL];
  float cu[4][KL];
  uint2 sched[2][KL];
  int32_t nch[2];
  int32_t ck[4];
  CandRange crange[4];
  int32_t flag;
  float red_v[NW];
  int32_t red_i[NW];
};

// rec (nullable): every list's candidates are kept there, [M][K] (x, y, frame,
// node; node -1 past the list).
template <int NW, bool DEGEN, int KL>
__device__ __forceinline__ DPResult dp_forward_few(FewShared<NW, KL>& sh, const MatchView& a, float* vtm,
                                                   float4* rec) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const bool producer = wv == NW;
  const int M = a.m.M, VS = a.vs;
  const int T = pair_limit(a.sp), TS = span_limit(a.sp);
  const float INF = __builtin_inff();
  const CandRange* ring = a.sp.node ? sh.crange : nullptr;

  struct List {
    Cands c;
    int32_t node;
  };
  struct Values {
    Cands c;
    float2 xy;
    int32_t t;
    float u;
    int32_t node = -1;
  };
  auto fetch_list = [&](int j) {
    List l;
    l.c = cands_of(a, j);
    l.node = l.c.list ? ro(l.c.list + (lane < a.cstride ? lane : 0)) : 0;
    return l;
  };
  auto fetch_values = [&](int j, const List& l) {
    Values f;
    f.c = l.c;
    if (lane < l.c.count()) {
      const int n = l.c.list ? l.node : cand_node(l.c.r, lane);
      f.xy = ro(a.s.xy + n);
      f.t = ro(a.s.t + n);
      f.u = ro(a.U + (long long)j * a.us + n);
      f.node = n;
    }
    return f;
  };
  auto commit = [&](int j, const Values& f) {
    const int k = f.c.count(), sl = j & 3;
    if (rec && lane < a.sp.K)
      rec[j * a.sp.K + lane] = make_float4(f.xy.x, f.xy.y, __int_as_float(f.t), __int_as_float(f.node));
    if (lane < k) {
      sh.cxy[sl][lane] = f.xy;
      sh.ctt[sl][lane] = f.t;
      sh.cu[sl][lane] = a.lambda1 * f.u;
    }
    if (lane == 0) {
      sh.ck[sl] = k;
      sh.crange[sl] = f.c.r;
    }
  };
  // the schedule of step i: rows list i - 1, columns list i, predecessors i - 2
  auto schedule = [&](int i) {
    const int sr = (i - 1) & 3, sc = i & 3, sp = i >= 2 ? (i - 2) & 3 : -1;
    build_schedule(sh.ctt[sr], sh.ck[sr], sh.ctt[sc], sh.ck[sc], sp >= 0 ? sh.ctt[sp] : nullptr,
                   sp >= 0 ? sh.ck[sp] : 0, T, sh.sched[i & 1], &sh.nch[i & 1], lane, nullptr, nullptr, ring, sr, sc,
                   sp);
  };
  // the (a_{i-2}, a_i) directions of step i, by the working waves
  auto directions = [&](int i) {
    const int s2 = (i - 2) & 3, s0 = i & 3, Kq = sh.ck[s2], Kn = sh.ck[s0];
    const int gap_min = a.sp.node ? 0 : 2;
    const int c = threadIdx.x & (KL - 1);
    if (c >= Kn) return;
    const int tc = sh.ctt[s0][c];
    const float2 pc = sh.cxy[s0][c];
    for (int k = threadIdx.x / KL; k < Kq; k += NW * 64 / KL) {
      const int gap = tc - sh.ctt[s2][k];
      if (gap >= gap_min && (T <= 0 || gap <= 2 * T - 2)) {
        if (TS > 0 && gap >= TS) {
          sh.ct[i & 1][k * KL + c] = INF;
          continue;
        }
        const float2 pk = sh.cxy[s2][k];
        if (!DEGEN && pk.x == pc.x && pk.y == pc.y) sh.flag = 1;
        sh.ct[i & 1][k * KL + c] = neg_dir<DEGEN>(pk, pc);
      }
    }
  };
  // angles and frames of 64 model points at a time, one per lane
  float2 th_l = make_float2(0.f, 0.f);
  int32_t tm_l = 0, tm_prev = 0;
  auto load_points = [&](int i0) {
    const int j = min(i0 + lane, M - 1);
    th_l = a.theta[j];
    tm_l = a.m.t[j];
  };

  List next_list;
  Values next;
  if (producer) {
    const List l0 = fetch_list(0), l1 = fetch_list(1), l2 = fetch_list(2);
    if (3 < M) next_list = fetch_list(3);
    const Values f0 = fetch_values(0, l0), f1 = fetch_values(1, l1), f2 = fetch_values(2, l2);
    if (3 < M) next = fetch_values(3, next_list);
    if (4 < M) next_list = fetch_list(4);
    if (lane == 0) sh.flag = 0;
    commit(0, f0);
    commit(1, f1);
    commit(2, f2);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    schedule(1);
  } else {
    load_points(0);
    tm_prev = __builtin_amdgcn_readlane(tm_l, 0);
  }
  __syncthreads();

  float bv = INF;  // first row-major minimum of the last step's cells
  int bi = 0x7fffffff;
  for (int i = 1; i < M; ++i) {
    if (producer) {
      if (i + 2 < M) commit(i + 2, next);
      if (i + 3 < M) next = fetch_values(i + 3, next_list);
      if (i + 4 < M) next_list = fetch_list(i + 4);
      if (i + 1 < M) schedule(i + 1);
    } else {
      const int s1 = (i - 1) & 3, s0 = i & 3, b = i & 1;
      if ((i & 63) == 0) load_points(i);
      const float2 th = make_float2(lane_value(th_l.x, i & 63), lane_value(th_l.y, i & 63));
      const int tm = __builtin_amdgcn_readlane(tm_l, i & 63);
      const int dtm = tm - tm_prev;
      tm_prev = tm;
      const float qw = a.lambda2 * (i <= M - 2 ? 2.f : 1.f);
      float* vt = i <= M - 2 ? vtable(vtm, a, i) : nullptr;
      const int nch = sh.nch[b];
      for (int ch = wv; ch < nch; ch += NW) {
        const Chunk c = unpack_chunk(sh.sched[b][ch]);
        int r, col;
        const bool valid = chunk_cell(c, lane, r, col);
        if (!valid) { r = c.r0; col = c.clo; }  // in-range reads; results unused
        const int tr = sh.ctt[s1][r], tp = sh.ctt[s0][col];
        const float2 xr = sh.cxy[s1][r], xa = sh.cxy[s0][col];
        const bool same = xa.x == xr.x && xa.y == xr.y;
        if (!DEGEN && same && valid) sh.flag = 1;
        const float anew = neg_dir<DEGEN>(xr, xa);
        float v;
        if (i == 1) {
          v = first_cell(sh.cu[s1][r], sh.cu[s0][col], a.lambda2, dtm, tp - tr);
        } else {
          float bm, be;
          cell_consts<false>(th, anew, bm, be);
          const float2* vcol = sh.va[b ^ 1] + r;
          const float* ccol = sh.ct[b] + col;
          const float w = a.w;
          float best = INF;
          int k = c.lo;
          for (; k + 3 < c.hi; k += 4) {
            const float2 v0 = vcol[k * KL], v1 = vcol[(k + 1) * KL];
            const float2 v2 = vcol[(k + 2) * KL], v3 = vcol[(k + 3) * KL];
            const float t0 = relax<DEGEN>(v0.x, v0.y, ccol[k * KL], bm, be, th, same, w);
            const float t1 = relax<DEGEN>(v1.x, v1.y, ccol[(k + 1) * KL], bm, be, th, same, w);
            const float t2 = relax<DEGEN>(v2.x, v2.y, ccol[(k + 2) * KL], bm, be, th, same, w);
            const float t3 = relax<DEGEN>(v3.x, v3.y, ccol[(k + 3) * KL], bm, be, th, same, w);
            best = fminf(fminf(best, fminf(fminf(t0, t1), t2)), t3);
          }
          for (; k < c.hi; ++k) {
            const float2 v0 = vcol[k * KL];
            best = fminf(best, relax<DEGEN>(v0.x, v0.y, ccol[k * KL], bm, be, th, same, w));
          }
          v = later_cell(sh.cu[s0][col], qw, dtm, tp - tr, best);
        }
        if (valid) {
          sh.va[b][r * KL + col] = make_float2(v, anew);
          if (vt) vt[col * VS + r] = v;
          const int idx = r * KL + col;
          if (i == M - 1 && (v < bv || (v == bv && idx < bi))) { bv = v; bi = idx; }
        }
      }
      if (i + 1 < M) directions(i + 1);
    }
    __syncthreads();
  }

  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(bv, off);
    const int oi = __shfl_xor(bi, off);
    if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (!producer && lane == 0) { sh.red_v[wv] = bv; sh.red_i[wv] = bi; }
  __syncthreads();
  bv = INF;
  bi = 0x7fffffff;
  for (int q = 0; q < NW; ++q) {
    const float ov = sh.red_v[q];
    const int oi = sh.red_i[q];
    if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  DPResult res;
  res.v = bv;
  res.idx = bi == 0x7fffffff ? 0 : bi;
  res.flag = DEGEN ? 0 : sh.flag;
  return res;
}

// ---- backtracking (Eq. 12), one wave per matching ---------------------------------
// From the optimal final pair (r, c) = (a_{M-2}, a_{M-1}), each step recomputes
// the terms of the optimal cell over its admissible predecessors (lanes) with
// the forward pass's arithmetic and keeps the lowest index of the minimum.
// With dummies r and c may be kEps; the epsilon predecessor comes last, so it
// is taken only when its term is strictly smaller.
//
// The candidates of a list do not depend on the path, so each lane holds one
// candidate (node, frame, coordinates) of the three lists of the current
// step; a list is read two steps and its nodes' data one step before their
// use.  The chosen cell is wave-uniform, so its data come from their lanes by
// readlane and the minimum by DPP: of the step's chain only the read of the
// chosen cell's values waits for memory.  1387 matchings of 75 points: 121 us,
// 228 with the lists' reads in the chain and shuffles.
struct LaneCand {
  int node;   // scene node of this lane's candidate, -1 past the list
  int t;      // its frame
  float2 xy;  // its coordinates
  int n;      // list length
};
struct LaneList {
  Cands c;
  int node;  // explicit lists: this lane's entry
};

template <bool LISTS>
__device__ __forceinline__ LaneList lane_list(const MatchView& a, int j, int lane) {
  LaneList l;
  l.c = cands_of<LISTS>(a, j);
  l.node = l.c.list ? ro(l.c.list + (lane < a.cstride ? lane : 0)) : 0;
  return l;
}

__device__ __forceinline__ LaneCand lane_cand(const MatchView& a, const LaneList& l, int lane) {
  LaneCand L;
  L.n = l.c.count();
  L.node = lane < L.n ? (l.c.list ? l.node : cand_node(l.c.r, lane)) : -1;
  L.t = L.node >= 0 ? ro(a.s.t + L.node) : 0;
  L.xy = L.node >= 0 ? ro(a.s.xy + L.node) : make_float2(0.f, 0.f);
  return L;
}

template <bool DEGEN, bool DUMMY = false, bool UNS = false, bool LISTS = false>
__device__ __forceinline__ void backtrack_wave(const MatchView& a, const float* vtm, int r_end, int c_end, int lane,
                               int32_t* out) {
  const int M = a.m.M, Kc = a.sp.K, VS = a.vs;
  const int T = pair_limit(a.sp), TS = span_limit(a.sp);
  const float INF = __builtin_inff();
  // candidate index idx of a list held in lanes -> its node (dummy: kDummyNode)
  auto node_at = [&](const LaneCand& L, int idx) {
    return DUMMY && idx == kEps ? kDummyNode : __builtin_amdgcn_readlane(L.node, idx);
  };
  int r = __builtin_amdgcn_readfirstlane(r_end), c = __builtin_amdgcn_readfirstlane(c_end);
  const LaneList l1 = lane_list<LISTS>(a, M - 1, lane), l2 = lane_list<LISTS>(a, M - 2, lane), l3 = lane_list<LISTS>(a, M - 3, lane);
  LaneList ln;
  if (M >= 4) ln = lane_list<LISTS>(a, M - 4, lane);
  LaneCand Lc = lane_cand(a, l1, lane);
  LaneCand Lr = lane_cand(a, l2, lane);
  LaneCand Lk = lane_cand(a, l3, lane);
  {
    const int nc0 = node_at(Lc, c), nr0 = node_at(Lr, r);
    if (lane == 0) {
      out[M - 1] = nc0;
      out[M - 2] = nr0;
    }
  }
  for (int i = M - 1; i >= 2; --i) {
    const int nk = Lk.n;
    const float* vp = vtable(vtm, a, i - 1);
    float tot = INF, teps = INF;
    const bool r_eps = DUMMY && r == kEps, c_eps = DUMMY && c == kEps;
    const int nr = __builtin_amdgcn_readlane(Lr.node, r), tr = __builtin_amdgcn_readlane(Lr.t, r);
    const int tc = __builtin_amdgcn_readlane(Lc.t, c);
    // the lanes with an admissible predecessor of the chosen cell, and their
    // values V_{i-1}(k, r)
    bool adm = lane < nk;
    if (!r_eps) adm = adm && (c_eps ? admissible(Lk.t, tr, T)
                                    : consecutive_ok(a.sp, T, Lk.node, Lk.t, nr, tr) && span_ok(Lk.t, tc, TS));
    float v = INF;
    if (adm) v = vp[(r_eps ? Kc : r) * VS + lane];
    if (DUMMY) teps = vp[(r_eps ? Kc : r) * VS + Kc];
    // the next lists, fetched while this step runs
    LaneCand Ln;
    if (i >= 3) Ln = lane_cand(a, ln, lane);
    if (i >= 4) ln = lane_list<LISTS>(a, i - 4, lane);
    if (r_eps || c_eps) {
      // V_i(eps, .) = ... + min(V_{i-1}(eps, eps), min_k V_{i-1}(k, eps)),
      // V_i(r, eps) = l1 W^d + min(V_{i-1}(eps, r), min_k V_{i-1}(k, r))
      tot = v;
    } else {
      // the cell's points are read from their lanes (of other lists) with every
      // lane active, not under the predecessors' mask
      const float2 xr = make_float2(lane_value(Lr.xy.x, r), lane_value(Lr.xy.y, r));
      const float2 xa = make_float2(lane_value(Lc.xy.x, c), lane_value(Lc.xy.y, c));
      const float2 th = ro(a.theta + i);
      const bool same = xa.x == xr.x && xa.y == xr.y;
      float bm, be;
      cell_consts<UNS>(th, neg_dir<DEGEN>(xr, xa), bm, be);
      if (adm)
        tot = relax<DEGEN, UNS>(v, neg_dir<DEGEN>(Lk.xy, xr), neg_dir<DEGEN>(Lk.xy, xa), bm, be, th, same, a.w);
    }
    const float best = wave_min(tot);
    int bk = __ffsll(static_cast<long long>(__ballot(tot == best))) - 1;
    if (DUMMY && teps < best) bk = kEps;
    const int nbk = node_at(Lk, bk);
    if (lane == 0) out[i - 2] = nbk;
    c = r;
    r = bk;
    Lc = Lr;
    Lr = Lk;
    if (i >= 3) Lk = Ln;
  }
}

// The same walk with the value tables and the candidates in LDS (dp_forward_few's
// vtm and rec; no dummies, plain angles): nothing of a step waits for memory.
template <bool DEGEN>
__device__ __forceinline__ void backtrack_lds(const MatchView& a, const float* vtm, const float4* rec, int r_end,
                                              int c_end, int lane, int32_t* out) {
  const int M = a.m.M, K = a.sp.K, VS = a.vs;
  const int T = pair_limit(a.sp), TS = span_limit(a.sp);
  const float INF = __builtin_inff();
  const int kl = lane < K ? lane : 0;
  int r = __builtin_amdgcn_readfirstlane(r_end);
  float4 pc = rec[(M - 1) * K + __builtin_amdgcn_readfirstlane(c_end)], pr = rec[(M - 2) * K + r];
  float4 pk = rec[(M - 3) * K + kl];
  if (lane == 0) {
    out[M - 1] = __float_as_int(pc.w);
    out[M - 2] = __float_as_int(pr.w);
  }
  float2 th_l = a.theta[min(((M - 1) & ~63) + lane, M - 1)];
  for (int i = M - 1; i >= 2; --i) {
    if ((i & 63) == 63) th_l = a.theta[min((i & ~63) + lane, M - 1)];
    const float2 th = make_float2(lane_value(th_l.x, i & 63), lane_value(th_l.y, i & 63));
    const int tr = __float_as_int(pr.z), nr = __float_as_int(pr.w), tc = __float_as_int(pc.z);
    const int tk = __float_as_int(pk.z), nk = __float_as_int(pk.w);
    const bool adm = lane < K && nk >= 0 && consecutive_ok(a.sp, T, nk, tk, nr, tr) && span_ok(tk, tc, TS);
    float tot = INF;
    if (adm) {
      const float v = vtable(vtm, a, i - 1)[r * VS + lane];
      const float2 xr = make_float2(pr.x, pr.y), xa = make_float2(pc.x, pc.y), xk = make_float2(pk.x, pk.y);
      const bool same = xa.x == xr.x && xa.y == xr.y;
      float bm, be;
      cell_consts<false>(th, neg_dir<DEGEN>(xr, xa), bm, be);
      tot = relax<DEGEN>(v, neg_dir<DEGEN>(xk, xr), neg_dir<DEGEN>(xk, xa), bm, be, th, same, a.w);
    }
    const float4 pn = rec[(i >= 3 ? i - 3 : 0) * K + kl];
    const float best = wave_min(tot);
    const int bk = __ffsll(static_cast<long long>(__ballot(tot == best))) - 1;
    pc = pr;
    pr = make_float4(lane_value(pk.x, bk), lane_value(pk.y, bk), lane_value(pk.z, bk), lane_value(pk.w, bk));
    if (lane == 0) out[i - 2] = __float_as_int(pr.w);
    r = bk;
    pk = pn;
  }
}

// ---- per-offset kernels: one workgroup per offset of a (model, scene) pair ------
__device__ __forceinline__ int part_of(const DPParts& b, int wg) {
  int q = 0;
#pragma unroll
  for (int x = 1; x < kDPParts; ++x) q += x < b.n && wg >= b.first[x];
  return q;
}

__device__ __forceinline__ MatchView view_of(const DPLaunch& a, int tl) {
  MatchView v;
  v.m = a.m;
  v.s = a.s;
  v.sp = a.sp;
  v.U = a.U;
  v.us = a.s.S;
  v.theta = a.theta;
  v.lambda1 = a.lambda1;
  v.lambda2 = a.lambda2;
  v.w = a.w;
  v.cw = a.cw;
  v.vs = a.sp.K + (a.dummy ? 1 : 0);
  v.tau = a.taus ? a.taus[tl] : a.tau0 + tl;
  v.cand = a.cand ? a.cand + (long long)tl * a.m.M * a.cstride : nullptr;
  v.ccount = a.cand ? a.ccount + (long long)tl * a.m.M : nullptr;
  v.cstride = a.cstride;
  return v;
}

__device__ __forceinline__ float* scratch_of(const DPLaunch& a, int tl) {
  const long long vs = a.sp.K + (a.dummy ? 1 : 0);
  return a.vt + (long long)tl * (a.m.M - 2) * vs * vs;
}

template <int NW, bool DEGEN, int KL, bool DUMMY = false, bool PACKED = false, bool UNS = false, bool LISTS = false>
__global__ __launch_bounds__(NW * 64)
__attribute__((amdgpu_waves_per_eu(KL < kMaxList || NW == 8 ? 4 : 1)))
void k_dp(DPParts parts) {
  __shared__ DPShared<NW, KL, DUMMY, PACKED, LISTS> sh;
  const int part = part_of(parts, blockIdx.x), tl = blockIdx.x - parts.first[part];
  const DPLaunch& a = parts.p[part];
  if (DEGEN && a.degen[tl] == 0) return;
  const DPResult r = dp_forward<NW, DEGEN, KL, DUMMY, PACKED, UNS, LISTS>(sh, view_of(a, tl), scratch_of(a, tl));
  if (threadIdx.x == 0) {
    constexpr int RS = KL + (DUMMY ? 1 : 0);
    a.e32[tl] = r.v;
    a.last2[tl] = make_int2(r.idx / RS, r.idx % RS);
    if (!DEGEN) a.degen[tl] = r.flag;
  }
}

// HIST: the value tables and the candidates stay in LDS and one wave of the
// workgroup backtracks from there.
template <int NW, bool DEGEN, int KL, bool HIST>
__global__ __launch_bounds__((NW + 1) * 64) void k_dp_few(DPParts parts) {
  __shared__ FewShared<NW, KL> sh;
  extern __shared__ __align__(16) float hist[];
  const int part = part_of(parts, blockIdx.x), tl = blockIdx.x - parts.first[part];
  const DPLaunch& a = parts.p[part];
  if (DEGEN && a.degen[tl] == 0) return;
  const MatchView v = view_of(a, tl);
  float* vt = hist + 4 * a.m.M * a.sp.K;  // behind the candidates
  float4* rec = reinterpret_cast<float4*>(hist);
  const DPResult r = HIST ? dp_forward_few<NW, DEGEN, KL>(sh, v, vt, rec)
                          : dp_forward_few<NW, DEGEN, KL>(sh, v, scratch_of(a, tl), nullptr);
  if (threadIdx.x == 0) {
    a.e32[tl] = r.v;
    if (!HIST) a.last2[tl] = make_int2(r.idx / KL, r.idx % KL);
    if (!DEGEN) a.degen[tl] = r.flag;
  }
  if (HIST && threadIdx.x < 64 && !r.flag) {
    const int lane = threadIdx.x, M = a.m.M;
    int32_t* out = a.assign + (long long)tl * M;
    if (r.v < __builtin_inff()) {
      backtrack_lds<DEGEN>(v, vt, rec, r.idx / KL, r.idx % KL, lane, out);
    } else {
      for (int i = lane; i < M; i += 64) out[i] = -1;
    }
  }
}

__global__ __launch_bounds__(64) void k_backtrack(DPParts parts) {
  const int part = part_of(parts, blockIdx.x), tl = blockIdx.x - parts.first[part], lane = threadIdx.x;
  const DPLaunch& a = parts.p[part];
  const int M = a.m.M;
  int32_t* out = a.assign + (long long)tl * M;
  if (!(a.e32[tl] < __builtin_inff())) {
    for (int i = lane; i < M; i += 64) out[i] = -1;
    return;
  }
  const MatchView v = view_of(a, tl);
  const int2 l2 = a.last2[tl];
  float* vt = scratch_of(a, tl);
  if (a.dummy) {
    if (a.degen[tl]) backtrack_wave<true, true>(v, vt, l2.x, l2.y, lane, out);
    else backtrack_wave<false, true>(v, vt, l2.x, l2.y, lane, out);
  } else if (a.sp.uns) {
    if (a.degen[tl]) backtrack_wave<true, false, true>(v, vt, l2.x, l2.y, lane, out);
    else backtrack_wave<false, false, true>(v, vt, l2.x, l2.y, lane, out);
  } else {
    if (a.degen[tl]) backtrack_wave<true>(v, vt, l2.x, l2.y, lane, out);
    else backtrack_wave<false>(v, vt, l2.x, l2.y, lane, out);
  }
}

// ---- batched persistent launch ------------------------------------------------------
// Workgroups pull (pair, offset) items from a cost-sorted list with an atomic
// counter until it runs out; each solves its item with the forward pass, re-runs
// the degenerate variant when coincident points were flagged, and backtracks in
// wave 0 from its own value-table scratch before taking the next item.
__device__ __forceinline__ MatchView view_of(const BatchLaunch& b, const PairDev& pd, int tau) {
  MatchView v;
  v.m = pd.m;
  v.s = pd.s;
  v.sp = b.sp;
  v.U = pd.U;
  v.us = pd.us;
  v.theta = pd.theta;
  v.lambda1 = b.lambda1;
  v.lambda2 = b.lambda2;
  v.w = b.w;
  v.cw = b.cw;
  v.vs = b.sp.K + (b.dummy ? 1 : 0);
  v.tau = tau;
  v.cand = pd.cand ? pd.cand + (long long)tau * pd.m.M * pd.cstride : nullptr;
  v.ccount = pd.cand ? pd.ccount + (long long)tau * pd.m.M : nullptr;
  v.cstride = pd.cstride;
  return v;
}

// A workgroup runs the forward passes of up to b.batch items (at most one per
// wave) one after the other, each into its own value tables, then wave q
// backtracks the q-th of them.  A backtracking walk is a
// chain of dependent memory reads, so the batch's walks overlap instead of
// each leaving the other waves idle.  The fast variant takes every item; an
// item whose matching has coincident points is appended to the degenerate
// list instead of being backtracked, and the degenerate variant (a second
// launch) takes the items of that list.  Occupancy target: two 8-wave
// workgroups per CU (four waves per SIMD), which leaves 128 registers per lane;
// the LDS of one matching would allow three, but at 80 registers the kernel
// spills and runs slower (1.3% on the realistic workload, 3.9% on the batched
// one).
template <int NW, bool DEGEN, int KL = kMaxList, bool DUMMY = false, bool PACKED = false, bool UNS = false,
          bool LISTS = false>
__global__ __launch_bounds__(NW * 64)
__attribute__((amdgpu_waves_per_eu(DUMMY || PACKED ? 4 : (NW >= 8 ? 4 : 3))))
void k_dp_persistent(BatchLaunch b) {
  __shared__ DPShared<NW, KL, DUMMY, PACKED, LISTS> sh;
  __shared__ int item_sh;
  __shared__ int bt_item[NW];  // item of each batch slot, -1: not backtracked here
  __shared__ int bt_idx[NW];   // its first minimising final pair, -1: infeasible
  constexpr int RS = KL + (DUMMY ? 1 : 0);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nb_max = b.batch < 1 ? 1 : (b.batch < NW ? b.batch : NW);
  float* vwg = b.vt + (long long)blockIdx.x * b.batch * b.vt_stride;
  const int n_items = DEGEN ? *b.degen_count : (b.list ? *b.list_count : b.n_items);
  int32_t* counter = DEGEN ? b.counter + 1 : b.counter;
  int slot = 0;  // forward passes waiting for their backtracking
  for (;;) {
    if (threadIdx.x == 0) item_sh = atomicAdd(counter, 1);
    __syncthreads();
    const bool done = item_sh >= n_items;
    if (!done) {
      const int item = DEGEN ? b.degen_items[item_sh] : b.list ? b.list[item_sh] : item_sh;
      const int2 it = b.items[item];
      const PairDev pd = b.pairs[it.x];
      const MatchView mv = view_of(b, pd, it.y);
      const DPResult r = dp_forward<NW, DEGEN, KL, DUMMY, PACKED, UNS, LISTS>(sh, mv, vwg + slot * b.vt_stride);
      if (threadIdx.x == 0) {
        if (!DEGEN && r.flag) {
          b.degen_items[atomicAdd(b.degen_count, 1)] = item;
          bt_item[slot] = -1;
        } else {
          b.e32[pd.row0 + it.y] = r.v;
          bt_item[slot] = item;
          bt_idx[slot] = r.v < __builtin_inff() ? r.idx : -1;
        }
      }
      ++slot;
    }
    if (slot == nb_max || (done && slot > 0)) {
      __syncthreads();
      if (wv < slot && bt_item[wv] >= 0) {
        const int2 it = b.items[bt_item[wv]];
        const PairDev pd = b.pairs[it.x];
        int32_t* out = b.assign + pd.assign0 + (long long)it.y * pd.m.M;
        const int idx = bt_idx[wv];
        if (idx >= 0) {
          backtrack_wave<DEGEN, DUMMY, UNS, LISTS>(view_of(b, pd, it.y), vwg + wv * b.vt_stride, idx / RS, idx % RS, lane,
                                       out);
        } else {
          for (int i = lane; i < pd.m.M; i += 64) out[i] = -1;
        }
      }
      slot = 0;
    }
    if (done) break;
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_collect_infeasible(const PairDev* __restrict__ pairs,
                                                           const int2* __restrict__ items, int n_items,
                                                           const float* __restrict__ e32, int32_t* __restrict__ list,
                                                           int32_t* __restrict__ count, int32_t* __restrict__ fell) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= n_items) return;
  const int2 it = items[q];
  const long long row = pairs[it.x].row0 + it.y;
  if (!(e32[row] < __builtin_inff())) {
    list[atomicAdd(count, 1)] = q;
    if (fell) fell[row] = 1;
  }
}

// Dense relaxations sum_i K_{i-2} K_{i-1} K_i of each item (one wave per item),
// the cost the work list is sorted by.
__global__ __launch_bounds__(64) void k_item_cost(const PairDev* __restrict__ pairs,
                                                 const int2* __restrict__ items, int n_items,
                                                 SearchParams sp, long long* __restrict__ cost) {
  const int item = blockIdx.x, lane = threadIdx.x;
  if (item >= n_items) return;
  const int2 it = items[item];
  const PairDev pd = pairs[it.x];
  const int M = pd.m.M, t0 = pd.m.t[0];
  long long acc = 0;
  for (int i = 2 + lane; i < M; i += 64) {
    long long prod = 1;
    for (int q = i - 2; q <= i; ++q) {
      const CandRange c = point_candidates(pd.s.fstart, pd.s.F, it.y + pd.m.t[q] - t0, sp);
      prod *= c.k1 + c.k2;
    }
    acc += prod;
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) cost[item] = acc;
}

__global__ void k_fill_i32(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---- FP64 re-score of an assignment from the definition (Eq. 1-8) ---------------
__device__ __forceinline__ double wrap64(double x) {
  const double two_pi = 6.283185307179586476925286766559;
  return x - two_pi * rint(x / two_pi);
}

// A workgroup re-scores the assignment z of one matching into e64[tl], eu64[tl].
// A dummy (kDummyNode) costs wd; a Delta term needs both of its points
// matched, D^g all three, and only matched consecutive points are checked.
// The descriptor distances are taken four points at a time, 16 lanes per
// point striding its descriptor (coalesced reads; partial sums joined by a
// 16-lane tree); the triangle terms one point per lane.  A chain of dependent
// reads bounds it, so four waves share a matching's points while the chip (8192
// waves) holds all of a launch at once, and one takes each above.  us with four
// waves / with one, models of 30 and 75 points, descriptors of 162:
//   matchings     512     1024       1536       2048       2560       4096
//   30 points   8 / 17   10 / 27   22 / 33    25 / 34    34 / 36    48 / 39
//   75 points  15 / 39   24 / 65   45 / 71    48 / 72    65 / 77    94 / 85
// (descriptors of 16 cross at 1500 for 30 points and at 2300 for 75, by 1 to 2 us.)
//
// The sums do not depend on W: with four waves the points' terms go through LDS
// and the first wave adds them as the single wave does, lane 16 g the distances
// of points g, g + 4, ... and lane l the triangles ending at l, l + 64, ...; fused
// products are spelled out, since the compiler picks either of two by itself.
constexpr int kRescoreMany = 2048;
constexpr int kRescoreBlock = 256;  // points of the terms held in LDS at a time
template <int W>
__device__ __forceinline__ void rescore(const ModelView& m, const SceneView& s, const SearchParams& sp, double l1, double l2,
                                        double l3, double wd, const int32_t* __restrict__ z, long long tl,
                                        double* __restrict__ e64, double* __restrict__ eu64) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int32_t T = pair_limit(sp), TS = span_limit(sp);
  const int M = m.M, dim = s.dim;
  const double inf = __builtin_inf();
  if (ro(z) == -1) {
    if (threadIdx.x == 0) {
      if (e64) e64[tl] = inf;
      if (eu64) eu64[tl] = inf;
    }
    return;
  }
  const int grp = lane >> 4, gl = lane & 15;
  // the descriptor distance of point i0 + grp, in lane gl = 0 of its 16
  const auto distance = [&](int i0) {
    const int i = i0 + grp;
    const int n = i < M ? ro(z + i) : kDummyNode;
    double acc = 0.0;
    if (n != kDummyNode) {
      const float* f = m.desc + (long long)i * dim;
      const float* g = s.desc + (long long)n * dim;
      for (int d = gl; d < dim; d += 16) {
        const double v = (double)ro(f + d) - (double)ro(g + d);
        acc = fma(v, v, acc);
      }
    }
    for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    return n == kDummyNode ? wd : sqrt(acc);
  };
  // the terms of the triangle ending at point i, added in this order (the second
  // one is 0 unless a point is a dummy); false where the assignment is infeasible
  const auto triangle = [&](int i, double& ta, double& tb) {
    bool ok = true;
    ta = tb = 0.0;
    const int n = ro(z + i);
    const int nj = i >= 1 ? ro(z + (i - 1)) : kDummyNode;
    const int nk = i >= 2 ? ro(z + (i - 2)) : kDummyNode;
    if (n != kDummyNode && nj != kDummyNode && !consecutive_ok(sp, T, nj, ro(s.t + nj), n, ro(s.t + n))) ok = false;
    // the span reading (no dummies): the triangle's first and last frames
    if (TS > 0 && i >= 2 && !span_ok(ro(s.t + ro(z + (i - 2))), ro(s.t + n), TS)) ok = false;
    if (i >= 2 && (n == kDummyNode || nj == kDummyNode || nk == kDummyNode)) {
      // the Delta terms whose points are both matched; no D^g
      if (n != kDummyNode && nj != kDummyNode) {
        const long d1 = (long)(ro(m.t + i) - ro(m.t + (i - 1))) - (long)(ro(s.t + n) - ro(s.t + nj));
        ta = (double)(d1 < 0 ? -d1 : d1);
      }
      if (nj != kDummyNode && nk != kDummyNode) {
        const long d2 = (long)(ro(m.t + (i - 1)) - ro(m.t + (i - 2))) - (long)(ro(s.t + nj) - ro(s.t + nk));
        tb = (double)(d2 < 0 ? -d2 : d2);
      }
    } else if (i >= 2) {
      const long dt1 = (long)(ro(m.t + i) - ro(m.t + (i - 1))) - (long)(ro(s.t + n) - ro(s.t + nj));
      const long dt2 = (long)(ro(m.t + (i - 1)) - ro(m.t + (i - 2))) - (long)(ro(s.t + nj) - ro(s.t + nk));
      const float2 pi = ro(m.xy + i), pj = ro(m.xy + (i - 1)), pk = ro(m.xy + (i - 2));
      const float2 qi = ro(s.xy + n), qj = ro(s.xy + nj), qk = ro(s.xy + nk);
      double mid_m = ang64(pi.x, pi.y, pj.x, pj.y, pk.x, pk.y);
      double mid_s = ang64(qi.x, qi.y, qj.x, qj.y, qk.x, qk.y);
      double end_m = ang64(pj.x, pj.y, pi.x, pi.y, pk.x, pk.y);
      double end_s = ang64(qj.x, qj.y, qi.x, qi.y, qk.x, qk.y);
      if (sp.uns) {  // the unsigned reading: magnitudes of the angles
        mid_m = fabs(mid_m);
        mid_s = fabs(mid_s);
        end_m = fabs(end_m);
        end_s = fabs(end_s);
      }
      const double d1 = wrap64(mid_m - mid_s), d2 = wrap64(end_m - end_s);
      ta = fma(l3, sqrt(fma(d1, d1, d2 * d2)), (double)(dt1 < 0 ? -dt1 : dt1) + (double)(dt2 < 0 ? -dt2 : dt2));
    }
    return ok;
  };
  double su = 0.0, sd = 0.0;
  int bad = 0;
  if constexpr (W == 1) {
    for (int i0 = 0; i0 < M; i0 += 4) {
      const double u = distance(i0);
      if (gl == 0 && i0 + grp < M) su += u;
    }
    for (int i = lane; i < M; i += 64) {
      double ta, tb;
      if (!triangle(i, ta, tb)) bad = 1;
      sd += ta;
      sd += tb;
    }
    for (int off = 32; off > 0; off >>= 1) bad |= __shfl_xor(bad, off);
  } else {
    __shared__ double tu[kRescoreBlock], ta[kRescoreBlock], tb[kRescoreBlock];
    for (int b0 = 0; b0 < M; b0 += kRescoreBlock) {
      const int n = min(kRescoreBlock, M - b0);
      for (int j0 = wv * 4; j0 < n; j0 += W * 4) {
        const double u = distance(b0 + j0);
        if (gl == 0) tu[j0 + grp] = u;  // (past the last point: not read)
      }
      for (int j = threadIdx.x; j < n; j += W * 64)
        if (!triangle(b0 + j, ta[j], tb[j])) bad = 1;
      bad = __syncthreads_or(bad);
      if (wv == 0) {
        if (gl == 0)
#pragma unroll 4
          for (int j = grp; j < n; j += 4) su += tu[j];
        for (int j = lane; j < n; j += 64) {
          sd += ta[j];
          sd += tb[j];
        }
      }
      if (b0 + kRescoreBlock < M) __syncthreads();
    }
    if (wv != 0) return;
  }
  for (int off = 32; off > 0; off >>= 1) {
    su += __shfl_xor(su, off);
    sd += __shfl_xor(sd, off);
  }
  if (lane == 0) {
    if (e64) e64[tl] = bad ? inf : fma(l1, su, l2 * sd);
    if (eu64) eu64[tl] = bad ? inf : l1 * su;
  }
}

template <int W>
__global__ __launch_bounds__(W * 64) void k_rescore(ModelView m, SceneView s, SearchParams sp, double l1, double l2,
                                               double l3, double wd, const int32_t* __restrict__ assign,
                                               double* __restrict__ e64, double* __restrict__ eu64) {
  const int tl = blockIdx.x;
  rescore<W>(m, s, sp, l1, l2, l3, wd, assign + (long long)tl * m.M, tl, e64, eu64);
}

template <int W>
__global__ __launch_bounds__(W * 64) void k_rescore_batch(const PairDev* __restrict__ pairs,
                                                     const int2* __restrict__ items, int n_items,
                                                     SearchParams sp, double l1, double l2, double l3, double wd,
                                                     const int32_t* __restrict__ assign,
                                                     double* __restrict__ e64, double* __restrict__ eu64) {
  const int item = blockIdx.x;
  if (item >= n_items) return;
  const int2 it = items[item];
  const PairDev pd = pairs[it.x];
  rescore<W>(pd.m, pd.s, sp, l1, l2, l3, wd, assign + pd.assign0 + (long long)it.y * pd.m.M,
          pd.row0 + it.y, e64, eu64);
}

// Lists of at most 32 candidates take dp_forward_few, with fewer working waves
// per matching the more matchings a launch has; many matchings of at most 16
// candidates one wave each without barriers to speak of.  Longer lists take the
// 64-slot layout with the requested number of waves, by default 8, or 16 where
// there is at most one matching per CU.  Whole calls of 30 points in us:
//   lists of 12 to 18       512   1024   2048   4096 matchings
//     dp_forward, 1 wave     370    398    461    537
//     dp_forward, 4 waves    253    283    414    591
//     3 working waves        233    256    358    545
//     4 working waves        224    304    452    726
//   lists of 20 to 32       256    512   1024   4096
//     dp_forward, 2 waves    589    595    732   1780
//     dp_forward, 8 waves    321    342    582   1855
//     3 working waves        352    366    480   1350
//     7 working waves        268    297    493   1507
//     12 working waves       247    352    583   1948
//   lists of 60             256    512
//     dp_forward, 8 waves    681    902
//     dp_forward, 16 waves   563    918
//     15 working waves       617   1007
// The arithmetic of every cell is the same, so the results do not depend on the
// variant.
DPParts dp_parts(const DPLaunch* a, int n_parts, int& n) {
  DPParts b;
  b.n = n_parts;
  n = 0;
  for (int q = 0; q < kDPParts; ++q) {
    b.p[q] = a[q < n_parts ? q : 0];
    b.first[q] = n;
    if (q < n_parts) n += a[q].n_tau;
  }
  return b;
}

// LDS of the value tables and candidates where short lists keep them there, 0
// where they do not fit beside the kernel's own in 64 KB or the launch has more
// matchings than two per CU, whose other workgroups they would keep out.  20
// points, lists of 16: 64 us, recursion and backtracking 53 + 27 through memory
// and a second launch.
size_t few_hist_bytes(const DPLaunch* a, int n_parts, int n) {
  const DPLaunch& p = a[0];
  if (p.dummy || p.sp.uns || p.sp.K > 32 || n > 2 * kCUs) return 0;
  int m = 0;
  for (int q = 0; q < n_parts; ++q) m = a[q].m.M > m ? a[q].m.M : m;
  const size_t bytes = (size_t)(m - 2) * p.sp.K * p.sp.K * sizeof(float) + (size_t)m * p.sp.K * sizeof(float4);
  const size_t own = p.sp.K <= 16 ? sizeof(FewShared<4, 16>) : sizeof(FewShared<12, 32>);
  return bytes + own <= 64 * 1024 ? bytes : 0;
}

template <bool DEGEN>
hipError_t launch_dp_waves(const DPLaunch* parts, int n_parts, hipStream_t st) {
  int n = 0;
  const DPParts b = dp_parts(parts, n_parts, n);
  if (n <= 0) return hipSuccess;
  const DPLaunch& a = parts[0];
  if (a.dummy) {  // dummies: one variant, 8 waves and the 64-slot layout
    hipLaunchKernelGGL((k_dp<8, DEGEN, 64, true>), dim3(n), dim3(8 * 64), 0, st, b);
    return hipGetLastError();
  }
  if (a.sp.uns) {  // unsigned angles: one variant, 8 waves, the 64-slot layout and dense schedules
    hipLaunchKernelGGL((k_dp<8, DEGEN, 64, false, false, true>), dim3(n), dim3(8 * 64), 0, st, b);
    return hipGetLastError();
  }
  if (a.packed && a.sp.K > 32) {  // sparse scenes, long lists: packed schedules
    if (a.runs)
      hipLaunchKernelGGL((k_dp<8, DEGEN, 64, false, true, false, true>), dim3(n), dim3(8 * 64), 0, st, b);
    else
      hipLaunchKernelGGL((k_dp<8, DEGEN, 64, false, true>), dim3(n), dim3(8 * 64), 0, st, b);
    return hipGetLastError();
  }
#define STM_DP_FEW(NW, KL, HIST) \
  hipLaunchKernelGGL((k_dp_few<NW, DEGEN, KL, HIST>), dim3(n), dim3((NW + 1) * 64), HIST ? hist : 0, st, b)
  const size_t hist = few_hist_bytes(parts, n_parts, n);
  if (a.sp.K <= 16) {
    if (n <= 2 * kCUs && hist)
      STM_DP_FEW(4, 16, true);
    else if (n <= 2 * kCUs)
      STM_DP_FEW(4, 16, false);
    else if (n <= 8 * kCUs)
      STM_DP_FEW(3, 16, false);
    else
      hipLaunchKernelGGL((k_dp<1, DEGEN, 16>), dim3(n), dim3(64), 0, st, b);
    return hipGetLastError();
  }
  if (a.sp.K <= 32) {
    if (n <= kCUs && hist)
      STM_DP_FEW(12, 32, true);
    else if (n <= kCUs)
      STM_DP_FEW(12, 32, false);
    else if (n <= 2 * kCUs && hist)
      STM_DP_FEW(7, 32, true);
    else if (n <= 2 * kCUs)
      STM_DP_FEW(7, 32, false);
    else
      STM_DP_FEW(3, 32, false);
    return hipGetLastError();
  }
#undef STM_DP_FEW
  switch (a.waves ? a.waves : n <= kCUs ? 16 : 8) {
    case 4:
      hipLaunchKernelGGL((k_dp<4, DEGEN, 64>), dim3(n), dim3(4 * 64), 0, st, b);
      break;
    case 16:
      hipLaunchKernelGGL((k_dp<16, DEGEN, 64>), dim3(n), dim3(16 * 64), 0, st, b);
      break;
    default:
      hipLaunchKernelGGL((k_dp<8, DEGEN, 64>), dim3(n), dim3(8 * 64), 0, st, b);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dp_fast(const DPLaunch* a, int n, hipStream_t st) { return launch_dp_waves<false>(a, n, st); }

hipError_t launch_dp_degenerate(const DPLaunch* a, int n, hipStream_t st) { return launch_dp_waves<true>(a, n, st); }

template <bool DEGEN>
hipError_t launch_persistent_variant(const BatchLaunch& b, int n_wg, hipStream_t st) {
  if (b.dummy) {  // dummies: 8 waves whatever the tuning says
    hipLaunchKernelGGL((k_dp_persistent<8, DEGEN, kMaxList, true>), dim3(n_wg), dim3(8 * 64), 0, st, b);
    return hipGetLastError();
  }
  if (b.sp.uns) {  // unsigned angles: one variant, 8 waves, dense schedules
    hipLaunchKernelGGL((k_dp_persistent<8, DEGEN, kMaxList, false, false, true>), dim3(n_wg), dim3(8 * 64), 0, st,
                       b);
    return hipGetLastError();
  }
  if (b.packed) {  // sparse scenes: packed schedules, 8 waves
    if (b.runs)
      hipLaunchKernelGGL((k_dp_persistent<8, DEGEN, kMaxList, false, true, false, true>), dim3(n_wg), dim3(8 * 64), 0,
                         st, b);
    else
      hipLaunchKernelGGL((k_dp_persistent<8, DEGEN, kMaxList, false, true>), dim3(n_wg), dim3(8 * 64), 0, st, b);
    return hipGetLastError();
  }
  switch (b.waves) {
    case 4:
      hipLaunchKernelGGL((k_dp_persistent<4, DEGEN>), dim3(n_wg), dim3(4 * 64), 0, st, b);
      break;
    case 16:
      hipLaunchKernelGGL((k_dp_persistent<16, DEGEN>), dim3(n_wg), dim3(16 * 64), 0, st, b);
      break;
    default:
      hipLaunchKernelGGL((k_dp_persistent<8, DEGEN>), dim3(n_wg), dim3(8 * 64), 0, st, b);
  }
  return hipGetLastError();
}

hipError_t launch_dp_persistent(const BatchLaunch& b, int n_wg, hipStream_t st) {
  hipError_t e = launch_persistent_variant<false>(b, n_wg, st);
  if (e != hipSuccess) return e;
  return launch_persistent_variant<true>(b, n_wg, st);
}

hipError_t launch_item_cost(const PairDev* pairs, const int2* items, int n_items, const SearchParams& sp,
                            long long* cost, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_item_cost, dim3(n_items), dim3(64), 0, st, pairs, items, n_items, sp, cost);
  return hipGetLastError();
}

hipError_t launch_collect_infeasible(const PairDev* pairs, const int2* items, int n_items, const float* e32,
                                     int32_t* list, int32_t* count, int32_t* fell, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_collect_infeasible, dim3((n_items + 255) / 256), dim3(256), 0, st, pairs, items, n_items, e32,
                     list, count, fell);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int* p, int n, int v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

hipError_t launch_rescore_batch(const PairDev* pairs, const int2* items, int n_items, const SearchParams& sp,
                                double lambda1, double lambda2, double lambda3, double w_dummy,
                                const int32_t* assign, double* e64, double* eu64, hipStream_t st) {
  if (n_items <= 0 || (!e64 && !eu64)) return hipSuccess;
  const bool many = n_items > kRescoreMany;
  hipLaunchKernelGGL((many ? k_rescore_batch<1> : k_rescore_batch<4>), dim3(n_items), dim3(many ? 64 : 256), 0, st, pairs, items, n_items, sp,
                     lambda1, lambda2, lambda3, w_dummy, assign, e64, eu64);
  return hipGetLastError();
}

hipError_t launch_backtrack(const DPLaunch* a, int n_parts, hipStream_t st) {
  int n = 0;
  const DPParts b = dp_parts(a, n_parts, n);
  if (n <= 0 || few_hist_bytes(a, n_parts, n)) return hipSuccess;  // the recursion backtracked
  hipLaunchKernelGGL(k_backtrack, dim3(n), dim3(64), 0, st, b);
  return hipGetLastError();
}

hipError_t launch_rescore(const ModelView& m, const SceneView& s, const SearchParams& sp, double lambda1,
                          double lambda2, double lambda3, double w_dummy, const int32_t* assign,
                          int32_t n_tau, double* e64, double* eu64, hipStream_t st) {
  if (n_tau <= 0 || (!e64 && !eu64)) return hipSuccess;
  const bool many = n_tau > kRescoreMany;
  hipLaunchKernelGGL((many ? k_rescore<1> : k_rescore<4>), dim3(n_tau), dim3(many ? 64 : 256), 0, st, m, s, sp, lambda1, lambda2, lambda3,
                     w_dummy, assign, e64, eu64);
  return hipGetLastError();
}

}  // namespace stm

// Valuations by their changed part (single games).
//
// Along a run most valuations follow a handful of switches.  A switch at w
// changes the play of exactly the vertices whose play passes w (with the
// strategy after the switch): call the union over all switched vertices A.
// Every other vertex keeps its play, hence its nearest greater vertex, its
// fate and its valuation, and any two of them keep their order.  A step here
// therefore
//   find    collects A from the switched vertices backwards over the game's
//           in-edges (u joins when its current successor is in A)
//   walk    recomputes ng for the vertices of A only, jumping over everyone
//           else's ng
//   fate    follows their ng chains to the sink or to top: fate and root
//   decide  evaluates the switching rule for the vertices whose row holds a
//           vertex of A: nobody else's options changed since it last did not
//           switch
// Nothing is ranked: keys are coarse (coarse_key), and a comparison of two
// vertices with the same one climbs their ng chains to the meeting point and
// decides there by signed priority, which is the order ranks list the tree
// in (pg_val.hip), so the switches are the same.  Full valuations of a run
// stop at the coarse keys too (pg_val.hip, enqueue_coarse).
//
// Count valuations take the same steps with rows instead of keys: a vertex
// of A walks its play out of A, counting, and adds the row it arrives at, so
// every row is up to date and comparisons are the rows' own (1M vertices, 4
// priorities, solve from arrays: 23.4 -> 9.4 ms).
//
// Decisions go to a list of {vertex, new successor} pairs (`dec`) that the
// next step applies, so a step that gives up (a hub with too many in-edges,
// a chain or walk longer than its bound, a full list) has changed nothing a
// full valuation does not recompute.
//
// Two forms: a few kernels over the whole device for large A, and one block
// that runs whole inner and outer iterations by itself while A stays small
// (no launches, no host in between).
//
// Every access is a random line, so a step costs its round trips (small A)
// or its lines (large A), a full valuation the whole game's lines whatever
// changed: on the 10M-vertex random game 18 of the 95 valuations stay full
// (0.4-0.9 ms each with coarse keys, 1.4-2.1 ms with ranks), 32 take the
// device form (0.1-0.4 ms mostly) and 45 the block form (25-40 us each).
// Solves, load included, against full valuations with ranks throughout:
// 153 -> 36 ms there, 15.5 -> 5.6 ms at 1M vertices, 58 -> 14 ms on the
// 2M-vertex chain, 5.9 -> 2.4 ms at 40,000 vertices.
#include <algorithm>

#include "pg_coarse.h"
#include "pg_rows.h"

namespace pgk {

// words of a step's counters (g->inc.ic)
enum IncCounter : int {
  I_ERR = 0,      // ERR_* bits (C_ERR's index: the walk sets it)
  I_STOP = 1,     // the step gave up: redo it as a full valuation
  I_NA = 2,       // vertices in A
  I_NC = 3,       // candidates of the decide kernel
  I_NDEC = 4,     // decisions
  // block form only
  I_STATE = 5, I_NVAL = 6, I_ODDSW = 7, I_EVENSW = 8, I_MAJOR = 9,
  I_INNER = 10, I_A0 = 11, I_CUR = 12, I_EPOCH = 13,
  I_NWIDE = 14,   // candidates with wide rows (device form)
  I_OPEN = 16,    // passes after the first: vertices left for them
  I_CLOCK = 32, I_CLOCK_END = 33,   // a step's start and end (clock32)
  I_WORDS = 64,   // the part copied to the host
  // the find's queue, a line each
  I_TICKET = 64, I_QTAIL = 96, I_QDONE = 128,
  I_ALL = 160,    // the part cleared before a step
  I_OFFROW = 160, // the last check of the rows that failed (its number); the
                  // host's copy follows the I_WORDS
  I_HUB = 161,    // the game has vertices of more than kHub in-edges (its
                  // copy next)
  I_SIZE = 162
};
static_assert((int)I_ERR == (int)C_ERR, "the ng walk reports through ctr[0]");
constexpr int kFindLevels = 512;     // levels of a device form's find
constexpr int kIncMaxDegree = 2048;  // in-edges of one vertex, else give up
// In-edges beyond which all threads of a block share a vertex's: two lanes
// to eight took a hub's 2,000 at 1.5 us a round trip, more than a full
// valuation (1M vertices with 500 such hubs: finds of up to 3.9 ms, 0.23 ms
// so).
constexpr uint32_t kHub = 128;
constexpr int kIncFate = 1024;       // ng steps of one fate
constexpr int kIncBlocks = 1024;
constexpr int32_t kEpochMax = 1 << 30;   // the marks are cleared at the start
                                         // of a run past it

// ---------------------------------------------------------------------------
// the in-edge lists
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_in_count(
    const int32_t *__restrict__ tgt, uint32_t *cnt, int64_t m) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < m) atomicAdd(&cnt[tgt[e]], 1u);
}

// An in-edge is its source with the owner in bit 31.
__global__ __launch_bounds__(kBlock) void k_in_fill(
    const int64_t *__restrict__ off, const int32_t *__restrict__ tgt,
    const uint8_t *__restrict__ owner, uint32_t *cursor, uint32_t *in,
    int32_t N) {
  __shared__ int32_t wide[kBlock], s_n;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t e0 = v < N ? off[v] : 0, end = v < N ? off[v + 1] : 0;
  if (end - e0 > kWideRow) wide[atomicAdd(&s_n, 1)] = (int32_t)v;
  __syncthreads();
  // wide rows by the whole block (see wide_rows)
  const int n = s_n;
  for (int k = 0; k < n; ++k) {
    const int32_t w = wide[k];
    const int64_t w0 = off[w], w1 = off[w + 1];
    if (w1 - w0 <= (int64_t)kWideShare * n) continue;
    const uint32_t x = (uint32_t)w | ((uint32_t)owner[w] << 31);
    for (int64_t e = w0 + threadIdx.x; e < w1; e += kBlock)
      in[atomicAdd(&cursor[tgt[e]], 1u)] = x;
  }
  if (v >= N || (end - e0 > kWideRow && end - e0 > (int64_t)kWideShare * n))
    return;
  const uint32_t x = (uint32_t)v | ((uint32_t)owner[v] << 31);
  for (int64_t e = e0; e < end; e += 4) {
    int32_t t[4];
    uint32_t at[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = e + j < end ? tgt[e + j] : -1;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      at[j] = t[j] >= 0 ? atomicAdd(&cursor[t[j]], 1u) : 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (t[j] >= 0) in[at[j]] = x;
  }
}

// the lists' starts (n + 1) as cursors, and whether one of them is a hub's
__global__ void k_in_cursors(const uint32_t *a, uint32_t *b, int64_t n,
                             int32_t *any_hub) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  b[i] = a[i];
  if (a[i + 1] - a[i] > kHub) *any_hub = 1;
}

// Large games: the edges partitioned by ranges of their targets first, then
// each range counted, placed and filled by one block in LDS.  The counters
// of the two passes above are random lines with an atomic on each; here an
// edge's pair goes to one of a thousand streams and from there to an address
// that stays in one L2.  10M vertices, 35M edges: 1.4 + 3.0 ms (and a scan
// and a copy of the counters) -> 0.10 + 0.67 + 0.45; 1M vertices, 6.5M edges:
// 0.24 + 0.45 -> 0.02 + 0.06 + 0.05 ms.  Below kInPartMin the counters stay in
// the L2 anyway and the two passes are fewer launches (40,000 vertices: 22
// us, 300,000 the same either way); past kInPartMax the ranges' counters
// outgrow a block's LDS.
constexpr int64_t kInPartMin = int64_t(1) << 17, kInPartMax = int64_t(1) << 26;
constexpr int kInPartThreads = 1024, kInRangeMax = 8192;
constexpr int kInRanges = (int)(kInPartMax / kInRangeMax);   // LDS counters

// edges per range of the block's vertices [vb b, vb (b + 1))
__global__ __launch_bounds__(kInPartThreads) void k_in_hist(
    const int64_t *__restrict__ off, const int32_t *__restrict__ tgt,
    int32_t N, int vb, int shift, int nr, uint32_t *hist) {
  __shared__ uint32_t c[kInRanges];
  for (int k = threadIdx.x; k < nr; k += kInPartThreads) c[k] = 0;
  __syncthreads();
  const int64_t v0 = (int64_t)blockIdx.x * vb;
  const int64_t e1 = off[min(v0 + vb, (int64_t)N)];
  for (int64_t e = off[v0] + threadIdx.x; e < e1; e += kInPartThreads)
    atomicAdd(&c[tgt[e] >> shift], 1u);
  __syncthreads();
  for (int k = threadIdx.x; k < nr; k += kInPartThreads)
    hist[(int64_t)k * gridDim.x + blockIdx.x] = c[k];
}

// {target inside its range, source}, range by range (at: hist scanned)
__global__ __launch_bounds__(kInPartThreads) void k_in_part(
    const int64_t *__restrict__ off, const int32_t *__restrict__ tgt,
    const uint8_t *__restrict__ owner, int32_t N, int vb, int shift, int nr,
    const uint32_t *__restrict__ at, uint2 *pairs) {
  __shared__ uint32_t c[kInRanges];
  __shared__ int32_t wide[kInPartThreads], s_n;
  if (threadIdx.x == 0) s_n = 0;
  for (int k = threadIdx.x; k < nr; k += kInPartThreads)
    c[k] = at[(int64_t)k * gridDim.x + blockIdx.x];
  __syncthreads();
  const int64_t v0 = (int64_t)blockIdx.x * vb;
  const int64_t v1 = min(v0 + vb, (int64_t)N);
  const uint32_t low = (1u << shift) - 1u;
  for (int64_t v = v0 + threadIdx.x; v < v1; v += kInPartThreads) {
    const uint32_t x = (uint32_t)v | ((uint32_t)owner[v] << 31);
    const int64_t e0 = off[v], end = off[v + 1];
    if (end - e0 > kWideRow) {
      const int k = atomicAdd(&s_n, 1);
      if (k < kInPartThreads) {
        wide[k] = (int32_t)v;
        continue;
      }
    }
    for (int64_t e = e0; e < end; e += 4) {
      int32_t t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] = e + j < end ? tgt[e + j] : -1;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (t[j] >= 0)
          pairs[atomicAdd(&c[t[j] >> shift], 1u)] =
              make_uint2((uint32_t)t[j] & low, x);
    }
  }
  __syncthreads();
  // wide rows by the whole block, or by a thread each (see wide_rows)
  const int n = min(s_n, kInPartThreads);
  for (int k = 0; k < n; ++k) {
    const int32_t w = wide[k];
    const int64_t e0 = off[w], end = off[w + 1];
    const bool all = end - e0 > (int64_t)kWideShare * n;
    if (!all && threadIdx.x != k) continue;
    const uint32_t x = (uint32_t)w | ((uint32_t)owner[w] << 31);
    for (int64_t e = e0 + (all ? threadIdx.x : 0); e < end;
         e += all ? kInPartThreads : 1) {
      const int32_t t = tgt[e];
      pairs[atomicAdd(&c[t >> shift], 1u)] = make_uint2((uint32_t)t & low, x);
    }
  }
}

// Adds one to *c for every active lane's counter c[x]; each gets its place.
// Lanes that share the first one's counter take one atomic: all in-edges of a
// hub meet in one block, and a wave's 64 atomics on one LDS word took their
// turns (333,000 in-edges of one vertex: k_in_range 298 -> 94 us).
__device__ __forceinline__ uint32_t lds_place(uint32_t *c, uint32_t x) {
  const uint32_t first = __builtin_amdgcn_readfirstlane(x);
  const uint64_t same = __ballot(x == first);
  const int lane = threadIdx.x & (kWave - 1);
  if (__popcll(same) < 8 || x != first) return atomicAdd(&c[x], 1u);
  const int lead = __ffsll((unsigned long long)same) - 1;
  uint32_t at = 0;
  if (lane == lead) at = atomicAdd(&c[x], (uint32_t)__popcll(same));
  return __shfl(at, lead) +
         (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
}

// a range's in-edge lists: range blockIdx.x, 1 << shift vertices, nb parts
__global__ __launch_bounds__(kInPartThreads) void k_in_range(
    const uint2 *__restrict__ pairs, const uint32_t *__restrict__ at, int nb,
    uint32_t M, int32_t N, int shift, uint32_t *in_off, uint32_t *in,
    int32_t *any_hub) {
  extern __shared__ uint32_t rc[];   // a counter per vertex
  __shared__ uint32_t s_w[kInPartThreads / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), R = 1 << shift;
  const int64_t k = blockIdx.x;
  const uint32_t p0 = at[k * nb];
  const uint32_t p1 = k + 1 < gridDim.x ? at[(k + 1) * nb] : M;
  for (int i = tid; i < R; i += kInPartThreads) rc[i] = 0;
  __syncthreads();
  // four pairs a round trip: a hub's are all this block's
  for (uint32_t p = p0 + tid; p < p1; p += 4 * kInPartThreads) {
    uint32_t x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      x[j] = p + j * kInPartThreads < p1 ? pairs[p + j * kInPartThreads].x
                                         : ~0u;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (x[j] != ~0u) (void)lds_place(rc, x[j]);
  }
  __syncthreads();
  // exclusive scan, R / kInPartThreads neighbours a thread
  const int per = R / kInPartThreads;
  uint32_t sum = 0;
  for (int j = 0; j < per; ++j) sum += rc[tid * per + j];
  uint32_t inc = sum;
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t o = __shfl_up(inc, d);
    if (lane >= d) inc += o;
  }
  if (lane == kWave - 1) s_w[tid / kWave] = inc;
  __syncthreads();
  uint32_t base = p0 + inc - sum;
  for (int w = 0; w < tid / kWave; ++w) base += s_w[w];
  for (int j = 0; j < per; ++j) {
    const uint32_t c = rc[tid * per + j];
    rc[tid * per + j] = base;
    const int64_t v = (k << shift) + tid * per + j;
    if (v < N) in_off[v] = base;
    if (c > kHub) *any_hub = 1;
    base += c;
  }
  __syncthreads();
  for (uint32_t p = p0 + tid; p < p1; p += 4 * kInPartThreads) {
    uint2 x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      x[j] = p + j * kInPartThreads < p1 ? pairs[p + j * kInPartThreads]
                                         : make_uint2(~0u, 0u);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (x[j].x != ~0u) in[lds_place(rc, x[j].x)] = x[j].y;
  }
}

// ---------------------------------------------------------------------------
// shared device code
// ---------------------------------------------------------------------------
struct IncP {
  int32_t N, n_oddpri;
  const int64_t *off;
  const int32_t *tgt, *pri;
  const uint32_t *in_off, *in;
  int2 *sp;
  int32_t *key, *ng, *cand;
  uint8_t *rs;
  int32_t *mark, *cmark;   // epoch of the last step that took the vertex
  int32_t *list;           // A of every step since the last All_Even
  int32_t list_cap;
  int32_t *cl;             // candidates (with repeats: cmark tells them)
  int32_t cl_cap;
  int32_t *q;              // the find's queue (kFindChunk-int chunks, -1)
  int32_t q_cap;           // chunks
  bool wide;               // the game has rows beyond kWideRow entries
  int32_t *wl;             // the candidates that have them
  bool hub;                // it has vertices of more than kHub in-edges
  // count valuations (kernels with D > 0)
  int32_t *cnt;
  const uint8_t *pidx;
  uint32_t odd_cols;
};

__device__ __forceinline__ CoarseP coarse(const IncP &P) {
  return CoarseP{P.N, P.n_oddpri, P.off, P.tgt, P.pri, P.ng, P.key};
}

template <bool F = false>
__device__ __forceinline__ bool inc_decide(const IncP &P, int32_t v, bool odd,
                                           int32_t *to, bool *stop) {
  const int2 me = P.sp[v];
  if (me.y == kTopMark) return false;   // known to stay top
  const CoarseP C = coarse(P);
  bool tie;
  const bool sw = coarse_row(C, v, me.x, odd, to, &tie);
  return tie ? coarse_exact<F>(C, v, me.x, odd, to, stop) : sw;
}

// The rule of a rank game (D = 0) or with count rows of D ints.
template <int D, bool F = false>
__device__ __forceinline__ bool rule(const IncP &P, int32_t v, bool odd,
                                     int32_t *to, bool *stop) {
  if constexpr (D == 0) {
    return inc_decide<F>(P, v, odd, to, stop);
  } else {
    const int2 me = P.sp[v];
    if (me.y == kTopMark) return false;   // known to stay top
    return odd ? cnt_decide_odd<D>(P.off, P.tgt, P.cnt, P.odd_cols, v, me, to)
               : cnt_decide_even<D>(P.N, P.off, P.tgt, P.cnt, P.odd_cols, v,
                                    me, to);
  }
}

// wide_rows for the vertices of the step's candidates (a vertex known to stay
// top keeps its choice).
template <int T>
__device__ __forceinline__ bool inc_wide(const IncP &P, bool live, int32_t v,
                                         bool odd, WideLds<T> &W, bool *sw,
                                         int32_t *to, bool *stop,
                                         unsigned long long most = ~0ull) {
  return wide_rows<T>(coarse(P), live && P.sp[v].y != kTopMark, v, odd, P.sp,
                      W, sw, to, stop, most);
}

// The ng of a vertex of A is open until its walk (count valuations walk
// plays: their ng is found again by the next full valuation).
__device__ __forceinline__ void inc_open(const IncP &P, int32_t v) {
  if (P.cnt) return;
  P.ng[v] = -1;
  P.cand[v] = -1;
}

// Applies a decision; the switched vertex is in A.
__device__ __forceinline__ void inc_apply(const IncP &P, int32_t epoch,
                                          int2 d) {
  P.sp[d.x] = make_int2(d.y, d.y == P.N ? 2147483647 : P.pri[d.y]);
  P.mark[d.x] = epoch;
  inc_open(P, d.x);
}

// The walk of one vertex of A (ng_walk of pg_val.hip on the changed part: an
// open vertex is one of A, everyone else's ng is jumped over).  False when
// the steps ran out (the candidate is kept).
__device__ __forceinline__ bool inc_walk(const IncP &P, int32_t *err,
                                         int32_t v, int steps) {
  const int32_t N = P.N;
  int32_t u = ld_relaxed(&P.cand[v]);
  if (u < 0) {
    const int2 me = P.sp[v];
    if (me.y == kTopMark) {
      st_relaxed(&P.ng[v], N + 1);
      return true;
    }
    u = me.x;
  }
  const int32_t pv = P.pri[v];
  int32_t res = -1;
  for (int s = 0; s < steps; ++s) {
    if (u == N) {
      res = N;
      break;
    }
    if (u == v) {
      // the largest vertex of its cycle, whose priority must be even for an
      // admissible sigma (section 3)
      if (pv & 1) atomicOr(err, ERR_INADMISSIBLE);
      res = N + 1;
      break;
    }
    if (P.pri[u] > pv) {
      res = u;
      break;
    }
    const int32_t r = ld_relaxed(&P.ng[u]);
    if (r >= N) {
      res = r;
      break;
    }
    if (r >= 0) {
      u = r;
      continue;
    }
    const int32_t c = ld_relaxed(&P.cand[u]);
    if (c >= 0) {
      u = c;
    } else {
      const int2 su = P.sp[u];
      if (su.y == kTopMark) {
        res = N + 1;
        break;
      }
      u = su.x;
    }
  }
  if (res >= 0) st_relaxed(&P.ng[v], res);
  else st_relaxed(&P.cand[v], u);
  return res >= 0;
}

// The fate and the coarse key of one vertex of A: along its ng chain to the
// sink, to top or to a vertex outside A, whose own stand.
__device__ __forceinline__ bool inc_fate(const IncP &P, int32_t epoch,
                                         int32_t v) {
  const int32_t N = P.N;
  int32_t a = v, r = P.ng[v], k = PG_KEY_TOP;
  int f = 0;
  for (int s = 0; s < kIncFate; ++s) {
    if (r >= N) {
      f = r == N ? 1 : 2;
      k = coarse_key(a);
      break;
    }
    if (P.mark[r] != epoch) {
      f = P.rs[r];
      k = P.key[r];
      break;
    }
    a = r;
    r = P.ng[r];
  }
  if (!f) return false;
  P.rs[v] = (uint8_t)f;
  P.key[v] = f == 2 ? PG_KEY_TOP : k;
  return true;
}

// The row and the fate of one vertex of A: along its play to a vertex outside
// A (or the sink), whose row stands.  A play that stays in A circles (Brent's
// detection) and is top; its cycle's largest priority must be even for an
// admissible sigma (section 3).  False when the steps run out.
template <int D>
__device__ __forceinline__ bool inc_row(const IncP &P, int32_t epoch,
                                        int32_t *err, int32_t v, int steps) {
  const int32_t N = P.N;
  int32_t acc[D] = {};
  add_unit<D>(acc, P.pidx[v], 1);
  int2 s = P.sp[v];
  int32_t u = s.x, mark = v;
  int lam = 1, power = 1, f = 0;
  for (int k = 0; k < steps; ++k) {
    if (s.y == kTopMark) {
      f = 2;
      break;
    }
    if (u == N || ld_relaxed(&P.mark[u]) != epoch) {
      int32_t r[D];
      f = load_val<D>(P.cnt, u, r) ? 2 : 1;
#pragma unroll
      for (int i = 0; i < D; ++i) acc[i] += r[i];
      break;
    }
    if (u == mark) {
      int32_t best = P.pri[u];
      for (int32_t x = P.sp[u].x; x != u; x = P.sp[x].x)
        best = max(best, P.pri[x]);
      if (best & 1) atomicOr(err, ERR_INADMISSIBLE);
      f = 2;
      break;
    }
    if (lam == power) {
      mark = u;
      power <<= 1;
      lam = 0;
    }
    ++lam;
    add_unit<D>(acc, P.pidx[u], 1);
    s = P.sp[u];
    u = s.x;
  }
  if (!f) return false;
  if (f == 2) {
#pragma unroll
    for (int i = 0; i < D; ++i) acc[i] = i == 0 ? -1 : 0;
  }
  store_vec<D>(P.cnt + (int64_t)v * D, acc);
  P.rs[v] = (uint8_t)f;
  return true;
}

// ---------------------------------------------------------------------------
// the device form: one step in a few kernels
// ---------------------------------------------------------------------------
// Applies the decisions: A starts with them.
__global__ __launch_bounds__(kBlock) void k_inc_begin(
    IncP P, int32_t epoch, int32_t a0, const int2 *__restrict__ dec,
    int32_t nsw, int32_t *ic) {
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nsw;
       i += gridDim.x * blockDim.x) {
    const int2 d = dec[i];
    inc_apply(P, epoch, d);
    P.list[a0 + i] = d.x;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ic[I_CLOCK] = clock32();
    ic[I_NA] = nsw;
  }
}

// One in-edge x of w in A: its source joins A when w is its successor; true
// once per source (a repeated edge or a switched vertex meets its mark; two
// lanes of w's group with the same source are told apart by shuffles).  Also
// returns the source's own in-edge range: the loads are independent, so a
// level of a find costs two round trips (the range was fetched with the
// level before).  A source that slips through twice is harmless: it is only
// walked twice.
__device__ __forceinline__ bool inc_edge(const IncP &P, int32_t epoch,
                                         int32_t w, uint32_t x, bool live,
                                         int L, uint2 *range) {
  const int32_t u = (int32_t)(x & 0x7fffffffu);
  bool a = false;
  *range = make_uint2(0u, 0u);
  if (live) {
    const int32_t su = P.sp[u].x;
    const int32_t mk = ld_relaxed(&P.mark[u]);
    range->x = P.in_off[u];
    range->y = P.in_off[u + 1];
    a = su == w && mk != epoch;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t ba = __ballot(a);
  if (L > 1 && __ballot(a && __popcll((ba >> (lane & ~(L - 1))) &
                                      ((1ull << L) - 1ull)) > 1)) {
    const int32_t mine = a ? u : -1;
    for (int k = 1; k < L; ++k) {
      const int32_t other = __shfl_up(mine, k);
      if ((lane & (L - 1)) >= k && a && other == u) a = false;
    }
  }
  if (a) {
    st_relaxed(&P.mark[u], epoch);
    inc_open(P, u);
  }
  return a;
}

// The same for an in-edge of a hub, whose sources the whole block looks at:
// the mark's exchange tells one source's edges apart.
__device__ __forceinline__ bool inc_hub_edge(const IncP &P, int32_t epoch,
                                             int32_t w, uint32_t x, bool live,
                                             uint2 *range) {
  const int32_t u = (int32_t)(x & 0x7fffffffu);
  bool a = false;
  *range = make_uint2(0u, 0u);
  if (live) {
    const int32_t su = P.sp[u].x;
    const int32_t mk = ld_relaxed(&P.mark[u]);
    range->x = P.in_off[u];
    range->y = P.in_off[u + 1];
    a = su == w && mk != epoch && atomicExch(&P.mark[u], epoch) != epoch;
  }
  if (a) inc_open(P, u);
  return a;
}

// Lanes per vertex of a find level of n vertices for T threads: a level is
// bound by its round trips, so few vertices spread their in-edges over up
// to 8 lanes.
__device__ __forceinline__ int find_lanes(int n, int T) {
  return n * 8 <= T ? 8 : n * 4 <= T ? 4 : n * 2 <= T ? 2 : 1;
}

// The find.  A block takes a chunk of A and follows the in-edges breadth
// first by itself, its part of A and its candidates (the Odd sources: they
// have an option in A) in LDS: plays inside A are tens of vertices long, so
// a kernel per level would be mostly launches, and a place in a global list
// per level mostly atomics' round trips.  A level costs a block two round
// trips (3 us), and per 64 vertices the rate at which one CU fetches random
// lines; trees are uneven (on the 10M-vertex game one switch can hold 200k
// vertices in 90 levels), so a level beyond kFindKeep vertices hands the
// rest on in chunks of a queue that idle blocks wait at.  Two blocks per CU
// with the queue took the longest finds of that game from 3.1 and 2.0 to 1.3
// and 0.77 ms (all 38: 11.4 -> 7.1 ms) against three launches that each
// handed their widest levels to the next; what is left are the levels.
// 256, 1024 and 2048 blocks were 0-4 % slower.
//
// Hubs are looked at by the whole block, and those of a level that have more
// than twice kFindHubs in-edges together go to the queue as well, with the
// level they are of (they are in A's list already).
//
// Chunk t is A's own t-th stretch for t < S, else place t - S of the queue.
// Blocks take tickets in order and wait for their chunk to come, or for all
// S + tail chunks to be done.  A waiting block needs nothing but the blocks
// that hold earlier tickets, and these run: no order of residency can stop
// it.  A queue place holds -1 until its writer stores the value, and again
// after its reader took it.
//
// The tail counts the places asked for, not those that are there: a wave past
// the LDS lists takes a chunk for the few sources it has just found, so a
// hub's in-edges can ask for more than the q_cap chunks that every vertex of
// the game once would need.  Whoever asks beyond them sets I_STOP, and no
// ticket names a place at or past q_cap; one that names a place nobody got to
// write ends its wait by I_STOP.
constexpr int kFindChunk = 64, kFindA = 1024, kFindC = 2048;
constexpr int kFindKeep = 128, kFindBlocks = 512;
constexpr int kFindHubs = 2048;   // in-edges of hubs a block keeps to itself
constexpr int kFindItems = kFindChunk - 1;   // of a queue chunk: word 0 is
                                             // its level, -2 no item
constexpr int kFindWait = 1 << 20;           // polls, then the step gives up

// the next chunk, or -1: all done, or the step gave up
__device__ __forceinline__ int32_t find_ticket(int32_t S, int32_t q_cap,
                                               int32_t *ic) {
  const int32_t t = atomicAdd(&ic[I_TICKET], 1);
  if (t < S) return t;
  if (t - S >= q_cap) return -1;
  for (int k = 0; k < kFindWait; ++k) {
    // done first (never negative: the tail's address waits for it): when it
    // has reached S + tail, no chunk was open then
    const int32_t done = ld_relaxed(&ic[I_QDONE]);
    const int32_t tail = ld_relaxed(&ic[I_QTAIL + (done < 0)]);
    if (tail > t - S) return t;
    if (done == S + tail || ld_relaxed(&ic[I_STOP])) return -1;
    __builtin_amdgcn_s_sleep(8);
  }
  atomicOr(&ic[I_STOP], 1);
  return -1;
}

// H: for games with hubs (the code for them slows the others' down, here and
// in the kernels with S and W below, by 3 to 15 %).
template <bool H>
__global__ __launch_bounds__(kBlock) void k_inc_find(IncP P, int32_t epoch,
                                                     int32_t a0, int32_t nsw,
                                                     int32_t *ic) {
  __shared__ int32_t la[kFindA], lc[kFindC];
  __shared__ uint2 lr[kFindA];   // in-edge ranges of la
  __shared__ int32_t s_na, s_nc, s_base, s_q, s_stop, s_t, s_level;
  __shared__ int32_t lh[kFindKeep], s_nh, s_hd;   // the level's hubs
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int32_t S = (nsw + kFindChunk - 1) / kFindChunk;
  if (tid == 0) s_stop = 0;
  // entries [from, to) of an LDS list to a global one (all threads)
  auto flush = [&](const int32_t *l, int from, int to, int32_t *ctr,
                   int32_t *out, int32_t cap) {
    if (from >= to) return;
    __syncthreads();
    if (tid == 0) s_base = atomicAdd(ctr, to - from);
    __syncthreads();
    for (int i = from + tid; i < to; i += kBlock) {
      const int32_t at = s_base + (i - from);
      if (at < cap) out[at] = l[i];
      else s_stop = 1;
    }
    __syncthreads();
  };
  // a source u joins A (a) with its in-edge range, or is a candidate (c); all
  // lanes of the wave
  auto place = [&](bool a, bool c, int32_t u, uint2 range, int level) {
    const int pc = wave_place(&s_nc, c);
    if (c && pc < kFindC) lc[pc] = u;
    const int pa = wave_place(&s_na, a);
    if (a && pa < kFindA) {
      la[pa] = u;
      lr[pa] = range;
    }
    // past the LDS lists (rare): to the global ones
    const bool oc = c && pc >= kFindC, oa = a && pa >= kFindA;
    if (__ballot(oc)) {
      const int32_t at = wave_place(&ic[I_NC], oc);
      if (oc && at < P.cl_cap) P.cl[at] = u;
      else if (oc) s_stop = 1;
    }
    const uint64_t bo = __ballot(oa);
    if (bo) {   // one or two chunks of the wave's own
      const int32_t at = wave_place(&ic[I_NA], oa);
      if (oa && a0 + at >= P.list_cap) s_stop = 1;
      else if (oa) P.list[a0 + at] = u;
      const int n = __popcll(bo), nq = (n + kFindItems - 1) / kFindItems;
      int32_t q0 = 0;
      if (lane == 0) q0 = atomicAdd(&ic[I_QTAIL], nq);
      q0 = __shfl(q0, 0);
      if (q0 + nq > P.q_cap) {
        if (lane == 0) atomicOr(&ic[I_STOP], 1);
      } else {
        int32_t *q = P.q + (int64_t)q0 * kFindChunk;
        for (int k = 0; k < nq; ++k)
          if (lane == 0 || k * kFindItems + lane - 1 >= n)
            st_relaxed(q + k * kFindChunk + lane,
                       lane == 0 ? level + 1 : -2);
        const int r = __popcll(bo & ((1ull << lane) - 1ull));
        if (oa)
          st_relaxed(q + r / kFindItems * kFindChunk + 1 +
                         r % kFindItems, u);
      }
    }
  };
  for (;;) {
    __syncthreads();
    if (tid == 0) s_t = find_ticket(S, P.q_cap, ic);
    __syncthreads();
    const int32_t t = s_t;
    if (t < 0) break;
    if (tid < kWave) {   // (a chunk is a wave)
      int32_t w = -2, lev = 0;
      if (t < S) {
        if (t * kFindChunk + lane < nsw) w = P.list[a0 + t * kFindChunk + lane];
      } else {
        int32_t *q = P.q + (int64_t)(t - S) * kFindChunk + lane;
        for (int k = 0; (w = ld_relaxed(q)) == -1; ++k)
          if (k >= kFindWait || ld_relaxed(&ic[I_STOP])) {
            w = -2;
            s_stop = 1;
            break;
          }
        st_relaxed(q, -1);
        lev = __shfl(w, 0);
        if (lane == 0) w = -2;
      }
      const uint64_t b = __ballot(w >= 0);
      if (w >= 0) {
        const int at = __popcll(b & ((1ull << lane) - 1ull));
        la[at] = w;
        lr[at] = make_uint2(P.in_off[w], P.in_off[w + 1]);
      }
      if (lane == 0) {
        s_na = __popcll(b);
        s_nc = 0;
        s_level = lev;
      }
    }
    __syncthreads();
    int beg = 0, end = s_na, level = s_level;
    int flushed = end;   // the chunk is in A's list already
    for (; beg < end; ++level) {
      if (level >= kFindLevels) {
        s_stop = 1;
        break;
      }
      const int L = find_lanes(end - beg, kBlock);
      int hubs = 0;
      if constexpr (H) {
        if (tid == 0) s_nh = s_hd = 0;
        __syncthreads();
        if (tid < end - beg) {
          const uint32_t d = lr[beg + tid].y - lr[beg + tid].x;
          if (d > (uint32_t)kIncMaxDegree) {
            s_stop = 1;
          } else if (d > kHub) {
            lh[atomicAdd(&s_nh, 1)] = beg + tid;
            atomicAdd(&s_hd, (int)d);
          }
        }
        __syncthreads();
        hubs = s_nh;
      }
      for (int i0 = beg; i0 < end; i0 += kBlock / L) {
        const int i = i0 + tid / L;
        uint32_t e = 0, e1 = 0;
        int32_t w = -1;
        if (i < end && (!H || lr[i].y - lr[i].x <= kHub)) {
          w = la[i];
          e = lr[i].x + tid % L;
          e1 = lr[i].y;
        }
        for (; __ballot(e < e1); e += L) {
          const bool live = e < e1;
          const uint32_t x = live ? P.in[e] : 0u;
          uint2 range;
          const bool a = inc_edge(P, epoch, w, x, live, L, &range);
          place(a, live && (x >> 31), (int32_t)(x & 0x7fffffffu), range,
                level);
        }
      }
      if (H && hubs > 0 && s_hd > 2 * kFindHubs) {
        // all but the first kFindHubs in-edges to the queue, as many in a
        // chunk by the average
        const int per =
            min(max((int)((int64_t)kFindHubs * hubs / s_hd), 1), kFindItems);
        const int nq = (hubs - per + per - 1) / per;
        __syncthreads();
        if (tid == 0) {
          s_q = atomicAdd(&ic[I_QTAIL], nq);
          if (s_q + nq > P.q_cap) atomicOr(&ic[I_STOP], 1);
        }
        __syncthreads();
        if (s_q + nq > P.q_cap) {
          s_stop = 1;
        } else {
          for (int i = tid; i < nq * kFindChunk; i += kBlock) {
            const int j = i % kFindChunk;
            const int h = per + i / kFindChunk * per + j - 1;
            st_relaxed(P.q + (int64_t)s_q * kFindChunk + i,
                       j == 0                      ? level
                       : j <= per && h < hubs ? la[lh[h]]
                                                   : -2);
          }
        }
        hubs = min(per, hubs);
      }
      for (int k = 0; H && k < hubs; ++k) {
        const int32_t w = la[lh[k]];
        const uint32_t e1 = lr[lh[k]].y;
        for (uint32_t e = lr[lh[k]].x + tid; __ballot(e < e1); e += kBlock) {
          const bool live = e < e1;
          const uint32_t x = live ? P.in[e] : 0u;
          uint2 range;
          const bool a = inc_hub_edge(P, epoch, w, x, live, &range);
          place(a, live && (x >> 31), (int32_t)(x & 0x7fffffffu), range,
                level);
        }
      }
      __syncthreads();
      const int na = min(s_na, kFindA), nc = min(s_nc, kFindC);
      __syncthreads();
      beg = end;
      end = na;
      if (nc > kFindC / 2) {
        flush(lc, 0, nc, &ic[I_NC], P.cl, P.cl_cap);
        if (tid == 0) s_nc = 0;
      }
      if (end - beg > kFindKeep || end > kFindA / 2) {
        flush(la, flushed, end, &ic[I_NA], P.list + a0, P.list_cap - a0);
        if (end - beg > kFindKeep) {
          // all but the first kFindChunk to 126 go to the queue
          const int nq = (end - beg - kFindChunk) / kFindItems;
          if (tid == 0) {
            s_q = atomicAdd(&ic[I_QTAIL], nq);
            if (s_q + nq > P.q_cap) atomicOr(&ic[I_STOP], 1);
          }
          __syncthreads();
          const int from = end - nq * kFindItems;
          if (s_q + nq > P.q_cap) {
            s_stop = 1;
          } else {
            for (int i = tid; i < nq * kFindChunk; i += kBlock) {
              const int k = i / kFindChunk, j = i % kFindChunk;
              st_relaxed(P.q + (int64_t)s_q * kFindChunk + i,
                         j == 0 ? level + 1
                                : la[from + k * kFindItems + j - 1]);
            }
          }
          end = from;
        }
        // the level moves to the front of the list
        const int n = end - beg;   // at most kFindKeep
        int32_t mv = 0;
        uint2 mr = make_uint2(0u, 0u);
        if (tid < n) {
          mv = la[beg + tid];
          mr = lr[beg + tid];
        }
        __syncthreads();
        if (tid < n) {
          la[tid] = mv;
          lr[tid] = mr;
        }
        beg = 0;
        end = flushed = n;
        if (tid == 0) s_na = n;
      }
      __syncthreads();
    }
    flush(la, flushed, end, &ic[I_NA], P.list + a0, P.list_cap - a0);
    __syncthreads();
    flush(lc, 0, min(s_nc, kFindC), &ic[I_NC], P.cl, P.cl_cap);
    __syncthreads();
    if (tid == 0) {
      if (s_stop) atomicOr(&ic[I_STOP], 1);
      atomicAdd(&ic[I_QDONE], 1);
    }
  }
}
static_assert(kFindChunk == kWave && kFindKeep <= kBlock, "k_inc_find");

__global__ __launch_bounds__(kBlock) void k_inc_walk(IncP P, int32_t a0,
                                                     int steps, int pass,
                                                     int last, int32_t *ic) {
  if (ic[I_STOP] || (pass > 0 && !ic[I_OPEN + pass])) return;
  const int32_t n = ic[I_NA];
  bool open = false;
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += gridDim.x * blockDim.x) {
    const int32_t v = P.list[a0 + i];
    if (pass > 0 && ld_relaxed(&P.ng[v]) >= 0) continue;
    open |= !inc_walk(P, &ic[I_ERR], v, steps);
  }
  if (open) atomicOr(last ? &ic[I_STOP] : &ic[I_OPEN + pass + 1],
                     1);
}

// Count valuations: rows and fates; the second pass takes the vertices whose
// steps ran out in the first (rs 0).
template <int D>
__global__ __launch_bounds__(kBlock) void k_inc_rows(IncP P, int32_t epoch,
                                                     int32_t a0, int steps,
                                                     int pass, int last,
                                                     int32_t *ic) {
  if (ic[I_STOP] || (pass > 0 && !ic[I_OPEN + pass])) return;
  const int32_t n = ic[I_NA];
  bool open = false;
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += gridDim.x * blockDim.x) {
    const int32_t v = P.list[a0 + i];
    if (pass > 0 && P.rs[v]) continue;
    if (!inc_row<D>(P, epoch, &ic[I_ERR], v, steps)) {
      P.rs[v] = 0;
      open = true;
    }
  }
  if (open) atomicOr(last ? &ic[I_STOP] : &ic[I_OPEN + pass + 1],
                     1);
}

__global__ __launch_bounds__(kBlock) void k_inc_fate(IncP P, int32_t epoch,
                                                     int32_t a0, int32_t *ic) {
  if (ic[I_STOP]) return;
  const int32_t n = ic[I_NA];
  bool open = false;
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += gridDim.x * blockDim.x)
    open |= !inc_fate(P, epoch, P.list[a0 + i]);
  if (open) atomicOr(&ic[I_STOP], 1);
}

// The rule for every candidate.
template <int D>
__global__ __launch_bounds__(kBlock) void k_inc_decide(IncP P, int32_t epoch,
                                                       int odd, int2 *dec,
                                                       int32_t *ic) {
  if (ic[I_STOP]) return;
  const int32_t n = ic[I_NC];
  bool stop = false;
  for (int32_t i0 = blockIdx.x * blockDim.x; i0 < n;
       i0 += gridDim.x * blockDim.x) {
    const int32_t i = i0 + threadIdx.x;
    bool sw = false, live = false;
    int32_t v = 0, to = 0;
    if (i < n) {
      v = P.cl[i];
      live = !odd || atomicExch(&P.cmark[v], epoch) != epoch;
    }
    if constexpr (D == 0) {
      if (P.wide) {   // wide rows are listed for k_inc_wide
        const bool wide = live && P.off[v + 1] - P.off[v] > kWideRow;
        const int32_t at = wave_place(&ic[I_NWIDE], wide);
        if (wide) P.wl[at] = v;
        live = live && !wide;
      }
    }
    if (live) sw = rule<D>(P, v, odd != 0, &to, &stop);
    const int32_t p = wave_place(&ic[I_NDEC], sw);
    if (sw) dec[p] = make_int2(v, to);
  }
  if (stop) atomicOr(&ic[I_STOP], 1);
}

// The rule for the candidates with wide rows, a block to each (the blocks of
// k_inc_decide would hold some of them in a row).
constexpr int kWideThreads = 1024, kWideBlocks = 512;
__global__ __launch_bounds__(kWideThreads) void k_inc_wide(IncP P, int odd,
                                                           int2 *dec,
                                                           int32_t *ic) {
  __shared__ WideLds<kWideThreads> W;
  // (one look for the block: a climb that outlasts its bound raises it)
  if (__syncthreads_or(threadIdx.x == 0 && ld_relaxed(&ic[I_STOP]))) return;
  const int32_t n = ic[I_NWIDE];
  bool stop = false;
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t v = P.wl[i];
    const int2 me = P.sp[v];
    int32_t to = 0;
    if (me.y != kTopMark &&
        coarse_wide<kWideThreads>(coarse(P), v, me.x, odd != 0, &to, &stop,
                                  W) &&
        threadIdx.x == 0)
      dec[atomicAdd(&ic[I_NDEC], 1)] = make_int2(v, to);
  }
  if (stop) atomicOr(&ic[I_STOP], 1);
}

// The Even vertices with an option among the vertices changed since the
// last All_Even (list[0..nd)).
__global__ __launch_bounds__(kBlock) void k_inc_even_cand(IncP P,
                                                          int32_t epoch,
                                                          int32_t nd,
                                                          int32_t *ic) {
  __shared__ uint2 hub[kBlock];
  __shared__ int32_t s_n;
  for (int32_t i0 = blockIdx.x * blockDim.x; i0 < nd;
       i0 += gridDim.x * blockDim.x) {
    const int32_t i = i0 + threadIdx.x;
    uint32_t e = 0, e1 = 0;
    if (i < nd) {
      const int32_t w = P.list[i];
      e = P.in_off[w];
      e1 = P.in_off[w + 1];
    }
    auto take = [&](uint32_t e, uint32_t e1) {
      const uint32_t x = e < e1 ? P.in[e] : 0x80000000u;
      const bool c =
          e < e1 && !(x >> 31) && atomicExch(&P.cmark[x], epoch) != epoch;
      const int32_t p = wave_place(&ic[I_NC], c);
      if (c) P.cl[p] = (int32_t)x;
    };
    if (P.hub) {   // a hub's by the whole block
      __syncthreads();
      if (threadIdx.x == 0) s_n = 0;
      __syncthreads();
      if (e1 - e > kHub) {
        hub[atomicAdd(&s_n, 1)] = make_uint2(e, e1);
        e1 = e;
      }
      __syncthreads();
      const int n = s_n;
      for (int k = 0; k < n; ++k)
        for (uint32_t q = hub[k].x + threadIdx.x; __ballot(q < hub[k].y);
             q += kBlock)
          take(q, hub[k].y);
    }
    for (; __ballot(e < e1); ++e) take(e, e1);
  }
}

// All_Even over every Even vertex; decisions only.
constexpr int even_block(int D) { return D >= 16 ? 256 : 1024; }
template <int D, bool W>
__global__ __launch_bounds__(even_block(D)) void k_inc_even_all(
    IncP P, int64_t count, const int32_t *__restrict__ ids, int2 *dec,
    int32_t *ic) {
  __shared__ int32_t n, base;
  if (threadIdx.x == 0) n = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool sw = false, stop = false, live = t < count;
  int32_t v = 0, to = 0;
  if (live) v = ids[t];
  if constexpr (W) {
    __shared__ WideLds<even_block(D)> wl;
    if (inc_wide(P, live, v, false, wl, &sw, &to, &stop)) live = false;
  }
  if (live) sw = rule<D, W>(P, v, false, &to, &stop);
  const int32_t at = wave_place(&n, sw);
  __syncthreads();
  if (threadIdx.x == 0 && n) base = atomicAdd(&ic[I_NDEC], n);
  __syncthreads();
  if (sw) dec[base + at] = make_int2(v, to);
  if (stop) atomicOr(&ic[I_STOP], 1);
}

// All_Odd for the vertices a coarse valuation left open: switched in place
// and listed, like the others' switches.
template <bool W>
__global__ __launch_bounds__(kBlock) void k_tie_decide(IncP P, int32_t *ctr,
                                                       int2 *dec) {
  if (ctr[C_ABORT]) return;
  const int32_t n = ctr[C_NTIE];
  for (int32_t i0 = blockIdx.x * blockDim.x; i0 < n;
       i0 += gridDim.x * blockDim.x) {
    const int32_t i = i0 + threadIdx.x;
    bool sw = false, stop = false, live = i < n;
    int32_t v = 0, to = 0;
    if (live) v = P.cl[i];
    if constexpr (W) {
      __shared__ WideLds<kBlock> wl;
      if (inc_wide(P, live, v, true, wl, &sw, &to, &stop)) live = false;
    }
    if (live) sw = inc_decide<W>(P, v, true, &to, &stop);
    if (sw) P.sp[v] = make_int2(to, P.pri[to]);
    // (the walks bound every chain: no climb stops)
    if (stop) atomicOr(&ctr[C_ERR], ERR_LISTWALK);
    list_block(&ctr[C_NDEC], dec, sw, v, to);
  }
}

// Stores `check` when a vertex's choice is no edge of its row (a strategy
// given at the C ABI may name any vertex): the find follows in-edges only.
// Bound by one read of the rows, before the run's first full valuation
// (300,000 vertices: 6 us); rows beyond kWideRow entries are read by the
// whole block, or a hub's would keep one thread.
__global__ __launch_bounds__(kBlock) void k_inc_rows_hold(IncP P,
                                                          int32_t check,
                                                          int32_t *word,
                                                          int32_t *host) {
  __shared__ int32_t wide[kBlock], s_n;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool off = false;
  const int32_t to = v < P.N ? P.sp[v].x : P.N;
  if (to != P.N) {
    const int64_t e0 = P.off[v], e1 = P.off[v + 1];
    if (e1 - e0 > kWideRow) {
      wide[atomicAdd(&s_n, 1)] = (int32_t)v;
    } else {
      off = true;
      for (int64_t e = e0; e < e1 && off; e += 4) {
        int32_t t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = e + j < e1 ? P.tgt[e + j] : -1;
#pragma unroll
        for (int j = 0; j < 4; ++j) off = off && t[j] != to;
      }
    }
  }
  __syncthreads();
  const int n = s_n;
  for (int k = 0; k < n; ++k) {
    const int32_t w = wide[k], cur = P.sp[w].x;
    bool hit = false;
    for (int64_t e = P.off[w] + threadIdx.x, e1 = P.off[w + 1]; e < e1;
         e += kBlock)
      hit |= P.tgt[e] == cur;
    off |= !__syncthreads_or(hit);
  }
  if (__ballot(off) && (threadIdx.x & (kWave - 1)) == 0 &&
      ld_relaxed(word) != check && atomicExch(word, check) != check)
    *host = check;
}

// Applies decisions before a full valuation or an export.
__global__ __launch_bounds__(kBlock) void k_inc_commit(
    const int2 *__restrict__ dec, int32_t n, const int32_t *__restrict__ pri,
    int32_t N, int2 *sp) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int2 d = dec[i];
  sp[d.x] = make_int2(d.y, d.y == N ? 2147483647 : pri[d.y]);
}

// ---------------------------------------------------------------------------
// the block form
// ---------------------------------------------------------------------------
// One block runs valuations and switch steps until nothing switches, a cap
// is reached, or a step outgrows it.  Every dependent access costs a
// round trip to the L2, so its steps are bound by the length of their
// chains (the depth of A, the ng chains), not by their size.
constexpr int32_t kBlockA = 4096;  // most vertices of its A (LDS)
constexpr int kBlockEven = 8192;   // most changed vertices of its All_Even
constexpr int kBlockWide = 8192;   // most entries of wide rows among 1,024
                                   // candidates: one CU reads them in some
                                   // 10 us, the device form the rest
constexpr int kBlockHubs = 256;    // most hubs of one of its levels
constexpr int kBlockIn = 32768;    // and most in-edges of those: 1,024 a round
                                   // trip, as long as a small device step
enum IncState : int {
  IS_GROWN = 0,    // the pending decisions need the device form (or full)
  IS_BR = 1,       // best response reached; All_Even is the host's
  IS_SOLVED = 2,   // All_Even switched nothing: the run is over
  IS_CAP = 3,      // an iteration cap: decisions pending
};

struct IncRun {
  int32_t epoch, a0, nsw, cur;   // pending decisions: dec[cur], nsw of them
  int32_t a_cap;                 // most vertices of one step's A
  int32_t val_cap;               // most valuations of this launch
  int32_t inner_cap, inner;      // valuations of this best response (0: none)
  int32_t major_cap, major;      // outer iterations (0: none)
  int32_t d_valid;               // list[0..a0) holds every change since the
                                 // last All_Even
  int32_t with_even;             // run All_Even and go on
};

// (wide count rows: fewer threads, so that the rows stay in registers)
constexpr int inc_threads(int D) { return D >= 16 ? 512 : 1024; }
template <int D, bool S>   // S: for games with hubs or wide rows
__global__ __launch_bounds__(inc_threads(D)) void k_inc_block(IncP P, IncRun R,
                                                              int2 *dec0,
                                                              int2 *dec1,
                                                              int32_t *ic) {
  constexpr int T = inc_threads(D);
  __shared__ int32_t la[kBlockA];   // A
  __shared__ uint2 lr[kBlockA];     // its in-edge ranges
  __shared__ int32_t s_na, s_nc, s_nd, s_stop, s_open, s_err;
  __shared__ WideLds<D == 0 && S ? T : kWave> wl;
  __shared__ int32_t lh[kBlockHubs], s_nh, s_hd;   // a level's hubs
  const int tid = threadIdx.x;
  int32_t nval = 0, oddsw = 0, evensw = 0, state = IS_GROWN;
  if (tid == 0) {
    ic[I_CLOCK] = clock32();
    s_err = 0;
  }
  for (;;) {
    if (nval >= R.val_cap) break;
    const int2 *din = R.cur ? dec1 : dec0;
    int2 *dout = R.cur ? dec0 : dec1;
    if (R.nsw > R.a_cap || R.a0 + R.a_cap > P.list_cap) break;
    const int32_t epoch = R.epoch++;
    if (tid == 0) {
      s_na = R.nsw;
      s_nc = 0;
      s_nd = 0;
      s_stop = 0;
    }
    for (int32_t i = tid; i < R.nsw; i += T) {
      const int2 d = din[i];
      inc_apply(P, epoch, d);
      la[i] = d.x;
      lr[i] = make_uint2(P.in_off[d.x], P.in_off[d.x + 1]);
    }
    __syncthreads();
    // find, level by level: a level is a stretch of the list
    int32_t beg = 0, end = R.nsw;
    while (beg < end) {
      const int L = find_lanes(end - beg, T);
      auto place = [&](bool a, bool c, int32_t u, uint2 range) {
        const int32_t pc = wave_place(&s_nc, c);
        if (c && pc < P.cl_cap) P.cl[pc] = u;
        const int32_t pa = wave_place(&s_na, a);
        if (a && pa < R.a_cap) {
          la[pa] = u;
          lr[pa] = range;
        }
      };
      int hubs = 0;
      if (S && P.hub) {
        if (tid == 0) s_nh = s_hd = 0;
        __syncthreads();
        for (int32_t i = beg + tid; i < end; i += T) {
          const uint32_t d = lr[i].y - lr[i].x;
          if (d <= kHub) continue;
          const int k = atomicAdd(&s_nh, 1);
          if (k < kBlockHubs) lh[k] = i;
          // (saturates: 4,096 of 2,048 at most)
          if (d > (uint32_t)kIncMaxDegree ||
              atomicAdd(&s_hd, (int)d) + (int)d > kBlockIn ||
              k >= kBlockHubs)
            s_stop = 1;
        }
        __syncthreads();
        hubs = s_stop ? 0 : s_nh;
      }
      for (int32_t i0 = beg; i0 < end; i0 += T / L) {
        const int32_t i = i0 + tid / L;
        uint32_t e = 0, e1 = 0;
        int32_t w = -1;
        if (i < end && (!S || lr[i].y - lr[i].x <= kHub)) {
          w = la[i];
          e = lr[i].x + tid % L;
          e1 = lr[i].y;
        }
        for (; __ballot(e < e1); e += L) {
          const bool live = e < e1;
          const uint32_t x = live ? P.in[e] : 0u;
          uint2 range;
          const bool a = inc_edge(P, epoch, w, x, live, L, &range);
          place(a, live && (x >> 31), (int32_t)(x & 0x7fffffffu), range);
        }
      }
      for (int k = 0; S && k < hubs; ++k) {
        const int32_t w = la[lh[k]];
        const uint32_t e1 = lr[lh[k]].y;
        for (uint32_t e = lr[lh[k]].x + tid; __ballot(e < e1); e += T) {
          const bool live = e < e1;
          const uint32_t x = live ? P.in[e] : 0u;
          uint2 range;
          const bool a = inc_hub_edge(P, epoch, w, x, live, &range);
          place(a, live && (x >> 31), (int32_t)(x & 0x7fffffffu), range);
        }
      }
      __syncthreads();
      beg = end;
      end = s_na;
      if (end > R.a_cap || s_nc > P.cl_cap || s_stop) break;
      __syncthreads();
    }
    // (every thread leaves the loop with the same beg and end)
    if (end > R.a_cap || s_nc > P.cl_cap || s_stop) break;
    const int32_t na = end;
    for (int32_t i = tid; i < na; i += T) P.list[R.a0 + i] = la[i];
    // walks: passes until none is open
    bool failed = true;
    for (int pass = 0; pass < (D == 0 ? 8 : 2); ++pass) {
      if (tid == 0) s_open = 0;
      __syncthreads();
      for (int32_t i = tid; i < na; i += T) {
        const int32_t v = la[i];
        if constexpr (D == 0) {
          if (ld_relaxed(&P.ng[v]) >= 0) continue;
          if (!inc_walk(P, &s_err, v, 64)) s_open = 1;
        } else {
          if (pass > 0 && P.rs[v]) continue;
          if (!inc_row<D>(P, epoch, &s_err, v, pass ? 1024 : 64)) {
            P.rs[v] = 0;
            s_open = 1;
          }
        }
      }
      __syncthreads();
      const bool open = s_open != 0;
      __syncthreads();
      if (!open) {
        failed = false;
        break;
      }
    }
    if (failed) break;
    if constexpr (D == 0)
      for (int32_t i = tid; i < na; i += T)
        if (!inc_fate(P, epoch, la[i])) s_stop = 1;
    __syncthreads();
    const int32_t nc = s_nc;
    const bool bad = s_stop || s_err;
    __syncthreads();   // the next phase writes s_stop
    if (bad) break;
    for (int32_t i0 = 0; i0 < nc; i0 += T) {
      const int32_t i = i0 + tid;
      bool sw = false, stop = false, live = false;
      int32_t v = 0, to = 0;
      if (i < nc) {
        v = P.cl[i];
        live = atomicExch(&P.cmark[v], epoch) != epoch;
      }
      if constexpr (D == 0 && S)
        if (P.wide &&
            inc_wide(P, live, v, true, wl, &sw, &to, &stop, kBlockWide))
          live = false;
      if (live) sw = rule<D, S>(P, v, true, &to, &stop);
      if (stop) s_stop = 1;
      const int32_t p = wave_place(&s_nd, sw);
      if (sw) dout[p] = make_int2(v, to);
    }
    __syncthreads();
    if (s_stop) break;
    // the valuation and its All_Odd step are done
    const int32_t nd = s_nd;
    __syncthreads();
    ++nval;
    ++R.inner;
    R.a0 += na;
    oddsw += nd;
    R.nsw = nd;
    R.cur ^= 1;
    if (nd > 0) {
      if (R.inner_cap > 0 && R.inner >= R.inner_cap) {
        state = IS_CAP;
        break;
      }
      continue;
    }
    // a best response
    state = IS_BR;
    if (!R.with_even || !R.d_valid || R.a0 > kBlockEven) break;
    const int32_t ep2 = R.epoch++;
    int2 *eout = R.cur ? dec1 : dec0;
    if (tid == 0) {
      s_nc = 0;
      s_nd = 0;
    }
    __syncthreads();
    for (int32_t i0 = 0; i0 < R.a0; i0 += T) {
      const int32_t i = i0 + tid;
      uint32_t e = 0, e1 = 0;
      if (i < R.a0) {
        const int32_t w = P.list[i];
        e = P.in_off[w];
        e1 = P.in_off[w + 1];
        if (S && e1 - e > kHub) {   // the device's All_Even shares them out
          s_stop = 1;
          e1 = e;
        }
      }
      for (; __ballot(e < e1); ++e) {
        const uint32_t x = e < e1 ? P.in[e] : 0x80000000u;
        const bool c =
            e < e1 && !(x >> 31) && atomicExch(&P.cmark[x], ep2) != ep2;
        const int32_t p = wave_place(&s_nc, c);
        if (c) P.cl[p] = (int32_t)x;
      }
    }
    __syncthreads();
    if (s_stop) break;   // (the host's All_Even starts over)
    const int32_t ne = s_nc;
    for (int32_t i0 = 0; i0 < ne; i0 += T) {
      const int32_t i = i0 + tid;
      bool sw = false, stop = false, live = i < ne;
      int32_t v = 0, to = 0;
      if (live) v = P.cl[i];
      if constexpr (D == 0 && S)
        if (P.wide &&
            inc_wide(P, live, v, false, wl, &sw, &to, &stop, kBlockWide))
          live = false;
      if (live) sw = rule<D, S>(P, v, false, &to, &stop);
      if (stop) s_stop = 1;
      const int32_t p = wave_place(&s_nd, sw);
      if (sw) eout[p] = make_int2(v, to);
    }
    __syncthreads();
    if (s_stop) break;   // the host's All_Even (it starts over)
    const int32_t sw = s_nd;
    __syncthreads();
    evensw += sw;
    R.nsw = sw;
    R.a0 = 0;
    if (sw == 0) {
      state = IS_SOLVED;
      break;
    }
    if (R.major_cap > 0 && R.major >= R.major_cap) {
      state = IS_CAP;
      R.inner = 0;
      break;
    }
    ++R.major;
    R.inner = 0;
    state = IS_GROWN;
  }
  __syncthreads();
  if (tid == 0) {
    ic[I_ERR] = s_err;
    ic[I_STATE] = state;
    ic[I_NVAL] = nval;
    ic[I_ODDSW] = oddsw;
    ic[I_EVENSW] = evensw;
    ic[I_MAJOR] = R.major;
    ic[I_INNER] = R.inner;
    ic[I_A0] = R.a0;
    ic[I_CUR] = R.cur;
    ic[I_NDEC] = R.nsw;
    ic[I_EPOCH] = R.epoch;
    ic[I_CLOCK_END] = clock32();
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// A step starts when at most one vertex in kIncSwitchShare switched, in the
// block form up to kBlockSwitches of them.  A is two to six times the
// switched vertices on the workloads, and its find follows plays of up to
// hundreds of vertices, level by level, where a full valuation with coarse
// keys takes 0.06 ms (40,000 vertices) to 0.8 ms (10M): one in 100 against
// one in 24 made solves 3-6 % faster, with the Odd region 20 %; one in 150
// and one in 400 were 2 % slower than that on some and faster on others.
// Full count valuations cost four times as much.
constexpr int64_t kIncSwitchShare = 100, kIncSwitchShareCounts = 24;
constexpr int32_t kBlockSwitches = 512;
constexpr int32_t kBlockVals = 64;

static IncP inc_params(const pg_game *g) {
  const int32_t N = (int32_t)g->n_aug;
  IncP P;
  P.N = N;
  P.n_oddpri = g->n_oddpri;
  P.off = g->off;
  P.tgt = g->tgt;
  P.pri = g->pri;
  P.in_off = g->inc.in_off;
  P.in = g->inc.in;
  P.sp = g->sp;
  P.key = g->key;
  P.ng = g->ng;
  P.cand = g->cand;
  P.rs = g->rs;
  P.cnt = g->dense ? g->cnt : nullptr;
  P.pidx = g->pidx;
  P.odd_cols = g->odd_cols;
  P.mark = g->inc.mark;
  P.cmark = g->inc.cmark;
  // the Euler list's records (4 N ints) and the parent sort's keys (N)
  // are free between full valuations
  P.list = reinterpret_cast<int32_t *>(g->aux);
  P.list_cap = 2 * N;
  P.cl = P.list + 2 * (int64_t)N;
  P.cl_cap = 2 * N;
  P.q = reinterpret_cast<int32_t *>(g->sk0);
  P.q_cap = N / kFindChunk;
  P.wide = g->wide;
  P.wl = g->rcand;   // (between full valuations)
  P.hub = g->inc.h && g->inc.h[I_WORDS + 1];
  return P;
}

// The decision lists live in the Euler list's elements (2 N pairs); the
// full valuation's All_Odd lists its switches in the first.
static int2 *inc_dec(const pg_game *g, int i) { return g->elem + i * g->n_aug; }

bool inc_eligible(const pg_game *g) {
  return (g->dense || g->relabeled) && !g->careful && !g->host_rl &&
         g->n_aug >= 2 && g->m_aug < (int64_t(1) << 31) &&
         (g->tsw || g->n_odd <= kIncRowOdd);
}

// The in-edge lists of a run's game (x.in_off and x.in).
static void in_lists(pg_game *g, hipStream_t s) {
  pg_game::Inc &x = g->inc;
  const int64_t N = g->n_aug, M = g->m_aug;
  if (N >= kInPartMin && N <= kInPartMax) {
    // about a thousand ranges; the parts are small enough that their counts
    // (one per range and part) are no more than the vertices
    int shift = 10;
    while ((N >> shift) >= 1024 && (1 << shift) < kInRangeMax) ++shift;
    const int nr = (int)((N + (1 << shift) - 1) >> shift);
    const int vb = N >= (int64_t(1) << 25)   ? 16384
                   : N >= (int64_t(1) << 22) ? 4096
                                             : 1024;
    const int nb = (int)((N + vb - 1) / vb);
    uint2 *pairs = nullptr;
    if (dev_alloc(&pairs, M) == PG_OK) {
      x.pairs = pairs;   // freed once the stream has been waited for
      uint32_t *hist = reinterpret_cast<uint32_t *>(g->aux);
      uint32_t *at = hist + (int64_t)nr * nb;
      hipLaunchKernelGGL(k_in_hist, dim3(nb), dim3(kInPartThreads), 0, s,
                         g->off, g->tgt, (int32_t)N, vb, shift, nr, hist);
      scan_excl_u32(hist, at, (int64_t)nr * nb, g->scan_tmp, s);
      hipLaunchKernelGGL(k_in_part, dim3(nb), dim3(kInPartThreads), 0, s,
                         g->off, g->tgt, g->owner, (int32_t)N, vb, shift, nr,
                         at, pairs);
      hipLaunchKernelGGL(k_in_range, dim3(nr), dim3(kInPartThreads),
                         sizeof(uint32_t) << shift, s, pairs, at, nb,
                         (uint32_t)M, (int32_t)N, shift, x.in_off, x.in,
                         x.ic + I_HUB);
      fill_i32((int32_t *)x.in_off + N, (int32_t)M, 1, s);
      return;
    }
    pg_fail(PG_OK, "");
  }
  fill_i32((int32_t *)x.in_off, 0, N, s);
  hipLaunchKernelGGL(k_in_count, dim3(grid_for(M)), dim3(kBlock), 0, s,
                     g->tgt, x.in_off, M);
  scan_excl_u32(x.in_off, x.in_off, N, g->scan_tmp, s);
  fill_i32((int32_t *)x.in_off + N, (int32_t)M, 1, s);
  uint32_t *cursor = reinterpret_cast<uint32_t *>(g->elem);
  hipLaunchKernelGGL(k_in_cursors, dim3(grid_for(N)), dim3(kBlock), 0, s,
                     x.in_off, cursor, N, x.ic + I_HUB);
  hipLaunchKernelGGL(k_in_fill, dim3(grid_for(N)), dim3(kBlock), 0, s,
                     g->off, g->tgt, g->owner, cursor, x.in, (int32_t)N);
}

// Builds the in-edge lists at the first solve of a game.  Without memory
// for them the game keeps full valuations.
bool inc_prepare(pg_game *g, hipStream_t s) {
  pg_game::Inc &x = g->inc;
  x.dirty = x.pending = x.d_valid = x.grown = x.even = x.exact = false;
  x.queue = x.offrow = false;
  x.nsw = x.a0 = 0;
  x.skip = x.back = x.ranks = x.ranks_back = 0;
  x.on = false;
  if (x.state < 0 || !inc_eligible(g)) return false;
  const int64_t N = g->n_aug, M = g->m_aug;
  if (x.state == 0) {
    pg_status st = dev_alloc(&x.in_off, N + 1);
    if (st == PG_OK) st = dev_alloc(&x.in, M);
    if (st == PG_OK) st = dev_alloc(&x.mark, N);
    if (st == PG_OK) st = dev_alloc(&x.cmark, N);
    if (st == PG_OK) st = dev_alloc(&x.ic, I_SIZE);
    if (st == PG_OK)
      st = host_alloc((void **)&x.h, sizeof(int32_t) * (I_WORDS + 2));
    if (st != PG_OK) {
      inc_release(g);
      x.state = -1;
      pg_fail(PG_OK, "");
      return false;
    }
    fill_i32(x.ic, 0, I_SIZE, s);
    in_lists(g, s);
    publish(x.h + I_WORDS + 1, x.ic + I_HUB, 1, s);
    fill_i32(x.mark, 0, N, s);
    fill_i32(x.cmark, 0, N, s);
    x.epoch = x.check = 0;
    x.state = 1;
  } else if (x.epoch >= kEpochMax) {
    fill_i32(x.mark, 0, N, s);
    fill_i32(x.cmark, 0, N, s);
    x.epoch = 0;
  }
  x.on = true;
  return true;
}

void inc_end(pg_game *g, hipStream_t s) {
  pg_game::Inc &x = g->inc;
  if (!x.pairs) return;
  (void)hipStreamSynchronize(s);
  dev_free(x.pairs);
  x.pairs = nullptr;
}

void inc_release(pg_game *g) {
  pg_game::Inc &x = g->inc;
  void *ptrs[] = {x.in_off, x.in, x.mark, x.cmark, x.ic, x.pairs};
  for (void *p : ptrs) dev_free(p);
  host_free(x.h);
  // a run that goes on without the lists keeps its counts
  const int32_t inner = x.inner, major = x.major;
  x = pg_game::Inc();
  x.inner = inner;
  x.major = major;
}

// direct: the kernel wrote its results to the host's words itself
static pg_status inc_read(pg_game *g, hipStream_t s, bool direct = false) {
  if (!direct) publish(g->inc.h, g->inc.ic, I_WORDS, s, I_CLOCK_END);
  PG_HIP(hipStreamSynchronize(s));
  if (g->prof.on) g->prof.flush();
  if (g->inc.h[I_ERR] & ERR_INADMISSIBLE)
    return pg_fail(PG_EINADMISSIBLE,
                   "the play graph has a cycle whose largest priority is odd");
  return PG_OK;
}

// Puts the pending decisions into the play graph.
void inc_commit(pg_game *g, hipStream_t s) {
  pg_game::Inc &x = g->inc;
  if (!x.on || !x.pending) return;
  x.pending = false;
  if (x.nsw > 0)
    PG_LAUNCH(&g->prof, K_OTHER, 24.0 * x.nsw, k_inc_commit,
              dim3(grid_for(x.nsw)), dim3(kBlock), 0, s, inc_dec(g, x.cur),
              x.nsw, g->pri, (int32_t)g->n_aug, g->sp);
}

// Looks whether every choice is an edge of its row; the answer is there after
// the stream's next synchronisation.
void inc_check_rows(pg_game *g, hipStream_t s) {
  pg_game::Inc &x = g->inc;
  if (!x.on) return;
  x.offrow = true;
  ++x.check;
  x.h[I_WORDS] = 0;
  const bool direct = host_pinned(x.h);
  PG_LAUNCH(&g->prof, K_OTHER, 24.0 * g->n_aug + 4.0 * g->m_aug,
            k_inc_rows_hold, dim3(grid_for(g->n_aug)), dim3(kBlock), 0, s,
            inc_params(g), x.check, x.ic + I_OFFROW,
            direct ? x.h + I_WORDS : x.ic + I_OFFROW);
  if (!direct) publish(x.h + I_WORDS, x.ic + I_OFFROW, 1, s);
}

bool inc_ready(const pg_game *g) {
  const pg_game::Inc &x = g->inc;
  return x.on && x.pending && x.skip == 0 && !x.exact && !x.offrow &&
         ((int64_t)x.nsw * (g->dense ? kIncSwitchShareCounts
                                     : kIncSwitchShare) <= g->n_aug ||
          g->n_aug <= kBlockA);
}

// Coarse keys serve the rank games of a run until something outgrows them.
bool inc_coarse(const pg_game *g) {
  return g->inc.on && !g->dense && g->inc.ranks == 0;
}

int32_t *tie_list(const pg_game *g) {
  return inc_params(g).cl;
}

void enqueue_ties(pg_game *g, hipStream_t s) {
  PG_LAUNCH(&g->prof, K_INC_DECIDE, 0.0,
            g->wide ? k_tie_decide<true> : k_tie_decide<false>, dim3(1024),
            dim3(kBlock), 0, s, inc_params(g), g->ctr, inc_dec(g, 0));
}

// Before a full valuation of a run (an exact one finds every fate again
// unless the last one was exact too, in the same inner loop).
void inc_before_full(pg_game *g, hipStream_t s, bool coarse) {
  pg_game::Inc &x = g->inc;
  if (!x.on) return;
  inc_commit(g, s);
  if (!coarse) {
    if (x.dirty || x.even) fates_reset(g, s);
    if (x.ranks > 0) --x.ranks;
  }
  if (x.skip > 0) --x.skip;
  x.even = false;
}

void inc_after_full(pg_game *g, hipStream_t s, int32_t switches, bool exact) {
  pg_game::Inc &x = g->inc;
  if (!x.on) return;
  x.dirty = !exact;
  x.exact = exact && !g->dense;
  if (exact) x.queue = false;
  else x.ranks_back = 0;
  x.d_valid = false;
  x.a0 = 0;
  x.grown = false;
  x.pending = true;   // already in the play graph: applying them is harmless
  dev_free(x.pairs);
  x.pairs = nullptr;
  x.cur = 0;
  x.nsw = switches;
  if (x.offrow) {   // (of the check before this valuation)
    x.offrow = x.h[I_WORDS] == x.check;
    if (x.offrow) inc_check_rows(g, s);
  }
}

// A step that gave up: full valuations for a while, on coarse keys all the
// same (a hub's in-edges stop the find, not the walks).
static void inc_backoff(pg_game *g) {
  pg_game::Inc &x = g->inc;
  x.back = x.back ? std::min(2 * x.back, 16) : 1;
  x.skip = x.back;
}

// A coarse valuation whose chains are too long: ranks for a while.
void inc_use_ranks(pg_game *g) {
  pg_game::Inc &x = g->inc;
  x.ranks_back = x.ranks_back ? std::min(2 * x.ranks_back, 16) : 1;
  x.ranks = x.ranks_back;
}

// One step (device form) or a run of steps (block form) from the pending
// decisions.
template <int D>
static pg_status inc_step_t(pg_game *g, hipStream_t s, bool with_even,
                   int32_t max_inner, int32_t max_major, IncOut *out) {
  pg_game::Inc &x = g->inc;
  const IncP P = inc_params(g);
  Prof *pf = &g->prof;
  const int32_t N = P.N;
  if (x.a0 > N) {   // no room for another step: forget the older changes
    x.a0 = 0;
    x.d_valid = false;
  }
  x.dirty = true;
  const bool block =
      !x.grown && (x.nsw <= kBlockSwitches || N <= kBlockA);
  x.grown = false;
  *out = IncOut();
  out->state = INC_MORE;
  if (block) {
    IncRun R;
    R.epoch = x.epoch + 1;
    R.a0 = x.a0;
    R.nsw = x.nsw;
    R.cur = x.cur;
    R.a_cap = std::min(kBlockA, N);
    R.val_cap = kBlockVals;
    R.inner_cap = max_inner;
    R.inner = x.inner;
    R.major_cap = max_major;
    R.major = x.major;
    R.d_valid = x.d_valid;
    R.with_even = with_even;
    PG_LAUNCH(pf, K_INC_BLOCK, 0.0,
              (P.hub || (D == 0 && P.wide) ? k_inc_block<D, true>
                                           : k_inc_block<D, false>),
              dim3(1), dim3(inc_threads(D)), 0, s, P, R, inc_dec(g, 0),
              inc_dec(g, 1), host_pinned(x.h) ? x.h : x.ic);
  } else {
    const int32_t epoch = ++x.epoch;
    const unsigned gb =
        std::min<unsigned>(kIncBlocks, grid_for(4 * (int64_t)x.nsw));
    const dim3 grid(std::max(gb, 64u)), blk(kBlock);
    if (!x.queue) fill_i32(P.q, -1, N, s, pf);
    x.queue = true;
    fill_i32(x.ic, 0, I_ALL, s, pf);
    PG_LAUNCH(pf, K_INC_FIND, 0.0, k_inc_begin, dim3(grid_for(x.nsw)), blk, 0,
              s, P, epoch, x.a0, inc_dec(g, x.cur), x.nsw, x.ic);
    PG_LAUNCH(pf, K_INC_FIND, 0.0, P.hub ? k_inc_find<true> : k_inc_find<false>,
              dim3(kFindBlocks), blk, 0, s, P, epoch, x.a0, x.nsw, x.ic);
    if constexpr (D == 0) {
      PG_LAUNCH(pf, K_INC_WALK, 0.0, k_inc_walk, grid, blk, 0, s, P, x.a0, 64,
                0, 0, x.ic);
      PG_LAUNCH(pf, K_INC_WALK, 0.0, k_inc_walk, grid, blk, 0, s, P, x.a0,
                256, 1, 1, x.ic);
      PG_LAUNCH(pf, K_INC_WALK, 0.0, k_inc_fate, grid, blk, 0, s, P, epoch,
                x.a0, x.ic);
    } else {
      PG_LAUNCH(pf, K_INC_WALK, 0.0, k_inc_rows<D>, grid, blk, 0, s, P, epoch,
                x.a0, 64, 0, 0, x.ic);
      PG_LAUNCH(pf, K_INC_WALK, 0.0, k_inc_rows<D>, grid, blk, 0, s, P, epoch,
                x.a0, 1024, 1, 1, x.ic);
    }
    PG_LAUNCH(pf, K_INC_DECIDE, 0.0, k_inc_decide<D>, grid, blk, 0, s, P,
              epoch, 1, inc_dec(g, x.cur ^ 1), x.ic);
    if (D == 0 && P.wide)
      PG_LAUNCH(pf, K_INC_DECIDE, 0.0, k_inc_wide, dim3(kWideBlocks),
                dim3(kWideThreads), 0, s, P, 1, inc_dec(g, x.cur ^ 1), x.ic);
  }
  const pg_status st = inc_read(g, s, block && host_pinned(x.h));
  // a refused run's epochs are used all the same: its marks stay
  if (st != PG_OK && st != PG_EINADMISSIBLE) {
    x.epoch = kEpochMax;
    return st;
  }
  g->last_ms = clock_ms(g, x.h[I_CLOCK], x.h[I_CLOCK_END]);
  if (block) {
    x.epoch = x.h[I_EPOCH];
    x.a0 = x.h[I_A0];
    x.cur = x.h[I_CUR];
    x.nsw = x.h[I_NDEC];
    x.inner = x.h[I_INNER];
    x.major = x.h[I_MAJOR];
    out->nval = x.h[I_NVAL];
    out->odd = x.h[I_ODDSW];
    out->even = x.h[I_EVENSW];
    if (st != PG_OK) return st;   // (what it had done is reported)
    switch (x.h[I_STATE]) {
      case IS_BR: out->state = INC_BR; break;
      case IS_SOLVED: out->state = INC_SOLVED; break;
      case IS_CAP:
        if (x.inner == 0) out->state = INC_CAP;
        break;
      default:
        if (out->nval >= kBlockVals) break;
        // the pending step is too large for one block (or, in a game that
        // always fits one, beyond another bound)
        if (N > kBlockA) x.grown = true;
        else inc_backoff(g);
        break;
    }
  } else if (st != PG_OK) {
    return st;
  } else if (x.h[I_STOP]) {
    x.queue = false;
    inc_backoff(g);
  } else {
    x.back = 0;
    x.a0 += x.h[I_NA];
    x.cur ^= 1;
    x.nsw = x.h[I_NDEC];
    ++x.inner;
    out->nval = 1;
    out->odd = x.nsw;
    if (x.nsw == 0) out->state = INC_BR;
  }
  return PG_OK;
}

// All_Even after a best response; its switches are pending afterwards.
template <int D>
static pg_status inc_even_t(pg_game *g, hipStream_t s, int32_t *count) {
  pg_game::Inc &x = g->inc;
  const IncP P = inc_params(g);
  Prof *pf = &g->prof;
  const int64_t ne = g->n_aug - g->n_odd;
  x.h[I_STOP] = 1;
  if (x.d_valid && (int64_t)x.a0 * 8 <= g->n_aug) {
    fill_i32(x.ic, 0, I_WORDS, s, pf);
    const dim3 grid(std::max(
        std::min<unsigned>(kIncBlocks, grid_for(4 * (int64_t)x.a0)), 64u));
    PG_LAUNCH(pf, K_INC_FIND, 0.0, k_inc_even_cand, grid, dim3(kBlock), 0, s,
              P, ++x.epoch, x.a0, x.ic);
    PG_LAUNCH(pf, K_INC_DECIDE, 0.0, k_inc_decide<D>, grid, dim3(kBlock), 0, s,
              P, x.epoch, 0, inc_dec(g, 0), x.ic);
    if (D == 0 && P.wide)
      PG_LAUNCH(pf, K_INC_DECIDE, 0.0, k_inc_wide, dim3(kWideBlocks),
                dim3(kWideThreads), 0, s, P, 0, inc_dec(g, 0), x.ic);
    PG_TRY(inc_read(g, s));
  }
  for (int pass = 0; x.h[I_STOP]; ++pass) {
    if (pass > 0) {   // a comparison outgrew its bound: ranks instead
      PG_TRY(ranks_device(g, s));
      x.dirty = x.queue = false;
      x.exact = true;
    }
    fill_i32(x.ic, 0, I_WORDS, s, pf);
    if (ne > 0)
      PG_LAUNCH(pf, K_EVEN_SWITCH, 28.0 * ne + 8.0 * (g->m_aug - g->m_odd),
                (D == 0 && P.wide ? k_inc_even_all<D, D == 0>
                                  : k_inc_even_all<D, false>),
                dim3(grid_for(ne, even_block(D))),
                dim3(even_block(D)), 0, s, P, ne, g->even_ids, inc_dec(g, 0),
                x.ic);
    PG_TRY(inc_read(g, s));
  }
  x.pending = x.even = true;
  x.grown = false;
  x.cur = 0;
  x.nsw = *count = x.h[I_NDEC];
  x.a0 = 0;
  x.d_valid = true;
  return PG_OK;
}

// The row width of a count game, 0 for rank keys.
pg_status inc_step(pg_game *g, hipStream_t s, bool with_even,
                   int32_t max_inner, int32_t max_major, IncOut *out) {
  switch (g->dense ? g->dw : 0) {
    case 0: return inc_step_t<0>(g, s, with_even, max_inner, max_major, out);
    case 4: return inc_step_t<4>(g, s, with_even, max_inner, max_major, out);
    case 8: return inc_step_t<8>(g, s, with_even, max_inner, max_major, out);
    case 16: return inc_step_t<16>(g, s, with_even, max_inner, max_major, out);
    default: return inc_step_t<32>(g, s, with_even, max_inner, max_major, out);
  }
}

pg_status inc_even(pg_game *g, hipStream_t s, int32_t *count) {
  switch (g->dense ? g->dw : 0) {
    case 0: return inc_even_t<0>(g, s, count);
    case 4: return inc_even_t<4>(g, s, count);
    case 8: return inc_even_t<8>(g, s, count);
    case 16: return inc_even_t<16>(g, s, count);
    default: return inc_even_t<32>(g, s, count);
  }
}

}  // namespace pgk

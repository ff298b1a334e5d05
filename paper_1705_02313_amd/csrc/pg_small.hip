// Small games (rank valuations): whole runs and valuations in one block.
//
// A valuation of a small game is some forty kernels of 2-8 us each on a chip
// that the game cannot fill, and a step in global memory is a chain of round
// trips to the L2.  A game of up to kSmallN vertices fits one CU's LDS (ids
// in 16 bits), where a dependent access costs a tenth of that, so one block
// runs Algorithm 1 from the strategies in the play graph to the end: ng
// walks with jumps over resolved vertices, fates, and the switching rules
// with each comparison decided on the two ng chains (pg_inc.hip's order), so
// no valuation needs ranks.  A whole solve of the 1,000-vertex game's 26-34
// valuations takes one launch.
//
// A single valuation (pg_valuation) needs the ranks themselves: subtree
// sizes by LDS atomics along the ng chains, the vertices sorted by (parent,
// signed position) in LDS, prefix sums of the sizes, and each vertex's rank
// as the sum of its offsets along its chain.
//
// Bound by LDS round trips and barriers.  Against the general path (forty
// kernels a valuation, or pg_inc.hip's block in global memory): pg_valuation
// at 1,000 vertices 158 -> 61 us a call, the load of a 1,000-vertex game 500
// -> 69 us, its solve from arrays 1.62 -> 0.42 ms, 4,099 vertices 2.6 -> 0.87
// ms.  The line at kSmallN is what 150 KB of LDS hold with up to 40,000
// edges; above it one block also stops paying (several vertices per thread in
// every step).
//
// ng chains longer than kSmallDepth (none of the random or chain workloads
// comes near) are left to the general path, before anything was switched.
#include <algorithm>

#include "pg_common.h"

namespace pgk {

constexpr int kSmallThreads = 1024;
constexpr int kSmallDepth = 256;          // longest ng chain
constexpr int kSmallPasses = 4096;        // walk passes before giving up
constexpr size_t kSmallLds = 150 * 1024;  // dynamic LDS of a block at most
constexpr uint32_t kOpen = 0x8000u;       // ng entry: still walking, low bits
                                          // its candidate

// words of g->hctr (g->ctr when that is not pinned) a small kernel reports in
enum SmallCounter : int {
  S_STATE = 8, S_NVAL, S_ODDSW, S_EVENSW, S_MAJOR, S_INNER, S_NFIN,
  S_CLOCK, S_CLOCK_END, S_END
};
static_assert((int)S_END <= (int)C_DIST_SW, "the small kernels' words");
enum SmallState : int {
  SS_MORE = 0,    // the launch's valuation budget is spent: go on
  SS_BR, SS_SOLVED,
  SS_CAP,         // an iteration cap
  SS_DEEP         // left to the general path at the start of a valuation
};

// The game's LDS arrays.  Ids: the sink is N, top is N + 1.
struct Small {
  int32_t N, n_oddpri;
  // per vertex and for the sink: rank by priority (the larger, the greater)
  // in the high half, ng in the low half, so that a step costs one access
  uint32_t *rec;
  uint16_t *succ;   // the play graph
  // the last vertex of the ng chain before the sink (the sink's own: N), or
  // N + 1 for top: two vertices with different ones compare by them
  uint16_t *root;
};

__device__ __forceinline__ int32_t rec_ng(uint32_t r) {
  return (int32_t)(r & 0xffffu);
}

__device__ __forceinline__ size_t small_align(size_t b) {
  return (b + 15) & ~size_t(15);
}

__device__ __forceinline__ uint16_t *lds_u16(char *&p, int64_t n) {
  uint16_t *r = reinterpret_cast<uint16_t *>(p);
  p += (2 * n + 15) & ~int64_t(15);
  return r;
}

// Sums of one value per thread over the block, one barrier each: three slots
// in turn, each cleared two sums ahead (every thread has read it by then).
// The slots start at zero; every thread takes part in every sum.
struct BlockSum {
  int32_t *slot;
  int k = 0;
  __device__ __forceinline__ int32_t operator()(int32_t x) {
    if (x) atomicAdd(&slot[k], x);
    __syncthreads();
    const int32_t r = slot[k];
    const int clear = k == 0 ? 2 : k - 1;
    if (threadIdx.x == 0) slot[clear] = 0;
    k = k == 2 ? 0 : k + 1;
    return r;
  }
};

// mag from the signed order (odd priorities descending, then even ones
// ascending): the position among its own parity plus the smaller ones of the
// other, by bisection of the other part.
__device__ __forceinline__ void small_mag(const Small &S, const int32_t *pri) {
  for (int32_t v = threadIdx.x; v < S.N; v += kSmallThreads) {
    const int32_t p = pri[v];
    const bool odd = v < S.n_oddpri;
    // the other part: indices lo..hi, ascending from the front (even) or
    // from the back (odd)
    int32_t lo = 0, hi = odd ? S.N - S.n_oddpri : S.n_oddpri;
    while (lo < hi) {
      const int32_t m = (lo + hi) >> 1;
      const int32_t q = odd ? pri[S.n_oddpri + m] : pri[S.n_oddpri - 1 - m];
      if (q < p) lo = m + 1;
      else hi = m;
    }
    S.rec[v] =
        (uint32_t)(lo + (odd ? S.n_oddpri - 1 - v : v - S.n_oddpri)) << 16;
  }
  if (threadIdx.x == 0) {   // the sink is greater than everything
    S.rec[S.N] = 0xffff0000u | (uint32_t)S.N;
    S.root[S.N] = (uint16_t)S.N;
  }
}

// ng and root of every vertex (all threads; barriers inside).  *err: a cycle
// with odd largest priority.  False when the walks do not end or a chain is
// longer than kSmallDepth.
__device__ __forceinline__ bool small_walks(const Small &S, BlockSum &sum,
                                            int32_t *err) {
  const int tid = threadIdx.x;
  const int32_t N = S.N;
  for (int32_t v = tid; v < N; v += kSmallThreads)
    S.rec[v] = (S.rec[v] & 0xffff0000u) | kOpen | S.succ[v];
  __syncthreads();
  for (int pass = 0;; ++pass) {
    int open = 0;
    for (int32_t v = tid; v < N; v += kSmallThreads) {
      const uint32_t mine = S.rec[v];
      if (!(mine & kOpen)) continue;
      int32_t u = (int32_t)(mine & (kOpen - 1u));
      int32_t res = -1;
      for (int s = 0; s < 64; ++s) {
        if (u >= N) {
          res = u;
          break;
        }
        if (u == v) {
          // the largest vertex of its cycle, whose priority must be even
          // for an admissible sigma (section 3)
          if (v < S.n_oddpri) *err = 1;
          res = N + 1;
          break;
        }
        const uint32_t r = *(volatile uint32_t *)&S.rec[u];
        if (r > mine) {   // (priority ranks differ: the low halves never
          res = u;        // decide)
          break;
        }
        // a resolved u's ng, or an open u's candidate: everything before it
        // is below u
        u = (int32_t)(r & (kOpen - 1u));
      }
      S.rec[v] = (mine & 0xffff0000u) |
                 (res >= 0 ? (uint32_t)res : kOpen | (uint32_t)u);
      open |= res < 0;
    }
    if (!sum(open)) break;
    if (pass >= kSmallPasses) return false;
  }
  int deep = 0;
  for (int32_t v = tid; v < N; v += kSmallThreads) {
    int32_t a = v, r = rec_ng(S.rec[v]);
    for (int s = 0; r < N && s < kSmallDepth; ++s) {
      a = r;
      r = rec_ng(S.rec[r]);
    }
    deep |= r < N;
    S.root[v] = (uint16_t)(r == N ? a : N + 1);
  }
  return !sum(deep);
}

// 1, 0 or -1: Val(x) above, equal to or below Val(y) (as
// coarse_climb of pg_coarse.h); rx and ry are their roots.
__device__ __forceinline__ int small_cmp(const Small &S, int32_t x, int32_t rx,
                                         int32_t y, int32_t ry) {
  const int32_t N = S.N;
  if (rx != ry) {
    // the sink lies above the odd and below the even ones of its children,
    // and everything below top
    if (rx == N) return ry >= S.n_oddpri ? -1 : 1;
    if (ry == N) return rx >= S.n_oddpri ? 1 : -1;
    return rx > ry ? 1 : -1;
  }
  if (x == y || rx >= N) return 0;
  int32_t a = x, b = y, ca = -1, cb = -1;
  uint32_t ra = S.rec[a], rb = S.rec[b];
  while (a != b) {
    if (ra < rb) {
      ca = a;
      a = rec_ng(ra);
      ra = S.rec[a];
    } else {
      cb = b;
      b = rec_ng(rb);
      rb = S.rec[b];
    }
  }
  if (ca < 0) return cb >= S.n_oddpri ? -1 : 1;
  if (cb < 0) return ca >= S.n_oddpri ? 1 : -1;
  return ca > cb ? 1 : -1;
}

struct SmallGame {
  int32_t N, n_oddpri, n_odd, M;
  const int64_t *off;
  const int32_t *tgt, *pri, *odd_ids, *even_ids;
  int2 *sp;
  uint8_t *rs;
  int32_t *ctr;
};

struct SmallRun {
  int32_t inner_cap, inner, major_cap, major;   // as pg_inc.hip's IncRun
  int32_t br_only, reset, val_cap;
};

// Algorithm 1 from the strategies in sp.
__global__ __launch_bounds__(kSmallThreads) void k_small_run(SmallGame G,
                                                             SmallRun R) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int32_t s_err, s_sum[3];
  const int tid = threadIdx.x;
  if (tid == 0) G.ctr[S_CLOCK] = clock32();
  const int32_t N = G.N;
  char *p = lds;
  Small S;
  S.N = N;
  S.n_oddpri = G.n_oddpri;
  S.rec = reinterpret_cast<uint32_t *>(p);
  p += small_align(4 * (size_t)(N + 1));
  S.succ = lds_u16(p, N);
  S.root = lds_u16(p, N + 1);
  uint16_t *ids = lds_u16(p, N);        // the Odd vertices, then the Even
  uint16_t *row = lds_u16(p, N + 1);    // row starts
  uint16_t *tgt = lds_u16(p, G.M);
  small_mag(S, G.pri);
  for (int32_t v = tid; v < N; v += kSmallThreads) {
    S.succ[v] = (uint16_t)G.sp[v].x;
    ids[v] = (uint16_t)(v < G.n_odd ? G.odd_ids[v] : G.even_ids[v - G.n_odd]);
  }
  for (int32_t v = tid; v <= N; v += kSmallThreads)
    row[v] = (uint16_t)G.off[v];
  for (int32_t e = tid; e < G.M; e += kSmallThreads)
    tgt[e] = (uint16_t)G.tgt[e];
  if (tid == 0) s_err = s_sum[0] = s_sum[1] = s_sum[2] = 0;
  BlockSum sum{s_sum};
  __syncthreads();
  // the switching rule of one player for every vertex of it; the number of
  // switches is returned.  The rule reads the ng chains and each vertex its
  // own choice: the new choices are written at once.
  auto all_switch = [&](bool odd) {
    const int32_t from = odd ? 0 : G.n_odd, to = odd ? G.n_odd : N;
    int32_t sw = 0;
    for (int32_t i = from + tid; i < to; i += kSmallThreads) {
      const int32_t v = ids[i];
      const int32_t cur = S.succ[v];
      int32_t best = odd ? -1 : N, rb = N;
      for (int32_t e = row[v], e1 = row[v + 1]; e < e1; ++e) {
        const int32_t u = tgt[e], ru = S.root[u];
        if (best >= 0) {
          const int c = small_cmp(S, u, ru, best, rb);
          if (odd ? c >= 0 : c <= 0) continue;
        }
        best = u;
        rb = ru;
      }
      const int c = best == cur ? 0 : small_cmp(S, best, rb, cur, S.root[cur]);
      if (odd ? c < 0 : c > 0) {
        S.succ[v] = (uint16_t)best;
        ++sw;
      }
    }
    return sum(sw);
  };
  int32_t nval = 0, oddsw = 0, evensw = 0, state = SS_MORE;
  while (nval < R.val_cap) {
    if (!small_walks(S, sum, &s_err)) {
      state = SS_DEEP;
      break;
    }
    if (s_err) break;
    const int32_t c = all_switch(true);
    ++nval;
    ++R.inner;
    oddsw += c;
    if (c > 0) {
      if (R.inner_cap > 0 && R.inner >= R.inner_cap) {
        state = SS_CAP;
        break;
      }
      continue;
    }
    state = SS_BR;
    if (R.br_only) break;
    const int32_t ce = all_switch(false);
    evensw += ce;
    if (ce == 0) {
      state = SS_SOLVED;
      break;
    }
    R.inner = 0;
    if (R.major_cap > 0 && R.major >= R.major_cap) {
      state = SS_CAP;
      break;
    }
    ++R.major;
    state = SS_MORE;
    if (R.reset) {   // SI-Reset: Odd back to the first entry of each row
      for (int32_t i = tid; i < G.n_odd; i += kSmallThreads)
        S.succ[ids[i]] = tgt[row[ids[i]]];
      __syncthreads();
    }
  }
  __syncthreads();
  for (int32_t v = tid; v < N; v += kSmallThreads) {
    const int32_t u = S.succ[v];
    G.sp[v] = make_int2(u, u == N ? 2147483647 : G.pri[u]);
    G.rs[v] = S.root[v] == N + 1 ? 2 : 1;
  }
  if (tid == 0) {
    G.ctr[C_ERR] = s_err ? ERR_INADMISSIBLE : 0;
    G.ctr[S_STATE] = state;
    G.ctr[S_NVAL] = nval;
    G.ctr[S_ODDSW] = oddsw;
    G.ctr[S_EVENSW] = evensw;
    G.ctr[S_MAJOR] = R.major;
    G.ctr[S_INNER] = R.inner;
    G.ctr[S_CLOCK_END] = clock32();
  }
}

// ---------------------------------------------------------------------------
// one valuation with ranks
// ---------------------------------------------------------------------------
struct SmallValue {
  // the caller's ids; null sigma: the play graph's own choices
  const int32_t *sigma, *tau;
  const uint8_t *owner;
  const int32_t *perm, *rvpos;
  int32_t *key;                 // [N+1], the caller's ids
  int32_t sort_n;               // power of two >= N
};

__global__ __launch_bounds__(kSmallThreads) void k_small_value(SmallGame G,
                                                               SmallValue V) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int32_t s_err, s_bad, s_sum[3];
  __shared__ uint32_t s_part[kSmallThreads / kWave];
  const int tid = threadIdx.x;
  const int32_t N = G.N;
  char *p = lds;
  Small S;
  S.N = N;
  S.n_oddpri = G.n_oddpri;
  S.rec = reinterpret_cast<uint32_t *>(p);
  p += small_align(4 * (size_t)(N + 1));
  S.succ = lds_u16(p, N);
  S.root = lds_u16(p, N + 1);
  uint16_t *off = lds_u16(p, N);         // offset within the parent's children
  uint16_t *first = lds_u16(p, N + 1);   // sizes before a node's children
  uint16_t *mid = lds_u16(p, N + 1);     // and before its even ones
  uint32_t *size = reinterpret_cast<uint32_t *>(p);
  p += small_align(4 * (size_t)N);
  uint32_t *srt = reinterpret_cast<uint32_t *>(p);
  if (tid == 0) s_err = s_bad = s_sum[0] = s_sum[1] = s_sum[2] = 0;
  BlockSum sum{s_sum};
  __syncthreads();
  small_mag(S, G.pri);
  for (int32_t i = tid; i < N; i += kSmallThreads) {
    const bool even = V.owner[i] == 0;
    const int32_t v = V.perm[i];
    int32_t s = !V.sigma ? G.sp[i].x : even ? V.sigma[v] : V.tau[v];
    if (!V.sigma) {
      // stored ids already
    } else if (even && s == PG_SINK) {
      s = N;
    } else if (s < 0 || s >= N) {
      s_bad = 1;
      s = N;
    } else {
      s = V.rvpos[s];
    }
    S.succ[i] = (uint16_t)s;
    size[i] = 1;
  }
  __syncthreads();
  const bool done = small_walks(S, sum, &s_err);
  const bool ok = done && !s_err && !s_bad;
  if (ok) {
    // subtree sizes
    for (int32_t v = tid; v < N; v += kSmallThreads)
      if (S.root[v] < N)
        for (int32_t a = rec_ng(S.rec[v]); a < N; a = rec_ng(S.rec[a]))
          atomicAdd(&size[a], 1u);
    // finite vertices by (parent, signed position)
    const uint32_t none = 0xffffffffu;
    for (int32_t v = tid; v < V.sort_n; v += kSmallThreads)
      srt[v] = v < N && S.root[v] < N ? (S.rec[v] << 16) | (uint32_t)v : none;
    __syncthreads();
    for (int32_t k = 2; k <= V.sort_n; k <<= 1)
      for (int32_t j = k >> 1; j > 0; j >>= 1) {
        for (int32_t t = tid; t < V.sort_n / 2; t += kSmallThreads) {
          const int32_t i = 2 * t - (t & (j - 1));   // bit j clear
          const uint32_t a = srt[i], b = srt[i + j];
          if ((a > b) == ((i & k) == 0)) {
            srt[i] = b;
            srt[i + j] = a;
          }
        }
        __syncthreads();
      }
    // sizes before each position, a stretch per thread
    const int32_t per = (V.sort_n + kSmallThreads - 1) / kSmallThreads;
    const int32_t i0 = tid * per;
    uint32_t sum = 0;
    for (int32_t i = i0; i < i0 + per && i < V.sort_n; ++i)
      if (srt[i] != none) sum += size[srt[i] & 0xffffu];
    const int lane = tid & (kWave - 1);
    uint32_t inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) s_part[tid / kWave] = inc;
    __syncthreads();
    uint32_t before = inc - sum;
    for (int w = 0; w < tid / kWave; ++w) before += s_part[w];
    for (int32_t i = i0; i < i0 + per && i < V.sort_n; ++i) {
      const uint32_t x = srt[i];
      if (x == none) break;
      const int32_t v = (int32_t)(x & 0xffffu), par = (int32_t)(x >> 16);
      const bool ev = v >= G.n_oddpri;
      const uint32_t px = i > 0 ? srt[i - 1] : none;
      const bool start = i == 0 || (int32_t)(px >> 16) != par;
      if (start) first[par] = (uint16_t)before;
      // the first even child, or the end when there is none
      if (ev && (start || (int32_t)(px & 0xffffu) < G.n_oddpri))
        mid[par] = (uint16_t)before;
      off[v] = (uint16_t)before;
      before += size[v];
      const uint32_t nx = i + 1 < V.sort_n ? srt[i + 1] : none;
      if (!ev && (nx == none || (int32_t)(nx >> 16) != par))
        mid[par] = (uint16_t)before;
    }
    __syncthreads();
  }
  // ranks: a vertex comes after its odd children, its even ones after it
  int32_t nfin = 0;
  for (int32_t v = tid; v <= N; v += kSmallThreads) {
    int32_t k = PG_KEY_TOP;
    if (ok && S.root[v] <= N) {
      ++nfin;
      // (the sink has children when any vertex is finite)
      const bool inner = v < N ? size[v] > 1 : srt[0] != 0xffffffffu;
      k = inner ? (int32_t)mid[v] - (int32_t)first[v] : 0;
      for (int32_t a = v; a < N;) {
        const int32_t q = rec_ng(S.rec[a]);
        k += (int32_t)off[a] - (int32_t)first[q] + (a >= G.n_oddpri ? 1 : 0);
        a = q;
      }
    }
    if (ok) V.key[v == N ? N : V.perm[v]] = k;
  }
  nfin = sum(nfin);
  if (tid == 0) {
    G.ctr[C_ERR] = (s_bad ? ERR_INVAL : 0) | (s_err ? ERR_INADMISSIBLE : 0);
    G.ctr[S_STATE] = !done ? SS_DEEP : SS_SOLVED;
    G.ctr[S_NFIN] = nfin;
  }
}

// ---------------------------------------------------------------------------
// loading
// ---------------------------------------------------------------------------
// pg_load_csr of a game of up to kSmallN vertices in one launch: validation,
// the signed-priority sort, X and its dummies (section 3), the modified game
// in signed order, the players' lists and the initial play graph, which the
// general path does in some seventy kernels and nine synchronisations.  A
// malformed game or repeated priorities are only reported: the general path
// then loads or refuses the game.
struct SmallLoad {
  int32_t n, m;
  const int64_t *off64;   // one of the two
  const int32_t *off32;
  const int32_t *tgt, *pri;
  const uint8_t *owner;
  int32_t preprocess;
  int32_t sort_n;         // power of two >= n
  // out (room for 2 n vertices)
  int64_t *off2;
  int32_t *tgt2, *pri2, *perm, *rvpos, *odd_ids, *even_ids;
  uint8_t *owner2;
  int2 *sp;
  int32_t *ctr;
};
// the words it reports in
enum LoadCounter : int {
  L_STATE = 8, L_NAUG, L_NODDPRI, L_NODD, L_MODD, L_WIDE, L_END
};
static_assert((int)L_END <= (int)C_DIST_SW, "the load kernel's words");

// Exclusive sum over the block of one value per thread (all threads);
// *total: the whole sum.
__device__ __forceinline__ int32_t block_excl(int32_t x, int32_t *part,
                                              int32_t *total) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  int32_t inc = x;
  for (int o = 1; o < kWave; o <<= 1) {
    const int32_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  __syncthreads();
  if (lane == kWave - 1) part[tid / kWave] = inc;
  __syncthreads();
  int32_t before = inc - x, all = 0;
  for (int w = 0; w < kSmallThreads / kWave; ++w) {
    if (w < tid / kWave) before += part[w];
    all += part[w];
  }
  *total = all;
  return before;
}

__global__ __launch_bounds__(kSmallThreads) void k_small_load(SmallLoad L) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int32_t part[kSmallThreads / kWave], s_sum[3], s_wide;
  const int tid = threadIdx.x;
  const int32_t n = L.n, m = L.m;
  if (tid < 3) s_sum[tid] = 0;
  if (tid == 0) s_wide = 0;
  __syncthreads();
  BlockSum sum{s_sum};
  char *p = lds;
  uint16_t *at = lds_u16(p, n);     // each vertex's stored position
  uint16_t *did = lds_u16(p, n);    // the dummy's number of a member of X'
  uint8_t *inx = reinterpret_cast<uint8_t *>(p);
  p += small_align((size_t)n);
  uint8_t *xp = reinterpret_cast<uint8_t *>(p);
  p += small_align((size_t)n);
  unsigned long long *srt = reinterpret_cast<unsigned long long *>(p);
  auto row = [&](int32_t v) -> int64_t {
    return L.off64 ? L.off64[v] : (int64_t)L.off32[v];
  };
  // validation
  int bad = 0;
  for (int32_t v = tid; v < n; v += kSmallThreads) {
    const int64_t a = row(v), b = row(v + 1);
    bad |= b <= a || b > m || a < 0 || (v == 0 && a != 0) ||
           (v == n - 1 && b != m) || L.owner[v] > 1 || L.pri[v] < 0;
    if (b - a > kWideRow) s_wide = 1;
    inx[v] = L.owner[v] == 1;
    xp[v] = 0;
  }
  for (int32_t e = tid; e < m; e += kSmallThreads)
    bad |= L.tgt[e] < 0 || L.tgt[e] >= n;
  if (sum(bad)) {
    if (tid == 0) L.ctr[L_STATE] = 0;
    return;
  }
  // signed-priority order of the original vertices (odd priorities
  // descending, then even ascending); the dummies' places follow from it
  for (int32_t i = tid; i < L.sort_n; i += kSmallThreads) {
    unsigned long long k = ~0ull;
    if (i < n) {
      const uint32_t q = (uint32_t)L.pri[i];
      k = ((unsigned long long)((q & 1u) ? 0x7fffffffu - q : 0x80000000u + q)
           << 16) | (unsigned long long)i;
    }
    srt[i] = k;
  }
  __syncthreads();
  for (int32_t k = 2; k <= L.sort_n; k <<= 1)
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      for (int32_t t = tid; t < L.sort_n / 2; t += kSmallThreads) {
        const int32_t i = 2 * t - (t & (j - 1));
        const unsigned long long a = srt[i], b = srt[i + j];
        if ((a > b) == ((i & k) == 0)) {
          srt[i] = b;
          srt[i + j] = a;
        }
      }
      __syncthreads();
    }
  int dup = 0, nodd = 0;
  for (int32_t i = tid; i < n; i += kSmallThreads) {
    dup |= i > 0 && (srt[i] >> 16) == (srt[i - 1] >> 16);
    nodd += (srt[i] >> 16) < 0x80000000ull;
  }
  if (sum(dup)) {
    if (tid == 0) L.ctr[L_STATE] = 0;
    return;
  }
  int32_t no = 0, nxp = 0;
  (void)block_excl(nodd, part, &no);
  if (L.preprocess) {
    // X: members without a successor in X leave until nobody does (in
    // place: any order ends at the same set).  A row is read on from the
    // entry last seen in X (X only shrinks); did holds the places meanwhile.
    for (int32_t v = tid; v < n; v += kSmallThreads) did[v] = 0;
    for (;;) {
      int drop = 0;
      for (int32_t v = tid; v < n; v += kSmallThreads) {
        if (!inx[v]) continue;
        bool any = false;
        const int64_t e0 = row(v), e1 = row(v + 1);
        int64_t e = e0 + did[v];
        for (; e < e1; ++e)
          if (*(volatile uint8_t *)&inx[L.tgt[e]]) {
            any = true;
            break;
          }
        if (any) did[v] = (uint16_t)(e - e0);   // (rows: below 65,536 entries)
        if (!any) {
          inx[v] = 0;
          drop = 1;
        }
      }
      if (!sum(drop)) break;
    }
    // X': members with a predecessor in X, numbered in increasing id
    for (int32_t v = tid; v < n; v += kSmallThreads)
      if (inx[v])
        for (int64_t e = row(v), e1 = row(v + 1); e < e1; ++e)
          if (inx[L.tgt[e]]) xp[L.tgt[e]] = 1;
    __syncthreads();
    const int32_t per = (n + kSmallThreads - 1) / kSmallThreads;
    const int32_t v0 = min(tid * per, n), v1 = min(v0 + per, n);
    int32_t c = 0;
    for (int32_t v = v0; v < v1; ++v) c += xp[v];
    int32_t k = block_excl(c, part, &nxp);
    for (int32_t v = v0; v < v1; ++v)
      if (xp[v]) did[v] = (uint16_t)k++;
    __syncthreads();
  }
  const int32_t N = n + nxp, K = nxp + (nxp & 1);
  // dummy i has priority i, below every original one: the odd ones
  // (descending) end the odd part, the even ones begin the even part
  auto dummy = [&](int32_t i) -> int32_t {
    return (i & 1) ? no + nxp / 2 - 1 - i / 2 : no + nxp / 2 + i / 2;
  };
  int over = 0;
  for (int32_t i = tid; i < n; i += kSmallThreads) {
    const int32_t v = (int32_t)(srt[i] & 0xffffull);
    const int32_t q = i < no ? i : i + nxp;
    at[v] = (uint16_t)q;
    L.perm[q] = v;
    L.rvpos[v] = q;
    L.owner2[q] = L.owner[v];
    over |= (int64_t)L.pri[v] + K > 2147483647LL;
    L.pri2[q] = L.pri[v] + K;
    if (L.preprocess && xp[v]) {
      const int32_t d = did[v], qd = dummy(d);
      L.perm[qd] = n + d;
      L.rvpos[n + d] = qd;
      L.owner2[qd] = 0;
      L.pri2[qd] = d;
    }
  }
  if (sum(over)) {
    if (tid == 0) L.ctr[L_STATE] = 0;
    return;
  }
  // row lengths, starts and the players' lists, a stretch of stored
  // vertices per thread
  const int32_t per = (N + kSmallThreads - 1) / kSmallThreads;
  const int32_t q0 = min(tid * per, N), q1 = min(q0 + per, N);
  int32_t len = 0, odd = 0, modd = 0;
  for (int32_t q = q0; q < q1; ++q) {
    const int32_t v = L.perm[q];
    const int32_t l = v < n ? (int32_t)(row(v + 1) - row(v)) : 1;
    len += l;
    if (L.owner2[q]) {
      ++odd;
      modd += l;
    }
  }
  int32_t M, n_odd, m_odd;
  int32_t e = block_excl(len, part, &M);
  int32_t o = block_excl(odd, part, &n_odd);
  (void)block_excl(modd, part, &m_odd);
  for (int32_t q = q0; q < q1; ++q) {
    const int32_t v = L.perm[q];
    L.off2[q] = e;
    const bool isodd = L.owner2[q] != 0;
    if (isodd) L.odd_ids[o++] = q;
    else L.even_ids[q - o] = q;
    e += v < n ? (int32_t)(row(v + 1) - row(v)) : 1;
  }
  if (tid == 0) {
    L.off2[N] = M;
    L.sp[N] = make_int2(N, 2147483647);
  }
  __syncthreads();
  // the rows: an edge inside X goes through its target's dummy
  for (int32_t v = tid; v < n; v += kSmallThreads) {
    const bool vx = L.preprocess && inx[v];
    const int32_t q = at[v];
    int64_t w = L.off2[q];
    const int64_t e0 = row(v), e1 = row(v + 1);
    int32_t t0 = 0;
    for (int64_t x = e0; x < e1; ++x) {
      const int32_t t = L.tgt[x];
      const int32_t u = vx && inx[t] ? dummy(did[t]) : at[t];
      if (x == e0) t0 = u;
      L.tgt2[w++] = u;
    }
    // sigma_init and the first entry of the row
    if (L.owner[v]) L.sp[q] = make_int2(t0, L.pri2[t0]);
    else L.sp[q] = make_int2(N, 2147483647);
    if (L.preprocess && xp[v]) {
      const int32_t qd = dummy(did[v]);
      L.tgt2[L.off2[qd]] = q;
      L.sp[qd] = make_int2(N, 2147483647);
    }
  }
  if (tid == 0) {
    L.ctr[L_STATE] = 1;
    L.ctr[L_NAUG] = N;
    L.ctr[L_NODDPRI] = no + nxp / 2;
    L.ctr[L_NODD] = n_odd;
    L.ctr[L_MODD] = m_odd;
    L.ctr[L_WIDE] = s_wide;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int32_t sort_size(int64_t N) {
  int32_t n = 2;
  while (n < N) n <<= 1;
  return n;
}
static size_t run_lds(int64_t N, int64_t M) {
  auto a = [](size_t b) { return (b + 15) & ~size_t(15); };
  return a(4 * (N + 1)) + 2 * a(2 * N) + 2 * a(2 * (N + 1)) + a(2 * M);
}
static size_t value_lds(int64_t N) {
  auto a = [](size_t b) { return (b + 15) & ~size_t(15); };
  return a(4 * (N + 1)) + 2 * a(2 * N) + 3 * a(2 * (N + 1)) + a(4 * N) +
         4 * (size_t)sort_size(N);
}

bool small_fits(int64_t N, int64_t M) {
  return N >= 1 && N <= kSmallN && M < 65536 && run_lds(N, M) <= kSmallLds &&
         value_lds(N) <= kSmallLds;
}

// More LDS than a kernel may use by default, once per device.
static pg_status small_ready(int device) {
  static std::mutex mu;
  static std::map<int, bool> ready;
  std::lock_guard<std::mutex> lock(mu);
  bool &r = ready[device];
  if (!r) {
    PG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_small_run),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kSmallLds));
    PG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_small_value),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kSmallLds));
    PG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_small_load),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kSmallLds));
    r = true;
  }
  return PG_OK;
}

static SmallGame small_game(const pg_game *g) {
  SmallGame G;
  G.N = (int32_t)g->n_aug;
  G.n_oddpri = g->n_oddpri;
  G.n_odd = (int32_t)g->n_odd;
  G.M = (int32_t)g->m_aug;
  G.off = g->off;
  G.tgt = g->tgt;
  G.pri = g->pri;
  G.odd_ids = g->odd_ids;
  G.even_ids = g->even_ids;
  G.sp = g->sp;
  G.rs = g->rs;
  G.ctr = host_pinned(g->hctr) ? g->hctr : g->ctr;
  return G;
}

static pg_status small_read(pg_game *g, hipStream_t s) {
  if (!host_pinned(g->hctr)) publish(g->hctr, g->ctr, S_END, s);
  PG_HIP(hipStreamSynchronize(s));
  if (g->prof.on) g->prof.flush();
  if (g->hctr[C_ERR] & ERR_INVAL)
    return pg_fail(PG_EINVAL,
                   "a strategy entry is out of range (Even: a vertex id or "
                   "PG_SINK, Odd: a vertex id)");
  if (g->hctr[C_ERR] & ERR_INADMISSIBLE)
    return pg_fail(PG_EINADMISSIBLE,
                   "the play graph has a cycle whose largest priority is odd");
  return PG_OK;
}

// Vertices and edges that small_load takes (the LDS of its sort).
bool small_load_fits(int64_t n, int64_t m) {
  return n >= 1 && n <= kSmallN && m < 65536;
}

pg_status small_load(pg_game *g, int64_t n, int64_t m, const void *offsets,
                     const int32_t *targets, const uint8_t *owner,
                     const int32_t *priority, uint32_t flags, hipStream_t s,
                     bool *done) {
  *done = false;
  PG_TRY(small_ready(g->device));
  const int64_t cap = (flags & PG_NO_PREPROCESS) ? n : 2 * n;
  PG_TRY(dev_alloc(&g->off, cap + 1));
  PG_TRY(dev_alloc(&g->tgt, m + cap - n));
  PG_TRY(dev_alloc(&g->owner, cap));
  PG_TRY(dev_alloc(&g->pri, cap));
  PG_TRY(alloc_state(g, cap));
  SmallLoad L;
  L.n = (int32_t)n;
  L.m = (int32_t)m;
  L.off32 = (flags & PG_OFFSETS_I32) ? (const int32_t *)offsets : nullptr;
  L.off64 = (flags & PG_OFFSETS_I32) ? nullptr : (const int64_t *)offsets;
  L.tgt = targets;
  L.pri = priority;
  L.owner = owner;
  L.preprocess = !(flags & PG_NO_PREPROCESS);
  L.sort_n = sort_size(n);
  L.off2 = g->off;
  L.tgt2 = g->tgt;
  L.pri2 = g->pri;
  L.perm = g->perm;
  L.rvpos = g->rvpos;
  L.odd_ids = g->odd_ids;
  L.even_ids = g->even_ids;
  L.owner2 = g->owner;
  L.sp = g->sp;
  L.ctr = host_pinned(g->hctr) ? g->hctr : g->ctr;
  auto a = [](size_t b) { return (b + 15) & ~size_t(15); };
  // (the launch's own status: the thread's last error may be another call's)
  void *args[] = {&L};
  PG_HIP(hipLaunchKernel(reinterpret_cast<const void *>(k_small_load), dim3(1),
                         dim3(kSmallThreads), args,
                         2 * a(2 * n) + 2 * a(n) + 8 * (size_t)L.sort_n, s));
  if (!host_pinned(g->hctr)) publish(g->hctr, g->ctr, L_END, s);
  PG_HIP(hipStreamSynchronize(s));
  if (!g->hctr[L_STATE]) return PG_OK;
  *done = true;
  g->n_aug = g->hctr[L_NAUG];
  g->m_aug = m + g->n_aug - n;
  g->n_oddpri = g->hctr[L_NODDPRI];
  g->n_odd = g->hctr[L_NODD];
  g->m_odd = g->hctr[L_MODD];
  g->wide = g->hctr[L_WIDE];
  g->sort_bits = 1;
  while ((int64_t(1) << g->sort_bits) <= g->n_aug + 1) ++g->sort_bits;
  g->relabeled = true;
  return PG_OK;
}

pg_status small_step(pg_game *g, hipStream_t s, bool br_only, bool reset,
                     int32_t max_inner, int32_t max_major, bool *deep,
                     IncOut *out) {
  PG_TRY(small_ready(g->device));
  SmallRun R;
  R.inner_cap = max_inner;
  R.inner = g->inc.inner;
  R.major_cap = max_major;
  R.major = g->inc.major;
  R.br_only = br_only;
  R.reset = reset;
  R.val_cap = 512;
  PG_LAUNCH(&g->prof, K_SMALL, 0.0, k_small_run, dim3(1), dim3(kSmallThreads),
            run_lds(g->n_aug, g->m_aug), s, small_game(g), R);
  *out = IncOut();
  *deep = false;
  const pg_status st = small_read(g, s);
  if (st != PG_OK && st != PG_EINADMISSIBLE) return st;
  // (a refused run reports what it had done, too)
  g->last_ms = clock_ms(g, g->hctr[S_CLOCK], g->hctr[S_CLOCK_END]);
  out->nval = g->hctr[S_NVAL];
  out->odd = g->hctr[S_ODDSW];
  out->even = g->hctr[S_EVENSW];
  g->inc.inner = g->hctr[S_INNER];
  g->inc.major = g->hctr[S_MAJOR];
  if (st != PG_OK) return st;
  switch (g->hctr[S_STATE]) {
    case SS_BR: out->state = INC_BR; break;
    case SS_SOLVED: out->state = INC_SOLVED; break;
    case SS_CAP:
      if (g->inc.inner == 0) out->state = INC_CAP;
      break;
    case SS_DEEP: *deep = true; break;
    default: break;
  }
  return PG_OK;
}

bool small_due(pg_game *g) {
  if (!g->small) return false;
  if (g->small_skip == 0) return true;
  --g->small_skip;
  return false;
}

pg_status small_valuation(pg_game *g, const int32_t *sigma, const int32_t *tau,
                          int32_t *key, hipStream_t s, bool *deep,
                          int64_t *n_finite) {
  PG_TRY(small_ready(g->device));
  SmallValue V;
  V.sigma = sigma;
  V.tau = tau;
  V.owner = g->owner;
  V.perm = g->perm;
  V.rvpos = g->rvpos;
  V.key = key;
  V.sort_n = sort_size(g->n_aug);
  PG_LAUNCH(&g->prof, K_SMALL, 0.0, k_small_value, dim3(1),
            dim3(kSmallThreads), value_lds(g->n_aug), s, small_game(g), V);
  PG_TRY(small_read(g, s));
  *deep = g->hctr[S_STATE] == SS_DEEP;
  g->small_back = !*deep ? 0
                  : g->small_back ? std::min(2 * g->small_back, 16)
                                  : 1;
  g->small_skip = g->small_back;
  if (n_finite) *n_finite = g->hctr[S_NFIN];
  return PG_OK;
}

}  // namespace pgk

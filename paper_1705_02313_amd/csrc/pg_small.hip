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
// at 1,000 vertices 158 -> 61 us a call, a 1,000-vertex solve from arrays
// 1.62 -> 1.08 ms (most of it the load), 4,099 vertices 2.6 -> 1.94 ms.  The
// line at kSmallN is what 150 KB of LDS hold with up to 40,000 edges; above
// it one block also stops paying (several vertices per thread in every step).
//
// ng chains longer than kSmallDepth (none of the random or chain workloads
// comes near) are left to the general path, before anything was switched.
#include "pg_common.h"

namespace pgk {

constexpr int kSmallThreads = 1024;
constexpr int kSmallDepth = 256;          // longest ng chain
constexpr int kSmallPasses = 4096;        // walk passes before giving up
constexpr size_t kSmallLds = 150 * 1024;  // dynamic LDS of a block at most
constexpr uint32_t kOpen = 0x8000u;       // ng entry: still walking, low bits
                                          // its candidate

// words of g->ctr a small kernel reports in (below C_DIST_SW)
enum SmallCounter : int {
  S_STATE = 8, S_NVAL, S_ODDSW, S_EVENSW, S_MAJOR, S_INNER, S_NFIN, S_END
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
  uint16_t *mag;    // rank by priority (the larger, the greater)
  uint16_t *succ;   // the play graph
  uint16_t *ng;
  uint8_t *fate;    // 1 finite, 2 top
};

__device__ __forceinline__ uint16_t *lds_u16(char *&p, int64_t n) {
  uint16_t *r = reinterpret_cast<uint16_t *>(p);
  p += (2 * n + 15) & ~int64_t(15);
  return r;
}

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
    S.mag[v] = (uint16_t)(lo + (odd ? S.n_oddpri - 1 - v : v - S.n_oddpri));
  }
}

// ng of every vertex (all threads; barriers inside).  *err: a cycle with odd
// largest priority.  False when the walks do not end.
__device__ __forceinline__ bool small_walks(const Small &S, int32_t *open,
                                            int32_t *err) {
  const int tid = threadIdx.x;
  const int32_t N = S.N;
  for (int32_t v = tid; v < N; v += kSmallThreads)
    S.ng[v] = (uint16_t)(kOpen | S.succ[v]);
  for (int pass = 0; pass < kSmallPasses; ++pass) {
    if (tid == 0) *open = 0;
    __syncthreads();
    for (int32_t v = tid; v < N; v += kSmallThreads) {
      const uint32_t mine = S.ng[v];
      if (!(mine & kOpen)) continue;
      int32_t u = (int32_t)(mine & ~kOpen);
      const uint32_t mv = S.mag[v];
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
        if (S.mag[u] > mv) {
          res = u;
          break;
        }
        // a resolved u's ng, or an open u's candidate: everything before it
        // is below u
        u = (int32_t)(*(volatile uint16_t *)&S.ng[u] & ~kOpen);
      }
      S.ng[v] = (uint16_t)(res >= 0 ? (uint32_t)res : kOpen | (uint32_t)u);
      if (res < 0) *open = 1;
    }
    __syncthreads();
    const bool more = *open != 0;
    __syncthreads();
    if (!more) return true;
  }
  return false;
}

// Fates; *deep when a chain is longer than kSmallDepth.
__device__ __forceinline__ void small_fates(const Small &S, int32_t *deep) {
  const int32_t N = S.N;
  for (int32_t v = threadIdx.x; v < N; v += kSmallThreads) {
    int32_t r = S.ng[v];
    int s = 0;
    for (; r < N && s < kSmallDepth; ++s) r = S.ng[r];
    if (r < N) *deep = 1;
    S.fate[v] = r == N ? 1 : 2;
  }
}

// 1, 0 or -1: Val(x) above, equal to or below Val(y) (pg_inc.hip, inc_climb)
__device__ __forceinline__ int small_cmp(const Small &S, int32_t x,
                                         int32_t y) {
  const int32_t N = S.N;
  if (x == y) return 0;
  const int fx = x == N ? 1 : S.fate[x], fy = y == N ? 1 : S.fate[y];
  if (fx != fy) return fx > fy ? 1 : -1;
  if (fx == 2) return 0;
  int32_t a = x, b = y, ca = -1, cb = -1;
  int32_t ma = a == N ? 0x10000 : S.mag[a], mb = b == N ? 0x10000 : S.mag[b];
  while (a != b) {
    if (ma < mb) {
      ca = a;
      a = S.ng[a];
      ma = a == N ? 0x10000 : S.mag[a];
    } else {
      cb = b;
      b = S.ng[b];
      mb = b == N ? 0x10000 : S.mag[b];
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

__device__ __forceinline__ size_t small_align(size_t b) {
  return (b + 15) & ~size_t(15);
}

// Algorithm 1 from the strategies in sp.
__global__ __launch_bounds__(kSmallThreads) void k_small_run(SmallGame G,
                                                             SmallRun R) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int32_t s_open, s_err, s_deep, s_sw;
  const int tid = threadIdx.x;
  const int32_t N = G.N;
  char *p = lds;
  Small S;
  S.N = N;
  S.n_oddpri = G.n_oddpri;
  S.mag = lds_u16(p, N);
  S.succ = lds_u16(p, N);
  S.ng = lds_u16(p, N);
  uint16_t *ids = lds_u16(p, N);        // the Odd vertices, then the Even
  uint16_t *row = lds_u16(p, N + 1);    // row starts
  uint16_t *tgt = lds_u16(p, G.M);
  S.fate = reinterpret_cast<uint8_t *>(p);
  small_mag(S, G.pri);
  for (int32_t v = tid; v < N; v += kSmallThreads) {
    S.succ[v] = (uint16_t)G.sp[v].x;
    ids[v] = (uint16_t)(v < G.n_odd ? G.odd_ids[v] : G.even_ids[v - G.n_odd]);
  }
  for (int32_t v = tid; v <= N; v += kSmallThreads)
    row[v] = (uint16_t)G.off[v];
  for (int32_t e = tid; e < G.M; e += kSmallThreads)
    tgt[e] = (uint16_t)G.tgt[e];
  if (tid == 0) s_err = s_deep = s_sw = 0;
  __syncthreads();
  // the switching rule of one player for every vertex of it; the number of
  // switches comes out in s_sw.  The rule reads the fates and ng chains and
  // each vertex its own choice: the new choices are written at once.
  auto all_switch = [&](bool odd) {
    const int32_t from = odd ? 0 : G.n_odd, to = odd ? G.n_odd : N;
    for (int32_t i = from + tid; i < to; i += kSmallThreads) {
      const int32_t v = ids[i];
      const int32_t cur = S.succ[v];
      int32_t best = odd ? -1 : N;
      for (int32_t e = row[v], e1 = row[v + 1]; e < e1; ++e) {
        const int32_t u = tgt[e];
        if (best >= 0) {
          const int c = small_cmp(S, u, best);
          if (odd ? c >= 0 : c <= 0) continue;
        }
        best = u;
      }
      const int c = best == cur ? 0 : small_cmp(S, best, cur);
      if (odd ? c < 0 : c > 0) {
        S.succ[v] = (uint16_t)best;
        atomicAdd(&s_sw, 1);
      }
    }
    __syncthreads();
    const int32_t n = s_sw;
    __syncthreads();
    if (tid == 0) s_sw = 0;
    return n;
  };
  int32_t nval = 0, oddsw = 0, evensw = 0, state = SS_MORE;
  while (nval < R.val_cap) {
    const bool done = small_walks(S, &s_open, &s_err);
    small_fates(S, &s_deep);
    __syncthreads();
    if (!done || s_deep) {
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
    G.rs[v] = S.fate[v];
  }
  if (tid == 0) {
    G.ctr[C_ERR] = s_err ? ERR_INADMISSIBLE : 0;
    G.ctr[S_STATE] = state;
    G.ctr[S_NVAL] = nval;
    G.ctr[S_ODDSW] = oddsw;
    G.ctr[S_EVENSW] = evensw;
    G.ctr[S_MAJOR] = R.major;
    G.ctr[S_INNER] = R.inner;
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
  __shared__ int32_t s_open, s_err, s_deep, s_bad;
  __shared__ uint32_t s_part[kSmallThreads / kWave];
  const int tid = threadIdx.x;
  const int32_t N = G.N;
  char *p = lds;
  Small S;
  S.N = N;
  S.n_oddpri = G.n_oddpri;
  S.mag = lds_u16(p, N);
  S.succ = lds_u16(p, N);
  S.ng = lds_u16(p, N);
  uint16_t *off = lds_u16(p, N);         // offset within the parent's children
  uint16_t *first = lds_u16(p, N + 1);   // sizes before a node's children
  uint16_t *mid = lds_u16(p, N + 1);     // and before its even ones
  uint32_t *size = reinterpret_cast<uint32_t *>(p);
  p += small_align(4 * (size_t)N);
  uint32_t *srt = reinterpret_cast<uint32_t *>(p);
  p += 4 * (size_t)V.sort_n;
  S.fate = reinterpret_cast<uint8_t *>(p);
  if (tid == 0) s_err = s_deep = s_bad = 0;
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
  const bool done = small_walks(S, &s_open, &s_err);
  small_fates(S, &s_deep);
  __syncthreads();
  const bool ok = done && !s_deep && !s_err && !s_bad;
  if (ok) {
    // subtree sizes
    for (int32_t v = tid; v < N; v += kSmallThreads)
      if (S.fate[v] == 1)
        for (int32_t a = S.ng[v]; a < N; a = S.ng[a]) atomicAdd(&size[a], 1u);
    // finite vertices by (parent, signed position)
    const uint32_t none = 0xffffffffu;
    for (int32_t v = tid; v < V.sort_n; v += kSmallThreads)
      srt[v] = v < N && S.fate[v] == 1
                   ? ((uint32_t)S.ng[v] << 16) | (uint32_t)v : none;
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
    if (ok && (v == N || S.fate[v] == 1)) {
      ++nfin;
      // the sink has children when any vertex is finite
      bool inner = v < N && size[v] > 1;
      if (v == N)
        for (int32_t u = 0; u < N && !inner; ++u) inner = S.fate[u] == 1;
      k = inner ? (int32_t)mid[v] - (int32_t)first[v] : 0;
      for (int32_t a = v; a < N; a = S.ng[a])
        k += (int32_t)off[a] - (int32_t)first[S.ng[a]] +
             (a >= G.n_oddpri ? 1 : 0);
    }
    if (ok) V.key[v == N ? N : V.perm[v]] = k;
  }
  if (tid == 0) s_open = 0;
  __syncthreads();
  if (nfin) atomicAdd(&s_open, nfin);
  __syncthreads();
  if (tid == 0) {
    G.ctr[C_ERR] = (s_bad ? ERR_INVAL : 0) | (s_err ? ERR_INADMISSIBLE : 0);
    G.ctr[S_STATE] = !done || s_deep ? SS_DEEP : SS_SOLVED;
    G.ctr[S_NFIN] = s_open;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static size_t run_lds(int64_t N, int64_t M) {
  auto a = [](size_t b) { return (b + 15) & ~size_t(15); };
  return 4 * a(2 * N) + a(2 * (N + 1)) + a(2 * M) + a(N);
}
static int32_t sort_size(int64_t N) {
  int32_t n = 2;
  while (n < N) n <<= 1;
  return n;
}
static size_t value_lds(int64_t N) {
  auto a = [](size_t b) { return (b + 15) & ~size_t(15); };
  return 4 * a(2 * N) + 2 * a(2 * (N + 1)) + a(4 * N) +
         4 * (size_t)sort_size(N) + a(N);
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
  G.ctr = g->ctr;
  return G;
}

static pg_status small_read(pg_game *g, hipStream_t s) {
  PG_HIP(hipMemcpyAsync(g->hctr, g->ctr, sizeof(int32_t) * S_END,
                        hipMemcpyDeviceToHost, s));
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
  if (g->timed && !g->ev_a) {
    PG_HIP(hipEventCreate(&g->ev_a));
    PG_HIP(hipEventCreate(&g->ev_b));
  }
  if (g->timed) PG_HIP(hipEventRecord(g->ev_a, s));
  PG_LAUNCH(&g->prof, K_SMALL, 0.0, k_small_run, dim3(1), dim3(kSmallThreads),
            run_lds(g->n_aug, g->m_aug), s, small_game(g), R);
  if (g->timed) PG_HIP(hipEventRecord(g->ev_b, s));
  PG_TRY(small_read(g, s));
  if (!g->timed ||
      hipEventElapsedTime(&g->last_ms, g->ev_a, g->ev_b) != hipSuccess)
    g->last_ms = 0.0f;
  *out = IncOut();
  out->nval = g->hctr[S_NVAL];
  out->odd = g->hctr[S_ODDSW];
  out->even = g->hctr[S_EVENSW];
  g->inc.inner = g->hctr[S_INNER];
  g->inc.major = g->hctr[S_MAJOR];
  *deep = false;
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
  if (n_finite) *n_finite = g->hctr[S_NFIN];
  return PG_OK;
}

}  // namespace pgk

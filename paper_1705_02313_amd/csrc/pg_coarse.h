// Coarse keys and the switching rules on them (rank games whose ids are in
// signed-priority order: relabeled single games, the batch's arena).
#ifndef PG_COARSE_H
#define PG_COARSE_H

#include "pg_common.h"

namespace pgk {

// Coarse keys: a finite vertex's key is that of the last vertex of its ng
// chain before the sink (its root, a child of the sink in the ng tree).
// Siblings are in signed-priority order, the order of a relabeled game's
// ids, and the sink lies between its odd and its even children, so vertices
// with different coarse keys compare as their ranks do.
__device__ __host__ __forceinline__ int32_t coarse_key(int32_t root) {
  return 2 * root + 1;
}
__device__ __host__ __forceinline__ int32_t coarse_sink(int32_t n_oddpri) {
  return 2 * n_oddpri;
}

constexpr int kClimb = 1024;   // ng steps of one comparison

// What a comparison and a row read: a game, ng and the coarse keys.
struct CoarseP {
  int32_t N, n_oddpri;
  const int64_t *off;
  const int32_t *tgt, *pri, *ng, *key;
};

// 1, 0 or -1: Val(x) above, equal to or below Val(y), for finite x and y.
// The ng chains meet at their least common ancestor; in the tree's listing
// order a vertex lies above its odd and below its even children's subtrees,
// and siblings are in signed-priority order, which is the order of the ids.
__device__ __forceinline__ int coarse_climb(const CoarseP &P, int32_t x,
                                            int32_t y, bool *stop) {
  const int32_t N = P.N;
  int32_t a = x, b = y, ca = -1, cb = -1;
  // a vertex's ng is fetched with its priority: one round trip a step
  int32_t pa = a >= N ? 2147483647 : P.pri[a], na = a >= N ? N : P.ng[a];
  int32_t pb = b >= N ? 2147483647 : P.pri[b], nb = b >= N ? N : P.ng[b];
  for (int s = 0; a != b; ++s) {
    if (s >= kClimb) {
      *stop = true;
      return 0;
    }
    if (pa < pb) {
      ca = a;
      a = na;
      pa = a >= N ? 2147483647 : P.pri[a];
      na = a >= N ? N : P.ng[a];
    } else {
      cb = b;
      b = nb;
      pb = b >= N ? 2147483647 : P.pri[b];
      nb = b >= N ? N : P.ng[b];
    }
  }
  if (ca < 0) return cb < 0 ? 0 : (cb >= P.n_oddpri ? -1 : 1);
  if (cb < 0) return ca >= P.n_oddpri ? 1 : -1;
  return ca > cb ? 1 : -1;
}

// the same for any two vertices (or the sink) with their coarse keys
__device__ __forceinline__ int coarse_cmp(const CoarseP &P, int32_t x,
                                          int32_t kx, int32_t y, int32_t ky,
                                          bool *stop) {
  if (kx != ky) return kx < ky ? -1 : 1;
  if (x == y || kx == PG_KEY_TOP) return 0;
  return coarse_climb(P, x, y, stop);
}

// All_Odd and All_Even (section 4, section 3) for a vertex with the current
// choice cur: true when it switches, to *to.  *tie: its best key is met on
// two vertices or is the current choice's too, so the row has to be read
// again with comparisons (coarse_exact).  Keys that are ranks never tie.
__device__ __forceinline__ bool coarse_row(const CoarseP &P, int32_t v,
                                           int32_t cur, bool odd, int32_t *to,
                                           bool *tie) {
  const int64_t e0 = P.off[v], e1 = P.off[v + 1];
  const int32_t kn = odd ? 0 : P.key[P.N];
  int32_t best = odd ? -1 : P.N, kb = kn, kc = kn;
  // the current choice's key comes with the row's gathers when it is there
  bool have = !odd && cur == P.N, two = false;
  for (int64_t q = e0; q < e1; q += 4) {
    int32_t u[4], k[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = q + j < e1 ? P.tgt[q + j] : -1;
#pragma unroll
    for (int j = 0; j < 4; ++j) k[j] = u[j] >= 0 ? P.key[u[j]] : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (u[j] < 0) continue;
      if (u[j] == cur) {
        kc = k[j];
        have = true;
      }
      if (odd ? best < 0 || k[j] < kb : k[j] > kb) {
        best = u[j];
        kb = k[j];
        two = false;
      } else {
        two |= k[j] == kb && u[j] != best;
      }
    }
  }
  if (!have) kc = P.key[cur];
  *to = best;
  // top never ties: the first top option is taken, a top minimum stays
  *tie = kb != PG_KEY_TOP && (two || (kb == kc && best != cur));
  return odd ? kb < kc : kb > kc;
}

// F: four entries a round trip, for kernels that meet long rows here (short
// ones are done sooner one by one: ties of the 10M-vertex game 25 against 28
// us a valuation).
template <bool F = false>
__device__ __forceinline__ bool coarse_exact(const CoarseP &P, int32_t v,
                                             int32_t cur, bool odd,
                                             int32_t *to, bool *stop) {
  const int64_t e0 = P.off[v], e1 = P.off[v + 1];
  int32_t best = odd ? -1 : P.N, kb = odd ? 0 : P.key[P.N];
  auto take = [&](int32_t u, int32_t k) {
    if (best >= 0) {
      const int c = coarse_cmp(P, u, k, best, kb, stop);
      if (!(odd ? c < 0 : c > 0)) return;
    }
    best = u;
    kb = k;
  };
  if constexpr (F) {
    for (int64_t q = e0; q < e1; q += 4) {
      int32_t u[4], k[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) u[j] = q + j < e1 ? P.tgt[q + j] : -1;
#pragma unroll
      for (int j = 0; j < 4; ++j) k[j] = u[j] >= 0 ? P.key[u[j]] : 0;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (u[j] >= 0) take(u[j], k[j]);
    }
  } else {
    for (int64_t q = e0; q < e1; ++q) {
      const int32_t u = P.tgt[q];
      take(u, P.key[u]);
    }
  }
  if (best == cur) return false;
  const int c = coarse_cmp(P, best, kb, cur, P.key[cur], stop);
  *to = best;
  return odd ? c < 0 : c > 0;
}

// ---------------------------------------------------------------------------
// wide rows
// ---------------------------------------------------------------------------
// One thread reads a row four entries a round trip: the rows of a few hubs
// kept every step of a run waiting, which full valuations over buckets
// (pg_switch.hip) share over a block.  Rows beyond kWideRow entries are
// decided by the whole block, one after the other; a row of a block with n of
// them only from kWideShare n entries on: below that its own thread is done
// before the block has come through all n, some 4 us each.  Solves of 1M
// vertices, load included, with a thread per row -> so: four Odd rows of
// 100,000 entries 1,212 -> 116 ms (nearly all of it the load), 200 of 5,000
// 133 -> 20 ms, four Even ones of 100,000 130 -> 43 ms; a batch of 20 games
// with two rows of 8,000 each 187 -> 16 ms.
constexpr int kWideShare = 16;

template <int T>
struct WideLds {
  int32_t v[T], to[T];   // the block's wide rows and their switches (-1: none)
  int32_t n;
  unsigned long long sum;
  int32_t k[T / kWave], c[T / kWave];
  int64_t at[T / kWave];
};

// The rule for v's row (current choice cur) by all T threads of the block,
// each of which gets the answer: the best key first, each thread its own
// entries'; then the entries that have it, by climbs.
template <int T>
__device__ bool coarse_wide(const CoarseP &P, int32_t v, int32_t cur, bool odd,
                            int32_t *to, bool *stop, WideLds<T> &W) {
  constexpr int U = 8;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t e0 = P.off[v], e1 = P.off[v + 1];
  const int32_t none = odd ? PG_KEY_TOP : -1;
  const int32_t kc = P.key[cur];
  int32_t best = -1, kb = none;
  int64_t at = 0;
  bool two = false;
  for (int64_t q = e0 + tid; q < e1; q += (int64_t)U * T) {
    int32_t u[U], k[U];
#pragma unroll
    for (int j = 0; j < U; ++j)
      u[j] = q + j * T < e1 ? P.tgt[q + j * T] : -1;
#pragma unroll
    for (int j = 0; j < U; ++j) k[j] = u[j] >= 0 ? P.key[u[j]] : 0;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (u[j] < 0) continue;
      if (best < 0 || (odd ? k[j] < kb : k[j] > kb)) {
        best = u[j];
        kb = k[j];
        at = q + j * T;
        two = false;
      } else {
        two |= k[j] == kb && u[j] != best;
      }
    }
  }
  int32_t g = kb;
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const int32_t x = __shfl_xor(g, o);
    if (odd ? x < g : x > g) g = x;
  }
  __syncthreads();   // (an earlier row's words)
  if (lane == 0) W.k[wave] = g;
  __syncthreads();
  for (int w = 0; w < T / kWave; ++w)
    if (odd ? W.k[w] < g : W.k[w] > g) g = W.k[w];
  // every thread has the row's best key now
  if (odd) {
    if (g == PG_KEY_TOP || g > kc) return false;
  } else {
    const int32_t kn = P.key[P.N];
    if (g <= kn) {
      *to = P.N;
      return kn > kc;
    }
    if (g < kc || kc == PG_KEY_TOP) return false;
    if (g == PG_KEY_TOP) {   // the first top entry
      int64_t f = kb == g ? at : e1;
      for (int o = kWave / 2; o > 0; o >>= 1) {
        const int64_t x = __shfl_xor(f, o);
        f = x < f ? x : f;
      }
      if (lane == 0) W.at[wave] = f;
      __syncthreads();
      for (int w = 0; w < T / kWave; ++w) f = W.at[w] < f ? W.at[w] : f;
      *to = P.tgt[f];
      return true;
    }
  }
  // a or b (-1: none), both with key g: the one the player prefers
  auto better = [&](int32_t a, int32_t b) {
    if (a < 0 || b < 0 || a == b) return a < 0 ? b : a;
    const int c = coarse_climb(P, a, b, stop);
    return (odd ? c <= 0 : c >= 0) ? a : b;
  };
  int32_t c = kb == g ? best : -1;
  if (c >= 0 && two)
    for (int64_t q = e0 + tid; q < e1; q += T) {
      const int32_t u = P.tgt[q];
      if (P.key[u] == g) c = better(c, u);
    }
  for (int o = kWave / 2; o > 0; o >>= 1) c = better(c, __shfl_xor(c, o));
  if (lane == 0) W.c[wave] = c;
  __syncthreads();
  c = -1;
  for (int w = 0; w < T / kWave; ++w) c = better(c, W.c[w]);
  *to = c;
  if (c == cur) return false;
  if (g != kc) return true;
  const int d = coarse_climb(P, c, cur, stop);
  return odd ? d < 0 : d > 0;
}

// Decides the wide rows among the vertices v (where live) of the block's
// threads; true for a thread whose row was: *sw and *to are its switch.
// Every thread of the block calls it.  With rows of more than `most` entries
// together it only raises *stop.
template <int T>
__device__ __forceinline__ bool wide_rows(const CoarseP &P, bool live,
                                          int32_t v, bool odd, const int2 *sp,
                                          WideLds<T> &W, bool *sw, int32_t *to,
                                          bool *stop,
                                          unsigned long long most = ~0ull) {
  const int64_t len = live ? P.off[v + 1] - P.off[v] : 0;
  const bool wide = len > kWideRow;
  if (!__syncthreads_or(wide)) return false;
  if (threadIdx.x == 0) {
    W.n = 0;
    W.sum = 0;
  }
  __syncthreads();
  int slot = 0;
  if (wide) {
    slot = atomicAdd(&W.n, 1);
    W.v[slot] = v;
    if (most != ~0ull) atomicAdd(&W.sum, (unsigned long long)len);
  }
  __syncthreads();
  if (W.sum > most) {
    *stop = true;
    return true;
  }
  const int n = W.n;
  for (int k = 0; k < n; ++k) {
    const int32_t w = W.v[k];
    if (P.off[w + 1] - P.off[w] <= (int64_t)kWideShare * n) continue;
    int32_t x = 0;
    const bool s = coarse_wide<T>(P, w, sp[w].x, odd, &x, stop, W);
    if (threadIdx.x == 0) W.to[k] = s ? x : -1;
  }
  __syncthreads();
  if (!wide || len <= (int64_t)kWideShare * n) return false;
  *to = W.to[slot];
  *sw = *to >= 0;
  return true;
}

}  // namespace pgk

#endif

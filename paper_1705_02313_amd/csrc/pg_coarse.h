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

__device__ __forceinline__ bool coarse_exact(const CoarseP &P, int32_t v,
                                             int32_t cur, bool odd,
                                             int32_t *to, bool *stop) {
  const int64_t e0 = P.off[v], e1 = P.off[v + 1];
  int32_t best = odd ? -1 : P.N, kb = odd ? 0 : P.key[P.N];
  for (int64_t q = e0; q < e1; ++q) {
    const int32_t u = P.tgt[q], k = P.key[u];
    if (best >= 0) {
      const int c = coarse_cmp(P, u, k, best, kb, stop);
      if (!(odd ? c < 0 : c > 0)) continue;
    }
    best = u;
    kb = k;
  }
  if (best == cur) return false;
  const int c = coarse_cmp(P, best, kb, cur, P.key[cur], stop);
  *to = best;
  return odd ? c < 0 : c > 0;
}

}  // namespace pgk

#endif

// Count rows (count valuations): D ints in registers, and the switching rules
// on them.
#pragma once

#include "pg_common.h"

namespace pgk {

// adds s at column col without indexing a register array at run time
template <int D>
__device__ __forceinline__ void add_unit(int32_t (&a)[D], int col,
                                         int32_t s) {
#pragma unroll
  for (int i = 0; i < D; ++i) a[i] += (i == col) ? s : 0;
}

template <int D>
__device__ __forceinline__ void load_vec(const int32_t *p, int32_t (&a)[D]) {
  const int4 *q = reinterpret_cast<const int4 *>(p);
#pragma unroll
  for (int i = 0; i < D / 4; ++i) {
    const int4 x = q[i];
    a[4 * i] = x.x;
    a[4 * i + 1] = x.y;
    a[4 * i + 2] = x.z;
    a[4 * i + 3] = x.w;
  }
}

template <int D>
__device__ __forceinline__ void store_vec(int32_t *p, const int32_t (&a)[D]) {
  int4 *q = reinterpret_cast<int4 *>(p);
#pragma unroll
  for (int i = 0; i < D / 4; ++i)
    q[i] = make_int4(a[4 * i], a[4 * i + 1], a[4 * i + 2], a[4 * i + 3]);
}

// -1: a below b, 0: equal, 1: above.  Top equals top and is above every
// count vector; otherwise the largest differing column decides: a larger
// count is better at an even priority, worse at an odd one.
template <int D>
__device__ __forceinline__ int vcmp(bool ta, const int32_t (&a)[D], bool tb,
                                    const int32_t (&b)[D], uint32_t odd_cols) {
  if (ta || tb) return ta == tb ? 0 : (ta ? 1 : -1);
  int r = 0;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    if (a[i] != b[i]) {
      const bool even = !((odd_cols >> i) & 1u);
      r = ((a[i] < b[i]) == even) ? -1 : 1;
    }
  }
  return r;
}

// the valuation of vertex u (u == N: the sink, the zero vector); returns
// whether it is top (the marker -1 in the first column)
template <int D>
__device__ __forceinline__ bool load_val(const int32_t *cnt, int32_t u,
                                         int32_t (&a)[D]) {
  load_vec<D>(cnt + (int64_t)u * D, a);
  return a[0] < 0;
}

// All_Odd (section 4): the first successor of least valuation, if strictly
// below the current choice.  True when v (whose record is me) switches, to
// *to.
template <int D>
__device__ __forceinline__ bool cnt_decide_odd(
    const int64_t *off, const int32_t *tgt, const int32_t *cnt,
    uint32_t odd_cols, int32_t v, int2 me, int32_t *to) {
  const int64_t e0 = off[v], e1 = off[v + 1];
  // the current choice is normally in the row: its valuation comes with
  // the row's loads (a strategy given at the C ABI may name another vertex)
  const int32_t cur = me.x;
  int32_t cv[D];
  bool ct = false, have_c = false;
  int32_t best = tgt[e0];
  int32_t bv[D];
  bool bt = load_val<D>(cnt, best, bv);
  if (best == cur) {
    ct = bt;
    have_c = true;
#pragma unroll
    for (int i = 0; i < D; ++i) cv[i] = bv[i];
  }
  for (int64_t e = e0 + 1; e < e1; ++e) {
    const int32_t u = tgt[e];
    int32_t uv[D];
    const bool ut = load_val<D>(cnt, u, uv);
    if (u == cur) {
      ct = ut;
      have_c = true;
#pragma unroll
      for (int i = 0; i < D; ++i) cv[i] = uv[i];
    }
    if (vcmp<D>(ut, uv, bt, bv, odd_cols) < 0) {
      best = u;
      bt = ut;
#pragma unroll
      for (int i = 0; i < D; ++i) bv[i] = uv[i];
    }
  }
  if (!have_c) ct = load_val<D>(cnt, cur, cv);
  *to = best;
  return vcmp<D>(bt, bv, ct, cv, odd_cols) < 0;
}

// All_Even, greedy all-switches (section 3): the sink first, then the row;
// the first option of greatest valuation, if strictly above the current one.
template <int D>
__device__ __forceinline__ bool cnt_decide_even(
    int32_t N, const int64_t *off, const int32_t *tgt, const int32_t *cnt,
    uint32_t odd_cols, int32_t v, int2 me, int32_t *to) {
  const int64_t e0 = off[v], e1 = off[v + 1];
  // the current choice is the sink (the zero vector) or normally in the
  // row (see All_Odd)
  const int32_t cur = me.x;
  int32_t cv[D] = {};
  bool ct = false, have_c = cur == N;
  int32_t best = N;
  int32_t bv[D] = {};
  bool bt = false;
  for (int64_t e = e0; e < e1; ++e) {
    const int32_t u = tgt[e];
    int32_t uv[D];
    const bool ut = load_val<D>(cnt, u, uv);
    if (u == cur) {
      ct = ut;
      have_c = true;
#pragma unroll
      for (int i = 0; i < D; ++i) cv[i] = uv[i];
    }
    if (vcmp<D>(ut, uv, bt, bv, odd_cols) > 0) {
      best = u;
      bt = ut;
#pragma unroll
      for (int i = 0; i < D; ++i) bv[i] = uv[i];
    }
  }
  if (!have_c) ct = load_val<D>(cnt, cur, cv);
  *to = best;
  return vcmp<D>(bt, bv, ct, cv, odd_cols) > 0;
}

}  // namespace pgk

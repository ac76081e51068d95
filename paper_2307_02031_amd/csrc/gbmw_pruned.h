// Device code of the layer step that looks only at what can still be minimal
// (Tables::runs != 0).  Internal; included by gbmw_kernels.hip.
//
// Along the budget axis every table is a non-increasing step function, and every layer leaves,
// per strategy and group of 64 budgets e' of its min-plus product, the value T + c at the
// group's first and at its last budget (Tables::Tsum).  For the group of budgets [wb, el] those
// words bound column s' of the previous table from above (its value at wb or earlier) and from
// below (at el or later), and with the smallest and the largest entry of row s' of R
// (Tables::Row) they bound its candidates C + R: a column whose lower bound exceeds the
// smallest upper bound of all columns is the minimiser of no cell of the group, whatever the
// output strategy.  fp32 addition is monotone, so the bounds hold for the rounded sums and the
// columns that are left (the candidates) decide every value and every lowest index, bit for bit.
// On the batched workloads 2 to 25 of 22 to 186 columns are left.
//
// One wave does that for up to four groups of 64 budgets, a lane per column.  Then:
//   - every candidate is constant over the group (95 % of the groups of the structured
//     workloads): the group's cells are computed once, a lane per output strategy;
//   - otherwise one wave takes the group (dense_group): the candidates' columns go to LDS, and,
//     a lane per output strategy, the sums at the group's first feasible and last budget give the
//     summary words and, per output, the candidates that can still be minimal somewhere in it
//     (mostly one: then a row is two additions and a store);
//   - more than kept() candidates (the groups where the first plans start to fit, where there is
//     no upper bound yet): the four waves of the workgroup share the group (big_group).
//
// What bounds it: the chain of one group (2 to 5 us of loads, 1 to 4 us of bounds, 5 to 18 us of cells)
// and the fetch of its 40 to 90 KB of code, neither bytes (46 MB per launch at B=64, S=44, E=32768:
// 1.1 TB/s) nor arithmetic.  Fills, before (all candidates unless a wave's columns are constant; no
// such shortcut beyond 64 strategies) -> with this step: B=64 S=44 E=32768 1.08 -> 0.80 ms, B=16
// L=96 S=64 E=65536 14.6 -> 7.2 ms, B=16 S=128 E=32768 4.8 -> 0.73 ms.  Everything unrolled over
// candidates is therefore sized to them (8 or kept()) and called from one place: at 84 to 215 KB of
// code the same step spilled scalar registers and took 30 to 40 % longer.
#pragma once
#include "gbmw_kernels.h"

namespace gbmw {

constexpr int kWaves = 4;              // waves per workgroup of the pruned step
constexpr int kUnit = 4;               // groups of 64 budgets that one wave classifies at once (at most)
// Candidates whose columns a wave's share of LDS holds, by strategies rounded up to a multiple of 4.
__host__ __device__ constexpr int kept(int SP) { return SP < 16 ? SP : SP <= 128 ? 16 : 24; }

// Summary of a table, laid out and indexed like the table itself: [S][EP / 64] pairs.
__device__ __forceinline__ float2* sum_table(const Tables& t, int inst, int row, int l) {
  const size_t slab = (size_t)t.S * (t.EP >> 6);
  return t.keep_all ? t.Tsum + (size_t)row * slab
                    : t.Tsum + ((size_t)(l & 1) * t.B + inst) * slab;
}

// The group records of table row `row`: [S][EP / 64] bytes (null without them).
__device__ __forceinline__ uint8_t* group_records(const Tables& t, int row) {
  return t.Asum ? t.Asum + (size_t)row * t.S * (t.EP >> 6) : nullptr;
}

__device__ __forceinline__ float* c_table(const Tables& t, int inst, int row, int l) {
  const size_t slab = (size_t)t.S * t.EP;
  return t.keep_all ? t.Cbuf + (size_t)row * slab
                    : t.Cbuf + ((size_t)(l & 1) * t.B + inst) * slab;
}

__device__ __forceinline__ float lane_f(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ int clamp_m(int m, int E) { return (m < 0 || m > E + 1) ? E + 1 : m; }

// Minimum over the wave's 64 lanes, in every lane (data-parallel shifts, no LDS round trips).
__device__ __forceinline__ float wave_min(float v) {
  constexpr int kInf = 0x7f800000;
#define GBMW_DPP(ctrl, rows) \
  v = __builtin_fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(kInf, __float_as_int(v), ctrl, rows, 0xf, false)))
  GBMW_DPP(0x111, 0xf);                // row_shr:1
  GBMW_DPP(0x112, 0xf);                // row_shr:2
  GBMW_DPP(0x114, 0xf);                // row_shr:4
  GBMW_DPP(0x118, 0xf);                // row_shr:8
  GBMW_DPP(0x142, 0xa);                // row_bcast:15
  GBMW_DPP(0x143, 0xc);                // row_bcast:31
#undef GBMW_DPP
  return lane_f(v, 63);
}
__device__ __forceinline__ int wave_min(int v) {
  constexpr int kMax = 0x7fffffff;
#define GBMW_DPP(ctrl, rows) \
  { const int o = __builtin_amdgcn_update_dpp(kMax, v, ctrl, rows, 0xf, false); v = o < v ? o : v; }
  GBMW_DPP(0x111, 0xf) GBMW_DPP(0x112, 0xf) GBMW_DPP(0x114, 0xf) GBMW_DPP(0x118, 0xf)
  GBMW_DPP(0x142, 0xa) GBMW_DPP(0x143, 0xc)
#undef GBMW_DPP
  return __builtin_amdgcn_readlane(v, 63);
}

// N rows of R from s0 on (one wave): copied to Rn, their smallest and largest entries with c and M
// of the layer to Row.  Returns false in a lane that read a negative entry or a NaN.
template <int N>
__device__ __forceinline__ bool row_limits(const float* __restrict__ R, int S, int s0, int lane,
                                           const float* __restrict__ c, const int* __restrict__ M,
                                           float* __restrict__ Rn, float4* __restrict__ Row) {
  float lo[N], hi[N];
  bool good = true;
#pragma unroll
  for (int i = 0; i < N; ++i) { lo[i] = INFINITY; hi[i] = -INFINITY; }
  for (int s = lane; s < S; s += 64) {
    float v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = s0 + i < S ? R[(size_t)(s0 + i) * S + s] : 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      good = good && v[i] >= 0.0f;
      lo[i] = __builtin_fminf(lo[i], v[i]);
      hi[i] = __builtin_fmaxf(hi[i], v[i]);
      if (s0 + i < S) Rn[(size_t)(s0 + i) * S + s] = v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float a = wave_min(lo[i]), b = -wave_min(-hi[i]);
    if (lane == 0 && s0 + i < S) Row[s0 + i] = make_float4(a, b, c[s0 + i], __int_as_float(M[s0 + i]));
  }
  return good;
}

// Keeps the values read across the lanes in one unrolled loop from being kept in scalar registers
// for the next, and from being read all at once (they spill).
__device__ __forceinline__ void forget(int& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void by_fours(int k) { if ((k & 3) == 3) __builtin_amdgcn_sched_barrier(0); }

// Orders a wave's LDS writes before its other lanes' reads (and reads before later writes).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// What one wave knows of the previous table's columns for one group of budgets: lane i of chunk c
// holds column s' = 64 c + i.
template <int NCH>
struct Columns {
  int m[NCH];                          // M(l-1, s'), clamped to 0..E+1
  float2 a[NCH], b[NCH];               // the summaries of the (at most two) groups its budgets fall in
  float2 rl[NCH];                      // smallest and largest R(l, s', .)
};

// Bounds of the columns over the budgets [wb, el], and the candidates.  varies: some candidate is
// not constant over the group.
template <int NCH>
__device__ __forceinline__ void bounds(const Columns<NCH>& q, int wb, int el, float (&ub)[NCH], float (&lb)[NCH],
                                       unsigned long long (&cand)[NCH], bool& varies) {
  float u = INFINITY;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int m = q.m[c];
    ub[c] = wb >= m ? q.a[c].x : INFINITY;
    lb[c] = el < m ? INFINITY : ((el - m) >> 6) != ((wb - m) >> 6) ? q.b[c].y : q.a[c].y;
    u = __builtin_fminf(u, ub[c] + q.rl[c].y);
  }
  float top = wave_min(u);
  // No column is bounded at wb: the first plans start to fit inside the group.  The column whose
  // second word is the first finite one (at budget e1) then bounds the budgets from e1 on; below
  // e1 only the columns count that may become finite there (176 -> 23 candidates on the cost-model
  // workloads, where many strategies need the same memory).
  unsigned early = 0;                                   // bit c: this lane's column of chunk c may be finite below e1
  if (top == INFINITY) {
    int second[NCH], e1 = 0x7fffffff;
    bool ends[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int m = q.m[c];
      second[c] = m + ((((wb - m) >> 6) + 1) << 6);
      ends[c] = el >= m && el >= second[c] && q.b[c].x < INFINITY;
      if (ends[c]) e1 = second[c] < e1 ? second[c] : e1;
    }
    e1 = wave_min(e1);
    u = INFINITY;
    early = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (ends[c] && second[c] == e1) u = __builtin_fminf(u, q.b[c].x + q.rl[c].y);
      if ((wb >= q.m[c] && q.a[c].y < INFINITY) || (second[c] < e1 && !ends[c])) early |= 1u << c;
    }
    top = wave_min(u);
  }
  varies = false;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const bool in = lb[c] < INFINITY && (lb[c] + q.rl[c].x <= top || ((early >> c) & 1));
    cand[c] = __builtin_amdgcn_ballot_w64(in);
    varies = varies || __builtin_amdgcn_ballot_w64(in && __float_as_int(ub[c]) != __float_as_int(lb[c])) != 0;
  }
}

// The columns of one group of budgets.
template <int NCH, bool FIRST>
__device__ __forceinline__ void load_columns(const Tables& t, int inst, int row, int l, int wb, int el, int lane,
                                             Columns<NCH>& q) {
  const int S = t.S, E = t.E, G = t.EP >> 6;
  const float2* __restrict__ Ts = FIRST ? nullptr : sum_table(t, inst, row - 1, l - 1);
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int s = 64 * c + lane;
    q.m[c] = 0;
    q.a[c] = q.b[c] = make_float2(INFINITY, INFINITY);
    q.rl[c] = make_float2(0.0f, 0.0f);
    if (s < S) {
      const int m = clamp_m(t.M[(size_t)(row - 1) * S + s], E);
      q.m[c] = m;
      const float4 info = t.Row[(size_t)row * S + s];
      q.rl[c] = make_float2(info.x, info.y);
      if (FIRST) {
        const float cv = t.c[(size_t)(row - 1) * S + s];
        q.a[c] = q.b[c] = make_float2(cv, cv);
      } else {
        const float2* __restrict__ w = Ts + (size_t)s * G;
        q.a[c] = w[(wb > m ? wb - m : 0) >> 6];
        q.b[c] = w[(el > m ? el - m : 0) >> 6];
      }
    }
  }
}

// The same for `unit` consecutive groups from budget `base`: w[c][g] and w[c][g + 1] are the two
// words of group g.  Ts, Mrow: summaries and M of the columns' table.
template <int NCH>
__device__ __forceinline__ void load_unit(const Tables& t, const float2* __restrict__ Ts, const int* __restrict__ Mrow,
                                          int base, int unit, int lane, int (&m)[NCH], float2 (&w)[NCH][kUnit + 1]) {
  const int S = t.S, E = t.E, G = t.EP >> 6;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int s = 64 * c + lane;
    m[c] = 0;
#pragma unroll
    for (int g = 0; g <= kUnit; ++g) w[c][g] = make_float2(INFINITY, INFINITY);
    if (s < S) m[c] = clamp_m(Mrow[s], E);
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int s = 64 * c + lane;
    if (s < S) {
      const int g0 = (base - m[c]) >> 6;                 // arithmetic: -1 and below lie before the table
      const float2* __restrict__ src = Ts + (size_t)s * G;
#pragma unroll
      for (int g = 0; g <= kUnit; ++g)
        if (g <= unit) {
          const int at = g0 + g;
          w[c][g] = src[at < 0 ? 0 : at > (E >> 6) ? (E >> 6) : at];
        }
    }
  }
}

// C(l-1, wb + lane, s') of one column (s' wave-uniform, cell = what memory holds there): +inf
// below M and beyond E, the group's word where its two ends are equal, else the cell.
template <int NCH, bool FIRST>
__device__ __forceinline__ float column_value(const Columns<NCH>& q, int s, float cell, int wb, int E, int lane) {
  int m = 0, c = 0;
  float2 a = make_float2(0.0f, 0.0f), b = a;
#pragma unroll
  for (; c < NCH; ++c)
    if (NCH == 1 || (s >> 6) == c) {
      m = __builtin_amdgcn_readlane(q.m[c], s & 63);
      a = make_float2(lane_f(q.a[c].x, s & 63), lane_f(q.a[c].y, s & 63));
      b = make_float2(lane_f(q.b[c].x, s & 63), lane_f(q.b[c].y, s & 63));
    }
  const int e = wb + lane;
  const int second = m + ((((wb - m) >> 6) + 1) << 6);   // first budget of the second group
  const bool ca = __float_as_int(a.x) == __float_as_int(a.y), cb = __float_as_int(b.x) == __float_as_int(b.y);
  float v;
  if (FIRST) v = a.x;
  else v = e < second ? (ca ? a.x : cell) : (cb ? b.x : cell);
  return (e < m || e > E) ? INFINITY : v;
}

// R(l, s', s) for the lane's output s of one row s' of R (wave-uniform): from the workgroup's copy of
// the layer's R in LDS (STAGED: up to 64 strategies) or from memory.
template <bool STAGED>
__device__ __forceinline__ float r_of(const float* __restrict__ rt, const float* __restrict__ Rrow, int S, int sp, int s) {
  return STAGED ? rt[sp * S + s] : Rrow[(size_t)sp * S + s];
}

// The group's cells where every candidate is constant over it (val: lane s' of chunk c holds its
// value): lane j of chunk oc forms min_s' (val[s'] + R[s'][s]) for output s = 64 oc + j, candidates
// in index order and a strict compare, so that the lowest minimiser (0 if all are +inf) is kept.
template <int NCH>
__device__ __forceinline__ void uniform_outputs(const float* __restrict__ rt, const float* __restrict__ Rrow, int S,
                                                int lane, const float (&val)[NCH],
                                                const unsigned long long (&cand)[NCH], float (&best)[NCH],
                                                int (&arg)[NCH]) {
  constexpr int NB = NCH == 1 ? 8 : 4;                   // rows of R in flight
#pragma unroll
  for (int oc = 0; oc < NCH; ++oc) { best[oc] = INFINITY; arg[oc] = 0; }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    unsigned long long mask = cand[c];
    while (mask) {
      int k[NB];
      float r[NB][NCH];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        k[i] = mask ? __builtin_ctzll(mask) : k[i > 0 ? i - 1 : 0];   // past the end: the last one again
        mask &= mask - 1;
#pragma unroll
        for (int oc = 0; oc < NCH; ++oc) {
          const int s = 64 * oc + lane;
          r[i][oc] = s < S ? r_of<NCH == 1>(rt, Rrow, S, 64 * c + k[i], s) : INFINITY;
        }
      }
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int oc = 0; oc < NCH; ++oc) {
          const float x = lane_f(val[c], k[i]) + r[i][oc];
          if (x < best[oc]) { best[oc] = x; arg[oc] = 64 * c + k[i]; }
        }
    }
  }
}

// Where the rows of 64 cells at e' = wb + lane go, a lane per output strategy: at e = e' + m of
// column s.  Beyond E nothing is stored.
struct RowStores {
  float* p;                                              // of this lane's output
  int e;
  unsigned long long fits, whole;                        // outputs with any / all 64 cells inside the table
  __device__ __forceinline__ RowStores(float* __restrict__ Cn, int EP, int E, int s, int wb, int m) {
    e = wb + m;
    p = Cn + (size_t)s * EP + (e <= E ? e : 0);
    fits = __builtin_amdgcn_ballot_w64(e <= E);
    whole = __builtin_amdgcn_ballot_w64(e + 63 <= E);
  }
  __device__ __forceinline__ void store(int j, int lane, int E, float out) const {
    if (!((fits >> j) & 1)) return;
    const unsigned long long a = (unsigned long long)(uintptr_t)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)a, j);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(a >> 32), j);
    typedef __attribute__((address_space(1))) float gf32;
    gf32* q = (gf32*)(((unsigned long long)hi << 32) | lo);
    if ((whole >> j) & 1) q[lane] = out;
    else if (__builtin_amdgcn_readlane(e, j) + lane <= E) q[lane] = out;
  }
};

// The records of one row: the group's byte where all records inside the table are equal, else
// kNoGroupRecord and the 64 bytes.
__device__ __forceinline__ int store_records(uint8_t* __restrict__ An, int EP, int s, int wb, int n_in, int lane, int a) {
  const int a0 = __builtin_amdgcn_readfirstlane(a);
  if (__builtin_amdgcn_ballot_w64(a != a0 && lane < n_in) == 0) return a0;
  An[(size_t)s * EP + wb + lane] = (uint8_t)a;
  return kNoGroupRecord;
}

// The two words of a group from its first and last value; true if they stand for its cells.  A zero does
// not: costs of -0.0 are accepted, minima of equal sums keep the sign of the lowest index, and that may
// change inside a group that begins and ends with the same zero.  Its words differ in sign, so that every
// reader takes the cells.
__device__ __forceinline__ bool words_of(float first, float last, float2& w) {
  w = make_float2(first, last);
  if (last == 0.0f) w = make_float2(first == 0.0f ? 0.0f : first, -0.0f);
  return __float_as_int(w.x) == __float_as_int(w.y);
}

// Cells, summaries and records of one group for the outputs s = sfirst + lane (valid lanes), given
// the columns of its K <= KEEP candidates in LDS: lane k holds candidate k's strategy (listv, in
// index order) and the place of its column (slotv).  estar: first budget of the group at which a
// candidate is finite.  The candidates' rows of R stay in registers, a lane per output, and so do
// the columns, a lane per budget: a row costs no memory round trip.
template <int KEEP, bool STAGED, bool ARG>
__device__ __forceinline__ void rows(const Tables& t, int inst, int row, int l, int wb, int n_in, int lane, int K,
                                     int listv, int slotv, int estar, const float* __restrict__ col,
                                     const float* __restrict__ rt, int sfirst, bool valid) {
  const int S = t.S, E = t.E, EP = t.EP, G = EP >> 6;
  const float* __restrict__ Rrow = t.Rn + (size_t)row * S * S;
  const int s = valid ? sfirst + lane : 0;
  const float4 info = t.Row[(size_t)row * S + s];
  float r[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k)
    r[k] = r_of<STAGED>(rt, Rrow, S, __builtin_amdgcn_readlane(listv, k), s);   // beyond K: the last one's
  const float fv = lane < K ? col[slotv * 64 + estar] : INFINITY, lv = lane < K ? col[slotv * 64 + n_in - 1] : INFINITY;
  const float cs = info.z;
  // T at the first feasible and at the last budget of the group
  float tf = INFINITY, tl = INFINITY;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    tf = __builtin_fminf(tf, lane_f(fv, k) + r[k]);
    tl = __builtin_fminf(tl, lane_f(lv, k) + r[k]);
    by_fours(k);
  }
  int lvb = __float_as_int(lv);
  forget(lvb);
  // T is non-increasing along the budgets, so beyond the first feasible budget it is at most tf: a
  // candidate that is above that even at its last budget is never the minimiser
  unsigned live = 0;
  float rk = 0.0f;                                       // of the first live candidate kk
  int kk = 0;
#pragma unroll
  for (int k = KEEP - 1; k >= 0; --k) {
    by_fours(k);
    const float x = lane_f(__int_as_float(lvb), k);
    const bool in = x < INFINITY && x + r[k] <= tf;
    live |= in ? 1u << k : 0u;
    rk = in ? r[k] : rk;
    kk = in ? k : kk;
  }
  float2 words;
  const bool same = words_of((estar == 0 ? tf : INFINITY) + cs, tl + cs, words);   // the cells are all equal
  const bool none = tl == INFINITY;                                  // no predecessor fits: +inf throughout, record 0
  const bool one = estar == 0 && tf < INFINITY && __builtin_popcount(live) == 1;
  if (valid) sum_table(t, inst, row, l)[(size_t)s * G + (wb >> 6)] = words;
  int rec = 0;
  if (ARG) {
    const int own = __builtin_amdgcn_ds_bpermute(kk << 2, listv);
    rec = none ? 0 : own;                                            // of the outputs with one candidate left
  }
  const unsigned long long single = __builtin_amdgcn_ballot_w64(valid && !none && one && !same);
  unsigned long long multi = __builtin_amdgcn_ballot_w64(valid && !none && !one && (ARG || !same));
  const unsigned long long flat = __builtin_amdgcn_ballot_w64(same);
  const RowStores out(c_table(t, inst, row, l), EP, E, s, wb, clamp_m(__float_as_int(info.w), E));
  // one candidate left: the row is its column plus two constants
  if (single) {
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
      unsigned long long todo = single & __builtin_amdgcn_ballot_w64(kk == k);
      if (!todo) continue;
      const float v = col[__builtin_amdgcn_readlane(slotv, k) * 64 + lane];
      while (todo) {
        const int j = __builtin_ctzll(todo);
        todo &= todo - 1;
        out.store(j, lane, E, (v + lane_f(rk, j)) + lane_f(cs, j));
      }
    }
  }
  if (!multi) {
    if (ARG && valid) group_records(t, row)[(size_t)s * G + (wb >> 6)] = (uint8_t)rec;
    return;
  }
  // several: in index order with a strict compare, four candidates at a time, fours without a live
  // one left out
  float cp[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    cp[k] = k < K ? col[__builtin_amdgcn_readlane(slotv, k) * 64 + lane] : INFINITY;
    by_fours(k);
  }
  uint8_t* __restrict__ An = ARG ? t.A + (size_t)row * S * EP : nullptr;
  do {
    const int j = __builtin_ctzll(multi);
    multi &= multi - 1;
    const unsigned lvj = (unsigned)__builtin_amdgcn_readlane((int)live, j);
    float best = INFINITY;
    int a = -1;
#pragma unroll
    for (int c = 0; c < KEEP; c += 4)
      if (lvj & (15u << c)) {
#pragma unroll
        for (int k = c; k < c + 4; ++k) {
          const float y = cp[k] + lane_f(r[k], j);
          if (y < best) { best = y; a = k; }
        }
      }
    if (!((flat >> j) & 1)) out.store(j, lane, E, best + lane_f(cs, j));
    if (ARG) {
      const int a0 = __builtin_amdgcn_readfirstlane(a);
      int g;
      if (__builtin_amdgcn_ballot_w64(a != a0 && lane < n_in) == 0) {
        g = a0 < 0 ? 0 : __builtin_amdgcn_readlane(listv, a0);
      } else {
        const int own = __builtin_amdgcn_ds_bpermute(a << 2, listv);
        An[(size_t)(sfirst + j) * EP + wb + lane] = (uint8_t)(a < 0 ? 0 : own);
        g = kNoGroupRecord;
      }
      rec = lane == j ? g : rec;
    }
  } while (multi);
  if (ARG && valid) group_records(t, row)[(size_t)s * G + (wb >> 6)] = (uint8_t)rec;
}

// The same where the candidates change at few budgets of the group (steps: a bit per budget at which
// one of them differs from the budget before, bit 0 set): between two steps all budgets have the
// same cells.  So the group is computed step by step with a lane per output, five instructions per
// step and candidate for all outputs together, and the rows are put together from the steps' values
// through LDS: about ten instructions per row.  buf: the wave's columns (read into registers
// first); the values of step i and output j lie at [i][j ^ i], so that neither the writes (a lane
// per output) nor the reads (a lane per budget) meet in a bank.
template <int KEEP> constexpr int kRuns = KEEP > 16 ? 12 : 16;      // steps: their records fill 64 bits
template <int KEEP, bool STAGED, bool ARG>
__device__ __forceinline__ void runs_of_rows(const Tables& t, int inst, int row, int l, int wb, int n_in, int lane,
                                             int K, int listv, unsigned long long steps, float* __restrict__ buf,
                                             const float* __restrict__ rt, int sfirst, bool valid, bool last_chunk) {
  constexpr int kBits = KEEP > 16 ? 5 : 4;
  const int S = t.S, E = t.E, EP = t.EP, G = EP >> 6;
  const float* __restrict__ Rrow = t.Rn + (size_t)row * S * S;
  const int s = valid ? sfirst + lane : 0;
  const float4 info = t.Row[(size_t)row * S + s];
  const float cs = info.z;
  float r[KEEP], cp[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k)
    r[k] = r_of<STAGED>(rt, Rrow, S, __builtin_amdgcn_readlane(listv, k), s);
#pragma unroll
  for (int k = 0; k < KEEP; ++k) cp[k] = k < K ? buf[k * 64 + lane] : INFINITY;
  wave_sync();
  unsigned long long args = 0;                           // of this lane's output, kBits per step
  unsigned inf = 0;                                      // a bit per step without a feasible predecessor: record 0
  float fo = INFINITY, lo = INFINITY;
  int i = 0, a0 = 0;
  bool same_arg = true;
  unsigned long long todo = steps;
  do {
    const int e = __builtin_ctzll(todo);
    todo &= todo - 1;
    float best = INFINITY;
    int a = 0;
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
      const float y = lane_f(cp[k], e) + r[k];
      if (y < best) { best = y; a = k; }
      by_fours(k);
    }
    lo = best + cs;
    if (i == 0) fo = lo;
    if (ARG) {
      const int id = best < INFINITY ? a : KEEP;
      if (i == 0) a0 = id;
      same_arg = same_arg && id == a0;
      args |= (unsigned long long)a << (kBits * i);
      inf |= best < INFINITY ? 0u : 1u << i;
    }
    buf[i * 64 + (lane ^ i)] = lo;
    ++i;
  } while (todo);
  wave_sync();
  float2 words;
  const bool same = words_of(fo, lo, words);
  const int first_arg = ARG ? __builtin_amdgcn_ds_bpermute(a0 << 2, listv) : 0;   // all lanes: inactive ones give nothing
  if (valid) {
    sum_table(t, inst, row, l)[(size_t)s * G + (wb >> 6)] = words;
    if (ARG) {
      group_records(t, row)[(size_t)s * G + (wb >> 6)] = (uint8_t)(!same_arg ? kNoGroupRecord : a0 == KEEP ? 0 : first_arg);
    }
  }
  // this lane's step
  const int mine = __builtin_popcountll(steps & ((2ull << lane) - 1)) - 1;
  const RowStores out(c_table(t, inst, row, l), EP, E, s, wb, clamp_m(__float_as_int(info.w), E));
  unsigned long long cells = __builtin_amdgcn_ballot_w64(valid && !same) & out.fits;
  while (cells) {
    int j[4];
    float v[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      j[x] = cells ? __builtin_ctzll(cells) : -1;
      cells &= cells - 1;
      v[x] = buf[mine * 64 + ((j[x] & 63) ^ mine)];
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
      if (j[x] >= 0) out.store(j[x], lane, E, v[x]);
  }
  if (ARG) {
    uint8_t* __restrict__ An = t.A + (size_t)row * S * EP;
    unsigned long long recs = __builtin_amdgcn_ballot_w64(valid && !same_arg);
    while (recs) {
      const int j = __builtin_ctzll(recs);
      recs &= recs - 1;
      const unsigned lo32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)args, j);
      const unsigned hi32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(args >> 32), j);
      const unsigned none = (unsigned)__builtin_amdgcn_readlane((int)inf, j);
      const int a = (int)((((unsigned long long)hi32 << 32 | lo32) >> (kBits * mine)) & ((1u << kBits) - 1));
      const int own = __builtin_amdgcn_ds_bpermute(a << 2, listv);
      An[(size_t)(sfirst + j) * EP + wb + lane] = (uint8_t)(((none >> mine) & 1) ? 0 : own);
    }
  }
  if (!last_chunk) {                                     // the next outputs read the columns again
    wave_sync();
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
      if (k < K) buf[k * 64 + lane] = cp[k];
    wave_sync();
  }
}

// The cells of one group, by one wave, once its K <= KB candidates (cand) are known.
template <int NCH, int KB, bool FIRST, bool ARG>
__device__ __forceinline__ void dense_cells(const Tables& t, int inst, int row, int l, int wb, int lane, int part,
                                            int parts, const Columns<NCH>& q, const unsigned long long (&cand)[NCH],
                                            int K, float* __restrict__ col, const float* __restrict__ rt) {
  const int S = t.S, E = t.E, EP = t.EP;
  const int el = wb + 63 < E ? wb + 63 : E, n_in = el - wb + 1;
  const float* __restrict__ Cp = FIRST ? nullptr : c_table(t, inst, row - 1, l - 1);
  // their columns, in index order; listv: lane k holds the k-th candidate's strategy (past the end
  // the last one again)
  int listv = 0;
  {
    int n = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int at = n + __builtin_popcountll(cand[c] & ((1ull << lane) - 1));
      // lane -> its place; the inverse permutation through the wave's own LDS
      if ((cand[c] >> lane) & 1) reinterpret_cast<int*>(col)[at] = 64 * c + lane;
      n += __builtin_popcountll(cand[c]);
    }
    wave_sync();
    listv = reinterpret_cast<const int*>(col)[lane < K ? lane : K - 1];
    wave_sync();
  }
  int estar = 63;                                        // (a candidate is finite at the last budget)
  unsigned long long steps = 1;                          // budgets at which some candidate differs from the budget before
  {
    float cell[KB];
    if (!FIRST) {
#pragma unroll
      for (int k = 0; k < KB; ++k)
        cell[k] = Cp[(size_t)__builtin_amdgcn_readlane(listv, k) * EP + wb + lane];
    }
    forget(listv);
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const float v = column_value<NCH, FIRST>(q, __builtin_amdgcn_readlane(listv, k), FIRST ? 0.0f : cell[k], wb, E, lane);
      col[k * 64 + lane] = v;
      const int b = __float_as_int(v), before = __builtin_amdgcn_update_dpp(b, b, 0x138, 0xf, 0xf, false);   // wave_shr:1
      steps |= __builtin_amdgcn_ballot_w64(b != before && lane < n_in);
      const unsigned long long fin = __builtin_amdgcn_ballot_w64(v < INFINITY);
      const int f = fin ? __builtin_ctzll(fin) : 63;
      estar = f < estar ? f : estar;
      by_fours(k);
    }
  }
  forget(listv);
  wave_sync();
  const bool few = __builtin_popcountll(steps) <= kRuns<KB>;
#pragma unroll 1
  for (int oc = NCH == 1 ? 0 : part; 64 * oc < S; oc += NCH == 1 ? 1 : parts) {
    const bool valid = 64 * oc + lane < S && (NCH > 1 || (lane & (parts - 1)) == part);
    if (few) {
      runs_of_rows<KB, NCH == 1, ARG>(t, inst, row, l, wb, n_in, lane, K, listv, steps, col, rt, 64 * oc, valid,
                                        NCH == 1 || 64 * (oc + parts) >= S);
      continue;
    }
    rows<KB, NCH == 1, ARG>(t, inst, row, l, wb, n_in, lane, K, listv, lane, estar, col, rt, 64 * oc, valid);
  }
}

// One group with at most KEEP candidates that are not all constant, by one wave; false if there
// are more.  parts: 1, 2 or 4 waves share the group, this one is `part` and computes every parts-th
// output (chunk of outputs beyond 64 strategies).  q: the columns' words.  col: KEEP columns of 64 budgets; rt: the layer's R (up to 64 strategies).
template <int NCH, int KEEP, bool FIRST, bool ARG>
__device__ __forceinline__ bool dense_group(const Tables& t, int inst, int row, int l, int wb, int lane, int part,
                                            int parts, const Columns<NCH>& q, float* __restrict__ col,
                                            const float* __restrict__ rt) {
  const int S = t.S, E = t.E;
  const int el = wb + 63 < E ? wb + 63 : E;
  const float* __restrict__ Rrow = t.Rn + (size_t)row * S * S;
  float ub[NCH], lb[NCH];
  unsigned long long cand[NCH];
  bool varies;
  bounds<NCH>(q, wb, el, ub, lb, cand, varies);
  int K = 0;
#pragma unroll
  for (int c = 0; c < NCH; ++c) K += __builtin_popcountll(cand[c]);
  if (K > KEEP) {
    // The same bound per output strategy instead of over all of them: a candidate stays if it can
    // be minimal for some output (two more reads of its row of R; 23 -> 11 candidates on the
    // structured workloads, where the costs differ by less than R does).
    float tub[NCH];
#pragma unroll
    for (int oc = 0; oc < NCH; ++oc) tub[oc] = INFINITY;
    constexpr int NB = NCH == 1 ? 8 : 4;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        unsigned long long mask = cand[c], keep = 0;
        while (mask) {
          int k[NB];
          float r[NB][NCH];
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            k[i] = mask ? __builtin_ctzll(mask) : k[i > 0 ? i - 1 : 0];
            mask &= mask - 1;
#pragma unroll
            for (int oc = 0; oc < NCH; ++oc) {
              const int s = 64 * oc + lane;
              r[i][oc] = s < S ? r_of<NCH == 1>(rt, Rrow, S, 64 * c + k[i], s) : INFINITY;
            }
          }
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            bool live = false;
#pragma unroll
            for (int oc = 0; oc < NCH; ++oc) {
              if (pass == 0) {
                tub[oc] = __builtin_fminf(tub[oc], lane_f(ub[c], k[i]) + r[i][oc]);
              } else {
                const float x = lane_f(lb[c], k[i]) + r[i][oc];
                live = live || (64 * oc + lane < S && x <= tub[oc]);
              }
            }
            if (pass == 1 && __builtin_amdgcn_ballot_w64(live) != 0) keep |= 1ull << k[i];
          }
        }
        if (pass == 1) cand[c] = keep;
      }
    K = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) K += __builtin_popcountll(cand[c]);
    if (K > KEEP) return false;
    // emptied only by entries of R that no comparison holds for (NaN: the solve is refused once it has
    // run): any one column will do
    if (K == 0) cand[0] = 1;
    K = K > 0 ? K : 1;
  }

  // sized to the candidates: the unrolled loops run for all of their slots
  if (KEEP > 8 && K <= 8) dense_cells<NCH, 8, FIRST, ARG>(t, inst, row, l, wb, lane, part, parts, q, cand, K, col, rt);
  else dense_cells<NCH, KEEP, FIRST, ARG>(t, inst, row, l, wb, lane, part, parts, q, cand, K, col, rt);
  return true;
}

// One group with any number of candidates, by the whole workgroup: the waves fetch a quarter of
// the columns each and then compute a quarter of the outputs each.  These are mostly the groups in
// which the first plans start to fit: their columns are +inf at the first budget, so that the
// summaries bound nothing from above.  The loaded columns do, from the first feasible budget on
// (176 -> 20 candidates on the cost-model workloads).  col: [S][64] floats; list: 256 words.
template <int NCH, int KEEP, bool FIRST, bool ARG>
__device__ __forceinline__ void big_group(const Tables& t, int inst, int row, int l, int wb, int wave, int lane,
                                          float* __restrict__ col, const float* __restrict__ rt,
                                          uint16_t* __restrict__ list, int* __restrict__ es) {
  constexpr bool STAGED = NCH == 1;
  const int S = t.S, E = t.E, EP = t.EP, G = EP >> 6;
  const int el = wb + 63 < E ? wb + 63 : E, n_in = el - wb + 1;
  const float* __restrict__ Rrow = t.Rn + (size_t)row * S * S;
  const float* __restrict__ Cp = FIRST ? nullptr : c_table(t, inst, row - 1, l - 1);
  Columns<NCH> q;
  load_columns<NCH, FIRST>(t, inst, row, l, wb, el, lane, q);
  float ub[NCH], lb[NCH];
  unsigned long long cand[NCH];
  bool varies;
  bounds<NCH>(q, wb, el, ub, lb, cand, varies);
  int K = 0;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {                        // every wave writes the same list
    const unsigned long long below = cand[c] & ((1ull << lane) - 1);
    if ((cand[c] >> lane) & 1) list[K + __builtin_popcountll(below)] = (uint16_t)(64 * c + lane);
    K += __builtin_popcountll(cand[c]);
  }
  __syncthreads();
  int estar = 63;
  constexpr int NB = 8;
#pragma unroll 1
  for (int k0 = wave; k0 < K; k0 += kWaves * NB) {
    int sp[NB];
    float cell[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int k = k0 + kWaves * i < K ? k0 + kWaves * i : k0;
      sp[i] = __builtin_amdgcn_readfirstlane((int)list[k]);
      cell[i] = FIRST ? 0.0f : Cp[(size_t)sp[i] * EP + wb + lane];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int k = k0 + kWaves * i < K ? k0 + kWaves * i : k0;
      const float v = column_value<NCH, FIRST>(q, sp[i], cell[i], wb, E, lane);
      col[k * 64 + lane] = v;
      const unsigned long long fin = __builtin_amdgcn_ballot_w64(v < INFINITY);
      const int f = fin ? __builtin_ctzll(fin) : 63;
      estar = f < estar ? f : estar;
    }
  }
  if (lane == 0) es[wave] = estar;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) estar = es[w] < estar ? es[w] : estar;
  estar = __builtin_amdgcn_readfirstlane(estar);

  // The bounds once more, from the loaded values and for every eight budgets by themselves (the
  // tables fall steeply where plans start to fit); a lane per candidate, every wave the same.
  int sk[NCH];                                           // strategy | place of its column << 8
  float last[NCH], lowest[NCH], highest[NCH];
  bool in[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int k = 64 * c + lane;
    sk[c] = k < K ? (int)list[k] | k << 8 : 0;
    const float4 info = t.Row[(size_t)row * S + (sk[c] & 255)];
    lowest[c] = info.x;
    highest[c] = info.y;
    in[c] = false;
  }
#pragma unroll 1
  for (int e = estar & ~7; e < n_in; e += 8) {
    const int from = e > estar ? e : estar, to = e + 7 < n_in ? e + 7 : n_in - 1;
    float u = INFINITY;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if (64 * c + lane < K) u = __builtin_fminf(u, col[(64 * c + lane) * 64 + from] + highest[c]);
    u = wave_min(u);
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if (64 * c + lane < K) {
        const float v = col[(64 * c + lane) * 64 + to];
        in[c] = in[c] || (v < INFINITY && v + lowest[c] <= u);
      }
  }
  __syncthreads();                                       // the list is read by now
  int K2 = 0;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const unsigned long long b = __builtin_amdgcn_ballot_w64(in[c]);
    if (in[c]) list[K2 + __builtin_popcountll(b & ((1ull << lane) - 1))] = (uint16_t)sk[c];
    K2 += __builtin_popcountll(b);
  }
  // A column's words may speak for budgets beyond this group.  If no column is finite inside it after all, the
  // list is as it was and its first one (+inf throughout) stands for them.
  K2 = K2 > 0 ? K2 : 1;
  __syncthreads();
  const int per = (S + kWaves - 1) / kWaves;             // at most 64
  const int sfirst = wave * per;
  const bool valid = lane < per && sfirst + lane < S;
  if (K2 <= KEEP) {
    const int v = (int)list[lane < K2 ? lane : K2 - 1];
    rows<KEEP, STAGED, ARG>(t, inst, row, l, wb, n_in, lane, K2, v & 255, v >> 8, estar, col, rt, sfirst, valid);
  } else {
    const int s = valid ? sfirst + lane : 0;
    const float4 info = t.Row[(size_t)row * S + s];
    const float cs = info.z;
    float tf = INFINITY, tl = INFINITY;
#pragma unroll 1
    for (int k0 = 0; k0 < K2; k0 += NB) {
      float r[NB];
      int v[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        v[i] = __builtin_amdgcn_readfirstlane((int)list[k0 + i < K2 ? k0 + i : K2 - 1]);
        r[i] = r_of<STAGED>(rt, Rrow, S, v[i] & 255, s);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        tf = __builtin_fminf(tf, col[(v[i] >> 8) * 64 + estar] + r[i]);
        tl = __builtin_fminf(tl, col[(v[i] >> 8) * 64 + n_in - 1] + r[i]);
      }
    }
    float2 words;
    const bool same = words_of((estar == 0 ? tf : INFINITY) + cs, tl + cs, words);
    const unsigned long long flat = __builtin_amdgcn_ballot_w64(same);
    if (valid) sum_table(t, inst, row, l)[(size_t)s * G + (wb >> 6)] = words;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int k = 64 * c + lane;
      sk[c] = k < K2 ? (int)list[k] : 0;
      last[c] = k < K2 ? col[(sk[c] >> 8) * 64 + n_in - 1] : INFINITY;
    }
    const RowStores out(c_table(t, inst, row, l), EP, E, s, wb, clamp_m(__float_as_int(info.w), E));
    uint8_t* __restrict__ An = ARG ? t.A + (size_t)row * S * EP : nullptr;
    int rec = 0;
    unsigned long long todo = __builtin_amdgcn_ballot_w64(valid && tl < INFINITY && (ARG || !same));
    constexpr int NR = 4;                                // rows whose entries of R are in flight
    while (todo) {
      int j[NR];
      float r[NR][NCH];
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        j[i] = todo ? __builtin_ctzll(todo) : -1;
        todo &= todo - 1;
        const int so = sfirst + (j[i] >= 0 ? j[i] : 0);
#pragma unroll
        for (int c = 0; c < NCH; ++c)
          r[i][c] = 64 * c + lane < K2 ? r_of<STAGED>(rt, Rrow, S, sk[c] & 255, so) : INFINITY;
      }
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        if (j[i] < 0) break;
        const float limit = lane_f(tf, j[i]);
        float best = INFINITY;
        int a = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          unsigned long long lv = __builtin_amdgcn_ballot_w64(64 * c + lane < K2 && last[c] + r[i][c] <= limit);
          while (lv) {
            int k[4], v[4];
            float x[4];
#pragma unroll
            for (int y = 0; y < 4; ++y) {
              k[y] = lv ? __builtin_ctzll(lv) : k[y > 0 ? y - 1 : 0];
              lv &= lv - 1;
              v[y] = __builtin_amdgcn_readlane(sk[c], k[y]);
              x[y] = col[(v[y] >> 8) * 64 + lane];
            }
#pragma unroll
            for (int y = 0; y < 4; ++y) {
              const float z = x[y] + lane_f(r[i][c], k[y]);
              if (z < best) { best = z; a = v[y] & 255; }
            }
          }
        }
        if (!((flat >> j[i]) & 1)) out.store(j[i], lane, E, best + lane_f(cs, j[i]));
        if (ARG) {
          const int g = store_records(An, EP, sfirst + j[i], wb, n_in, lane, a);
          rec = lane == j[i] ? g : rec;
        }
      }
    }
    if (ARG && valid) group_records(t, row)[(size_t)s * G + (wb >> 6)] = (uint8_t)rec;
  }
  __syncthreads();                                       // the columns are overwritten by the next group
}

// Measurement only: which groups of the unit read one and the same column of the previous table
// at all their budgets.  counts[0] / [3]: whole units of 256 budgets and the groups inside the
// table that they cover; [1]: other such groups.  ([2]: see pruned_step.)
template <bool FIRST>
__device__ __forceinline__ void count_runs(const Tables& t, int inst, int row, int l, int base, int lane) {
  const int S = t.S, E = t.E;
  const float* __restrict__ Cp = FIRST ? nullptr : c_table(t, inst, row - 1, l - 1);
  const float2* __restrict__ Tp = FIRST ? nullptr : sum_table(t, inst, row - 1, l - 1);
  const int* __restrict__ Mp = t.M + (size_t)(row - 1) * S;
  auto value = [&](int s, int e) {
    if (FIRST) return e >= clamp_m(Mp[s], E) ? t.c[(size_t)(row - 1) * S + s] : INFINITY;
    return table_cell(t, Cp, Tp, Mp, s, e);
  };
  int inside = 0, runs = 0;
  bool whole = true;
  for (int g = 0; g < kUnit; ++g) {
    const int wb = base + 64 * g;
    if (wb > E) break;
    ++inside;
    bool run = true;
    for (int s = 0; s < S; ++s) {
      const int e = wb + lane;
      const int v = __float_as_int(value(s, e <= E ? e : E));
      run = run && __builtin_amdgcn_ballot_w64(v != __builtin_amdgcn_readfirstlane(v)) == 0;
      whole = whole && v == __float_as_int(value(s, base));
    }
    runs += run ? 1 : 0;
    whole = __builtin_amdgcn_ballot_w64(!whole) == 0;
  }
  if (lane != 0 || inside == 0) return;
  if (whole) {
    atomicAdd(t.counts, 1ull);
    atomicAdd(t.counts + 3, (unsigned long long)inside);
  } else {
    atomicAdd(t.counts + 1, (unsigned long long)runs);
  }
}

// Columns of 64 floats of LDS that a wave has: its candidates, or the values of 16 steps.
__host__ __device__ constexpr int wave_columns(int keep) { return keep > 16 ? keep : 16; }
// LDS of a workgroup of the pruned step, in floats: the layer's R (up to 64 strategies), then the
// columns.
__host__ __device__ inline int pruned_lds_head(int S) { return S <= 64 ? (S * S + 63) / 64 * 64 : 0; }
__host__ __device__ inline int pruned_lds_floats(int S, int keep) {
  const int own = kWaves * wave_columns(keep) * 64, shared = S > keep ? S * 64 : 0;
  return pruned_lds_head(S) + (own > shared ? own : shared);
}

// The layer step of one workgroup: four waves, `unit` groups of 64 budgets each.  The waves' units
// lie a quarter of the budget axis apart: the groups that are not constant cluster (at the low
// budgets on the structured workloads), and the workgroup's waves share them.  unit == 0: small
// launches, where the time of one group counts: the four waves share one group from the start.
// who: the instance and its first table row.
template <int NCH, int KEEP, bool FIRST, bool ARG, bool COUNT>
__device__ __forceinline__ void pruned_step(const Tables& t, int l, int2 who, int place, int places, int unit,
                                            float* __restrict__ lds) {
  constexpr bool MAY_BE_BIG = NCH > 1 || COUNT || KEEP >= 16;   // else never more candidates than strategies
  __shared__ int x_n[2], x_group[kWaves * kUnit], x_big[kWaves * kUnit], x_es[kWaves];
  __shared__ uint16_t x_list[256];
  const int S = t.S, E = t.E, EP = t.EP, G = EP >> 6;
  const int inst = who.x, row = who.y + l;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool split = unit == 0;
  const int base = split ? place * 64 : (place + wave * places) * unit * 64;
  const bool present = base <= E;
  const bool share = !split && (NCH > 1 || unit > 1);    // else the wave that finds a group computes it
  const int groups = split ? 1 : unit;
  int mine = -1;                                         // the last group of this wave that is not constant
  if (threadIdx.x < 2) x_n[threadIdx.x] = 0;
  const float* __restrict__ Rrow = t.Rn + (size_t)row * S * S;
  float* __restrict__ rt = lds;                          // NCH == 1: [S][S]
  float* __restrict__ cols = lds + pruned_lds_head(S);
  // R, M and the summaries (whose place depends on M) are all asked for before anything is waited for
  constexpr int NSTG = NCH == 1 ? 16 : 1;                // 64 x 64 floats / 256 threads
  float stg[NSTG];
  if (NCH == 1) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i) {
      const int at = threadIdx.x + i * 64 * kWaves;
      if (i * 64 * kWaves < S * S) stg[i] = at < S * S ? Rrow[at] : 0.0f;
    }
  }
  Columns<NCH> q;
  float2 w[NCH][kUnit + 1];
  float cs[NCH];
  if (present) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int s = 64 * c + lane;
      const float4 info = s < S ? t.Row[(size_t)row * S + s] : make_float4(0.0f, 0.0f, INFINITY, 0.0f);
      q.rl[c] = make_float2(info.x, info.y);
      cs[c] = info.z;
    }
    if (FIRST) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int s = 64 * c + lane;
        q.m[c] = s < S ? clamp_m(t.M[(size_t)(row - 1) * S + s], E) : 0;
        const float cv = s < S ? t.c[(size_t)(row - 1) * S + s] : INFINITY;
#pragma unroll
        for (int g = 0; g <= kUnit; ++g) w[c][g] = make_float2(cv, cv);
      }
    } else {
      load_unit<NCH>(t, sum_table(t, inst, row - 1, l - 1), t.M + (size_t)(row - 1) * S, base, groups, lane, q.m, w);
    }
  }
  if (NCH == 1) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i) {
      const int at = threadIdx.x + i * 64 * kWaves;
      if (i * 64 * kWaves < S * S && at < S * S) rt[at] = stg[i];
    }
  }
  __syncthreads();
  if (present) {
    if (COUNT) count_runs<FIRST>(t, inst, row, l, base, lane);
    float2* __restrict__ Tn = sum_table(t, inst, row, l);
    uint8_t* __restrict__ Ag = ARG ? group_records(t, row) : nullptr;
    float best[NCH], val[NCH];
    int arg[NCH];
    unsigned long long have[NCH];
    bool any = false;
#pragma unroll
    for (int c = 0; c < NCH; ++c) { best[c] = val[c] = INFINITY; arg[c] = 0; have[c] = 0; }
#pragma unroll 1
    for (int g = 0; g < groups; ++g) {
      const int wb = base + 64 * g;
      if (wb > E) break;
      const int el = wb + 63 < E ? wb + 63 : E;
#pragma unroll
      for (int c = 0; c < NCH; ++c) { q.a[c] = w[c][0]; q.b[c] = w[c][1]; }
      float ub[NCH], lb[NCH];
      unsigned long long cand[NCH];
      bool varies;
      bounds<NCH>(q, wb, el, ub, lb, cand, varies);
      if (COUNT) {                                       // measurement only: the sums that the bounds leave
        int left = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) left += __builtin_popcountll(cand[c]);
        if (lane == 0) atomicAdd(t.counts + 2, (unsigned long long)left * S * (varies ? el - wb + 1 : 1));
      }
      if (varies) {
        mine = wb;
        if (share && lane == 0) x_group[atomicAdd(&x_n[0], 1)] = wb;
      } else {
        // the groups of a unit mostly carry the same column: its outputs are computed once
        bool again = !any;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
          again = again || cand[c] != have[c] ||
                  __builtin_amdgcn_ballot_w64(((cand[c] >> lane) & 1) && __float_as_int(ub[c]) != __float_as_int(val[c])) != 0;
        if (again) {
          uniform_outputs<NCH>(rt, Rrow, S, lane, ub, cand, best, arg);
#pragma unroll
          for (int c = 0; c < NCH; ++c) { have[c] = cand[c]; val[c] = ub[c]; }
          any = true;
        }
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const int s = 64 * c + lane;
          const float out = best[c] + cs[c];
          if (s < S && !(split && wave != 0)) {
            Tn[(size_t)s * G + (wb >> 6)] = make_float2(out, out);
            if (ARG) Ag[(size_t)s * G + (wb >> 6)] = (uint8_t)arg[c];
          }
        }
      }
#pragma unroll
      for (int c = 0; c < NCH; ++c)                      // the next group's words
#pragma unroll
        for (int x = 0; x < kUnit; ++x) w[c][x] = w[c][x + 1];
    }
  }
  // one or two groups: four or two waves share each, and divide its outputs
  int n = mine >= 0 ? 1 : 0, at = 0, step = 1, parts = split ? kWaves : 1;
  if (share) {
    __syncthreads();
    n = x_n[0];
    parts = n == 1 ? 4 : n == 2 ? 2 : 1;
    at = wave / parts;
    step = kWaves / parts;
  }
#pragma unroll 1
  for (; at < n; at += step) {
    if (share) {
      mine = __builtin_amdgcn_readfirstlane(x_group[at]);
      load_columns<NCH, FIRST>(t, inst, row, l, mine, mine + 63 < E ? mine + 63 : E, lane, q);
    }
    if (!dense_group<NCH, KEEP, FIRST, ARG>(t, inst, row, l, mine, lane, wave & (parts - 1), parts, q,
                                            cols + wave * wave_columns(KEEP) * 64, rt) && lane == 0 && (wave & (parts - 1)) == 0)
      x_big[atomicAdd(&x_n[1], 1)] = mine;
  }
  if (!MAY_BE_BIG || (NCH == 1 && S <= KEEP)) return;
  __syncthreads();
  const int nbig = x_n[1];
  for (int i = 0; i < nbig; ++i)
    big_group<NCH, KEEP, FIRST, ARG>(t, inst, row, l, __builtin_amdgcn_readfirstlane(x_big[i]), wave, lane, cols, rt, x_list,
                                     x_es);
}

}  // namespace gbmw

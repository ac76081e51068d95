// gfx950 kernels of the batched layer-wise strategy search (Section 4.1.2,
// Eq. 3; Appendix A, Algorithm 3 of the paper).  See gbmw_kernels.h for the
// device layout.  (min,+) is not a multiply-accumulate, so the matrix cores
// are not used: the work is fp32 VALU adds and mins with wave-uniform R
// operands, streamed along the budget axis.
#include "gbmw_kernels.h"
#include "gbmw_pruned.h"

#include <math.h>

namespace gbmw {

#define GBMW_AS4 __attribute__((address_space(4)))
typedef const GBMW_AS4 float* cf32_t;   // uniform, read-only -> scalar loads
typedef const GBMW_AS4 int* ci32_t;

template <typename T>
__device__ __forceinline__ const GBMW_AS4 T* as_const(const T* p) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
  return (const GBMW_AS4 T*)(p);
#pragma clang diagnostic pop
}

// ---------------------------------------------------------------------------
// prepare: Rt[row][s][0..SP) = R[row][.][s] (zero padding), Rt[row][s][SP] = c,
// Rt[row][s][SP+1] = bits of M; + input validation.  c and M are read from the caller's
// arrays (src_c, src_M) and, where those are not the context's own (device-resident inputs),
// copied into the context's (t.c, t.M), which is what every later kernel and every later call
// reads: the caller's arrays are not touched again once this kernel has run.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_prepare(Tables t, const float* __restrict__ R, int sumL,
                                                 int validate, float* __restrict__ Rt,
                                                 const float* __restrict__ src_c,
                                                 const int* __restrict__ src_M) {
  const int SP = t.SP, S = t.S, RS = t.RS;
  const size_t n = (size_t)sumL * S * RS;
  const bool copy = src_c != t.c;
  int bad = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const int sp = (int)(i % RS);
    const int s = (int)((i / RS) % S);
    const size_t row = i / ((size_t)RS * S);
    float v = 0.0f;
    if (sp < S) {
      v = R[(row * S + sp) * S + s];
    } else if (sp == SP) {
      v = src_c[row * S + s];
      if (validate && !(v >= 0.0f)) bad |= 1;
      if (copy) const_cast<float*>(t.c)[row * S + s] = v;
    } else if (sp == SP + 1) {
      const int m = src_M[row * S + s];
      if (validate && m < 0) bad |= 2;
      if (copy) const_cast<int*>(t.M)[row * S + s] = m;
      v = __int_as_float(m);
    }
    Rt[i] = v;
  }
  if (validate && bad) atomicOr(t.status, bad);
}

// The same for the pruned layer step (t.runs != 0): R is kept as it comes, a row s' of a layer being
// the S costs of leaving s' (what the step's lanes, one per output strategy, read), and every row
// leaves its smallest and largest entry beside c and M (t.Row).  The l == 0 slab of R is ignored by contract and
// may hold anything: it is neither read nor checked.  One wave per row, four rows in flight.
__global__ __launch_bounds__(256) void k_prepare_runs(Tables t, const float* __restrict__ R, int validate,
                                                      float* __restrict__ Rn, float4* __restrict__ Row,
                                                      const float* __restrict__ src_c, const int* __restrict__ src_M) {
  const int l = blockIdx.x, inst = blockIdx.y, S = t.S;
  if (l >= t.L[inst]) return;
  const size_t row = (size_t)t.off[inst] + l;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int bad = 0;
  if (blockIdx.z == 0 && (int)threadIdx.x < S) {   // S < 256
    const size_t i = row * S + threadIdx.x;
    const float v = src_c[i];
    const int m = src_M[i];
    if (!(v >= 0.0f)) bad |= 1;
    if (m < 0) bad |= 2;
    if (src_c != t.c) {
      const_cast<float*>(t.c)[i] = v;
      const_cast<int*>(t.M)[i] = m;
    }
  }
  if (l > 0) {
    const int s0 = ((int)blockIdx.z * 4 + wave) * 4;
    if (s0 < S && !row_limits<4>(R + row * S * S, S, s0, lane, src_c + row * S, src_M + row * S, Rn + row * S * S,
                                   Row + row * S))
      bad |= 4;
  }
  if (validate && bad) atomicOr(t.status, bad);
}

// R is validated per instance because the l == 0 slab is ignored by contract
// and may hold anything.
__global__ __launch_bounds__(256) void k_validate_R(Tables t, const float* __restrict__ R) {
  const int inst = blockIdx.y;
  const int S = t.S;
  const int Lb = t.L[inst];
  const size_t base = ((size_t)t.off[inst] + 1) * S * S;   // skip layer 0
  const size_t n = (size_t)(Lb - 1) * S * S;
  int bad = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    if (!(R[base + i] >= 0.0f)) bad = 4;
  if (bad) atomicOr(t.status, bad);
}

__global__ void k_clear_status(int* status) { *status = 0; }

__global__ void k_clear_counts(unsigned long long* counts, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) counts[i] = 0;
}

void launch_clear_counts(unsigned long long* counts, int n, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(k_clear_counts, dim3((n + 255) / 256), dim3(256), 0, st, counts, n);
}

void launch_prepare(const Tables& t, const float* R, const float* src_c, const int* src_M, int sumL,
                    int Lmax, bool validate, hipStream_t st) {
  // a fill kernel rather than a memset node, so that the sequence can be captured
  hipLaunchKernelGGL(k_clear_status, dim3(1), dim3(1), 0, st, t.status);
  if (t.runs != 0) {
    hipLaunchKernelGGL(k_prepare_runs, dim3(Lmax, t.B, (t.S + 15) / 16), dim3(256), 0, st, t, R, validate ? 1 : 0,
                       const_cast<float*>(t.Rn), const_cast<float4*>(t.Row), src_c, src_M);
    return;
  }
  const size_t n = (size_t)sumL * t.S * t.RS;
  int blocks = (int)((n + 255) / 256);
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_prepare, dim3(blocks), dim3(256), 0, st, t, R, sumL, validate ? 1 : 0,
                     const_cast<float*>(t.Rt), src_c, src_M);
  if (validate) hipLaunchKernelGGL(k_validate_R, dim3(64, t.B), dim3(256), 0, st, t, R);
}

// ---------------------------------------------------------------------------
// layer 0:  C(0, e, s) = e >= M(0, s) ? c(0, s) : +inf
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init_layer0(Tables t, int first) {
  const int inst = t.perm[first + blockIdx.z].x, s = blockIdx.y;
  const int e = (blockIdx.x * 256 + threadIdx.x) * 4;     // EP is a multiple of 256: whole float4s
  if (e >= t.EP) return;
  const int row = t.off[inst];
  const int m = t.M[(size_t)row * t.S + s];
  const float cs = t.c[(size_t)row * t.S + s];
  float* C0 = c_table(t, inst, row, 0);
  float4 v;                                                // padding rows: +inf
  v.x = (m >= 0 && e >= m && e <= t.E) ? cs : INFINITY;
  v.y = (m >= 0 && e + 1 >= m && e + 1 <= t.E) ? cs : INFINITY;
  v.z = (m >= 0 && e + 2 >= m && e + 2 <= t.E) ? cs : INFINITY;
  v.w = (m >= 0 && e + 3 >= m && e + 3 <= t.E) ? cs : INFINITY;
  *reinterpret_cast<float4*>(C0 + (size_t)s * t.EP + e) = v;
  // T + c of layer 0 is c(0, s) at every budget: the same summary for every group of 64
  if (t.runs != 0 && (e & 63) == 0 && e <= t.E)
    sum_table(t, inst, row, 0)[(size_t)s * (t.EP >> 6) + (e >> 6)] = make_float2(cs, cs);
}

void launch_init_layer0(const Tables& t, int first, int count, hipStream_t st) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_init_layer0, dim3((t.EP + 1023) / 1024, t.S, count), dim3(256), 0, st, t, first);
}

// ---------------------------------------------------------------------------
// min-plus + argmin + shift-add, register-blocked.
//   wave: 64*K consecutive budgets e' of one instance; lane owns e' = e0 + 64*j.
//   The SP values C_{l-1}[e'][0..SP) of each owned e' stay in VGPRs for the
//   whole kernel.  The layer's R tile (with c and M riding in each row) is
//   staged once per workgroup in LDS; every output strategy s reads its row
//   with wave-uniform 128-bit LDS reads (broadcast, conflict-free, returned in
//   order so the reads pipeline ahead of the adds).
//
//   Value pass: the SP candidates x = C + R are folded into chunk minima of CH
//   candidates (3-input min), and the chunk minima into a running prefix
//   minimum P[k] = min(P[k-1], chunk 2k-1, chunk 2k); T is the last prefix.
//   One add and half a min per candidate, no compare in the chain.  The R row is
//   consumed quad by quad as it arrives and only the prefix minima stay live.
//   Argmin: P[k] == T is monotone in k, so the lowest-index minimiser lies in
//   the first block k whose prefix equals T.  The block tests are independent
//   compares into wave masks; a block is re-scanned only when some lane of
//   the wave first hits it, which for neighbouring budgets is usually one; the
//   re-scan redoes the block's sums from the LDS row (same operands, same bits,
//   so equality with T is exact).
//   ARG = false leaves the argmin out altogether (values-only fill).
// ---------------------------------------------------------------------------
// Word 3 of a gfx9-family raw buffer descriptor: 32-bit data format, no swizzle.
constexpr int kBufWord3 = 0x00020000;
// Cache policy of a buffer store: non-temporal.  The argmin records of an unsplit launch are
// written once and not read again before the solve ends, and the previous table is read once
// (streaming loads): keeping both out of the way leaves the L2 to the fp32 stores, whose
// shifted rows meet their neighbours' in shared cache lines and are merged there (the same
// hint on those stores costs 20 %: the halves of a line are then written back separately).
constexpr int kStreaming = 2;

__device__ __forceinline__ float fmin3(float a, float b, float c) {
  return __builtin_fminf(__builtin_fminf(a, b), c);
}

// How a launch's workgroups map to (instance, tile): the divisors of that mapping come with
// floor(2^32 / d) from the host, so that a workgroup finds its place with a multiply, a
// subtract and one correction per division (the quotient estimate is never more than one
// short) instead of the thirty-instruction sequence of a division by a run-time value: every
// wave pays for them before it can ask for its first byte.
struct Deal {
  int n;                                                 // instances in the launch
  unsigned inv_tiles, inv_n;                             // of the tiles of an instance, and of n
  int unit;                                              // pruned step: groups of 64 budgets per wave
};

__device__ __forceinline__ void divmod(unsigned p, unsigned d, unsigned inv, int& q, int& r) {
  unsigned qq = __umulhi(p, inv), rr = p - qq * d;
  if (rr >= d) { ++qq; rr -= d; }
  q = (int)qq; r = (int)rr;
}

static unsigned inv_of(unsigned d) { return d <= 1 ? 0xffffffffu : (unsigned)((1ull << 32) / d); }

static Deal make_deal(int tiles, int n, int unit = 1) {
  return Deal{n, inv_of((unsigned)tiles), inv_of((unsigned)n), unit};
}

// RUNS: the pruned step (gbmw_pruned.h) instead of the dense arithmetic.
// COUNT: the same with counts of the groups that read one column (t.counts), for measurements.
template <int SP, int K, int NW, int CH, int MINW, bool FIRST, bool ARG, bool SPLIT, bool RUNS, bool COUNT = false>
__global__ __launch_bounds__(64 * NW, MINW) void k_minplus(Tables t, int l, int tiles, int first, Deal deal) {
  constexpr bool split = SPLIT;
  static_assert(!(SPLIT && RUNS), "the pruned step has no split mode");
  static_assert(RUNS || !COUNT, "only the run paths are counted");
  extern __shared__ float4 rt_lds[];                     // [S][RQ], or the pruned step's columns
  if constexpr (RUNS) {
    // all instances' low budgets first: the groups that are not constant lie there, and they take
    // the longest
    int place, slot;
    divmod(blockIdx.x, (unsigned)deal.n, deal.inv_n, place, slot);
    pruned_step<1, (COUNT ? 4 : kept(SP)), FIRST, ARG, COUNT>(t, l, t.perm[first + slot], place, tiles, deal.unit,
                                                                 reinterpret_cast<float*>(rt_lds));
  } else {
  constexpr int NC = (SP + CH - 1) / CH;                 // chunks (last may be short)
  constexpr int NP = NC / 2 + 1;                         // prefix minima / blocks
  constexpr int RS = (SP + 2 + 3) / 4 * 4;               // row: SP x R, c, M, padding
  constexpr int RQ = RS / 4;
  int slot, tile;
  divmod(blockIdx.x, (unsigned)tiles, deal.inv_tiles, slot, tile);
  const int inst = t.perm[first + slot].x;
  const int S = t.S, E = t.E, EP = t.EP;
  const int row = t.off[inst] + l;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, scalar
  const int lane = threadIdx.x & 63;
  // Normal mode: the workgroup's waves take consecutive row tiles and every
  // output strategy.  Split mode (small problems, too few workgroups to fill the
  // chip): the waves share one row tile and divide the output strategies, which
  // shortens the serial chain per wave NW-fold at the price of loading the tile
  // NW times (from L2).
  const int wbase = (split ? tile : tile * NW + wave) * (64 * K);
  const bool present = wbase <= E;                       // else: whole wave beyond the table

  {
    const float4* __restrict__ src = reinterpret_cast<const float4*>(t.Rt + (size_t)row * S * RS);
    constexpr int NSTG = (SP * RQ + 64 * NW - 1) / (64 * NW);
    float4 stg[NSTG];
#pragma unroll
    for (int k = 0; k < NSTG; ++k) {
      const int i = threadIdx.x + k * 64 * NW;
      stg[k] = (i < S * RQ) ? src[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
#pragma unroll
    for (int k = 0; k < NSTG; ++k) {
      const int i = threadIdx.x + k * 64 * NW;
      if (i < S * RQ) rt_lds[i] = stg[k];
    }
  }
  __syncthreads();
  if (!present) return;
  const int s_begin = split ? (wave * S) / NW : 0;
  const int s_end = split ? ((wave + 1) * S) / NW : S;
  const float* __restrict__ Cp = c_table(t, inst, row - 1, l - 1);
  float* __restrict__ Cn = c_table(t, inst, row, l);
  uint8_t* __restrict__ An = ARG ? t.A + (size_t)row * S * EP : nullptr;
  const int e0 = wbase + lane;

  // EP is a multiple of 64*K and wbase <= E < EP, so rows e0 + 64*j < EP are
  // inside the allocation; rows in (E, EP) are padding whose results are
  // never stored into the table proper.
  float cp[K][SP];
  if (FIRST) {
    // l == 1: layer 0 is a closed form, C(0, e, s') = e >= M(0, s') ? c(0, s') : +inf,
    // built here instead of being written to and read back from HBM.
    cf32_t c0 = as_const(t.c) + (size_t)(row - 1) * S;
    ci32_t m0 = as_const(t.M) + (size_t)(row - 1) * S;
#pragma unroll
    for (int sp = 0; sp < SP; ++sp) {
      const bool col = (sp < SP - 3 || sp < S);
      const float cv = col ? c0[sp] : INFINITY;
      const int mv = col ? m0[sp] : 0;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int e = e0 + 64 * j;
        cp[j][sp] = (mv >= 0 && e >= mv && e <= E) ? cv : INFINITY;
      }
    }
  } else {
#pragma unroll
    for (int sp = 0; sp < SP; ++sp) {
#pragma unroll
      for (int j = 0; j < K; ++j)
        {
        // a large launch reads every table value exactly once: streaming loads leave the
        // caches to the stores; a split launch is small enough to find its table in cache
        const float* src = &Cp[(size_t)sp * EP + e0 + 64 * j];
        cp[j][sp] = !(sp < SP - 3 || sp < S) ? INFINITY : SPLIT ? *src : __builtin_nontemporal_load(src);
      }
    }
  }

  if (!ARG) {
    // Values only: the argmin records are not materialised (the walkers recompute the
    // one record they need per layer from the kept tables).  One add and half a
    // three-input min per candidate; the R row is consumed quad by quad as it arrives.
    static_assert(K == 1 || ARG, "the values-only path handles one budget per lane");
#pragma unroll 1
    for (int s = s_begin; s < s_end; ++s) {
      float acc = INFINITY, cs = 0.0f;
      int m_raw = 0;
#pragma unroll
      for (int q = 0; q < RQ; ++q) {
        const float4 v = rt_lds[s * RQ + q];
        const float rq[4] = {v.x, v.y, v.z, v.w};
        float xq[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) xq[i] = (4 * q + i < SP) ? cp[0][(4 * q + i < SP) ? 4 * q + i : 0] + rq[i] : INFINITY;
        if (4 * q + 3 < SP) {
          acc = fmin3(acc, xq[0], xq[1]);
          acc = fmin3(acc, xq[2], xq[3]);
        }
        // SP is a multiple of 4: c(l,s) and M(l,s) sit in the quad after the last candidates
        if (4 * q == SP) {
          cs = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(rq[0])));
          m_raw = __builtin_amdgcn_readfirstlane(__float_as_int(rq[1]));
        }
      }
      const int m = (m_raw < 0 || m_raw > E + 1) ? E + 1 : m_raw;
      float* Cs = Cn + (size_t)s * EP;
      const __amdgpu_buffer_rsrc_t bc = __builtin_amdgcn_make_buffer_rsrc(Cs, 0, (E + 1) * 4, kBufWord3);
      const __amdgpu_buffer_rsrc_t binf = __builtin_amdgcn_make_buffer_rsrc(Cs, 0, m * 4, kBufWord3);
      const int outb = __float_as_int(acc + cs);
      __builtin_amdgcn_raw_buffer_store_b32((unsigned)outb, bc, (e0 + m) * 4, 0, 0);
      if (wbase < m)                                       // wave-uniform: some lane is below M
        __builtin_amdgcn_raw_buffer_store_b32(0x7f800000u, binf, e0 * 4, 0, 0);
    }
    return;
  }

  static_assert(K == 1, "one budget per lane");
#pragma unroll 1
  for (int s = s_begin; s < s_end; ++s) {
    // ---- value pass, streaming: the R row is consumed quad by quad as it arrives from LDS,
    // candidates fold into chunk minima and those into the prefix minima at once, so that
    // only the prefix minima stay live (the sums are not kept: the rescan redoes the few it
    // needs).  c(l,s) and M(l,s) sit in the quad after the last candidates (SP % 4 == 0).
    float P[NP];
    float xs[CH], cm_odd = INFINITY;
    float cs = 0.0f;
    int m_raw = 0;
#pragma unroll
    for (int q = 0; q < RQ; ++q) {
      const float4 v = rt_lds[s * RQ + q];
      const float rq[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int i = 4 * q + i4;
        if (i < SP) {
          const int c = i / CH, pos = i % CH;
          xs[pos] = cp[0][i] + rq[i4];
          const int hi = ((c + 1) * CH < SP) ? (c + 1) * CH : SP;     // end of chunk c
          if (i == hi - 1) {                                          // chunk c complete
            const int len = hi - c * CH;
            const float cmv = len == 3 ? fmin3(xs[0], xs[1], xs[2])
                              : len == 2 ? __builtin_fminf(xs[0], xs[1]) : xs[0];
            if (c == 0) P[0] = cmv;
            else if (c % 2 == 1) {
              cm_odd = cmv;
              if (c == NC - 1) P[(c + 1) / 2] = __builtin_fminf(P[(c - 1) / 2], cm_odd);
            } else {
              P[c / 2] = fmin3(P[c / 2 - 1], cm_odd, cmv);
            }
          }
        }
      }
      if (4 * q == SP) {
        cs = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(rq[0])));
        m_raw = __builtin_amdgcn_readfirstlane(__float_as_int(rq[1]));
      }
    }
    const float T = P[NP - 1];
    // invalid (negative) M: the column is infeasible; beyond E + 1 nothing changes
    const int m = (m_raw < 0 || m_raw > E + 1) ? E + 1 : m_raw;
    // Stores go through buffer descriptors of column s: the address is a scalar base
    // plus the lane's byte offset (no per-lane pointer arithmetic in the loop), and
    // the hardware range check drops what lies outside [0, num_records):
    //   bc:   rows 0..E of column s         -> the shifted store at e' + m is dropped
    //                                          beyond E without a compare
    //   binf: rows 0..m-1 of column s       -> the +inf prefix
    //   ba:   rows 0..EP-1 of column s of A (padding rows are harmless)
    float* Cs = Cn + (size_t)s * EP;
    const __amdgpu_buffer_rsrc_t bc = __builtin_amdgcn_make_buffer_rsrc(Cs, 0, (E + 1) * 4, kBufWord3);
    const __amdgpu_buffer_rsrc_t binf = __builtin_amdgcn_make_buffer_rsrc(Cs, 0, m * 4, kBufWord3);
    const __amdgpu_buffer_rsrc_t ba = __builtin_amdgcn_make_buffer_rsrc(An + (size_t)s * EP, 0, EP, kBufWord3);
    {
      constexpr int j = 0;
      // ---- argmin: first block whose prefix minimum reaches T
      int arg = 0;
      bool prev = false;
      unsigned long long prevm = 0;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const bool eq = (k == NP - 1) ? true : (P[k] == T);
        const unsigned long long eqm = (k == NP - 1) ? ~0ull : __builtin_amdgcn_ballot_w64(eq);
        if (__builtin_expect((eqm & ~prevm) != 0, 0)) {  // wave-uniform: a lane first hits block k
          if (eq && !prev) {
            const int clo = (k == 0) ? 0 : 2 * k - 1;    // chunks of block k
            const int chi = (k == 0) ? 1 : ((2 * k + 1 < NC) ? 2 * k + 1 : NC);
            const int lo = clo * CH, hi = (chi * CH < SP) ? chi * CH : SP;
            int a = hi - 1;                              // implied when no earlier one matches
            {
              // The sums are not kept: redo them from the R row (same operands, same
              // bits).  The row offset goes through an opaque register so that these
              // reads are not merged with the value pass's (which would keep the whole
              // row live), yet can be issued together.
              int roff = s * RS;
              asm volatile("" : "+v"(roff));
              const float* rl = reinterpret_cast<const float*>(rt_lds) + roff;
              float rr[2 * CH];
#pragma unroll
              for (int i = lo; i < hi - 1; ++i) rr[i - lo] = rl[i];
#pragma unroll
              for (int i = hi - 2; i >= lo; --i) a = (cp[j][i] + rr[i - lo] == T) ? i : a;
            }
            arg = a;
          }
        }
        prev = eq;
        prevm = eqm;
      }

      const int e = e0 + 64 * j;                         // pre-shift budget e'
      __builtin_amdgcn_raw_buffer_store_b8((unsigned char)arg, ba, e, 0, SPLIT ? 0 : kStreaming);
      const int outb = __float_as_int(T + cs);
      __builtin_amdgcn_raw_buffer_store_b32((unsigned)outb, bc, (e + m) * 4, 0, 0);
      if (wbase + 64 * j < m)                            // wave-uniform: some lane is below M
        __builtin_amdgcn_raw_buffer_store_b32(0x7f800000u, binf, e * 4, 0, 0);
    }
  }
  }
}

// Any S up to 256 (used above 128): the C_{l-1} tile of 64 budgets is staged in LDS as
// [S][64]; wave w handles output strategies w, w+4, ...
__global__ __launch_bounds__(256) void k_minplus_generic(Tables t, int l, int tiles, int first) {
  extern __shared__ float lds[];
  const int inst = t.perm[first + blockIdx.x / tiles].x;
  const int tile = blockIdx.x % tiles;
  const int S = t.S, RS = t.RS, E = t.E, EP = t.EP;
  const int row = t.off[inst] + l;
  const float* __restrict__ Cp = c_table(t, inst, row - 1, l - 1);
  float* __restrict__ Cn = c_table(t, inst, row, l);
  uint8_t* __restrict__ An = t.A ? t.A + (size_t)row * S * EP : nullptr;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = tile * 64 + lane;

  for (int sp = wave; sp < S; sp += 4)
    lds[sp * 64 + lane] = (e <= E) ? Cp[(size_t)sp * EP + e] : INFINITY;
  __syncthreads();

  cf32_t Rrow = as_const(t.Rt) + (size_t)row * S * RS;
  for (int s = wave; s < S; s += 4) {
    float tmin = INFINITY;
    int arg = 0;
    for (int sp = 0; sp < S; ++sp) {
      const float x = lds[sp * 64 + lane] + Rrow[s * RS + sp];
      if (x < tmin) { tmin = x; arg = sp; }
    }
    const int m = t.M[(size_t)row * S + s];
    const float cs = t.c[(size_t)row * S + s];
    if (e <= E) {
      if (An) An[(size_t)s * EP + e] = (uint8_t)arg;
      if (m >= 0 && m <= E - e) Cn[(size_t)s * EP + e + m] = tmin + cs;
      if (m < 0 || e < m) Cn[(size_t)s * EP + e] = INFINITY;
    }
  }
}

template <int SP>
struct Blocking {                       // budgets per lane for a given strategy count
  static constexpr int K = 1;
  // waves per workgroup.  Beyond 64 strategies the R tile takes 20 to 68 KB of LDS, so that one or
  // two workgroups fit a compute unit: they are made large enough to bring the waves per SIMD
  // that the registers allow (4 up to 96 strategies, 3 up to 128)
  static constexpr int NW = (SP <= 64) ? 4 : (SP <= 96) ? 8 : 12;
  static constexpr int CH = 3;          // candidates per chunk minimum
  // waves per SIMD the register allocation must allow: SP live table values plus about 20
  // working registers out of 512 (the value pass streams the R row and keeps only the
  // prefix minima; the candidate sums are not kept)
  static constexpr int MINW = (SP <= 44) ? 8 : (SP <= 56) ? 6 : (SP <= 64) ? 5 : (SP <= 96) ? 4 : 3;
  static constexpr int MINW_SPLIT = 4;
  // the layer-1 variant builds layer 0 from c and M and needs a few registers more
  static constexpr int MINW_FIRST = (SP > 40 && SP <= 44) ? 7 : MINW;
  // without the argmin pass: the SP table values plus about 16 working registers
  static constexpr int MINW_VALUES = (SP <= 44) ? 8 : (SP <= 52) ? 7 : (SP <= 60) ? 6 : (SP <= 64) ? 5 : (SP <= 96) ? 4 : 3;
  // the pruned step: up to 32 KB of LDS per workgroup leave five workgroups per compute unit
  // (the layer-1 variant needs a few registers more: at five waves per SIMD it spills two)
  static constexpr int MINW_RUNS = 5, MINW_RUNS_FIRST = 4;
};

// Groups of 64 budgets per launch from which a wave takes a group of its own instead of a fourth of one:
// where workgroups of one group would come in more than two rounds of the five (beyond 64 strategies four or
// three) that a compute unit holds.  A solve, four waves per group -> one: S=20, 2624 groups 244 -> 198 us and
// 3078 groups 234 -> 177; S=255, 2052 groups 842 -> 640; below the line S=36, 2064 groups 215 -> 227 and S=66,
// 1026 groups 177 -> 199.  (S=64 gains from 2800 on: 365 -> 383 at 2624, 324 -> 278 at 3078.)
static long long wave_groups(int S) { return S <= 64 ? 2560 : 2048; }

// The shape of a pruned launch: groups of 64 budgets per wave and workgroups per instance.
struct PrunedShape { int unit, places; size_t lds; };
static PrunedShape pruned_shape(const Tables& t, int n_active) {
  const int groups = (t.E + 64) / 64;
  PrunedShape p;
  const long long all = (long long)groups * n_active;
  p.unit = (t.counts || all >= 16384) ? kUnit : all >= wave_groups(t.S) ? 1 : 0;
  p.places = p.unit == 0 ? groups : (groups + kWaves * p.unit - 1) / (kWaves * p.unit);
  p.lds = (size_t)pruned_lds_floats(t.S, kept(t.SP)) * sizeof(float);
  return p;
}

template <int SP>
static void launch_minplus_sp(const Tables& t, int l, int first, int n_active, hipStream_t st) {
  constexpr int K = Blocking<SP>::K, NW = Blocking<SP>::NW, CH = Blocking<SP>::CH,
                MINW = Blocking<SP>::MINW;
  if (t.runs != 0) {
    static_assert(NW == kWaves, "the pruned step's workgroup");
    constexpr int MR = Blocking<SP>::MINW_RUNS, MR1 = Blocking<SP>::MINW_RUNS_FIRST;
    const PrunedShape p = pruned_shape(t, n_active);
#define GBMW_LAUNCH(MW, FIRST_, ARG_, COUNT_)                                                                  \
  hipLaunchKernelGGL((k_minplus<SP, K, NW, CH, MW, FIRST_, ARG_, false, true, COUNT_>),                        \
                     dim3((unsigned)p.places * n_active), dim3(64 * NW), p.lds, st, t, l, p.places, first,     \
                     make_deal(p.places, n_active, p.unit))
    if (t.counts) {                                      // the counting twin
      if (t.A == nullptr) { if (l == 1) GBMW_LAUNCH(2, true, false, true); else GBMW_LAUNCH(2, false, false, true); }
      else { if (l == 1) GBMW_LAUNCH(2, true, true, true); else GBMW_LAUNCH(2, false, true, true); }
    } else if (t.A == nullptr) {
      if (l == 1) GBMW_LAUNCH(MR1, true, false, false); else GBMW_LAUNCH(MR, false, false, false);
    } else {
      if (l == 1) GBMW_LAUNCH(MR1, true, true, false); else GBMW_LAUNCH(MR, false, true, false);
    }
#undef GBMW_LAUNCH
    return;
  }
  int tiles = (t.E + 1 + 64 * K * NW - 1) / (64 * K * NW);
  // fewer than two and a half workgroups per compute unit: split the strategies over the waves
  const int split = ((long long)tiles * n_active < 640) ? 1 : 0;
  if (split) tiles = (t.E + 1 + 64 * K - 1) / (64 * K);
  constexpr int RS = (SP + 2 + 3) / 4 * 4;
  const dim3 grid((unsigned)tiles * n_active), block(64 * NW);
  const size_t lds = (size_t)t.S * RS * sizeof(float);
  // Split launches are the small ones, where a wave's own latency counts and registers are
  // plentiful: a low occupancy target lets the compiler keep the whole R row in flight.
  constexpr int MS = Blocking<SP>::MINW_SPLIT;
#define GBMW_LAUNCH(MW, FIRST_, ARG_, SPLIT_)                                                               \
  hipLaunchKernelGGL((k_minplus<SP, K, NW, CH, MW, FIRST_, ARG_, SPLIT_, false>), grid, block, lds, st, t, l, \
                     tiles, first, make_deal(tiles, n_active))
  if (t.A == nullptr) {
    constexpr int MW = Blocking<SP>::MINW_VALUES;
    if (l == 1) { if (split) GBMW_LAUNCH(MS, true, false, true); else GBMW_LAUNCH(MW, true, false, false); }
    else { if (split) GBMW_LAUNCH(MS, false, false, true); else GBMW_LAUNCH(MW, false, false, false); }
  } else {
    constexpr int M1 = Blocking<SP>::MINW_FIRST;
    if (l == 1) { if (split) GBMW_LAUNCH(MS, true, true, true); else GBMW_LAUNCH(M1, true, true, false); }
    else { if (split) GBMW_LAUNCH(MS, false, true, true); else GBMW_LAUNCH(MINW, false, true, false); }
  }
#undef GBMW_LAUNCH
}

// The pruned step beyond 64 strategies: a lane holds NCH columns (and NCH outputs).
template <int NCH, bool FIRST, bool ARG, bool COUNT>
__global__ __launch_bounds__(64 * kWaves, NCH == 2 ? 4 : 3) void k_pruned_wide(Tables t, int l, int places, int first, Deal deal) {
  extern __shared__ float pruned_lds[];
  int place, slot;
  divmod(blockIdx.x, (unsigned)deal.n, deal.inv_n, place, slot);
  pruned_step<NCH, (COUNT ? 4 : kept(64 * NCH)), FIRST, ARG, COUNT>(t, l, t.perm[first + slot], place, places, deal.unit, pruned_lds);
}

template <int NCH>
static void launch_pruned_wide(const Tables& t, int l, int first, int n_active, hipStream_t st) {
  const PrunedShape p = pruned_shape(t, n_active);
#define GBMW_LAUNCH(FIRST_, ARG_, COUNT_)                                                                      \
  hipLaunchKernelGGL((k_pruned_wide<NCH, FIRST_, ARG_, COUNT_>), dim3((unsigned)p.places * n_active),          \
                     dim3(64 * kWaves), p.lds, st, t, l, p.places, first, make_deal(p.places, n_active, p.unit))
  if (t.counts) {
    if (t.A == nullptr) { if (l == 1) GBMW_LAUNCH(true, false, true); else GBMW_LAUNCH(false, false, true); }
    else { if (l == 1) GBMW_LAUNCH(true, true, true); else GBMW_LAUNCH(false, true, true); }
  } else if (t.A == nullptr) {
    if (l == 1) GBMW_LAUNCH(true, false, false); else GBMW_LAUNCH(false, false, false);
  } else {
    if (l == 1) GBMW_LAUNCH(true, true, false); else GBMW_LAUNCH(false, true, false);
  }
#undef GBMW_LAUNCH
}

// 65 to 128 strategies: the same register-blocked kernel, every lane with its S' table values
// in registers (148 to 168 of them at 128 strategies: three waves per SIMD), in larger workgroups
// (see Blocking::NW).  No split shape, layer 0 read from memory.
template <int SP>
static void launch_minplus_big(const Tables& t, int l, int first, int n_active, hipStream_t st) {
  constexpr int NW = Blocking<SP>::NW, CH = Blocking<SP>::CH;
  const int tiles = (t.E + 1 + 64 * NW - 1) / (64 * NW);
  constexpr int RS = (SP + 2 + 3) / 4 * 4;
  const dim3 grid((unsigned)tiles * n_active), block(64 * NW);
  const size_t lds = (size_t)t.S * RS * sizeof(float);
  if (t.A == nullptr)
    hipLaunchKernelGGL((k_minplus<SP, 1, NW, CH, Blocking<SP>::MINW_VALUES, false, false, false, false>), grid, block, lds,
                       st, t, l, tiles, first, make_deal(tiles, n_active));
  else
    hipLaunchKernelGGL((k_minplus<SP, 1, NW, CH, Blocking<SP>::MINW, false, true, false, false>), grid, block, lds, st, t,
                       l, tiles, first, make_deal(tiles, n_active));
}

hipError_t launch_minplus(const Tables& t, int l, int first, int n_active, hipStream_t st) {
  if (n_active <= 0) return hipSuccess;
  if (t.runs != 0 && t.S > 64) {
    if (t.S <= 128) launch_pruned_wide<2>(t, l, first, n_active, st);
    else launch_pruned_wide<4>(t, l, first, n_active, st);
    return hipSuccess;
  }
  switch (t.SP) {
#define GBMW_CASE(N) case N: launch_minplus_sp<N>(t, l, first, n_active, st); return hipSuccess;
    GBMW_CASE(4) GBMW_CASE(8) GBMW_CASE(12) GBMW_CASE(16) GBMW_CASE(20) GBMW_CASE(24)
    GBMW_CASE(28) GBMW_CASE(32) GBMW_CASE(36) GBMW_CASE(40) GBMW_CASE(44) GBMW_CASE(48)
    GBMW_CASE(52) GBMW_CASE(56) GBMW_CASE(60) GBMW_CASE(64)
#undef GBMW_CASE
  // (a launch of fewer waves than the chip has SIMDs is better off with the generic kernel below,
  // whose waves divide the output strategies: four times the waves)
#define GBMW_CASE(N) case N: if ((long long)((t.E + 64) / 64) * n_active < 1024) break; launch_minplus_big<N>(t, l, first, n_active, st); return hipSuccess;
    GBMW_CASE(68) GBMW_CASE(72) GBMW_CASE(76) GBMW_CASE(80) GBMW_CASE(84) GBMW_CASE(88)
    GBMW_CASE(92) GBMW_CASE(96) GBMW_CASE(100) GBMW_CASE(104) GBMW_CASE(108) GBMW_CASE(112)
    GBMW_CASE(116) GBMW_CASE(120) GBMW_CASE(124) GBMW_CASE(128)
#undef GBMW_CASE
    default: break;
  }
  if (t.runs != 0) return hipErrorInvalidDeviceFunction;   // the generic kernel reads t.Rt, which is not there
  const int tiles = (t.E + 64) / 64;
  hipLaunchKernelGGL(k_minplus_generic, dim3((unsigned)tiles * n_active), dim3(256),
                     (size_t)t.S * 64 * sizeof(float), st, t, l, tiles, first);
  return hipSuccess;
}

bool layer0_in_registers(const Tables& t) { return t.runs != 0 || t.S <= 64; }

// When the pruned step is taken (else the dense kernels; the results are the same).  S == 256: a
// strategy index of 255 would read as kNoGroupRecord.  Beyond 64 strategies the dense kernels take 1.1 to 30
// times as long, but for up to 80 strategies over at most three groups of 64 budgets (S=65, E=64: 262 us per
// solve dense, 321 pruned; S=80, E=128: 347 and 366; S=96, E=64: 464 and 315; S=65, E=200: 268 and 250).
// Up to 64 the pruned step takes 10 to 17 us per layer however small the launch is (a chain of memory round
// trips per group), a split dense launch about 10 us plus its updates at 1.75e13 per second.  Where they meet
// depends on the costs: at 1.3e8 updates per layer with transformations up to a tenth of the layer costs
// (S=24, E=16384, B=12: 168 us per solve dense, 163 pruned), at 6e8 to 1.3e9 with transformations above the
// layer costs, which leave little out (S=64, E=5200, B=64: 852 and 829); 4e8 lies between.  From 2560 groups
// per launch on, dense launches are no longer split and the pruned ones hold a group per wave: level at S=4
// (150 and 145 us at 4160 groups), 1.3 times as fast at S=16.
bool pruned_step_takes(int S, int E, int n, long long most_dense_updates) {
  if (S >= 256) return false;
  if (S > 64) return S > 80 || E >= 192;
  return (long long)((E + 64) / 64) * n >= wave_groups(S) || (long long)n * (E + 1) * S * S >= most_dense_updates;
}

// ---------------------------------------------------------------------------
// final reduce: best(e) = min_s C(L_b - 1, e, s), lowest-index argmin
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_final(Tables t, int first) {
  const int inst = t.perm[first + blockIdx.y].x;
  const int e = t.final_from + blockIdx.x * 256 + threadIdx.x;
  if (e > t.E) return;
  const int l = t.L[inst] - 1;
  const float* __restrict__ C = c_table(t, inst, t.off[inst] + l, l);
  float b = INFINITY;
  int a = 0;
  // eight loads in flight, then the compares in strategy order
  int s = 0;
  for (; s + 8 <= t.S; s += 8) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __builtin_nontemporal_load(&C[(size_t)(s + i) * t.EP + e]);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (x[i] < b) { b = x[i]; a = s + i; }
  }
  for (; s < t.S; ++s) {
    const float x = C[(size_t)s * t.EP + e];
    if (x < b) { b = x; a = s; }
  }
  t.best[(size_t)inst * t.EP + e] = b;
  t.best_s[(size_t)inst * t.EP + e] = (uint8_t)a;
}

// The same from the summaries: a wave takes up to four groups of 64 budgets, a lane per column, and
// where the columns that can be the smallest are constant the group's minimum is one number;
// elsewhere their cells are read (the bounds are those of the layer step with R = 0).
template <int NCH>
__global__ __launch_bounds__(256) void k_final_pruned(Tables t, int first, int unit) {
  const int inst = t.perm[first + blockIdx.y].x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int base = t.final_from + (int)(blockIdx.x * 4 + wave) * unit * 64;
  const int S = t.S, E = t.E, EP = t.EP;
  if (base > E) return;
  const int l = t.L[inst] - 1, row = t.off[inst] + l;
  const float* __restrict__ C = c_table(t, inst, row, l);
  Columns<NCH> q;
  float2 w[NCH][kUnit + 1];
  load_unit<NCH>(t, sum_table(t, inst, row, l), t.M + (size_t)row * S, base, unit, lane, q.m, w);
#pragma unroll
  for (int c = 0; c < NCH; ++c) q.rl[c] = make_float2(0.0f, 0.0f);
#pragma unroll
  for (int g = 0; g < kUnit; ++g) {
    const int wb = base + 64 * g;
    if (g >= unit || wb > E) break;
    const int el = wb + 63 < E ? wb + 63 : E;
#pragma unroll
    for (int c = 0; c < NCH; ++c) { q.a[c] = w[c][g]; q.b[c] = w[c][g + 1]; }
    float ub[NCH], lb[NCH];
    unsigned long long cand[NCH];
    bool varies;
    bounds<NCH>(q, wb, el, ub, lb, cand, varies);
    float b = INFINITY;
    int a = 0;
    if (!varies) {
#pragma unroll
      for (int c = NCH - 1; c >= 0; --c) {
        if (cand[c] == 0) continue;
        const bool in = (cand[c] >> lane) & 1;
        const float v = wave_min(in ? ub[c] : INFINITY);
        if (v <= b) {                                    // (b: as the lowest index has it, -0.0 and 0.0 are equal)
          const int k = __builtin_ctzll(__builtin_amdgcn_ballot_w64(in && ub[c] == v));
          b = lane_f(ub[c], k);
          a = 64 * c + k;
        }
      }
    } else {
      constexpr int NB = 8;
      const int at = wb + lane <= E ? wb + lane : E;     // final_from need not be a multiple of 64
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        unsigned long long mask = cand[c];
        while (mask) {
          int k[NB];
          float cell[NB];
#pragma unroll
          for (int i = 0; i < NB; ++i) {                 // past the end: the last one again (no strict minimum)
            k[i] = mask ? __builtin_ctzll(mask) : k[i > 0 ? i - 1 : 0];
            mask &= mask - 1;
            cell[i] = C[(size_t)(64 * c + k[i]) * EP + at];
          }
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const float x = column_value<NCH, false>(q, 64 * c + k[i], cell[i], wb, E, lane);
            if (x < b) { b = x; a = 64 * c + k[i]; }
          }
        }
      }
    }
    if (wb + lane <= E) {
      t.best[(size_t)inst * EP + wb + lane] = b;
      t.best_s[(size_t)inst * EP + wb + lane] = (uint8_t)a;
    }
  }
}

void launch_final(const Tables& t, int first, int count, hipStream_t st) {
  if (count <= 0) return;
  if (t.runs != 0) {
    const int groups = (t.E - t.final_from + 64) / 64;
    const int unit = (long long)groups * count >= 16384 ? kUnit : 1;
    const dim3 grid((groups + 4 * unit - 1) / (4 * unit), count);
    if (t.S <= 64) hipLaunchKernelGGL(k_final_pruned<1>, grid, dim3(256), 0, st, t, first, unit);
    else if (t.S <= 128) hipLaunchKernelGGL(k_final_pruned<2>, grid, dim3(256), 0, st, t, first, unit);
    else hipLaunchKernelGGL(k_final_pruned<4>, grid, dim3(256), 0, st, t, first, unit);
    return;
  }
  hipLaunchKernelGGL(k_final, dim3((t.E - t.final_from + 256) / 256, count), dim3(256), 0, st, t, first);
}

// ---------------------------------------------------------------------------
// backtrack: one lane per query walks the argmin records from the last layer
// down; each step is one dependent byte gather.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_backtrack(Tables t, int nq, const int* __restrict__ q_inst,
                                                  const int* __restrict__ q_e, int Lmax,
                                                  uint8_t* __restrict__ plan,
                                                  float* __restrict__ cost,
                                                  int* __restrict__ mem_used) {
  const int q = blockIdx.x * 64 + threadIdx.x;
  if (q >= nq) return;
  const int inst = q_inst[q];
  int e = q_e[q];
  uint8_t* p = plan + (size_t)q * Lmax;
  const int Lb = t.L[inst];
  const float b = t.best[(size_t)inst * t.EP + e];
  cost[q] = b;
  if (b == INFINITY) {
    for (int l = 0; l < Lmax; ++l) p[l] = 0xFF;
    mem_used[q] = -1;
    return;
  }
  for (int l = Lb; l < Lmax; ++l) p[l] = 0xFF;
  int s = t.best_s[(size_t)inst * t.EP + e];
  const int row0 = t.off[inst];
  int mem = 0;
  for (int l = Lb - 1; l >= 1; --l) {
    p[l] = (uint8_t)s;
    const int m = t.M[(size_t)(row0 + l) * t.S + s];
    mem += m;
    e -= m;                                            // budget left for layers < l
    if (m < 0 || e < 0) { mem = -2; break; }           // only reachable with invalid inputs
    s = pred_strategy(t, row0 + l, s, e);
  }
  if (mem != -2) {
    p[0] = (uint8_t)s;
    mem += t.M[(size_t)row0 * t.S + s];
  }
  mem_used[q] = mem;
}

// The same walk without argmin records: every step has to redo the minimum over the S
// predecessors from the kept table of the layer below, so a whole wave takes one query, its
// lanes over the predecessors (pred_strategy_wave), and lane 0 writes the plan.
__global__ __launch_bounds__(256) void k_backtrack_wave(Tables t, int nq, const int* __restrict__ q_inst,
                                                        const int* __restrict__ q_e, int Lmax,
                                                        uint8_t* __restrict__ plan, float* __restrict__ cost,
                                                        int* __restrict__ mem_used) {
  const int q = blockIdx.x * 4 + (threadIdx.x >> 6);      // wave-uniform
  const int lane = threadIdx.x & 63;
  if (q >= nq) return;
  const int inst = q_inst[q];
  int e = q_e[q];
  uint8_t* p = plan + (size_t)q * Lmax;
  const int Lb = t.L[inst];
  const float b = t.best[(size_t)inst * t.EP + e];
  if (b == INFINITY) {
    for (int l = lane; l < Lmax; l += 64) p[l] = 0xFF;
    if (lane == 0) { cost[q] = b; mem_used[q] = -1; }
    return;
  }
  for (int l = Lb + lane; l < Lmax; l += 64) p[l] = 0xFF;
  int s = t.best_s[(size_t)inst * t.EP + e];
  const int row0 = t.off[inst];
  int mem = 0;
  for (int l = Lb - 1; l >= 1; --l) {
    if (lane == 0) p[l] = (uint8_t)s;
    const int m = t.M[(size_t)(row0 + l) * t.S + s];
    mem += m;
    e -= m;                                              // budget left for layers < l
    if (m < 0 || e < 0) { mem = -2; break; }             // only reachable with invalid inputs
    s = pred_strategy_wave(t, row0 + l, s, e, lane);
  }
  if (mem != -2) {
    if (lane == 0) p[0] = (uint8_t)s;
    mem += t.M[(size_t)row0 * t.S + s];
  }
  if (lane == 0) { cost[q] = b; mem_used[q] = mem; }
}

void launch_backtrack(const Tables& t, int nq, const int* q_inst, const int* q_e, int Lmax,
                      uint8_t* plan, float* cost, int* mem_used, hipStream_t st) {
  if (nq <= 0) return;
  if (t.A == nullptr) {
    hipLaunchKernelGGL(k_backtrack_wave, dim3((nq + 3) / 4), dim3(256), 0, st, t, nq, q_inst, q_e, Lmax, plan, cost,
                       mem_used);
    return;
  }
  hipLaunchKernelGGL(k_backtrack, dim3((nq + 63) / 64), dim3(64), 0, st, t, nq, q_inst, q_e, Lmax,
                     plan, cost, mem_used);
}

// ---------------------------------------------------------------------------
// Algorithm 3's outer loop.  walk_plan follows the argmin records of instance
// `inst` from budget e down and evaluates Eq. 2 on the way.  Going from the last
// layer to the first, the forward prefix of layer i is F - suf_i with F the sum
// of all O_f and suf_i the sum over the layers above i, so
//   E_all = F + max_i (O_b(i) - suf_i) + sum O_ms.
// ---------------------------------------------------------------------------
// WAVE: all lanes of the wave walk the same plan and lane 0 writes it.
template <bool WAVE>
__device__ long long walk_plan(const Tables& t, int inst, int e, const int* __restrict__ Of,
                               const int* __restrict__ Ob, const int* __restrict__ Oms,
                               uint8_t* plan, int lane) {
  const int Lb = t.L[inst], row0 = t.off[inst], S = t.S;
  int s = t.best_s[(size_t)inst * t.EP + e];
  long long suf = 0, ms = 0, mx = 0;
  for (int l = Lb - 1; l >= 0; --l) {
    const size_t cell = (size_t)(row0 + l) * S + s;
    if (plan && (!WAVE || lane == 0)) plan[l] = (uint8_t)s;
    const long long here = (long long)Ob[cell] - suf;
    mx = (l == Lb - 1 || here > mx) ? here : mx;
    suf += Of[cell];
    ms += Oms[cell];
    if (l > 0) {
      const int m = t.M[cell];
      e -= m;                                            // budget left for layers < l
      if (m < 0 || e < 0) return -2;                     // only reachable with invalid inputs
      s = WAVE ? pred_strategy_wave(t, row0 + l, s, e, lane) : pred_strategy(t, row0 + l, s, e);
    }
  }
  return suf + mx + ms;
}

__global__ void k_select_init(int B, int* first_bad) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) first_bad[b] = 0x7fffffff;
}

// one lane per (instance, budget of its window): record the lowest budget
// whose plan does not fit the overall memory
__global__ __launch_bounds__(64) void k_select_check(Tables t, const int* __restrict__ Of,
                                                     const int* __restrict__ Ob,
                                                     const int* __restrict__ Oms,
                                                     const int* __restrict__ bup,
                                                     int* __restrict__ first_bad) {
  const int inst = blockIdx.y;
  const int base = t.E - bup[inst];                      // last budget that needs no check
  const int lo = (base < 0 ? -1 : base) + 1;
  const int e = lo + blockIdx.x * 64 + threadIdx.x;
  // budgets above a failure already recorded have nothing to add
  if (*(volatile const int*)&first_bad[inst] < lo + (int)blockIdx.x * 64) return;
  if (e > t.E) return;
  if (t.best[(size_t)inst * t.EP + e] == INFINITY) return;   // no plan: nothing to check
  const long long ea = walk_plan<false>(t, inst, e, Of, Ob, Oms, nullptr, 0);
  if (ea > (long long)t.E || ea < 0) atomicMin(&first_bad[inst], e);
}

// One wave per instance: all lanes walk the chosen plan together and, without records, share the
// recomputation of each step (pred_strategy_wave); lane 0 writes.  One lane per instance took
// 0.78 ms for 64 instances of up to 24 layers and 44 strategies without records (latency: every step
// is S dependent candidates), a wave takes 0.06 ms.
__global__ __launch_bounds__(64) void k_select_pick(Tables t, const int* __restrict__ Of,
                                                    const int* __restrict__ Ob,
                                                    const int* __restrict__ Oms,
                                                    const int* __restrict__ bup,
                                                    const int* __restrict__ first_bad, int Lmax,
                                                    int* __restrict__ e_opt,
                                                    float* __restrict__ cost,
                                                    uint8_t* __restrict__ plan,
                                                    int* __restrict__ e_all) {
  const int inst = blockIdx.x, lane = threadIdx.x;
  const int base = t.E - bup[inst];
  const int init = base < 0 ? -1 : base;
  const int fb = first_bad[inst];
  const int last = (fb == 0x7fffffff) ? t.E : fb - 1;
  int opt = init;
  if (last > init && t.best[(size_t)inst * t.EP + last] != INFINITY) opt = last;
  uint8_t* p = plan + (size_t)inst * Lmax;
  float cst = INFINITY;
  long long ea = -1;
  if (opt >= 0) cst = t.best[(size_t)inst * t.EP + opt];
  const bool any = cst != INFINITY;
  for (int l = (any ? t.L[inst] : 0) + lane; l < Lmax; l += 64) p[l] = 0xFF;
  if (any) ea = walk_plan<true>(t, inst, opt, Of, Ob, Oms, p, lane);
  if (lane == 0) {
    e_opt[inst] = opt;
    cost[inst] = cst;
    e_all[inst] = (int)ea;
  }
}

void launch_select(const Tables& t, const int* Of, const int* Ob, const int* Oms, const int* bup,
                   int max_window, int Lmax, int* first_bad, int* e_opt, float* cost,
                   uint8_t* plan, int* e_all, hipStream_t st) {
  hipLaunchKernelGGL(k_select_init, dim3((t.B + 63) / 64), dim3(64), 0, st, t.B, first_bad);
  if (max_window > 0)
    hipLaunchKernelGGL(k_select_check, dim3((max_window + 63) / 64, t.B), dim3(64), 0, st, t, Of,
                       Ob, Oms, bup, first_bad);
  hipLaunchKernelGGL(k_select_pick, dim3(t.B), dim3(64), 0, st, t, Of, Ob, Oms, bup,
                     first_bad, Lmax, e_opt, cost, plan, e_all);
}

// ---------------------------------------------------------------------------
// Pipeline time (Eq. 5 / Eq. 8).  One lane per stage walks its plan down the
// argmin records into a scratch row, then re-evaluates it upward with the costs
// without gradient synchronisation; R(l, s', s) is read from the transposed
// table Rt[row][s][s'].
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_stage_cost(Tables t, int n_stage,
                                                   const int* __restrict__ st_inst,
                                                   const int* __restrict__ st_e,
                                                   const float* __restrict__ c_ns,
                                                   uint8_t* __restrict__ plan_scratch, int Lmax,
                                                   float* __restrict__ st_C,
                                                   float* __restrict__ st_Cns) {
  const int q = blockIdx.x * 64 + threadIdx.x;
  if (q >= n_stage) return;
  const int inst = st_inst[q];
  int e = st_e[q];
  float C = INFINITY, Cns = INFINITY;
  if (e >= 0) C = t.best[(size_t)inst * t.EP + e];
  if (C != INFINITY) {
    if (!c_ns) {
      Cns = C;
    } else {
      const int Lb = t.L[inst], row0 = t.off[inst], S = t.S;
      uint8_t* plan = plan_scratch + (size_t)q * Lmax;
      int s = t.best_s[(size_t)inst * t.EP + e];
      bool ok = true;
      for (int l = Lb - 1; l >= 1; --l) {
        plan[l] = (uint8_t)s;
        e -= t.M[(size_t)(row0 + l) * S + s];
        if (e < 0) { ok = false; break; }                // only reachable with invalid inputs
        s = pred_strategy(t, row0 + l, s, e);
      }
      if (ok) {
        plan[0] = (uint8_t)s;
        float v = c_ns[(size_t)row0 * S + s];
        for (int l = 1; l < Lb; ++l) {
          const int sn = plan[l];
          const float r = r_entry(t, row0 + l, s, sn);
          v = (v + r) + c_ns[(size_t)(row0 + l) * S + sn];
          s = sn;
        }
        Cns = v;
      }
    }
  }
  st_C[q] = C;
  st_Cns[q] = Cns;
}

__global__ __launch_bounds__(64) void k_pipeline_cost(int n_pipe, const int* __restrict__ st_begin,
                                                      const int* __restrict__ mb,
                                                      const float* __restrict__ st_C,
                                                      const float* __restrict__ st_Cns,
                                                      float* __restrict__ cost) {
  const int p = blockIdx.x * 64 + threadIdx.x;
  if (p >= n_pipe) return;
  const int b = st_begin[p], e = st_begin[p + 1];
  float total = st_C[b], mx = st_Cns[b];
  for (int i = b + 1; i < e; ++i) {
    total = total + st_C[i];
    mx = st_Cns[i] > mx ? st_Cns[i] : mx;
  }
  float out = INFINITY;
  if (total != INFINITY && mx != INFINITY) {
    const float head = (float)(mb[p] - 1) * mx;
    out = head + total;
  }
  cost[p] = out;
}

void launch_pipeline_cost(const Tables& t, int n_stage, const int* st_inst, const int* st_e,
                          const float* c_ns, uint8_t* plan_scratch, int Lmax, float* st_C,
                          float* st_Cns, int n_pipe, const int* st_begin, const int* mb,
                          float* cost, hipStream_t st) {
  hipLaunchKernelGGL(k_stage_cost, dim3((n_stage + 63) / 64), dim3(64), 0, st, t, n_stage, st_inst,
                     st_e, c_ns, plan_scratch, Lmax, st_C, st_Cns);
  hipLaunchKernelGGL(k_pipeline_cost, dim3((n_pipe + 63) / 64), dim3(64), 0, st, n_pipe, st_begin,
                     mb, st_C, st_Cns, cost);
}

// ---------------------------------------------------------------------------
// export: device [n][S][EP] -> logical [n][E+1][S] through a 64x64 LDS tile
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_export(const T* __restrict__ src, T* __restrict__ dst, int S,
                                                int E, int EP) {
  __shared__ T tile[64][65];
  const int n = blockIdx.z;
  const int e0 = blockIdx.x * 64, s0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const T* in = src + (size_t)n * S * EP;
  T* out = dst + (size_t)n * (E + 1) * S;
  for (int i = ty; i < 64; i += 4) {
    const int s = s0 + i, e = e0 + tx;
    if (s < S && e <= E) tile[i][tx] = in[(size_t)s * EP + e];
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int e = e0 + i, s = s0 + tx;
    if (s < S && e <= E) out[(size_t)e * S + s] = tile[tx][i];
  }
}

__global__ __launch_bounds__(256) void k_argmin_row(Tables t, int row, uint8_t* __restrict__ dst) {
  const int e = blockIdx.x * 256 + threadIdx.x, s = blockIdx.y;
  if (e >= t.EP) return;
  dst[(size_t)s * t.EP + e] = (e <= t.E) ? (uint8_t)pred_strategy(t, row, s, e) : 0;
}

void launch_argmin_row(const Tables& t, int row, uint8_t* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_argmin_row, dim3(t.EP / 256, t.S), dim3(256), 0, st, t, row, dst);
}

__global__ __launch_bounds__(256) void k_export_c(Tables t, const float* __restrict__ Ctab,
                                                  const float2* __restrict__ Tsum_tab, const int* __restrict__ Mrow,
                                                  float* __restrict__ dst) {
  const int e = blockIdx.x * 256 + threadIdx.x, s = blockIdx.y;
  if (e > t.E) return;
  dst[(size_t)e * t.S + s] = table_cell(t, Ctab, Tsum_tab, Mrow, s, e);
}
void launch_export_c(const Tables& t, const float* Ctab, const float2* Tsum_tab, const int* Mrow, float* dst,
                     hipStream_t st) {
  hipLaunchKernelGGL(k_export_c, dim3((t.E + 256) / 256, t.S), dim3(256), 0, st, t, Ctab, Tsum_tab, Mrow, dst);
}
void launch_export_u8(const uint8_t* src, uint8_t* dst, int n, int S, int E, int EP,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_export<uint8_t>, dim3((E + 64) / 64, (S + 63) / 64, n), dim3(256), 0, st,
                     src, dst, S, E, EP);
}

}  // namespace gbmw

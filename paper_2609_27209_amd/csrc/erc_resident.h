// Resident CG for small graphs on gfx950 (Section 3.1.3, column-wise CG; Eq. 5).
//
// The columns of a block are independent, and on a graph of up to a few ten thousand nodes
// one column's search direction fits the LDS of one CU (160 KB) and its other vectors fit
// the registers.  One workgroup therefore solves one column from its right-hand side to the
// stop without leaving the CU: p in LDS, where every neighbour gather is served, z, r and
// q in registers, the two inner products of an iteration by workgroup reductions.  No
// launch, grid-wide reduction or host poll sits between iterations.
//
// What bounds it: on the smallest graphs in fp32 the chain of reductions, barriers and LDS
// round trips of an iteration (2000 rows, 22,000 entries: 3.7 us; vector units and LDS busy 36%
// of the time each), in fp64 the vector instructions of the double-double products and folds
// (4.8 us; vector units 68%), on larger graphs the LDS gathers, whose random banks collide
// (64-lane gathers take 7 cycles instead of 2), and the vector instructions around them (20,000
// rows, 220,000 entries: 20.7 us; LDS busy 58% of the time, over half of it conflicts, vector
// units 64%), with the operator's stream from the L2 (2 bytes of position and the weight per
// entry) behind them.  The block kernels took 28, 28 and 54 us for these iterations of 32, 64
// and 64 columns, as three or four dependent launches each.  Whole steps: 2000 rows fp64 1.20 ->
// 0.34 ms, 2000 rows and 1024 columns 16.7 -> 0.79 ms, 20,000 rows 2.00 -> 0.97 ms, 12,305 rows
// fp64 Jacobi 4.7 -> 1.27 ms.
//
// The recurrence is Hestenes-Stiefel CG with the stopping rule of the block kernels, and no sum
// is less precise than theirs: fp32 or fp64 vectors; a thread's part of an inner product in fp64
// or double-double, the threads' parts folded as compensated pairs; in fp32 a row's entries in
// fours, and the fours (of rows above kResHeavy entries each entry) added in fp64.  (fp32 chains
// over the row put weighted rows of about 100 entries 1.7 times as far from the fp64 solution
// as the block kernels; with plain folds they saved 0.4-0.7 us an iteration up to 16,384 rows
// and 1.1-1.5 us above.)  In fp64 beta also has their expanded form, so that rows which both sum
// one entry after the other give the same bits from both (fp64 CG is where a caller looks for
// agreement beyond the stopping tolerance, and a few ten iterations amplify the last bit of a
// beta to 1e-8 of the solution); fp32 takes r.r of the stored r, which needs slightly fewer
// iterations on power-law graphs than the expansion and lies no further from the fp64 solution.
#pragma once

#include <hip/hip_runtime.h>

#include "erc_common.h"

namespace erc {

struct ResArgs {
  ResPlan p;
  int32_t n;
  const void* csr_w;
  void* y;       // n x kb: right-hand sides, replaced by the solutions
  int kb;
  int max_iter;
  double delta, tol2;
  void* q;           // n per column, by position (only where q does not fit the LDS)
  const void* minv;  // by position (Jacobi variant)
  ResOut* out;
};

// The kernels of one working precision (erc_resident_f32.hip, erc_resident_f64.hip).
hipError_t res_solve_f32(const ResArgs& a, int ncols, size_t lds, hipStream_t s);
hipError_t res_solve_f64(const ResArgs& a, int ncols, size_t lds, hipStream_t s);

// Workgroup sizes and slots that a kernel exists for, smallest first.  512 threads up to 2048
// rows: there an iteration is mostly reductions, whose instructions every wavefront of a SIMD
// issues in turn, against the latency that more wavefronts hide (2000 rows, 38 iterations of
// fp32 and 42 of fp64, us per solve with 256 / 512 / 1024 threads: 205 / 142 / 163 and
// 227 / 173 / 196, the latter with one inner product less than now).
inline constexpr ResForm kForms32[] = {{512, 2}, {512, 4}, {1024, 4}, {1024, 6}, {1024, 8}, {1024, 12},
                                       {1024, 16}, {1024, 20}, {1024, 24}, {1024, 28}, {1024, 32}};
inline constexpr ResForm kForms64[] = {{512, 2}, {512, 4}, {1024, 4}, {1024, 6}, {1024, 8},
                                       {1024, 10}, {1024, 13}, {1024, 16}};
// Quads that a wavefront of a 512-thread form can keep in registers for the whole solve.
constexpr int kResRegQuads = 16;
// Sums of a workgroup that the LDS has room for: four of an update and p.q.
constexpr int kResSums = 5;
// Sums that a workgroup folds at once, of which the LDS holds a part per thread where res_parts.
constexpr int kResFolds = 2;

// Forms whose partial sums go through the LDS to one wavefront per sum (fp32 up to 16,384 rows)
// rather than being folded by every wavefront in registers: 120 instructions per sum and
// wavefront, four wavefronts to a SIMD, of a short iteration.  Up to 12,288 rows that saves
// 0.5-0.8 us of an iteration (8000 rows, 88,000 entries: 9.85 -> 9.1 us, with Jacobi 12.3 ->
// 11.0), at 16,000 0.5 of 16.5 us, above nothing (20,000 rows with Jacobi 27.4 -> 29.6 us, as q
// no longer fits beside the parts); fp64's pairs would need twice the LDS.
constexpr bool res_parts(ResForm f, size_t elem) { return elem == 4 && f.nt * f.rpt <= 16 * 1024; }

// Places for q that a form's kernels exist for: beside p in the LDS (a form's last rows may be
// missing, which leaves room), and outside it.
constexpr bool res_q_inside(ResForm f, size_t elem) { return f.nt * f.rpt * elem <= 84 * 1024; }
constexpr bool res_q_outside(ResForm f, size_t elem) { return f.nt * f.rpt * elem > 64 * 1024; }

namespace {

struct DD {
  double s, c;  // value s + c
};

__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
#pragma clang fp contract(off)
  s = a + b;
  const double z = s - a;
  e = (a - (s - z)) + (b - z);
}

__device__ __forceinline__ DD dd_add(DD a, DD b) {
#pragma clang fp contract(off)
  double s, e;
  two_sum(a.s, b.s, s, e);
  return DD{s, (a.c + b.c) + e};
}
__device__ __forceinline__ double dd_value(DD a) { return a.s + a.c; }
__device__ __forceinline__ DD dd_times(DD a, double b) {
#pragma clang fp contract(off)
  const double p = a.s * b;
  const double pe = fma(a.s, b, -p);
  const double c = pe + a.c * b;
  DD r;
  two_sum(p, c, r.s, r.c);
  return r;
}

// Inner products in twice the working precision, as in the block kernels: a thread adds
// exact fp32 products in fp64, or exactly split fp64 products in double-double, and the threads'
// sums are folded as compensated pairs.
template <typename T>
struct Acc;
template <>
struct Acc<float> {
  typedef double L;
  __device__ __forceinline__ static L zero() { return 0.0; }
  __device__ __forceinline__ static L mac(L a, float x, float y) {
    return fma(static_cast<double>(x), static_cast<double>(y), a);
  }
  __device__ __forceinline__ static DD pair(L a) { return DD{a, 0.0}; }
};
template <>
struct Acc<double> {
  typedef DD L;
  __device__ __forceinline__ static L zero() { return DD{0.0, 0.0}; }
  __device__ __forceinline__ static L mac(L a, double x, double y) {
#pragma clang fp contract(off)
    const double p = x * y;
    const double pe = fma(x, y, -p);
    double t, e;
    two_sum(a.s, p, t, e);
    return DD{t, a.c + (e + pe)};
  }
  __device__ __forceinline__ static DD pair(L a) { return a; }
};

// Lane exchanges within 16-lane rows by DPP (a few cycles each, against an LDS round trip
// for a shuffle): quad permutations, then mirrors of 8 and 16 lanes, which pair equal sums.
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
template <int CTRL>
__device__ __forceinline__ DD dpp(DD x) {
  return DD{dpp<CTRL>(x.s), dpp<CTRL>(x.c)};
}
__device__ __forceinline__ double plus(double a, double b) { return a + b; }
__device__ __forceinline__ DD plus(DD a, DD b) { return dd_add(a, b); }

// Sum over each row of 16 (or 8) lanes, in every lane of the row (the same bits in each).
template <int LANES, typename V>
__device__ __forceinline__ V row_sum(V x) {
  x = plus(x, dpp<0xB1>(x));   // lanes xor 1
  x = plus(x, dpp<0x4E>(x));   // lanes xor 2
  x = plus(x, dpp<0x141>(x));  // the other four of eight
  if constexpr (LANES == 16) x = plus(x, dpp<0x140>(x));  // the other eight of sixteen
  return x;
}
// a, b: x of a lane's row of 16 and of the row beside it (K = 16), or of its half of the
// wavefront and of the other (K = 32), in one order for both; a lane swap gives both words at
// once.  across: their sum.
template <int K>
__device__ __forceinline__ void swapped(double x, double& a, double& b) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = static_cast<unsigned>(v), hi = static_cast<unsigned>(v >> 32);
  if constexpr (K == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    a = __longlong_as_double((static_cast<long long>(h[0]) << 32) | l[0]);
    b = __longlong_as_double((static_cast<long long>(h[1]) << 32) | l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __longlong_as_double((static_cast<long long>(h[0]) << 32) | l[0]);
    b = __longlong_as_double((static_cast<long long>(h[1]) << 32) | l[1]);
  }
}
template <int K>
__device__ __forceinline__ double across(double x) {
  double a, b;
  swapped<K>(x, a, b);
  return a + b;
}
template <int K>
__device__ __forceinline__ DD across(DD x) {
  DD a, b;
  swapped<K>(x.s, a.s, b.s);
  swapped<K>(x.c, a.c, b.c);
  return dd_add(a, b);
}
template <typename V>
__device__ __forceinline__ V wave_sum(V x) {
  return across<32>(across<16>(row_sum<16>(x)));
}

// The sum of N parts as a compensated pair, by halves.
template <int N>
__device__ __forceinline__ DD pair_of(const double (&x)[N]) {
  static_assert(N == 8 || N == 16, "parts per lane");
  DD t[N / 2];
#pragma unroll
  for (int k = 0; k < N / 2; ++k) two_sum(x[k], x[k + N / 2], t[k].s, t[k].c);
#pragma unroll
  for (int h = N / 4; h > 0; h >>= 1) {
#pragma unroll
    for (int k = 0; k < h; ++k) t[k] = dd_add(t[k], t[k + h]);
  }
  return t[0];
}

// Makes a uniform address opaque, so that loads through it are not kept in registers across
// the point (hoisted out of the iteration, or shared between its start and its end): the
// registers hold z, r and q, and the reloads hit the caches.  The result names its address
// space (global memory), which the compiler would no longer see.
template <typename P>
using Global = P __attribute__((address_space(1)))*;
__device__ __forceinline__ uint64_t opaque(const void* p) {
  uint64_t u = reinterpret_cast<uint64_t>(p);
  asm volatile("" : "+s"(u));
  return u;
}
template <typename P>
__device__ __forceinline__ Global<P> fresh(P* p) {
  return reinterpret_cast<Global<P>>(opaque(p));
}
__device__ __forceinline__ int fresh_lane(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Computes x here: not later, where its operands would have to be kept until then.
__device__ __forceinline__ double here(double x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ DD here(DD x) { return DD{here(x.s), here(x.c)}; }

// Four entries of one row: positions and weights (unit weights are not stored).
template <typename T, bool W>
struct Quad {
  uint32_t j[2];
  T w[4];
};
template <typename T, bool W>
__device__ __forceinline__ Quad<T, W> load_quad(Global<const uint16_t> idx, Global<const T> w,
                                                int t, int lane) {
  typedef uint32_t U2 __attribute__((ext_vector_type(2)));
  typedef T T4 __attribute__((ext_vector_type(4)));
  Quad<T, W> q;
  // a uniform base plus a 32-bit lane offset: the address costs no vector instruction
  const auto bi = reinterpret_cast<Global<const char>>(idx) + static_cast<int64_t>(t) * 512;
  const U2 j = *reinterpret_cast<Global<const U2>>(bi + static_cast<uint32_t>(lane) * 8u);
  q.j[0] = j[0];
  q.j[1] = j[1];
  if constexpr (W) {
    constexpr uint32_t kLane = 4 * sizeof(T);
    const auto bw = reinterpret_cast<Global<const char>>(w) + static_cast<int64_t>(t) * (64 * kLane);
    const T4 x = *reinterpret_cast<Global<const T4>>(bw + static_cast<uint32_t>(lane) * kLane);
#pragma unroll
    for (int k = 0; k < 4; ++k) q.w[k] = x[k];
  }
  return q;
}

// p at the position in half `hi` of j: the half is picked and scaled to bytes in one
// instruction.
template <typename T>
__device__ __forceinline__ T at_position(const T* s_p, uint32_t j, int hi) {
  uint32_t o;
  if (hi)
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
        : "=v"(o) : "v"(sizeof(T) == 4 ? 2 : 3), "v"(j));
  else
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
        : "=v"(o) : "v"(sizeof(T) == 4 ? 2 : 3), "v"(j));
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(s_p) + o);
}

template <int N>
struct Count {
  static constexpr int value = N;
};

// One workgroup of NT threads per column.  RPT: rows per thread, so that z and r are indexed
// by constants and stay in registers and a row's place in LDS is a constant offset.  q is
// stored in LDS behind p where both fit (QL), else in global memory by position.
// NQ > 0: a wavefront's quads (at most NQ) stay in registers for the whole solve; else they are
// streamed from the L2 in every iteration.
template <typename T, int NT, int RPT, bool W, bool PC, bool QL, int NQ>
__global__ __launch_bounds__(NT) void k_resident(ResArgs a) {
  typedef Acc<T> A;
  constexpr int NW = NT / 64;
  constexpr int D = W && sizeof(T) == 8 ? 2 : 4;  // quads in flight per wavefront
  static_assert(D <= kResPadQuads, "the stream is read D quads past its end");
  __shared__ T s_p[RPT * NT];
  extern __shared__ __attribute__((aligned(16))) char smem[];
  DD (*s_red)[NW] = reinterpret_cast<DD (*)[NW]>(smem);
  double* s_h = reinterpret_cast<double*>(&s_red[kResSums][0]);
  constexpr bool PARTS = res_parts(ResForm{NT, RPT}, sizeof(T));
  double* s_part = s_h + ((a.p.nchunk + 1) & ~1);  // kResFolds x NT where PARTS
  T* s_q = reinterpret_cast<T*>(s_part + (PARTS ? kResFolds * NT : 0));

  int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = blockIdx.x;
  const T* __restrict__ Y = static_cast<const T*>(a.y) + c;
  // the wavefront's quads: lane s holds the end of slot s
  const int t0 = a.p.off[wv * RPT];
  const int ends = a.p.off[wv * RPT + min(lane + 1, RPT)];

  // sums over the workgroup of K values at once, in every thread; partial set b is free
  // again when the barrier after the next has passed (set 0: up to four sums, set 1: one).
  // Every wavefront folds its lanes' pairs and then the wavefronts', or (PARTS) one wavefront per
  // value adds NT / 64 threads' parts per lane before it folds.
  auto block_sums = [&](const typename A::L* x, DD* sum, auto kk, int b) {
    constexpr int K = decltype(kk)::value;
    if constexpr (PARTS) {
      static_assert(K <= kResFolds, "room for the parts");
#pragma unroll
      for (int k = 0; k < K; ++k) s_part[k * NT + tid] = x[k];
      __syncthreads();
      if (wv < K) {
        double part[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) part[k] = s_part[wv * NT + k * 64 + lane];
        const DD t = wave_sum(pair_of(part));
        if (lane == 0) s_red[4 * b + wv][0] = t;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < K; ++k) sum[k] = s_red[4 * b + k][0];
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const DD t = wave_sum(A::pair(x[k]));
        if (lane == 0) s_red[4 * b + k][wv] = t;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < K; ++k) sum[k] = row_sum<NW>(s_red[4 * b + k][lane & (NW - 1)]);
    }
  };
  static_assert(NW == 8 || NW == 16, "row_sum adds 8 or 16 partials");

  Quad<T, W> own[NQ > 0 ? NQ : 1];
  if constexpr (NQ > 0) {
    const int last = a.p.off[wv * RPT + RPT] - 1;
#pragma unroll
    for (int k = 0; k < NQ; ++k)
      own[k] = load_quad<T, W>(fresh(a.p.idx), fresh(static_cast<const T*>(a.p.w)),
                               max(min(t0 + k, last), 0), lane);
  }

  T z[RPT], r[RPT];
  // r.r, then r.M^-1 r with the Jacobi variant, then r.q and q.q of the expanded beta
  // (weighted by M^-1 with the Jacobi variant)
  constexpr bool X = sizeof(T) == 8;
  constexpr int R = PC ? 2 : 1;
  constexpr int ND = X ? R + 2 : R;
  typename A::L dot[4] = {A::zero(), A::zero(), A::zero(), A::zero()};
  DD sum[4];
#pragma unroll
  for (int s = 0; s < RPT; ++s) {
    const int pos = s * NT + tid;
    z[s] = T(0);
    r[s] = pos < a.n ? Y[static_cast<int64_t>(a.p.row[pos]) * a.kb] : T(0);
    T p0 = r[s];
    if constexpr (PC) {
      p0 = static_cast<const T*>(a.minv)[pos] * r[s];
      dot[1] = A::mac(dot[1], r[s], p0);
    }
    dot[0] = here(A::mac(dot[0], r[s], r[s]));
    s_p[pos] = p0;
    if (s % 4 == 3) asm volatile("" ::: "memory");  // no more than four slots' addresses at once
  }
  block_sums(dot, sum, Count<R>(), 0);  // its barrier also completes p
  const double rho0 = dd_value(sum[0]);
  double rr = rho0;
  double rho = PC ? dd_value(sum[1]) : rho0;
  const double thr = a.tol2 * rho0;
  int iters = 0, status = 0;
  bool active = rr > 0.0;

  while (active && iters < a.max_iter) {
    tid = fresh_lane(tid);
    // 1. chunks of the long rows, one per wavefront at a time, in fp64
    for (int h = wv; h < a.p.nchunk; h += NW) {
      const int b = a.p.hbeg[h], len = a.p.hlen[h];
      const double pi = static_cast<double>(s_p[a.p.hpos[h]]);
      double acc = 0.0;
      // all of a lane's entries of the chunk are loaded before the first is used; lanes past
      // the end take the row itself (a zero term)
      constexpr int K = kResChunk / 64;
      uint16_t j[K];
      T w[K];
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int k = u * 64 + lane;
        const bool in = k < len;
        j[u] = in ? a.p.cpos[b + k] : static_cast<uint16_t>(a.p.hpos[h]);
        w[u] = W && in ? static_cast<const T*>(a.csr_w)[b + k] : T(1);
      }
#pragma unroll
      for (int u = 0; u < K; ++u)
        acc += static_cast<double>(w[u]) * (pi - static_cast<double>(s_p[j[u]]));
      acc = wave_sum(acc);
      if (lane == 0) s_h[h] = acc;
    }
    if (a.p.nchunk > 0) __syncthreads();
    // 2. q = (L + delta I) p, one row per lane: the wavefront's quads are one stream through
    // its slots, D of them in flight; at a slot's end its rows are finished
    typename A::L pq[1] = {A::zero()};
    {
      const Global<const uint16_t> idx = fresh(a.p.idx);
      const Global<const T> wq = fresh(static_cast<const T*>(a.p.w));
      const Global<T> gq = fresh(static_cast<T*>(a.q)) + static_cast<int64_t>(c) * a.n;
      Quad<T, W> buf[D];
#pragma unroll
      for (int k = 0; NQ == 0 && k < D; ++k) {
        buf[k] = load_quad<T, W>(idx, wq, t0 + k, lane);
        __builtin_amdgcn_sched_barrier(0);  // in the order they are waited for
      }
      int t = t0, slot = 0;
      int te = __builtin_amdgcn_readlane(ends, 0);
      // an fp32 row adds the sums of its quads in fp64, an fp64 row its entries one by one
      double acc = 0.0;
      T pi = s_p[tid], pn = s_p[min(1, RPT - 1) * NT + tid];  // this slot's p and the next's
      auto finish = [&]() {
        const int pos = slot * NT + tid;
        if (slot * NT < a.p.nheavy && pos < a.p.nheavy) {
          acc = 0.0;
          for (int h = a.p.hc0[pos]; h < a.p.hc0[pos + 1]; ++h) acc += s_h[h];
        }
        const T q = static_cast<T>(a.delta * static_cast<double>(pi) + acc);
        if (pos < a.n) {
          if (QL) s_q[pos] = q;
          else gq[pos] = q;
        }
        pq[0] = A::mac(pq[0], pi, q);
        acc = 0.0;
        ++slot;
        te = __builtin_amdgcn_readlane(ends, slot);
        pi = pn;
        pn = s_p[min(slot + 1, RPT - 1) * NT + tid];
      };
      auto add = [&](const Quad<T, W>& e) {
        T x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = at_position<T>(s_p, e.j[u / 2], u & 1);
        if constexpr (X) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if constexpr (W) acc += e.w[u] * (pi - x[u]);
            else acc += pi - x[u];
          }
        } else if constexpr (W) {
          T t = e.w[0] * (pi - x[0]);
#pragma unroll
          for (int u = 1; u < 4; ++u) t += e.w[u] * (pi - x[u]);
          acc += static_cast<double>(t);
        } else {
          acc += static_cast<double>(((pi - x[0]) + (pi - x[1])) + ((pi - x[2]) + (pi - x[3])));
        }
      };
      // (one way into the loop and gotos out of it: every path to a step then has the same
      // loads in flight, and the step waits for its own quad alone)
      while (t == te) {
        finish();
        if (slot == RPT) goto done;
      }
      if constexpr (NQ > 0) {
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
          add(own[k]);
          ++t;
          while (t == te) {
            finish();
            if (slot == RPT) goto done;
          }
        }
      } else {
        for (;;) {
#pragma unroll
          for (int k = 0; k < D; ++k) {
            add(buf[k]);
            buf[k] = load_quad<T, W>(idx, wq, t + D, lane);
            ++t;
            while (t == te) {
              finish();
              if (slot == RPT) goto done;
            }
          }
        }
      }
    done:;
    }
    block_sums(pq, sum, Count<1>(), 1);
    const double pqv = dd_value(sum[0]);
    active = pqv > 0.0 && isfinite(pqv);
    status = active ? 0 : 1;
    if (active) {
      // 3. z += alpha p, r -= alpha q, and r.r (and r.M^-1 r) of the stored r
      const T al = static_cast<T>(rho / pqv);
      Global<const T> mv = fresh(static_cast<const T*>(a.minv));
      const Global<const T> gq = fresh(static_cast<const T*>(a.q)) + static_cast<int64_t>(c) * a.n;
      dot[0] = dot[1] = dot[2] = dot[3] = A::zero();
#pragma unroll
      for (int s = 0; s < RPT; ++s) {
        const int pos = s * NT + tid;
        T q = T(0);
        if (pos < a.n) q = QL ? s_q[pos] : gq[pos];
        z[s] += al * s_p[pos];
        if constexpr (X) {
          const T m = PC ? mv[pos] : T(1);
          dot[R] = here(A::mac(dot[R], PC ? r[s] * m : r[s], q));
          dot[R + 1] = here(A::mac(dot[R + 1], PC ? q * m : q, q));
        }
        r[s] -= al * q;
        dot[0] = A::mac(dot[0], r[s], r[s]);
        if constexpr (X) dot[0] = here(dot[0]);
        if constexpr (PC) dot[1] = here(A::mac(dot[1], r[s], mv[pos] * r[s]));
        if (s % (X ? 2 : 8) == (X ? 1 : 7)) asm volatile("" ::: "memory");
      }
      block_sums(dot, sum, Count<ND>(), 0);
      rr = dd_value(sum[0]);
      const double rs = PC ? dd_value(sum[1]) : rr;
      ++iters;
      if (!(rr > thr)) {
        active = false;
        if (!isfinite(rr)) status = 1;
      } else if (!(rs > 0.0) || !isfinite(rs)) {
        active = false;
        status = 1;
      }
      // 4. p = r + beta p (p = M^-1 r + beta p; an explicit fma, so that both variants round
      // alike); unused after the last iteration
      double rn = rs;
      if constexpr (X) {
        const double a1 = rho / pqv;
        const DD t = dd_add(dd_add(DD{rho, 0.0}, dd_times(sum[R], -2.0 * a1)), dd_times(dd_times(sum[R + 1], a1), a1));
        rn = dd_value(t) > 0.0 ? dd_value(t) : 0.0;
      }
      const T be = static_cast<T>(rn / rho);
      rho = rs;
      mv = fresh(static_cast<const T*>(a.minv));
      tid = fresh_lane(tid);
#pragma unroll
      for (int s = 0; s < RPT; ++s) {
        const T sv = PC ? mv[s * NT + tid] * r[s] : r[s];
        s_p[s * NT + tid] = fma(be, s_p[s * NT + tid], sv);
        if (s % 8 == 7) asm volatile("" ::: "memory");
      }
    }
    __syncthreads();
  }

  const Global<T> Z = fresh(static_cast<T*>(a.y)) + c;
  const Global<const int32_t> row = fresh(a.p.row);
  tid = fresh_lane(tid);
#pragma unroll
  for (int s = 0; s < RPT; ++s) {
    const int pos = s * NT + tid;
    if (pos < a.n) Z[static_cast<int64_t>(row[pos]) * a.kb] = z[s];
    if (s % 4 == 3) asm volatile("" ::: "memory");
  }
  if (tid == 0) a.out[c] = ResOut{rr, rho0, iters, active ? 1 : 0, status, 0};
}

template <typename T, int NT, int RPT, bool W, bool PC, bool QL, int NQ>
hipError_t res_go(const ResArgs& a, int ncols, size_t lds, hipStream_t s) {
  const auto kernel = &k_resident<T, NT, RPT, W, PC, QL, NQ>;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(ncols), dim3(NT), lds, s, a);
  return hipGetLastError();
}
template <typename T, int NT, int RPT, bool QL, int NQ>
hipError_t res_kind(const ResArgs& a, int ncols, size_t lds, hipStream_t s) {
  if (a.p.w != nullptr)
    return a.minv != nullptr ? res_go<T, NT, RPT, true, true, QL, NQ>(a, ncols, lds, s)
                             : res_go<T, NT, RPT, true, false, QL, NQ>(a, ncols, lds, s);
  return a.minv != nullptr ? res_go<T, NT, RPT, false, true, QL, NQ>(a, ncols, lds, s)
                           : res_go<T, NT, RPT, false, false, QL, NQ>(a, ncols, lds, s);
}
// The kernel of form F[I] for the plan's workgroup size and slots.
template <typename T, size_t I = 0>
hipError_t res_dispatch(const ResArgs& a, int ncols, size_t lds, hipStream_t s) {
  constexpr const auto& F = *[]() {
    if constexpr (sizeof(T) == 4) return &kForms32;
    else return &kForms64;
  }();
  if constexpr (I < sizeof(F) / sizeof(F[0])) {
    constexpr ResForm f = F[I];
    if (a.p.nt != f.nt || a.p.rpt != f.rpt) return res_dispatch<T, I + 1>(a, ncols, lds, s);
    if (a.q == nullptr) {
      if constexpr (f.nt == 512)
        if (a.p.quads <= kResRegQuads) return res_kind<T, f.nt, f.rpt, true, kResRegQuads>(a, ncols, lds, s);
      if constexpr (res_q_inside(f, sizeof(T))) return res_kind<T, f.nt, f.rpt, true, 0>(a, ncols, lds, s);
    } else {
      if constexpr (res_q_outside(f, sizeof(T))) return res_kind<T, f.nt, f.rpt, false, 0>(a, ncols, lds, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace erc

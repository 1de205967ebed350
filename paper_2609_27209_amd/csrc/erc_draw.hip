// Curvature-guided subgraph draws on gfx950.
//
// Section 3.2 turns the normalised node scores of Eq. 7 and edge scores of Eq. 8 into
// sampling distributions; Section 4 trains on GraphSAINT-style subgraphs drawn from
// them.  This file draws indices from such a distribution and assembles the subgraph.
//
//   k_weight_sums, k_tile_scan, k_draw   W_i = floor(P_i 2^62) summed over tiles of 4096
//        items, exclusive prefix sums of the tiles and, within each, of its subtiles of 16,
//        and per draw the target t = floor(X T / 2^128) from two SplitMix64 words and the
//        item i with C_i <= t < C_{i+1}, found tile, subtile, item
//   k_mark (k_flag and k_pack for many draws), k_bits_up, k_bits_down   the drawn items as a
//        bitmap, its population counts, and from it the kept ids in increasing order and the
//        rank of every kept node
//   k_count_edges, k_count_up, k_count_down, k_emit_edges   the subgraph induced on the kept
//        nodes, from their rows alone
//   k_edge_bits, k_kept_ends             the same from the list of all edges, where a good part
//        of the nodes is kept
//   k_endpoints_of, k_renumber           the endpoints of the kept edges
//
// What bounds it: a draw reads every probability once (31M edges: 250 MB) and writes 1/16 of
// that, where the full prefix sums took two reads and a write; a subgraph touches the bitmaps
// (m / 8 or n / 8 bytes) and the rows of the kept nodes, where flags per edge took seven
// passes over 4 m bytes and two walks over all rows.  One draw and its subgraph, 12,000 nodes
// of 1.2M (31M edges) 0.75 -> 0.19 ms, 31,000 edges of 15.5M 0.53 -> 0.16 ms.
//
// Every sum here is an exact integer sum, so no result depends on the order in which
// partial sums are combined: draws and subgraphs repeat bit for bit and match any other
// exact evaluation of the same definition.
#include <hip/hip_runtime.h>

#include "erc_common.h"

namespace erc {
namespace {

constexpr int kSub = kDrawSub;             // items of a subtile
constexpr int kTile = kScanTile;           // items (or words) of a tile
constexpr int kSubs = kTile / kSub;        // subtiles of a tile
constexpr int kPerThread = kTile / kBlock; // consecutive counts of a thread
constexpr int kWords = kBitTile / kBlock;  // consecutive bitmap words of a thread
static_assert(kSub == 16 && kSubs == kBlock && kWords == 4, "lane layouts below");

// SplitMix64 output finaliser (Steele, Lea & Flood 2014), as for the projection signs.
__device__ __forceinline__ uint64_t sm_final(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;

// A probability's integer weight; `bad` is set by a value outside [0, 1] or NaN.  p * 2^62 is
// exact (a power-of-two scaling) and below 2^63; the conversion of its integer part is too.
__device__ __forceinline__ uint64_t weight_of(double p, bool& bad) {
  if (!(p >= 0.0 && p <= 1.0)) {
    bad = true;
    return 0;
  }
  return static_cast<uint64_t>(p * 0x1p62);
}

template <typename U>
__device__ __forceinline__ U wave_sum(U x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

// Sum of one value per thread over the block, in every thread.
template <typename U>
__device__ __forceinline__ U block_sum(U x) {
  __shared__ U s[kWavesPerBlock];
  x = wave_sum(x);
  __syncthreads();  // a previous call's values may still be read
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = x;
  __syncthreads();
  U t = 0;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) t += s[w];
  return t;
}

// Exclusive scan of one value per thread over a block of NW wavefronts, in thread order;
// `total` receives the block sum.
template <int NW, typename U>
__device__ __forceinline__ U block_exclusive_scan(U x, U& total) {
  __shared__ U s_wave[NW];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  U inc = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const U y = __shfl_up(inc, off);
    if (lane >= off) inc += y;
  }
  __syncthreads();
  if (lane == 63) s_wave[wv] = inc;
  __syncthreads();
  U before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const U s = s_wave[w];
    if (w < wv) before += s;
    total += s;
  }
  return before + inc - x;
}

// ---- draws -----------------------------------------------------------------------------

// One block per tile: the exclusive prefix sums of its subtiles' weights within the tile ->
// sub, the tile's weight sum -> tsum, and the fp64 sum of its probabilities -> psum (a fixed
// order).  A wavefront reads 128 consecutive items per load (16 bytes per lane where the array
// is 16-byte aligned), eight subtiles of eight lanes each.
__global__ __launch_bounds__(kBlock) void k_weight_sums(const double* __restrict__ P, int64_t N,
                                                        uint64_t* __restrict__ sub,
                                                        uint64_t* __restrict__ tsum,
                                                        double* __restrict__ psum,
                                                        uint32_t* status) {
  constexpr int kLoads = kTile / kBlock / 2;  // pairs per thread
  __shared__ uint64_t s_sub[kSubs];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTile + wv * (kTile / kWavesPerBlock);
  const bool wide = t0 + kTile / kWavesPerBlock <= N && (reinterpret_cast<uintptr_t>(P) & 15) == 0;
  typedef double D2 __attribute__((ext_vector_type(2)));
  D2 p[kLoads];
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const int64_t i = t0 + k * 128 + 2 * lane;
    if (wide) {
      p[k] = *reinterpret_cast<const D2*>(P + i);
    } else {
      p[k].x = i < N ? P[i] : 0.0;
      p[k].y = i + 1 < N ? P[i + 1] : 0.0;
    }
  }
  bool bad = false;
  double pall = 0.0;
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    uint64_t w = weight_of(p[k].x, bad) + weight_of(p[k].y, bad);
    pall += p[k].x + p[k].y;
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) w += __shfl_xor(w, off);
    if ((lane & 7) == 0) s_sub[wv * (kSubs / kWavesPerBlock) + k * 8 + (lane >> 3)] = w;
  }
  if (__ballot(bad) != 0 && lane == 0) atomicOr(status, kDrawBadProb);
  __syncthreads();
  uint64_t all;
  const uint64_t before = block_exclusive_scan<kWavesPerBlock>(s_sub[threadIdx.x], all);
  sub[static_cast<int64_t>(blockIdx.x) * kSubs + threadIdx.x] = before;
  pall = block_sum(pall);
  if (threadIdx.x == 0) {
    tsum[blockIdx.x] = all;
    psum[blockIdx.x] = pall;
  }
}

// One block of 1024 threads: tile sums to their exclusive prefix sums in place, total to
// tsum[nb].  Each thread takes consecutive tiles, so that the block scans once.  The fp64 sum must not
// exceed 1.5 (the integer weights then sum below 2^63, so no 64-bit sum above can have
// wrapped) and the weights must not be all zero.
constexpr int kMidThreads = 1024;
__global__ __launch_bounds__(kMidThreads) void k_tile_scan(uint64_t* __restrict__ tsum, int64_t nb,
                                                           const double* __restrict__ psum,
                                                           uint32_t* status) {
  __shared__ double s_d[kMidThreads / 64];
  const int64_t per = (nb + kMidThreads - 1) / kMidThreads;
  const int64_t a = threadIdx.x * per;
  const int64_t b = a + per < nb ? a + per : nb;
  uint64_t mine = 0;
  double d = 0.0;
  for (int64_t i = a; i < b; ++i) {
    mine += tsum[i];
    d += psum[i];
  }
  uint64_t total;
  uint64_t run = block_exclusive_scan<kMidThreads / 64>(mine, total);
  for (int64_t i = a; i < b; ++i) {
    const uint64_t x = tsum[i];
    tsum[i] = run;
    run += x;
  }
  d = wave_sum(d);
  if ((threadIdx.x & 63) == 0) s_d[threadIdx.x >> 6] = d;
  __syncthreads();
  if (threadIdx.x == 0) {
    tsum[nb] = total;
    double all = 0.0;
    for (int w = 0; w < kMidThreads / 64; ++w) all += s_d[w];
    if (!(all <= 1.5)) atomicOr(status, kDrawSumTooLarge);
    if (total == 0) atomicOr(status, kDrawAllZero);
  }
}

// One thread per draw, draws first .. first + draws - 1.  X = x_hi 2^64 + x_lo from outputs 2d and 2d+1 of SplitMix64 started
// at `base`; t = floor(X T / 2^128) = hi64(x_hi T + hi64(x_lo T)) is uniform on [0, T), and
// the drawn item is the last i with C_i <= t: the tile, then its subtile by binary searches of
// their prefix sums, then the item among the subtile's 16 (two cache lines).  (A group of 16
// lanes per draw with 16-way searches took 6 us instead of 9 for a few thousand draws but 1.1
// ms instead of 0.6 for 4.8M, at 16 cache lines a step.)
__global__ __launch_bounds__(kBlock) void k_draw(const double* __restrict__ P, int64_t N,
                                                 const uint64_t* __restrict__ sub,
                                                 const uint64_t* __restrict__ tsum, int64_t nb,
                                                 int64_t first, int64_t draws, uint64_t base,
                                                 const uint32_t* __restrict__ status,
                                                 int64_t* __restrict__ idx) {
  const uint32_t st = *status;
  const uint64_t T = tsum[nb];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t d = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; d < draws; d += stride) {
    if (st != 0u) {
      idx[d] = -1;
      continue;
    }
    const uint64_t ctr = 2ull * static_cast<uint64_t>(first + d);
    const uint64_t xh = sm_final(base + (ctr + 1ull) * kGolden);
    const uint64_t xl = sm_final(base + (ctr + 2ull) * kGolden);
    const uint64_t a_lo = xh * T;
    const uint64_t a_hi = __umul64hi(xh, T);
    const uint64_t s = a_lo + __umul64hi(xl, T);
    uint64_t t = a_hi + (s < a_lo ? 1ull : 0ull);
    // last i of [0, n) with c[i] <= t (c[0] <= t); t becomes the rest beyond c[i]
    auto search = [&](const uint64_t* __restrict__ c, int64_t n) {
      int64_t lo = 0, hi = n;
      uint64_t at = c[0];
      while (hi - lo > 1) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        const uint64_t x = c[mid];
        if (x <= t) {
          lo = mid;
          at = x;
        } else {
          hi = mid;
        }
      }
      t -= at;
      return lo;
    };
    const int64_t tile = search(tsum, nb);
    const int64_t i0 = tile * kTile + search(sub + tile * kSubs, kSubs) * kSub;
    double p[kSub];
#pragma unroll
    for (int k = 0; k < kSub; ++k) p[k] = P[i0 + k < N ? i0 + k : N - 1];
    // the last item whose exclusive prefix is <= t; items past N cannot be reached, as the
    // subtile's weights sum above t
    bool bad = false;
    uint64_t c = 0;
    int last = 0;
#pragma unroll
    for (int k = 0; k < kSub; ++k) {
      if (i0 + k < N && c <= t) last = k;
      c += weight_of(p[k], bad);
    }
    idx[d] = i0 + last;
  }
}

// ---- subgraphs -------------------------------------------------------------------------

// Sets a bit unless it is seen set already: hubs are marked over and over, and atomics on one
// word go one after the other (endpoints of 3M edges of a 1.2M-node graph: 7.9 ms without the
// look, 0.52 ms with it, and one of a run of equal u marking).  A stale zero costs an atomic and nothing else.
__device__ __forceinline__ void set_bit(uint32_t* bits, int64_t i) {
  uint32_t* w = bits + (i >> 5);
  const uint32_t b = 1u << (i & 31);
  if ((__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & b) == 0u) atomicOr(w, b);
}

__global__ __launch_bounds__(kBlock) void k_mark(const int64_t* __restrict__ idx,
                                                 int64_t count, int64_t N,
                                                 uint32_t* __restrict__ bits,
                                                 uint32_t* status) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t d = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; d < count;
       d += stride) {
    const int64_t i = idx[d];
    if (i < 0 || i >= N) atomicOr(status, kSubBadIndex);
    else set_bit(bits, i);
  }
}

// Marks of many items: a plain store into a byte per item, which k_pack makes bits of.  Atomics
// run at about 15 per ns (4.8M draws of 1.2M nodes: 312 us to mark bits, where stores take
// about 55), but bytes have to be cleared and read.
__global__ __launch_bounds__(kBlock) void k_flag(const int64_t* __restrict__ idx,
                                                 int64_t count, int64_t N,
                                                 uint8_t* __restrict__ flags,
                                                 uint32_t* status) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t d = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; d < count;
       d += stride) {
    const int64_t i = idx[d];
    if (i < 0 || i >= N) atomicOr(status, kSubBadIndex);
    else flags[i] = 1;
  }
}

// One thread per bitmap word: 32 bytes of 0 or 1 to its bits, four bytes to four bits by one
// product (the ten partial products fall on different bits).
__global__ __launch_bounds__(kBlock) void k_pack(const uint8_t* __restrict__ flags,
                                                 uint32_t* __restrict__ bits) {
  const int64_t w = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  const uint4* f = reinterpret_cast<const uint4*>(flags) + w * 2;
  const uint4 a = f[0], b = f[1];
  const uint32_t x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t out = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) out |= ((x[k] * 0x01020408u) >> 24) << (4 * k);
  bits[w] = out;
}

// One block per bitmap tile, four words (a 16-byte load) per thread; the bitmaps are 16-byte
// aligned and padded to whole tiles by the host layout.  Tiles of 1024 words spread the few
// set bits of a draw over enough blocks (nodes of the 1.2M-node case: 6.4 us against 16.0 with
// tiles of 4096).
__global__ __launch_bounds__(kBlock) void k_bits_up(const uint32_t* __restrict__ bits,
                                                    uint32_t* __restrict__ tile) {
  const uint4 v = reinterpret_cast<const uint4*>(bits)[static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x];
  const uint32_t c = block_sum(static_cast<uint32_t>(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w)));
  if (threadIdx.x == 0) tile[blockIdx.x] = c;
}

// The sum of tile[0 .. blockIdx.x): each block adds the counts before it itself (a few
// hundred tiles at 10^8 bits), which saves a launch for their scan.
__device__ __forceinline__ uint32_t tiles_before(const uint32_t* __restrict__ tile) {
  uint32_t c = 0;
  for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kBlock) c += tile[k];
  return block_sum(c);
}

// One block per tile of words: the ids of its set bits, in increasing order, to out (rank
// order), and with `prefix` the rank of each word's first bit.  The last block writes the
// total.
template <typename Id>
__global__ __launch_bounds__(kBlock) void k_bits_down(const uint32_t* __restrict__ bits,
                                                      const uint32_t* __restrict__ tile,
                                                      uint32_t* __restrict__ prefix,
                                                      Id* __restrict__ out, uint32_t* total) {
  const uint32_t before = tiles_before(tile);
  const int64_t w0 = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * kWords;
  const uint4 x4 = *reinterpret_cast<const uint4*>(bits + w0);
  const uint32_t v[kWords] = {x4.x, x4.y, x4.z, x4.w};
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kWords; ++k) c += __popc(v[k]);
  uint32_t all;
  uint32_t at = before + block_exclusive_scan<kWavesPerBlock>(c, all);
#pragma unroll
  for (int k = 0; k < kWords; ++k) {
    if (prefix != nullptr) prefix[w0 + k] = at;
    for (uint32_t x = v[k]; x != 0; x &= x - 1)
      out[at++] = static_cast<Id>((w0 + k) * 32 + (__ffs(x) - 1));
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = before + all;
}

__device__ __forceinline__ bool is_set(const uint32_t* __restrict__ bits, int32_t i) {
  return (bits[i >> 5] >> (i & 31)) & 1u;
}
__device__ __forceinline__ uint32_t rank_of(const uint32_t* __restrict__ bits,
                                            const uint32_t* __restrict__ prefix, int32_t i) {
  return prefix[i >> 5] + __popc(bits[i >> 5] & ((1u << (i & 31)) - 1u));
}

// The upper (u < v) entries of the kept nodes' rows whose other end is kept too.  A wavefront
// takes one kept node; f is called with every lane's entry in order.  A row of more than 64
// entries is read kRows * 64 at a time, the next ones while these are looked up, and no load
// sits behind a branch, so that a hub's thousands of entries do not wait for one load after
// the other (1.2M-node case, longest row 8000 entries: 37 us to count and 54 to emit with a
// branch per load, 23 and 37 without).
constexpr int kRows = 16;
template <typename F>
__device__ __forceinline__ void for_kept_entries(const DevGraph& g, const uint32_t* __restrict__ bits,
                                                 int u, F f) {
  const int lane = threadIdx.x & 63;
  const int64_t end = g.rowptr[u + 1];
  const int64_t e0 = g.ubase[u];
  const int64_t beg = end - (g.ubase[u + 1] - e0);
  if (beg == end) return;
  auto entry = [&](int64_t pos) {
    const int64_t p = pos + lane;
    return g.col[p < end ? p : end - 1];
  };
  if (end - beg <= 64) {
    const int32_t v = entry(beg);
    f(is_set(bits, v) & (beg + lane < end), v, e0 + lane);
    return;
  }
  int32_t next[kRows];
#pragma unroll
  for (int k = 0; k < kRows; ++k) next[k] = entry(beg + k * 64);
  for (int64_t pos = beg; pos < end; pos += kRows * 64) {
    int32_t v[kRows];
    bool keep[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) v[k] = next[k];
#pragma unroll
    for (int k = 0; k < kRows; ++k) next[k] = entry(pos + (kRows + k) * 64);
#pragma unroll
    for (int k = 0; k < kRows; ++k) keep[k] = is_set(bits, v[k]) & (pos + k * 64 + lane < end);
#pragma unroll
    for (int k = 0; k < kRows; ++k)
      if (pos + k * 64 < end) f(keep[k], v[k], e0 + (pos - beg) + k * 64 + lane);
  }
}

__global__ __launch_bounds__(kBlock) void k_count_edges(DevGraph g, const uint32_t* __restrict__ bits,
                                                        const int32_t* __restrict__ nodes,
                                                        const uint32_t* __restrict__ nkept,
                                                        uint32_t* __restrict__ cnt) {
  const int64_t n = *nkept;
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kWavesPerBlock;
  for (int64_t i = blockIdx.x + static_cast<int64_t>(threadIdx.x >> 6) * gridDim.x; i < n; i += nw) {
    uint32_t c = 0;
    for_kept_entries(g, bits, nodes[i], [&](bool keep, int32_t, int64_t) { c += __popcll(__ballot(keep)); });
    if ((threadIdx.x & 63) == 0) cnt[i] = c;
  }
}

// Exclusive prefix sums of the kept nodes' counts in two launches, as for the bitmaps (the
// grid covers the most nodes that can be kept; tiles past the last are empty).
__global__ __launch_bounds__(kBlock) void k_count_up(const uint32_t* __restrict__ cnt,
                                                     const uint32_t* __restrict__ nkept,
                                                     uint32_t* __restrict__ tile) {
  const int64_t n = *nkept;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTile;
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kPerThread; ++k) {
    const int64_t i = t0 + k * kBlock + threadIdx.x;
    if (i < n) c += cnt[i];
  }
  c = block_sum(c);
  if (threadIdx.x == 0) tile[blockIdx.x] = c;
}
__global__ __launch_bounds__(kBlock) void k_count_down(uint32_t* __restrict__ cnt,
                                                       const uint32_t* __restrict__ nkept,
                                                       const uint32_t* __restrict__ tile,
                                                       uint32_t* total) {
  const int64_t n = *nkept;
  const uint32_t before = tiles_before(tile);
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kTile + threadIdx.x * kPerThread;
  uint32_t v[kPerThread], c = 0;
#pragma unroll
  for (int k = 0; k < kPerThread; ++k) {
    v[k] = i0 + k < n ? cnt[i0 + k] : 0u;
    c += v[k];
  }
  uint32_t all;
  uint32_t at = before + block_exclusive_scan<kWavesPerBlock>(c, all);
#pragma unroll
  for (int k = 0; k < kPerThread; ++k) {
    if (i0 + k < n) cnt[i0 + k] = at;
    at += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = before + all;
}

__global__ __launch_bounds__(kBlock) void k_emit_edges(DevGraph g, const uint32_t* __restrict__ bits,
                                                       const uint32_t* __restrict__ prefix,
                                                       const int32_t* __restrict__ nodes,
                                                       const uint32_t* __restrict__ nkept,
                                                       const uint32_t* __restrict__ off,
                                                       int64_t* __restrict__ edges,
                                                       int32_t* __restrict__ uo,
                                                       int32_t* __restrict__ vo) {
  const int64_t n = *nkept;
  const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kWavesPerBlock;
  for (int64_t i = blockIdx.x + static_cast<int64_t>(threadIdx.x >> 6) * gridDim.x; i < n; i += nw) {
    uint32_t at = off[i];
    for_kept_entries(g, bits, nodes[i], [&](bool keep, int32_t v, int64_t e) {
      const uint64_t m = __ballot(keep);
      if (keep) {
        const uint32_t k = at + __popcll(m & below);
        edges[k] = e;
        uo[k] = static_cast<int32_t>(i);
        vo[k] = static_cast<int32_t>(rank_of(bits, prefix, v));
      }
      at += __popcll(m);
    });
  }
}

// Bits of the edges whose ends are both kept, for draws that keep a good part of the nodes: every
// edge once, in order, where the rows' upper parts are short and uneven.  A wavefront takes
// 256 edges, four per lane; every word of the bitmap is written.  What bounds it: the list
// (8 bytes per edge) and the lookups, which hit the caches.
__global__ __launch_bounds__(kBlock) void k_edge_bits(DevGraph g, const uint32_t* __restrict__ bits,
                                                      uint64_t* __restrict__ ebits) {
  const int lane = threadIdx.x & 63;
  const int64_t e0 = (static_cast<int64_t>(blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6)) * 256;
  int32_t u[4], v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t e = e0 + k * 64 + lane;
    u[k] = g.eu[e < g.m ? e : g.m - 1];
    v[k] = g.ev[e < g.m ? e : g.m - 1];
  }
  uint64_t mine = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t m = __ballot(is_set(bits, u[k]) & is_set(bits, v[k]) & (e0 + k * 64 + lane < g.m));
    if (lane == k) mine = m;
  }
  if (lane < 4) ebits[e0 / 64 + lane] = mine;
}

// New numbers of the kept edges' ends.
__global__ __launch_bounds__(kBlock) void k_kept_ends(DevGraph g, const int64_t* __restrict__ edges,
                                                      const uint32_t* __restrict__ mkept,
                                                      const uint32_t* __restrict__ bits,
                                                      const uint32_t* __restrict__ prefix,
                                                      int32_t* __restrict__ uo,
                                                      int32_t* __restrict__ vo) {
  const int64_t m = *mkept;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; k < m; k += stride) {
    const int64_t e = edges[k];
    uo[k] = static_cast<int32_t>(rank_of(bits, prefix, g.eu[e]));
    vo[k] = static_cast<int32_t>(rank_of(bits, prefix, g.ev[e]));
  }
}

// Endpoints of the kept edges (old numbering) and their marks, bits or (FLAGS) bytes.
template <bool FLAGS>
__global__ __launch_bounds__(kBlock) void k_endpoints_of(DevGraph g, const int64_t* __restrict__ edges,
                                                         const uint32_t* __restrict__ mkept,
                                                         int32_t* __restrict__ uo,
                                                         int32_t* __restrict__ vo,
                                                         uint32_t* __restrict__ bits,
                                                         uint8_t* __restrict__ flags) {
  const int64_t m = *mkept;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; k < m; k += stride) {
    const int64_t e = edges[k];
    const int32_t lo = g.eu[e], v = g.ev[e];
    uo[k] = lo;
    vo[k] = v;
    // edges run by u: one of a run of equal u marks it
    const int prev = __shfl_up(lo, 1);
    const bool first = (threadIdx.x & 63) == 0 || prev != lo;
    if constexpr (FLAGS) {
      if (first) flags[lo] = 1;
      flags[v] = 1;
    } else {
      if (first) set_bit(bits, lo);
      set_bit(bits, v);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_renumber(const uint32_t* __restrict__ bits,
                                                     const uint32_t* __restrict__ prefix,
                                                     const uint32_t* __restrict__ mkept,
                                                     int32_t* __restrict__ uo,
                                                     int32_t* __restrict__ vo) {
  const int64_t m = *mkept;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; k < m; k += stride) {
    uo[k] = static_cast<int32_t>(rank_of(bits, prefix, uo[k]));
    vo[k] = static_cast<int32_t>(rank_of(bits, prefix, vo[k]));
  }
}

int blocks_for(int64_t count, int64_t per_block) {
  const int64_t g = (count + per_block - 1) / per_block;
  return static_cast<int>(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

#define ERC_DLAUNCH(kernel, grid, stream, ...) \
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), 0, stream, __VA_ARGS__)

}  // namespace

hipError_t launch_draw_sums(const double* prob, int64_t N, const DrawWork& w, hipStream_t s) {
  const int64_t nb = scan_blocks(N);
  hipError_t e = launch_fill_u32(w.status, 0u, 1, s);
  if (e != hipSuccess) return e;
  ERC_DLAUNCH(k_weight_sums, nb, s, prob, N, w.sub, w.tsum, w.psum, w.status);
  hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(kMidThreads), 0, s, w.tsum, nb, w.psum, w.status);
  return hipGetLastError();
}

hipError_t launch_draw(const double* prob, int64_t N, int64_t first, int64_t draws, uint64_t base,
                       const DrawWork& w, int64_t* idx, hipStream_t s) {
  if (draws <= 0) return hipSuccess;
  ERC_DLAUNCH(k_draw, blocks_for(draws, kBlock), s, prob, N, w.sub, w.tsum, scan_blocks(N), first, draws,
              base, w.status, idx);
  return hipGetLastError();
}

// Whether `count` marks of N items go through bytes: where their atomics (15 per ns) take
// longer than clearing and packing the bytes (2 N at 4 TB/s) and two launches.  Whole subgraph
// calls, bits against bytes: 310,200 draws of 31M edges 0.18 against 0.10 ms, 3.1M 0.67 against
// 0.25; 480,000 of 4.8M 0.17 against 0.09; 33,000 of 110,000 (bits either way) 0.08.
constexpr int64_t kFlagMin = 65536;
static bool by_flags(int64_t count, int64_t N) { return count > kFlagMin && count > N / 64; }

// The marks that `mark` leaves (bits into `bits`, or bytes into w.flags) as a bitmap of N items.
template <typename Mark>
static hipError_t marked(bool flags, int64_t N, const SubgraphWork& w, uint32_t* bits, hipStream_t s, Mark mark) {
  if (flags) {
    const hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(w.flags), 0u, sub_words(N) * 8, s);
    if (e != hipSuccess) return e;
  }
  mark();
  if (flags) ERC_DLAUNCH(k_pack, sub_words(N) / kBlock, s, w.flags, bits);
  return hipGetLastError();
}

// Node draws of at least this share of the nodes look at every edge, fewer at the rows of the
// kept nodes.  Whole calls, rows against every edge: 1.2M nodes and 31M edges, draws of 1/100 of
// the nodes 0.12 against 0.16 ms, 1/10 0.23 against 0.21, as many as nodes 0.71 against 0.45,
// four times as many 1.18 against 0.67 (with marks by bits, and rows, 1.47; flags per edge and
// two walks over all rows had taken 1.32); 1.2M nodes and 4.8M edges, 1/100 0.08 either way,
// 1/10 0.15 against 0.09, four times as many 0.70 against 0.17 (0.98; 0.42).
constexpr int64_t kEveryEdge = 16;

hipError_t launch_subgraph(const DevGraph& g, int items, const int64_t* idx, int64_t count,
                           const SubgraphWork& w, int32_t* nodes, int64_t* edges, int32_t* uo,
                           int32_t* vo, hipStream_t s) {
  const int64_t ntile = sub_words(g.n) / kBitTile, mtile = sub_words(g.m) / kBitTile;
  uint32_t* status = w.head;      // status, kept nodes, kept edges
  uint32_t* nkept = w.head + 1;
  uint32_t* mkept = w.head + 2;
  // the head and the bitmaps follow each other: one fill
  hipError_t err = launch_fill_u32(w.head, 0u, w.clear_words, s);
  if (err != hipSuccess) return err;
  auto mark = [&](int64_t N, uint32_t* bits) {
    const bool flags = by_flags(count, N);
    return marked(flags, N, w, bits, s, [&]() {
      if (flags) ERC_DLAUNCH(k_flag, blocks_for(count, kBlock), s, idx, count, N, w.flags, status);
      else if (count > 0) ERC_DLAUNCH(k_mark, blocks_for(count, kBlock), s, idx, count, N, bits, status);
    });
  };
  if (items == 0) {
    if ((err = mark(g.n, w.nbits)) != hipSuccess) return err;
    ERC_DLAUNCH(k_bits_up, ntile, s, w.nbits, w.tile);
    ERC_DLAUNCH(k_bits_down<int32_t>, ntile, s, w.nbits, w.tile, w.nprefix, nodes, nkept);
    const int64_t most = count < g.n ? count : g.n;
    if (most > 0 && g.m > 0 && count >= g.n / kEveryEdge) {
      ERC_DLAUNCH(k_edge_bits, sub_words(g.m) * 32 / (256 * kWavesPerBlock), s, g, w.nbits,
                  reinterpret_cast<uint64_t*>(w.ebits));
      ERC_DLAUNCH(k_bits_up, mtile, s, w.ebits, w.tile);
      ERC_DLAUNCH(k_bits_down<int64_t>, mtile, s, w.ebits, w.tile, static_cast<uint32_t*>(nullptr), edges, mkept);
      ERC_DLAUNCH(k_kept_ends, blocks_for(g.m, kBlock), s, g, edges, mkept, w.nbits, w.nprefix, uo, vo);
    } else if (most > 0 && g.m > 0) {
      const int grid = blocks_for(most, kWavesPerBlock);
      ERC_DLAUNCH(k_count_edges, grid, s, g, w.nbits, nodes, nkept, w.cnt);
      ERC_DLAUNCH(k_count_up, scan_blocks(most), s, w.cnt, nkept, w.tile);
      ERC_DLAUNCH(k_count_down, scan_blocks(most), s, w.cnt, nkept, w.tile, mkept);
      ERC_DLAUNCH(k_emit_edges, grid, s, g, w.nbits, w.nprefix, nodes, nkept, w.cnt, edges, uo, vo);
    }
  } else if (count > 0) {  // (the host refuses drawn edges of a graph without any)
    const int64_t most = count < g.m ? count : g.m;
    const int grid = blocks_for(most, kBlock);
    if ((err = mark(g.m, w.ebits)) != hipSuccess) return err;
    ERC_DLAUNCH(k_bits_up, mtile, s, w.ebits, w.tile);
    ERC_DLAUNCH(k_bits_down<int64_t>, mtile, s, w.ebits, w.tile, static_cast<uint32_t*>(nullptr), edges,
                mkept);
    const bool flags = by_flags(most, g.n);
    err = marked(flags, g.n, w, w.nbits, s, [&]() {
      if (flags) ERC_DLAUNCH(k_endpoints_of<true>, grid, s, g, edges, mkept, uo, vo, w.nbits, w.flags);
      else ERC_DLAUNCH(k_endpoints_of<false>, grid, s, g, edges, mkept, uo, vo, w.nbits, w.flags);
    });
    if (err != hipSuccess) return err;
    ERC_DLAUNCH(k_bits_up, ntile, s, w.nbits, w.tile);
    ERC_DLAUNCH(k_bits_down<int32_t>, ntile, s, w.nbits, w.tile, w.nprefix, nodes, nkept);
    ERC_DLAUNCH(k_renumber, grid, s, w.nbits, w.nprefix, mkept, uo, vo);
  }
  return hipGetLastError();
}

}  // namespace erc

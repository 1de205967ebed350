// Plan, LDS size and launches of the resident CG (erc_resident.h).
#include <hip/hip_runtime.h>

#include "erc_common.h"
#include "erc_resident.h"

namespace erc {
namespace {

constexpr size_t kMaxLds = 160 * 1024;

// Entries of the plan's slots from the CSR arrays: one wavefront per slot.
template <typename T>
__global__ __launch_bounds__(64) void k_res_fill(DevGraph g, uint16_t* __restrict__ idx,
                                                 T* __restrict__ wq) {
  const int lane = threadIdx.x;
  const int wv = blockIdx.x / g.res.rpt, s = blockIdx.x % g.res.rpt;
  const int pos = s * g.res.nt + wv * 64 + lane;
  const int t0 = g.res.off[blockIdx.x], t1 = g.res.off[blockIdx.x + 1];
  int64_t b = 0;
  int deg = 0;
  if (pos >= g.res.nheavy && pos < g.n) {
    const int i = g.res.row[pos];
    b = g.rowptr[i];
    deg = static_cast<int>(g.rowptr[i + 1] - b);
  }
  const T* __restrict__ w = static_cast<const T*>(g.w);
  for (int t = t0; t < t1; ++t) {
    for (int u = 0; u < 4; ++u) {
      const int k = (t - t0) * 4 + u;
      const int64_t o = (static_cast<int64_t>(t) * 64 + lane) * 4 + u;
      idx[o] = k < deg ? g.res.pos[g.col[b + k]] : static_cast<uint16_t>(pos);
      if (wq != nullptr) wq[o] = k < deg ? w[b + k] : T(0);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_res_cpos(DevGraph g, uint16_t* __restrict__ cpos) {
  for (int64_t e = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; e < g.nnz;
       e += static_cast<int64_t>(gridDim.x) * kBlock)
    cpos[e] = g.res.pos[g.col[e]];
}

// M^-1 by position, zero past the last row.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_res_minv(DevGraph g, double delta,
                                                     T* __restrict__ minv) {
  const int pos = blockIdx.x * kBlock + threadIdx.x;
  if (pos >= g.res.rpt * g.res.nt) return;
  minv[pos] = pos < g.n ? static_cast<T>(1.0 / (g.deg[g.res.row[pos]] + delta)) : T(0);
}

}  // namespace

ResForm res_form(erc_dtype dt, int64_t n) {
  if (dt == ERC_F32) {
    for (const ResForm& f : kForms32)
      if (int64_t{f.nt} * f.rpt >= n) return f;
  } else {
    for (const ResForm& f : kForms64)
      if (int64_t{f.nt} * f.rpt >= n) return f;
  }
  return ResForm{0, 0};
}

int res_q_place(ResForm f, int64_t n, int nchunk, erc_dtype dt, size_t* lds) {
  const size_t sz = dt == ERC_F32 ? 4 : 8;
  const size_t red = kResSums * static_cast<size_t>(f.nt / 64) * 2 * sizeof(double);
  const size_t p = static_cast<size_t>(f.nt) * f.rpt * sz;
  const size_t parts = res_parts(f, sz) ? kResFolds * static_cast<size_t>(f.nt) * 8 : 0;
  *lds = red + static_cast<size_t>((nchunk + 1) & ~1) * 8 + parts;
  if (res_q_inside(f, sz) && p + *lds + n * sz <= kMaxLds) {
    *lds += n * sz;
    return 1;
  }
  return res_q_outside(f, sz) && p + *lds <= kMaxLds ? 2 : 0;
}

hipError_t launch_res_fill(const DevGraph& g, erc_dtype dt, hipStream_t s) {
  uint16_t* idx = const_cast<uint16_t*>(g.res.idx);
  void* w = const_cast<void*>(g.res.w);
  const int slots = g.res.nt / 64 * g.res.rpt;
  if (dt == ERC_F32)
    hipLaunchKernelGGL(k_res_fill<float>, dim3(slots), dim3(64), 0, s, g, idx, static_cast<float*>(w));
  else
    hipLaunchKernelGGL(k_res_fill<double>, dim3(slots), dim3(64), 0, s, g, idx, static_cast<double*>(w));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || g.res.nchunk == 0) return e;
  const int64_t grid = ceil_div(g.nnz, kBlock);
  hipLaunchKernelGGL(k_res_cpos, dim3(static_cast<unsigned>(grid < 2048 ? grid : 2048)), dim3(kBlock), 0, s,
                     g, const_cast<uint16_t*>(g.res.cpos));
  return hipGetLastError();
}

hipError_t launch_res_minv(const DevGraph& g, erc_dtype dt, double delta, void* minv, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(ceil_div(g.res.rpt * g.res.nt, kBlock)));
  if (dt == ERC_F32)
    hipLaunchKernelGGL(k_res_minv<float>, grid, dim3(kBlock), 0, s, g, delta, static_cast<float*>(minv));
  else
    hipLaunchKernelGGL(k_res_minv<double>, grid, dim3(kBlock), 0, s, g, delta, static_cast<double*>(minv));
  return hipGetLastError();
}

hipError_t launch_resident(const DevGraph& g, erc_dtype dt, void* y, void* q, int kb, int ncols,
                           double delta, double tol2, int max_iter, const void* minv_pos,
                           ResOut* out, hipStream_t s) {
  ResArgs a;
  a.p = g.res;
  a.n = g.n;
  a.csr_w = g.w;
  a.y = y;
  a.q = q;
  a.kb = kb;
  a.max_iter = max_iter;
  a.delta = delta;
  a.tol2 = tol2;
  a.minv = minv_pos;
  a.out = out;
  size_t lds = 0;
  if (res_q_place(ResForm{g.res.nt, g.res.rpt}, g.n, g.res.nchunk, dt, &lds) != g.res.on ||
      (g.res.on == 2) != (q != nullptr))
    return hipErrorInvalidValue;
  return dt == ERC_F32 ? res_solve_f32(a, ncols, lds, s) : res_solve_f64(a, ncols, lds, s);
}

}  // namespace erc

// Internal declarations shared by the host library and the HIP kernels.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime_api.h>

#include "../../include/erc.h"

namespace erc {

// Threads per block of every kernel (4 wavefronts of 64).
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / 64;
// Fan-in of one level of the deterministic grid reduction tree.
constexpr int kTreeFan = 32;
// Largest grid of a launch that reduces through the ticket tree directly.
constexpr int kMaxTreeGrid = 2048;

// Device view of the graph operator (all pointers are device memory inside the
// caller's graph buffer).
// A light row of the SpMM plan with its CSR range, so that one 16-byte load gives a
// lane group everything it needs to start on the row.
struct alignas(16) LightRow {
  int64_t beg;  // rowptr[row]
  int32_t row;
  int32_t deg;  // rowptr[row + 1] - rowptr[row]
};

// Plan of the resident CG (erc_resident.hip), kept for graphs of up to a few ten thousand
// nodes.  Rows sit at positions 0 .. n-1: first the rows of more than kResHeavy entries,
// then the others by decreasing degree.  Thread t of a workgroup of nt threads owns the
// positions t, t + nt, ... (one per slot).  The entries of the 64 rows of
// wavefront v's slot s are stored as quads off[v * rpt + s] .. off[v * rpt + s + 1] - 1:
// quad t of lane l holds four (position, weight) pairs at (t * 64 + l) * 4, padded with the
// row's own position and weight zero.
constexpr int kResHeavy = 128;   // rows above this many entries are summed by whole wavefronts
constexpr int kResChunk = 256;  // in chunks of this many entries
constexpr int kResPadQuads = 4;  // readable quads past the last one
struct ResPlan {
  int32_t on;             // 0: no such plan; else where q is kept: 1 in LDS, 2 in memory
  int32_t nt;             // threads of a workgroup
  int32_t rpt;            // slots
  int32_t nheavy;         // positions below this are rows of more than kResHeavy entries
  int32_t nchunk;         // chunks of those rows
  int32_t quads;          // most quads of one wavefront
  const int32_t* row;     // rpt * nt: row at each position (0 beyond n)
  const uint16_t* pos;    // n: position of each row
  const int32_t* off;     // nt / 64 * rpt + 1
  const uint16_t* idx;    // quads x 64 x 4
  const void* w;          // the same shape, working precision (weighted graphs)
  const uint16_t* cpos;   // nnz: position of each CSR entry's column (the chunks read it)
  const int32_t* hpos;    // nchunk: position of each chunk's row
  const int32_t* hbeg;    // nchunk: first entry in CSR
  const int32_t* hlen;    // nchunk
  const int32_t* hc0;     // nheavy + 1: first chunk of each long row
};

// What the resident CG reports for each column.
struct ResOut {
  double rr, rho0;
  int32_t iters, active, status, pad;
};

struct DevGraph {
  int32_t n;
  int64_t nnz;
  int64_t m;
  int weighted;              // 0: unit weights, w == nullptr
  const int64_t* rowptr;     // n+1
  const int32_t* col;        // nnz, ascending per row
  const void* w;             // nnz, working precision
  const int32_t* eid;        // nnz, canonical edge id of each entry
  const double* sw;          // m, sqrt(w_e) rounded once from fp64(w_e)
  int sw_from_w;             // 1 if w holds the input weights exactly (sqrt on the fly)
  const int64_t* ubase;      // n+1, id of the first edge (u, v>u) of row u
  const double* deg;         // n, d_i = sum_j w_ij in fp64 (diagonal of L)

  // SpMM plan: per-wave ranges over `light`, plus block-cooperative tasks for long rows
  int32_t grid;              // blocks of the SpMM kernel
  const LightRow* light;     // light rows, ascending, with their CSR ranges
  const int32_t* wave_lo;    // grid*4 + 1 boundaries into `light`
  int32_t ntask;             // block tasks (task t runs on block t % grid)
  const int32_t* task_row;
  const int32_t* task_mega;  // -1, or index of the multi-chunk row this chunk belongs to
  const int32_t* task_chunk; // chunk index within its row (0 for single-chunk rows)
  const int64_t* task_beg;   // CSR range of the task
  const int64_t* task_end;
  int32_t nmega;
  const int32_t* mega_row;     // row of each multi-chunk row
  const int32_t* mega_nchunk;
  const int32_t* mega_chunk0;  // first chunk slot of each multi-chunk row
  int32_t nchunk_slots;

  // Endpoints u < v of every edge, in canonical order: the per-edge kernels run over edges
  // rather than rows, whose upper parts are short and uneven
  const int32_t* eu;  // m
  const int32_t* ev;  // m

  ResPlan res;
};

// Per-column CG state of one block, in the workspace.
struct ColState {
  double* rho;      // current r.r, or r.M^-1 r with the Jacobi variant (fp64)
  double* rr;       // current r.r (stopping test and final relative residual)
  double* rho0;     // r.r of the right-hand side
  double* thr;      // tol^2 * rho0
  double* alpha;    // step of the current iteration
  double* beta;     // direction update of the current iteration
  int32_t* active;  // 1 while the column iterates
  int32_t* iters;   // iterations taken
  int32_t* status;  // 0 ok, 1 breakdown
  int32_t* n_active;  // one int: number of active columns (polled by the host)
  int32_t* upd_pending;  // one int: an update ran whose r.r is not yet reduced
  int32_t* pred_done;  // one int: every active column is predicted to stop after the
                       // pending update, so its exact test runs before the next SpMM
  int32_t* nspmm;      // one int: SpMM launches of this block that found active columns
  unsigned long long* fin_word;  // finishing-step counter word: active columns, columns
                                 // predicted to go on and blocks done; zero between launches
  int32_t* one;       // one int holding 1 (keeps debug launches from exiting early)
};

// Reduction scratch for one kernel family: level buffers and tickets.
struct Tree {
  double* lvl0;     // grid * nval
  double* lvl1;     // ceil(grid/32) * nval
  double* lvl2;     // ceil(grid/1024) * nval
  uint32_t* tick;   // ceil(grid/32) + ceil(grid/1024) + 1 counters, zero between launches
};

// Workspace of one column block of padded width kb.
struct Work {
  int kb;            // padded width
  void* z;           // n x kb
  void* r;
  void* p;
  void* q;
  void* chunkbuf;    // nchunk_slots x kb fp64 partial sums of multi-chunk rows
  double* mega_dots; // nmega x 3 x kb compensated (s, c) pairs
  ColState cs;
  double* part;      // block partials of the SpMM / RHS launch: grid x 3 x kb pairs
  double* part_u;    // block partials of the update launch: grid_upd x kb pairs
  Tree tree;         // tickets and levels of the small finishing launches
  unsigned long long* bad;  // count of resistances that are <= 0 or not finite
  void* minv;        // n: 1 / (d_i + delta) in the working precision (Jacobi variant)
  int pc;            // 1: Jacobi-preconditioned CG, 0: plain CG
  int fin2;          // 1: enqueue the early exact stopping test after each update
  int32_t grid_rhs, grid_upd, grid_ed;
};

// Launchers (erc_kernels.hip).  All return hipSuccess or the launch error.
hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t count, hipStream_t s);
hipError_t launch_rhs(const DevGraph& g, const Work& w, erc_dtype dt, int K, int col0, int ncols,
                      uint64_t base, double inv_sqrt_k, double tol, hipStream_t s);
// the right-hand sides alone, into w.r (no CG state)
hipError_t launch_rhs_only(const DevGraph& g, const Work& w, erc_dtype dt, int K, int col0,
                           int ncols, uint64_t base, double inv_sqrt_k, hipStream_t s);
// tickets and counters to zero, the constant gate to one
hipError_t launch_prepare(const Work& w, hipStream_t s);
hipError_t launch_spmm(const DevGraph& g, const Work& w, erc_dtype dt, double delta,
                       const void* p, const void* r, void* q, const int32_t* gate,
                       hipStream_t s);
hipError_t launch_update(const DevGraph& g, const Work& w, erc_dtype dt, hipStream_t s);
// w.minv[i] = 1 / (d_i + delta), rounded to the working precision
hipError_t launch_minv(const DevGraph& g, const Work& w, erc_dtype dt, double delta, hipStream_t s);
hipError_t launch_fin_iter(const DevGraph& g, const Work& w, int mode, hipStream_t s);
hipError_t launch_edge_dist(const DevGraph& g, const Work& w, erc_dtype dt, double* R,
                            int accumulate, hipStream_t s);
hipError_t launch_count_bad(const double* x, int64_t count, const Work& w, hipStream_t s);
hipError_t launch_copy_cols(const DevGraph& g, const void* src, int kb, erc_dtype dt, int ncols,
                            void* dst, hipStream_t s);
hipError_t launch_node_p(const DevGraph& g, erc_dtype dt, const double* R, double* p,
                         hipStream_t s);
hipError_t launch_edge_kappa(const DevGraph& g, const double* R, const double* p, double* kappa,
                             hipStream_t s);
// u[e], v[e] from the CSR arrays (erc_create fills eu and ev with it)
hipError_t launch_endpoints(const DevGraph& g, int32_t* u, int32_t* v, hipStream_t s);
hipError_t launch_eids(const DevGraph& g, int32_t* out, hipStream_t s);

// Resident CG (erc_resident.hip).  Workgroup size and slots for n rows (slots 0: too many
// rows).
struct ResForm {
  int nt, rpt;
};
ResForm res_form(erc_dtype dt, int64_t n);
// Where the resident CG of n rows keeps q: 1 in the LDS, 2 in global memory, 0 if the plan
// does not fit a CU at all; *lds receives the launch's dynamic LDS bytes.
int res_q_place(ResForm f, int64_t n, int nchunk, erc_dtype dt, size_t* lds);
// The plan's device-side arrays; M^-1 by position; the solve of the ncols columns of an
// n x kb block whose right-hand sides are in y (solutions replace them).
hipError_t launch_res_fill(const DevGraph& g, erc_dtype dt, hipStream_t s);
hipError_t launch_res_minv(const DevGraph& g, erc_dtype dt, double delta, void* minv, hipStream_t s);
hipError_t launch_resident(const DevGraph& g, erc_dtype dt, void* y, void* q, int kb, int ncols,
                           double delta, double tol2, int max_iter, const void* minv_pos,
                           ResOut* out, hipStream_t s);

struct SampleWork {
  double* part_mm;   // grid x 3 block partials (-kappa_min, kappa_max, non-finite flag),
                     // then grid edge-weight block sums
  double* part_n;    // grid_n node-weight block sums
  double* totals;    // [0] -kappa_min, [1] kappa_max, [2] node sum, [3] edge sum, [4] bad flag
  int32_t grid;      // blocks of the per-edge passes
  int32_t grid_n;    // blocks of the per-node pass, a multiple of eight
};
hipError_t launch_sampling(const DevGraph& g, const double* kappa, double eta, int64_t nonisolated,
                           const SampleWork& sw, double* pn, double* pe, hipStream_t s);

// Fixed device scratch (erc_static.hip) of erc_sampling_probs_static.
constexpr size_t kStaticScratchBytes = 64 << 10;
// Looks up this process's copy of the array on `device`, which must be current; once
// per device, later calls return at once.
hipError_t static_scratch_setup(int device);
// The looked-up device address, or nullptr before static_scratch_setup succeeded.
void* static_scratch_ptr(int device);

// Gather probe (erc_probe.hip): rows of sums it stores for `count` indices, and launch.
int64_t probe_out_rows(int64_t count);
hipError_t launch_probe_gather(const int32_t* idx, int64_t count, const void* table, int64_t rows,
                               int row_bytes, int slices, void* out, hipStream_t s);

// Tree sizing helpers (host).
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t tree_ticks(int grid) {
  return ceil_div(grid, kTreeFan) + ceil_div(grid, kTreeFan * kTreeFan) + 1;
}

// Subgraph draws (erc_draw.hip).  Status bits a launch leaves in its status word.
constexpr uint32_t kDrawBadProb = 1u;      // a probability outside [0, 1] or NaN
constexpr uint32_t kDrawSumTooLarge = 2u;  // probabilities sum above 1.5
constexpr uint32_t kDrawAllZero = 4u;      // every integer weight is zero
constexpr uint32_t kSubBadIndex = 8u;      // a drawn index outside the node or edge range
constexpr int64_t kScanTile = 4096;        // items per block of a scan
constexpr int64_t kBitTile = 1024;         // bitmap words per block
constexpr int64_t kDrawSub = 16;           // items of a subtile of a draw's weights
constexpr int64_t kDrawSome = 32768;       // draws at a time where they replace the probabilities
inline int64_t scan_blocks(int64_t items) { return ceil_div(items, kScanTile); }
// Words of a bitmap over `items`, in whole tiles of at least one.
inline int64_t sub_words(int64_t items) {
  return kBitTile * (items > 0 ? ceil_div(items, 32 * kBitTile) : 1);
}

struct DrawWork {
  uint64_t* sub;     // scan_blocks(N) x kScanTile / kDrawSub: prefix sums within each tile
  uint64_t* tsum;    // scan_blocks(N) + 1: tile sums, then their prefix sums and the total
  double* psum;      // scan_blocks(N) fp64 tile sums of the probabilities
  uint32_t* status;  // one word
  int64_t* some;     // kDrawSome draws, where idx overlaps the probabilities
};
struct SubgraphWork {
  uint32_t* head;       // status, kept nodes, kept edges (followed by the bitmaps)
  uint32_t* nbits;      // bitmap of the kept nodes
  uint32_t* ebits;      // bitmap of the kept edges (edge draws)
  int64_t clear_words;  // words from head that a call starts from zero
  uint32_t* nprefix;    // rank of each node word's first bit
  uint32_t* cnt;        // up to n: edges per kept node, then their prefix sums (node draws)
  uint32_t* tile;       // tile sums
  uint8_t* flags;       // a byte per item (32 per bitmap word), for marks of many items
};
// The sums of prob that the draws search; then draws first .. first + draws - 1 into idx, which
// must not overlap prob (the draws read it).
hipError_t launch_draw_sums(const double* prob, int64_t N, const DrawWork& w, hipStream_t s);
hipError_t launch_draw(const double* prob, int64_t N, int64_t first, int64_t draws, uint64_t base,
                       const DrawWork& w, int64_t* idx, hipStream_t s);
// items 0: subgraph induced on the nodes in idx; 1: the edges in idx and their endpoints
hipError_t launch_subgraph(const DevGraph& g, int items, const int64_t* idx, int64_t count,
                           const SubgraphWork& w, int32_t* nodes, int64_t* edges, int32_t* uo,
                           int32_t* vo, hipStream_t s);

}  // namespace erc

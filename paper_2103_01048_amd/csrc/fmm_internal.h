// Internal structures of the MI355X FMM library (host planner + kernels).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "../../include/fmmbem.h"

namespace fmm {

constexpr int MAXLEVEL = 21;
constexpr int GEMM_NT = 64;   // columns per GEMM task (4 MFMA column blocks)
constexpr int M2L_WIDE_TASKS = 160;  // segmented M2L launches of fewer 64-column tasks use 16-column ones
constexpr int M2L_FEW_COLUMNS = 1024;
constexpr int MAX_NR = 4;     // density columns handled by one kernel pass

// Surface radii, in units of the box half-width (upward equivalent, upward
// check, downward equivalent, downward check).
constexpr double ALPHA_UE = 1.05, ALPHA_UC = 2.95, ALPHA_DE = 2.95, ALPHA_DC = 1.05;

void set_error(const std::string &msg);
int plan_upload(fmm_plan *P, void **ptr, const void *h, size_t bytes);
hipEvent_t prof_begin(fmm_plan *P, int phase, hipStream_t s);
void prof_end(fmm_plan *P, int phase, hipEvent_t begin, hipStream_t s);
// Timing events for a phase that is a single kernel launch: the launch
// carries them (hipExtLaunchKernelGGL), so no marker goes on the stream
// beside it.  Both null when the phase is not being timed.
void prof_launch(fmm_plan *P, int phase, hipEvent_t *begin, hipEvent_t *end);
// Near-field items of a pair evaluation that start at once on the second
// side stream: near_early per mille of the items (the shortest, at the tail
// of the item list), with pass order 3 or 4 and a far field only.
inline int near_early_items(const fmm_tuning_t &t, int nitems, bool far) {
  return (far && t.pair_order >= 3 && t.near_early > 0)
             ? (int)std::min<int64_t>(nitems, (int64_t)nitems * t.near_early / 1000)
             : 0;
}
void matmul_rect(int m, int k, int p, const double *A, int lda, const double *B, int ldb, double *C, int ldc);
void pinv_tsvd(int n, const double *A, double tau, double *out);
int tsvd_factors(int n, const double *A, double tau, double *UT, double *VS, int nthreads);
int tsvd_factors_parity(int n, const double *grid, const double *A, double tau, double *UT, double *VS, int ldv,
                        unsigned char *code);
int tsvd_split(int rows, int cols, const double *A, double tau, double *L, int ldl, double *R, int ldr);

// Which operator set an evaluation of plan P takes.  Set 0 (segmented M2L) is
// the faster one but adds a target's sources in another order than set 1
// (pairwise M2L).  Set 1 serves the factored operators and, in single
// precision, two kinds of evaluation that keep their order of summation and
// with it every bit (`keeps_order`): one column of one plan, whose gradients
// autograd.py hands on in the caller's double precision (the last column of
// nrhs = 5, 9, ... is evaluated as one column, and so to the same bits as on its
// own), and monopole + dipole sources (the boundary-element products).  The
// plans of a boundary-element operator take set 1 for every evaluation: one
// that a caller takes out by bem_fmm_plan finds the operators that its setup
// built, and no evaluation builds operators.  Plans of few M2L columns (fewer than
// M2L_FEW_COLUMNS, whatever the number of densities) take set 1 too: its launch
// spreads V pairs over the chip where the segmented one walks up to eight
// segments in a few workgroups.  Pair passes at p = 8, pairwise / segmented: bf16x3
// 120 / 135 us at 85 columns, 183 / 190 at 284, within 2% of each other from 960 to
// 2000 (p = 5 and 6: within 3.5% from 960 to 2400), 217 / 210 at 2272; FP32 133 /
// 149 us at 85, 208 / 205 at 284, 244 / 233 at 1589.
inline int op_set(const fmm_plan *P, bool keeps_order);

#define FMM_HIP_TRY(call)                                                        \
  do {                                                                           \
    hipError_t e_ = (call);                                                      \
    if (e_ != hipSuccess) {                                                      \
      ::fmm::set_error(std::string(#call) + ": " + hipGetErrorString(e_));       \
      return FMM_EHIP;                                                           \
    }                                                                            \
  } while (0)

// One GEMM work item: Y[dst[c]] (op)= alpha * A[mat] * concat_s X[src[c*S+s]]
// for columns c in [col0, col0 + ncol), ncol <= GEMM_NT.
struct GemmTask {
  int32_t mat;
  int32_t col0;
  int32_t ncol;
  int32_t nrb;     // 16-row blocks this task computes (0: the batch's nrb)
  int32_t klen;    // k-values this task reads (0: the batch's klen)
  double alpha;
};

enum GemmMode { GEMM_STORE = 0, GEMM_ADD = 1 };

// Everything one gather-GEMM batch needs on the device; a launch takes two
// (the second with ntask = 0 when unused) so that the same pass of two plans
// sharing a tree runs as one launch.
struct GemmArgs {
  const GemmTask *tasks;
  const void *pool;     // matrix pool (elements of the work type; uint4 units for bf16x3)
  int64_t mstride;      // one matrix, in pool units
  const int32_t *src;   // ncols*S row indices into X
  const int32_t *dst;   // ncols row indices into Y
  const void *X;
  void *Y;
  int ntask, nrb, klen, ldx, ldy, S, seg, KQ, mode;
};

// A batch of GEMM tasks that can run in one launch (no two tasks write the
// same output rows).
struct GemmBatch {
  int S = 1;                   // K segments per column
  int nrb = 0;                 // 16-row blocks of A that are computed
  int klen = 0;                // K extent actually read (multiple of 16)
  int seg = 0;                 // K length of one segment (0: the work-array row length)
  int kq_stride = 0;           // 16-wide k groups per stored row block (0: row length / 16)
  int ldy = 0;                 // leading dimension of the output rows (0: the work-array row length)
  int mode = GEMM_STORE;
  int set = 0;                 // operator set
  int pool = 0;                // 0: matrix pool, 2: bf16x3 split pool
  int ldx = 0;                 // row length of X (0: the work-array row length)
  int ntask = 0;
  GemmTask *d_tasks = nullptr;
  int32_t *d_src = nullptr;    // ncols*S  (row index into X, already * nr + r)
  int32_t *d_dst = nullptr;    // ncols    (row index into Y)
  int ncols = 0;
  // host copies kept until upload
  std::vector<GemmTask> h_tasks;
  std::vector<int32_t> h_src, h_dst;
};

// One workgroup of the segmented M2L (k_m2l): columns col0 .. col0 + ncol - 1
// (one slot row each) of one (level, shape),
//   slot[c] = F_c^d sum_{s < nseg} pool[mat[s]] F_c^u X[src[src0 + s * nt + c]],
// F_c the signs of column c's reflection; a source of -1 is absent.
struct M2LTask {
  int32_t col0, ncol, nseg;
  int32_t nrb;       // 16-row blocks (the level's downward rank)
  int32_t klen;      // k-values per segment (the level's upward rank)
  int32_t src0;
  int32_t tab;       // the level's tables: sign bytes at tab * ld, zero-tile masks at tab * 8 * (ld / 16)
  int32_t pad;
  uint64_t blocks;   // bit 8 s + b: some column of 16-column block b holds segment s
  int32_t mat[8];
  uint8_t zero[8];   // per segment, the axes along which its offset is zero
};

// Tasks of the segmented M2L.
struct M2LBatch {
  int ntask = 0, nt = GEMM_NT;  // tasks; columns per task
  int split = 0;                // the first task of the two finest levels
  int nrb = 0, nrbk = 0;        // most row blocks and 16-wide k groups of a task
  int ldy = 0;                  // slot row length
  M2LTask *d_tasks = nullptr;
  int32_t *d_src = nullptr;     // per task, nseg * nt source rows
  uint8_t *d_flip = nullptr;    // per column, its reflection (bit 2: x, 1: y, 0: z)
};

// One plan's half of a segmented M2L launch.
struct M2LArgs {
  const M2LTask *tasks;
  const int32_t *src;
  const uint8_t *flip;
  const uint8_t *par_u, *par_d;  // [level][ld] sign bytes of the upward and downward coordinates
  const uint32_t *tiles;         // [level][zero axes][row block]: bit q set when the 16 x 16 tile of k group q is not zero
  const void *pool;
  int64_t mstride;               // one operator, in pool units (elements; uint4 for bf16x3)
  const void *X;
  void *Y;
  int64_t xlo;                   // bf16x3: from the high to the low parts in X
  // nrbk: 16-wide k groups of the largest klen; rbg: row blocks per grid row; zrow: a zero row of X
  int ntask, nrb, nrbk, rbg, ldx, ldy, zrow, kstride;  // kstride: 16-wide (bf16x3: 32-wide) k groups per stored row block
};

// Per-nrhs-chunk task lists.  Row indices in the work arrays are
// box * nr + r, so the lists depend on nr.
// One task of a chained launch (k_chain): kind 0 runs GEMM task idx >> 4,
// row group idx & 15, of GemmArgs arg; kind 1 sums the M2M slots of the
// four boxes idx .. idx + 3 of ReduceArgs arg.  Tasks of phase p > 0 start
// once every task of phase p - 1 has finished.
struct ChainTask {
  int32_t kind, phase, arg, idx;
};

// Device task list of a chained launch and what it was built from.
struct Chain {
  std::vector<const void *> key;  // plans, column count and work arrays it was built for
  int ntask = 0, nphase = 0, kch = 0;
  void *tasks = nullptr, *gargs = nullptr, *rargs = nullptr, *need = nullptr;
};

// Device buffers that plans on the same points share (a tree's sorted order,
// boxes, lists and leaf items; a set of operators; the surface grid); freed
// when the last plan holding them is.
struct SharedAllocs {
  std::vector<void *> ptrs;
  ~SharedAllocs() {
    for (void *p : ptrs) (void)hipFree(p);
  }
};

// Translation operators of a plan in one basis of singular coordinates.  Set 0
// takes singular vectors of one reflection class each (tsvd_factors_parity):
// one M2L operator serves every reflection of its offset and the segmented
// M2L applies it.  Set 1 takes them as the SVD leaves them, with one M2L
// operator per offset (or its two factors), for the pairwise M2L.
// A plan's sets are built or taken from another plan during its setup and
// never change afterwards: other threads' setups read them, and plans that
// took them outlive the plan that built them.
struct OpSet {
  bool built = false;
  std::shared_ptr<SharedAllocs> mem;  // its device buffers
  void *pool1 = nullptr;           // swizzled ld x ld matrices
  int64_t pool1_count = 0, poolbf_count = 0;
  void *pool_bf = nullptr;         // bf16x3 mode: split M2L operators
  int bf_kb = 0;                   // 32-wide k blocks per row block in pool_bf
  // matrix ids (pool1 unless noted) per level; -1 when absent
  std::vector<int> utu_id, vsu_id, utd_id, vsd_id;  // truncated-SVD factors
  std::vector<int> rank_u, rank_d;                  // their ranks
  std::vector<std::vector<int>> m2m_id;             // [parent level][octant]
  std::vector<std::vector<int>> l2l_id;             // [parent level][octant]
  std::vector<std::vector<int>> m2l_id;             // [level][343 offset code] (set 0: offsets with no negative
                                                    // component; factored: the left factor L)
  std::vector<std::vector<int>> m2l_r_id;           // factored M2L: the right factor R, same indexing
  std::vector<std::vector<int>> m2l_k;              // factored M2L: rank k per (level, offset)
  int m2l_ldt = 0;                                  // factored M2L: row length of the per-pair intermediate
  uint8_t *d_par = nullptr;                         // set 0: sign bytes, [upward, downward][maxlevel + 1][ld]
  uint32_t *d_tiles = nullptr;                      // set 0: M2LArgs::tiles
  std::vector<double> vs_alpha;                     // Laplace level scaling
};

struct PassLists {
  int nr = 0;
  // per level l (index l, levels >= 2), in singular coordinates c = U^T chk
  std::vector<GemmBatch> m2m;   // per-child M2M slots of the parents at level l
  GemmBatch ut_u_all;           // leaf upward check -> c_u, all levels
  std::vector<GemmBatch> l2l;   // child c_d += L2L * parent c_d (levels >= 3)
  GemmBatch vs_u;               // c_u -> upward equivalent (M2P sources), all levels
  GemmBatch ut_dx;              // P2L check -> its own c_d array (added by the M2L sums), all levels
  GemmBatch vs_d;               // c_d -> downward equivalent (leaves), all levels
  M2LBatch m2lc;                // segmented M2L: all levels, c_u -> column slots of c_d
  GemmBatch m2l;                // pairwise M2L: c_u -> pair slots (factored: per-pair intermediate -> slots)
  GemmBatch m2l_r;              // factored M2L: c_u -> per-pair intermediate (R factors)
  // per level (0 .. maxlevel + 1): the first task of that level in m2l (tasks
  // ascend by level; entry maxlevel + 1 = the task count)
  std::vector<int> m2l_t0;
  int32_t *d_m2l_rows = nullptr;  // per box: rows of its M2L sums (its level's downward rank, to 16)
};

struct DevTree {
  int64_t n = 0;
  int nbox = 0, nleaf = 0, maxlevel = 0;
  // sorted points relative to their leaf's centre; xyz + density slot, in T
  void *pts = nullptr;
  int32_t *perm = nullptr;      // sorted -> caller index
  // boxes
  void *box_geom = nullptr;     // T4: centre xyz (relative to the molecule's root centre), half width
  int32_t *box_begin = nullptr, *box_end = nullptr;
  int32_t *leaves = nullptr;    // leaf box ids
  // leaf work items: (leaf slot, first target | split << 24, part or -1, 0)
  int32_t *items = nullptr;
  int nitems = 0;
  int32_t *near_off = nullptr;  // per item, into near_rng
  int32_t *near_rng = nullptr;  // (begin, end) point ranges of near sources, one leaf each
  void *near_o = nullptr;       // T4 per range: source leaf centre - target leaf centre
  void *far_o = nullptr;        // T4 per far entry: surface box centre - target leaf centre, radius
  int32_t *far_off = nullptr;   // per item, into far_idx
  int32_t *far_idx = nullptr;   // surface boxes (bit 30: own downward surface)
  int32_t *split_tiles = nullptr;  // (slot, code, first part, nparts) per split tile
  int nsplit = 0, nparts = 0;
  void *parts = nullptr;        // partial sums of split tiles
  int32_t *x_box = nullptr;     // boxes with a non-empty X list
  int32_t *x_off = nullptr, *x_idx = nullptr;
  void *x_o = nullptr;          // T4 per X entry: source leaf centre - target box centre
  int nxbox = 0;
  int32_t *v_tgt = nullptr;     // boxes at level >= 2 (M2L sums)
  int32_t *v_off = nullptr;     // M2L columns of each such box (CSR)
  int32_t *v_pair = nullptr;
  int nvbox = 0;
  int64_t nvcol = 0;
  // per level: non-leaf boxes, CSR of their children (for the M2M sums)
  std::vector<int32_t *> m2m_tgt, m2m_off, m2m_kid;
  std::vector<int> m2m_n;
};

}  // namespace fmm

struct fmm_plan {
  int kernel = 0, p = 0, ncrit = 0, precision = 0;
  double kappa = 0;
  int64_t n = 0;
  int nsurf = 0, ld = 0;           // surface points, padded leading dimension
  double lo[3] = {0, 0, 0}, W = 1, shift[3] = {0, 0, 0};
  int device = 0;
  // host tree
  std::vector<int64_t> keys, perm;
  std::vector<int32_t> level, nchild;
  std::vector<int64_t> anchor, begin, end, parent, child_begin;
  std::vector<int64_t> level_begin;  // size maxlevel+2
  std::vector<int32_t> mol;          // molecule of each box
  std::vector<int64_t> mol_off;      // point ranges of the molecules (input order)
  std::vector<double> mol_lo;        // lower corner of each molecule's root cube
  std::vector<int64_t> loff[4];      // U, V, W, X CSR offsets (nbox+1)
  std::vector<int64_t> lidx[4];
  std::vector<int32_t> leaf_ids;
  std::vector<int32_t> vpair_src, vpair_pos;  // pairwise M2L: V pairs in GEMM order (sort_pairs)
  std::vector<int64_t> vpair_first;
  // M2L columns in GEMM order: eight source boxes (-1: absent), level * 27 +
  // shape, reflection
  std::vector<int32_t> mcol_src, mcol_key;
  std::vector<uint8_t> mcol_flip;
  std::vector<int32_t> p2l_boxes;             // boxes whose X list goes through P2L
  int64_t p2p_inter = 0, far_inter = 0;
  std::vector<int64_t> item_pairs;  // pair interactions (targets x near sources) per leaf item, in launch order
  // device
  fmm::DevTree dt;
  void *surf = nullptr;            // T4 grid offsets in [-1,1]^3, nsurf entries
  fmm::OpSet ops[2];               // translation operators (OpSet)
  // work arrays, sized for work_nr columns
  int work_nr = 0, cub_nr = 0;
  void *qs = nullptr, *equ = nullptr, *chk = nullptr, *eqd = nullptr, *chku = nullptr,
       *cu = nullptr, *yd = nullptr, *m2lbuf = nullptr, *cub = nullptr, *mslot = nullptr, *m2l_t = nullptr;
  // m2lbuf: M2L slots, one per V pair (pairwise) or per column (segmented)
  // cub: cu split into bf16 high and low parts (bf16x3, segmented M2L), for cub_nr columns
  // cu: upward check in singular coordinates (U_u^T chk); yd: downward
  // check in singular coordinates (M2L sums + U_d^T chk)
  void *ydx[fmm::MAX_NR + 1] = {};  // P2L projections, by the number of columns
  fmm::PassLists lists[2][fmm::MAX_NR + 1];  // task lists per operator set and column count
  // P2M targets (leaves at level >= 2) and per-leaf flags
  int p2m_count = 0;
  int32_t *d_p2m_box = nullptr;   // box ids
  int32_t *d_p2m_off = nullptr;   // 0..p2m_count (each box is its own source)
  int32_t *d_has_local = nullptr; // per leaf slot: level >= 2
  int32_t *d_vp_off = nullptr, *d_vp_pair = nullptr;  // pairwise M2L: pair slots of each box at level >= 2
  // profiling: event pairs per phase, recorded during fmm_eval
  int profiling = 0;               // bit k set: time phase k
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> prof_events;
  std::vector<hipEvent_t> event_pool;
  // pair evaluation (this plan as the Laplace half): side stream, fork and
  // join events, and the near-field running sums of both kernels
  // the device's shared side streams: far passes; early near items; early M2L levels
  hipStream_t aux = nullptr, aux2 = nullptr, aux3 = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr, ev_up = nullptr, ev_m2l = nullptr, ev_near = nullptr;
  hipEvent_t ev_m2m = nullptr, ev_m2lf = nullptr;  // the first M2M level done; the early M2L levels done
  size_t m2lbuf_bytes = 0, m2l_t_bytes = 0;
  void *pair_acc = nullptr;
  size_t pair_acc_bytes = 0;
  void *dips = nullptr;             // monopole + dipole sources: dipole records in Morton order
  // chained launches of a pair evaluation led by this plan: the M2M levels
  // and the L2L levels of both plans, each in one launch; counters (ticket,
  // finished tasks per phase, error flag) cleared before each launch
  fmm::Chain chain_up[2], chain_down[2];  // [monopole + dipole sources]
  int32_t *chain_ctr = nullptr;
  int chain_ctr_n = 0;
  uint64_t coord_hash = 0;          // checksum of the FP64 input coordinates (per molecule, chained)
  uint64_t tree_hash = 0;           // fingerprint of coordinates, points, boxes and leaf items
  void *adj = nullptr;              // adjoint scratch: psi and grad psi
  size_t adj_bytes = 0;
  int64_t device_bytes = 0;
  double setup_ms = 0;
  double setup_split[5] = {0, 0, 0, 0, 0};  // sort, tree, lists, items, operators (ms)
  int tree_on_device = 0, tree_shared = 0;
  int products = 0;                 // a boundary-element operator's plan
  fmm_tuning_t tune{32, 16, 512, 16384, 1.15, 0, 0, 4, 0, 512, 0, 64, 0, 0, 1024, 0, 0};  // tunables in force at setup
  std::vector<void *> allocs;      // everything to free
  std::shared_ptr<fmm::SharedAllocs> tree_mem;  // the tree's device buffers (shared with plans on the same points)
  std::shared_ptr<fmm::SharedAllocs> geom_mem;  // surface grid and box geometry (shared with plans of the same kernel on the same tree)
  std::vector<void *> *alloc_sink = nullptr;    // where dev_alloc records a buffer (null: allocs)
};

namespace fmm {
inline int op_set(const fmm_plan *P, bool keeps_order) {
  return P->tune.m2l_factored ||
                 (P->precision != FMM_FP64 && (P->products || keeps_order || P->dt.nvcol < M2L_FEW_COLUMNS))
             ? 1
             : 0;
}
}  // namespace fmm

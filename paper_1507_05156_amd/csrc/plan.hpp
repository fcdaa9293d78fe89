// Plan object behind the opaque fockmi_plan handle (host side only).
#pragma once

#include <hip/hip_runtime.h>

#include <functional>
#include <initializer_list>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/fockmi.h"
#include "kernels.hpp"
#include "pairs.hpp"
#include "tune.hpp"

namespace fockmi {

fock_status fail(fock_status st, const char* fmt, ...);
// looks up the current device's copy of the allocation-free call's scratch array (noalloc.hip)
fock_status noalloc_setup(int device);
fock_status hip_fail(hipError_t e, const char* where);

// Device allocation owned by the plan, grown on demand. A graph captured from a call refers to the
// allocations that the call used: these are held, so that growth replaces them and keeps them until
// the plan is destroyed.
struct DevBuf {
  void* ptr = nullptr;
  size_t bytes = 0;
  bool held = false;
  std::vector<void*> kept;  // held allocations that a larger one has replaced
  fock_status ensure(size_t need, size_t cap, const char* what);
  void hold();     // the call in progress uses the buffer as it is (ensure does this by itself)
  void drop();     // without an allocation from here on
  void release();  // frees everything
};

// whether the stream is being captured into a graph
bool stream_captures(hipStream_t st);
// whether that of this thread's call in progress is
extern thread_local bool g_capturing;

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
inline bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const char* x = (const char*)a;
  const char* y = (const char*)b;
  return x < y + nb && y < x + na;
}

// The k-points a pair sum runs over: targets X at ntk k-points, sources P and
// M (stored contiguously) at nsk k-points, and qidx[t][s] the kernel-table row
// of that (target, source) pair.
struct PairSet {
  int ntk = 0, nsk = 0;
  const int* qidx = nullptr;  // device [ntk][nsk]
  int ntk_all = 0;            // target k-points of the whole application (a k-range runs part of them)
};

struct Cell {
  Geom geom{};
  int nr = 0, nk = 0, nb = 0;
  double a[3][3]{}, vol = 0.0, omega = 0.0, gs = 2.0;
  std::vector<double> kpts;   // [nk][3]
  int nq = 0;                 // distinct q = k_t - k_s
  std::vector<int> qidx_host; // [nk][nk]
  DevBuf qidx, qvec, qzero;   // int[nk*nk], double[nq*3], int[nq]
  DevBuf Kt;                  // float[nq][nr], fused-kernel layout (FP32 plans)
  DevBuf SD;                  // float[nq][nr/2][2], (S, D) pairs of the split 32^3 form (FP32 plans, n = 32)
  DevBuf Kp;                  // float or double [nq][nr], order of the pair kernels and the fused FP64 kernel (cubes of 16-32)
  DevBuf Kpl;                 // double[nq][nr] as [l1][l3][l2], for the plane passes (grids without a one-CU kernel)
  bool f64f = false;          // this cell runs the fused FP64 kernel
  bool f32plain = false;      // an FP32-form cell on a grid that is not cubic: complex64 plane passes, FP64 sums
  DevBuf kvec;                // double[nk][3] k-points on the device
  // down-sampling: the source sub-mesh S (all k-points when ds is false)
  bool ds = false;
  std::vector<int> src;       // [nsrc] k indices of S
  int nsrc = 0;
  DevBuf qidx_ts, qidx_st;    // int[nk][nsrc] (target k, source s), int[nsrc][nk] (source s as target, k)
  // forward sums: all k-points as targets, S as sources
  PairSet fwd() const { return {nk, nsrc, (const int*)(ds ? qidx_ts.ptr : qidx.ptr), nk}; }
  // the reverse role of the adjoint: S as targets, all k-points as sources
  PairSet rev() const { return {nsrc, nk, (const int*)(ds ? qidx_st.ptr : qidx.ptr), nsrc}; }
};

// the batched form used when no tuned choice exists: the forked cells (three
// cells 16^3/27 k/8 b, 20^3/64 k/12 b, 24^3/125 k/16 b: 257.5 ms, against 261.8
// in sequence and 282.2 for the persistent kernel)
constexpr int kDefaultBatchForm = 1;

// state of the batched persistent launch (fock_apply_batched): buffers whose
// addresses a captured graph refers to, and the graph itself
struct BatchState {
  std::vector<const void*> key;  // u, phi, vphi pointers and nphi of every cell
  DevBuf shadow_u[kMaxBatchCells], shadow_x[kMaxBatchCells], comp[kMaxBatchCells];
  DevBuf accs, queue, counters;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipStream_t cap = nullptr;
  BatchArgs args{};
  int nthreads = 0, nwg = 0, entries = 0;
  // form 0: the persistent kernel; form 1: each cell's own fused kernel on a
  // stream of its own, forked from and joined to the caller's stream; form 2:
  // those kernels one after another, costliest cell first
  int form = kDefaultBatchForm;
  hipStream_t side[kMaxBatchCells] = {};
  hipEvent_t fork = nullptr, join[kMaxBatchCells] = {};
  bool ready = false;
  void reset_graph();
  void release();
};

// The mirror side of a two-sided pair sum: dst[j] = (accumulate ? dst[j] : 0) +
// (scale + i scale_im) sum_i F_i conj(W_ji) over the targets i. dst NULL: one-sided. tri: the targets are the
// sources, every pair of fields is transformed once and the mirror adds the other half.
template <typename T>
struct Mirror {
  const cx<T>* F = nullptr;
  c128* dst = nullptr;
  double scale = 0.0, scale_im = 0.0;
  bool accumulate = false;
  bool tri = false;
};

// The targets per row and sources per block of a two-stage pair sum within `budget` bytes of W
// (whole_partials: blocks of at least one FP32 partial sum of at most 16 bands).
void pairs_block_shape(int nt, int nj, int ns, int nr, size_t fb, size_t budget, bool whole_partials, bool tri,
                       int* rows, long* njmax);
// The scratch of such a sum, one allocation: the batch of W fields, then (256-byte aligned, at these
// offsets) the sums kept between the blocks of a row if it has several and, when two-sided, the mirror sums of each
// group of a row's targets and in FP32 their compensation. One instead of four: an allocation takes
// longer than a small sum (first application on a new plan, 16^3 / 8 k / 4 bands in FP64: 531 us with
// one per piece, 181 us, of which the sum is 42).
struct PairsLayout {
  int rows = 0, groups = 0;
  long njmax = 0;
  size_t run = 0, mir = 0, mcomp = 0, end = 0;
  size_t largest = 0;  // bytes of its largest piece
};
PairsLayout pairs_layout(int nr, int nt, int nj, int ns, size_t fb, size_t budget, bool sums32, bool two, bool tri);
// Stage 1 of a two-stage pair sum: W of a block's pairs into the batch.
template <typename TW>
using PairStage = std::function<hipError_t(const PairBlock&, cx<TW>*)>;
// one pair per workgroup pass, on a cubic grid whose field fits on a CU; Kt: tables in the
// pair kernel's order
template <typename T>
PairStage<T> cube_stage(int n, int num_cus, const PairSet& ps, const cx<T>* X, int nx, const cx<T>* P, int ns,
                        const T* Kt, hipStream_t st);
// the plane passes, any grid; K: tables in the plane passes' order
template <typename T>
PairStage<T> plane_stage(const Geom& g, int num_cus, const PairSet& ps, const c128* X, int nx, const c128* P, int ns,
                         const double* K, hipStream_t st);
// The blocks of a two-stage pair sum (nt targets, nj sources of ns per k-point) over buffers of
// the caller's: W holds rows * njmax fields, run rows * nr sums (complex64 for FP32 sums,
// complex128 for FP64 ones). TW: the type of W, TM: of the products and sums; np: n2 * n3 when
// M and F are in the paired order of the FP32 one-CU kernel, else 0.
template <typename TW, typename TM>
fock_status pairs_blocks(int nr, int np, int nt, int nj, int ns, const PairStage<TW>& stage, const cx<TM>* M,
                         const Mirror<TM>& mr, c128* out, double scale, bool accumulate, int rows, long njmax,
                         cx<TW>* W, void* run, c128* mir, c64* mcomp, hipStream_t st);

// bytes of the fixed scratch array of fock_apply_noalloc, and what a sum needs of it
// (x_is_u: the targets are the sources' array)
constexpr size_t kNoAllocBytes = size_t(64) << 20;
size_t noalloc_bytes(const Cell& c, const PairSet& ps, int nx, int ns, bool x_is_u);

// work arrays of the block eigensolver (eig_api.hip)
struct EigState {
  DevBuf x, hx, w, hw, p, hp, xn, hxn, pn, hpn;  // [nk][nb][N_r] blocks and their images under h
  DevBuf S, A, C, lam, status;                    // Rayleigh-Ritz matrices, coefficients, values, flags
  void release();
};

struct Plan {
  static constexpr unsigned kMagic = 0xF0C4C0DEu;
  unsigned magic = kMagic;
  fock_prec prec = FOCK_FP64;
  int device = 0;
  std::string tune_path;
  std::vector<Cell> cells;
  size_t workspace_cap = 0;                 // 0 = no cap (FOCKMI_WORKSPACE_CAP overrides)
  int xcd_map = 1;
  DevBuf ktmp;                              // one cell's tables in natural order, read while its forms' copies are made
  DevBuf shadow_x, shadow_p, shadow_m, comp, accs, vu, partial, dotres, srcbuf, srcout;
  DevBuf psi0, phiA, phiB, predb, srcbuf2, kin, vxb, lam, lam2, gtmp, ftmp, phis, norms, red6, vloc_buf;
  DevBuf sync;                              // lockstep counters of the persistent fused form
  DevBuf parts;                             // FP64 part sums of the lockstep form's k' split
  DevBuf xbuf, sflags, sstatus;             // exchange buffers, rendezvous counters, abort word of the split form
  DevBuf fallbacks;                         // split launches that fell back (counted while profiling)
  long split_wait_ticks = 5000000;          // rendezvous bound of the split form, 50 ms (FOCKMI_SPLIT_WAIT_TICKS)
  // pair symmetry of the split form: mirror copies (FP32 partial, FP64 sum, compensation),
  // their push counters, and the push order and counts for (nwg, nk, nb) = sym_key
  DevBuf mpart, msum, mcomp, mdone, sym_rank, sym_cnt;
  int sym_key[4] = {-1, -1, -1, -1};
  int split_stagger_shift = 1;              // the bands' order of the symmetric form (FOCKMI_SPLIT_STAGGER_SHIFT)
  int split_sym = 1;                        // 0: every form runs every pair (FOCKMI_SPLIT_SYM=0)
  DevBuf pscratch;                          // scratch of the two-stage pair form (PairsLayout)
  DevBuf gramb;                             // Gram matrices and their factors (fock_orthonormalize)
  size_t pair_batch = size_t(8) << 30;      // bytes of one batch
  int split_form = 0;                       // 1: a split-form variable is set, 32^3 runs the split form
  std::vector<double> host_norms;
  double* host_pinned = nullptr;            // 4 doubles for reductions
  bool profiling = false;
  // autotuning: the cache is read at plan creation when a path is given; missing
  // keys are measured on first use and the file is rewritten
  TuneCache tune;
  bool tuning = false;
  int use_graph = 1;
  BatchState bstate;
  EigState eig;
  int num_cus = 0;
  std::mutex calls;                         // one call at a time (PlanCall)
  hipEvent_t done = nullptr;                // recorded behind the last ordered call's work (PlanCall)
  bool done_recorded = false;

  std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_events;
  double prof_ms = 0.0;
  long long prof_launches = 0;
  hipError_t prof_begin(hipStream_t st);
  hipError_t prof_end(hipStream_t st);
  void prof_drop();                         // forgets a prof_begin whose launches did not happen
  fock_status prof_collect();

  fock_status init_cell(Cell& c, const fock_cell_desc& d, int index);
  fock_status check_ready(int cell) const;
  void destroy();

  // out[t][x] = (accumulate ? out : 0) + scale * sum_{s, b} M[s][b] W(P[s][b], X[t][x]; K_{qidx[t][s]})
  // over the targets and sources of ps
  fock_status general(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M, int ns,
                      c128* out, double scale, bool accumulate, hipStream_t st);
  fock_status run_plain(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M, int ns,
                        c128* out, double scale, bool accumulate, hipStream_t st);
  fock_status run_fused(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M, int ns,
                        c128* out, double scale, bool accumulate, hipStream_t st);
  fock_status run_fused64(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M,
                          int ns, c128* out, double scale, bool accumulate, hipStream_t st);
  // a sum in the two-stage pair form, its batch at most `batch` bytes; others: the caller has another form
  template <typename TW, typename TM>
  fock_status run_pairs(int nr, int np, int nt, int nj, int ns, const PairStage<TW>& stage, const cx<TM>* M, c128* out,
                        double scale, bool accumulate, const Mirror<TM>& mr, size_t batch, hipStream_t st, bool others = true);
  // whether the sum runs in the two-stage pair form (cubic grids up to 24), and with the pair symmetry
  struct PairRule {
    bool pairs = false, tri = false;
    bool shared = false;  // fock_apply_noalloc serves the same sum, by the same rule
    double fused_ns = 0.0, pairs_ns = 0.0;  // modelled cost of the one-sided sum per source (0: no fused form)
    double ns = 0.0;                        // and of the form chosen
  };
  PairRule pair_rule(const Cell& c, const PairSet& ps, int nx, int ns, bool same, bool f32) const;
  // FP32 cells of 16^3 to 24^3 with every k-point a source: whether they are faster one after another, in
  // the pair form where that is the rule, than as the batched launch's forked streams
  bool batch_in_sequence(const void* const* u, const void* const* phi, const int* nphi) const;
  // whether the scratch of such a sum can be had: under capture, where nothing can be allocated, what is
  // there has to hold it, if in smaller blocks
  bool pairs_ready(int nr, int nt, int nj, int ns, size_t field_bytes, bool sums32, bool two, bool tri) const;
  // the scratch of a sum with a batch of at most `batch` bytes, less where a piece would exceed the
  // workspace cap (a smaller batch has rows of fewer groups) or the whole `room`; false: none fits
  bool pairs_fit(int nr, int nt, int nj, int ns, size_t fb, size_t batch, bool sums32, bool two, bool tri,
                 PairsLayout* l, size_t room = ~size_t(0)) const;
  // whether that of a symmetric sum over nt fields of nb per k-point fits
  bool pairs_tri_fits(int nt, int nb, int nr, bool f32) const;
  // the orbitals of the source k-points, contiguous: `arr` itself without
  // down-sampling, else a copy of its S blocks ([nsrc][nper][nr]) in buf
  fock_status sources(Cell& c, const c128* arr, int nper, DevBuf& buf, hipStream_t st, const c128** out);
  // V_x[u] phi for the output k-points k0 .. k0 + nkout - 1 only (phi, out: those k-points)
  fock_status apply_krange(Cell& c, const c128* u, int k0, int nkout, const c128* phi, int nphi, c128* out,
                           hipStream_t st);
  // V_x[u] phi into out (forward sums over S, weight 1/|S|)
  fock_status apply_op(Cell& c, const c128* u, const c128* phi, int nphi, c128* out, hipStream_t st);
  // Both sides of one set of pairs, each transformed once: the forward sum out = scale *
  // sum_j u_j W_ji over targets X ([nk][nx] fields, sources us as in Plan::sources), and
  // gu[j] (+)= (mre + i mim) sum_i F_i conj(W_ji) over the source orbitals. *done = false (and
  // nothing written): two separate sums are the faster way.
  fock_status two_sided(Cell& c, const c128* X, int nx, const c128* us, double scale, c128* out, const c128* F,
                        double mre, double mim, bool maccumulate, c128* gu, hipStream_t st, bool* done);
  // complex64 copy of src in buf; np > 0: in the pair form's order (np = n2 * n3)
  fock_status shadow(DevBuf& buf, const c128* src, size_t count, const char* what, hipStream_t st, int np,
                     const c64** out);
  // sum conj(a) b over count elements in FP64 (fixed order); synchronises st
  fock_status dot(const c128* a, const c128* b, size_t count, hipStream_t st, double* re, double* im);
  // the same sum as double-double: out = (re.hi, re.lo, im.hi, im.lo)
  fock_status dot_dd(const c128* a, const c128* b, size_t count, hipStream_t st, double out[4]);

  // propagator pieces (prop_api.hip)
  fock_status kinetic(Cell& c, const c128* x, int nf, c128* y, const double a[3], hipStream_t st);
  // vx_ready: vxb holds V_x x already; with acc, acc = acc_src + out as well
  fock_status h_apply(Cell& c, const c128* us, const c128* us2, const c128* x, c128* out, const c128* base,
                      double cre, double cim, const double* vloc, const double a[3], double alpha, hipStream_t st,
                      bool vx_ready = false, const c128* acc_src = nullptr, c128* acc = nullptr);
  // acc <- x0 + sum_{m=1}^{order} phi_m, phi_m = (-i dt/m) h phi_{m-1}, phi_0 = x0 (acc distinct from x0)
  fock_status taylor_sum(Cell& c, const c128* us, const c128* us2, const c128* x0, c128* acc, const double* vloc,
                         const double a[3], double dt, double alpha, int order, hipStream_t st);
  // max over (k, b) of |(Omega/N_r) ||psi_kb||^2 - 1|; synchronises st
  fock_status norm_dev(Cell& c, const c128* psi, hipStream_t st, double* dev);
  fock_status field_bufs(Cell& c, std::initializer_list<DevBuf*> bufs, int nfields_per_k);

  // eigenstates of h (Eq. (25)) and the excited-electron density (Eq. (26)) (eig_api.hip)
  fock_status eigensolve(Cell& c, const c128* u, c128* phi, const double* vloc, const double a[3], double alpha,
                         double tol, int maxit, double* eig_host, double* res_host, int* iters_host, hipStream_t st);
  fock_status excited_density(Cell& c, const c128* phi, const c128* psi, hipStream_t st, double* nex);

  // batched persistent launch (batched.hip)
  fock_status run_batched(const void* const* u, const void* const* phi, const int* nphi, void* const* vphi,
                          hipStream_t st);
  std::string key_for(const Cell& c, const PairSet& ps, int nx, const char* what) const;
  void save_tune();
};

// One call of the ABI on a plan: calls of other threads wait for it to return. Where it uses scratch
// that calls on other streams may use at the same time (order()), its work waits for that of the last
// such call, and an event is recorded at its end for the next. While the stream is being captured
// nothing is ordered (the graph runs later), and the buffers that the call uses are held for it.
class PlanCall {
 public:
  PlanCall(Plan* p, hipStream_t st);
  ~PlanCall();
  PlanCall(const PlanCall&) = delete;
  PlanCall& operator=(const PlanCall&) = delete;
  static void order();  // of this thread's call in progress
  // frees the plan's pair scratch, which the next pair sum sizes anew, where another buffer finds no
  // device memory; false: there is none to free
  static bool give_back(const DevBuf* asking);

 private:
  Plan* p_;
  hipStream_t st_;
  std::lock_guard<std::mutex> lock_;
  bool ordered_ = false;
};

}  // namespace fockmi

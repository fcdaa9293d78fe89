// Host side of the two-stage pair form (pairs.hip): blocks of pairs, buffers, launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "../../include/fockmi.h"
#include "pairs.hpp"
#include "plan.hpp"

using namespace fockmi;

namespace fockmi {

extern thread_local std::string g_last_error;

// Targets of one row of blocks. Stage 2 runs nr/64 waves per target tile, and a grid of
// about 8,192 waves fills the 256 CUs twice over; two-sided blocks take multiples of 64
// targets, whose mirror sums meet in one workgroup. At 32^3 that is 128 targets; with the
// 8 GiB batch a block then runs 16,384 to 32,768 pairs, so that its last round costs under 2%
// (32^3 / 216 k / 16 bands: 1,159 ms with batches of 512 MiB, 1,110 with 4 GiB, 1,088 with 8).
static int row_targets(int nt, int nr, size_t field_bytes, size_t budget, int least, bool tri) {
  long want = std::max<long>(64, ((1L << 22) / nr + 63) / 64 * 64);
  if (tri) {
    while (want > 64 && (size_t)want * want * field_bytes > budget) want -= 64;
  } else {
    while (want > kPairTile && (size_t)want * 16 * field_bytes > budget) want -= want > 64 ? 64 : kPairTile;
    while (want > 1 && (size_t)want * least * field_bytes > budget) --want;
  }
  return (int)std::min<long>(want, nt);
}

void pairs_block_shape(int nt, int nj, int ns, int nr, size_t fb, size_t budget, bool whole_partials, bool tri,
                       int* rows, long* njmax) {
  const int least = whole_partials ? std::min(16, ns) : 1;
  *rows = row_targets(nt, nr, fb, budget, least, tri);
  long m = std::min<long>((long)(budget / ((size_t)*rows * fb)), nj);
  m = std::max<long>(m, least);
  *njmax = tri ? std::max<long>(m, *rows) : m;
}

bool Plan::pairs_fit(int nr, int nt, int nj, int ns, size_t fb, size_t batch, bool sums32, bool two, bool tri,
                     PairsLayout* l, size_t room) const {
  for (size_t budget = workspace_cap ? std::min(workspace_cap, batch) : batch;; budget /= 2) {
    *l = pairs_layout(nr, nt, nj, ns, fb, budget, sums32, two, tri);
    if ((!workspace_cap || l->largest <= workspace_cap) && l->end <= room) return true;
    if (budget < fb) return false;
  }
}

bool Plan::pairs_tri_fits(int nt, int nb, int nr, bool f32) const {
  PairsLayout l;
  return pairs_fit(nr, nt, nt, nb, (size_t)nr * (f32 ? sizeof(c64) : sizeof(c128)), pair_batch, f32, true, true, &l);
}

// Measured costs of the forms on a 256-CU device, cubic grids (64 k-points of 16 bands, phi apart
// from u at 64 to 1,024 targets): `wg[m - 1]` us per source with m workgroups of a fused kernel
// on every CU, one target each (fewer targets than CUs leave CUs idle); the pair form `pair` ns per
// pair one-sided and `sym` ns per pair of the sum with the pair symmetry, whatever the shape of
// the sum. Per source, 128 targets of 20^3: FP32 8.1 us fused and 4.4 in pairs, FP64 9.9 and 8.1;
// 256: 8.3 and 8.3, 10.7 and 15.9.
struct FormCost {
  int n, per_cu;  // grid length, workgroups of the fused kernel that a CU holds
  double wg[4], pair, sym;
};
constexpr FormCost kCost64[] = {{16, 2, {4.8, 6.9}, 27.5, 17.0}, {20, 1, {10.7}, 62.5, 35.0}, {24, 1, {31.9}, 126.0, 67.5}};
constexpr FormCost kCost32[] = {
    {16, 4, {4.2, 4.8, 7.0, 8.9}, 13.6, 10.5}, {20, 2, {8.3, 13.4}, 33.0, 20.5}, {24, 1, {13.1}, 62.5, 35.5}};

static const FormCost* form_cost(int n, bool f32) {
  for (const FormCost& x : f32 ? kCost32 : kCost64)
    if (x.n == n) return &x;
  return nullptr;
}

Plan::PairRule Plan::pair_rule(const Cell& c, const PairSet& ps, int nx, int ns, bool same, bool f32) const {
  PairRule r;
  const long nt = (long)(ps.ntk_all ? ps.ntk_all : ps.ntk) * nx, nj = (long)ps.nsk * ns;
  const FormCost* fc = form_cost(c.geom.n1, f32);
  if (!fc) return r;
  same = same && nx == ns && !c.ds;
  // a cap without room for one FP32 partial sum's pairs (FP64: one pair) of one target
  if (workspace_cap && (size_t)(f32 ? std::min(ns, 16) : 1) * c.nr * (f32 ? sizeof(c64) : sizeof(c128)) > workspace_cap)
    return r;
  r.pairs_ns = nt * fc->pair * 256.0 / num_cus;
  const long per_cu = (nt + num_cus - 1) / num_cus;  // targets of the busiest CU
  const int rest = (int)(per_cu % fc->per_cu);
  const double fused = 1e3 * ((double)(per_cu / fc->per_cu) * fc->wg[fc->per_cu - 1] + (rest ? fc->wg[rest - 1] : 0.0));
  r.fused_ns = r.ns = fused;
  // below 4 tiles the triangle is nearly the whole square, and the mirror sums cost a launch
  const bool tri_ok = split_sym && same && ps.ntk == c.nk && ps.nsk == c.nk && ps.qidx == (const int*)c.qidx.ptr &&
                      nt > 3 * kPairTile &&
                      pairs_tri_fits((int)nt, ns, c.nr, f32);
  if (f32) {
    // what the allocation-free call needs where the targets could be u itself, also when they are not:
    // a k-range of u, or a copy of it, goes the way of the application to u and gives its bits
    const size_t need = noalloc_bytes(c, ps, nx, ns, nx == ns && !c.ds);
    r.shared = need <= kNoAllocBytes;
    if (r.shared) {
      // fock_apply_noalloc serves this sum with the same bits: one-sided in both (its sums do
      // not depend on the blocks), and only where its 64 MiB hold a batch that is still the
      // faster form
      const size_t least = (size_t)std::min(ns, 16) * c.nr * sizeof(c64);
      r.pairs = nt * nj <= (fc->n == 24 ? 96 * 96 : 128 * 128) && r.pairs_ns < fused &&
                need + least <= kNoAllocBytes;
      if (r.pairs) r.ns = r.pairs_ns;
      return r;
    }
  }
  const double sym = nt * fc->sym * 256.0 / num_cus;
  if (tri_ok && sym < fused) r.pairs = r.tri = true;
  else r.pairs = r.pairs_ns < fused;
  if (r.pairs) r.ns = r.tri ? sym : r.pairs_ns;
  return r;
}

// The forked streams run four cells' kernels at a time (the device's hardware queues), whose workgroups
// share CUs although others are idle: of four cells of 16^3 three to a CU, of 20^3 two. Both estimates
// leave out some 13 us per cell for its launches; the forked one is within 16% of these sets' times
// but for that. Measured, forked and in sequence (us): 8 cells of 16^3 / 8 k with
// 16, 8 and 4 bands 1,821 and 2,019, 1,002 and 587, 512 and 233; 8 of 24^3 / 8 k / 12 b 4,496 and
// 4,453, of 24^3 / 4 k / 8 b 889 and 640; 4 of 20^3 / 8 k / 8 b 913 and 604; 16^3 / 64 k / 16 b with
// 16^3 / 8 k / 16 b 9,281 and 9,467; 24^3 / 125 k / 16 b with two smaller 225,600 and 152,100. The
// sequence has to win by 15% in the estimate.
bool Plan::batch_in_sequence(const void* const* u, const void* const* phi, const int* nphi) const {
  constexpr int kQueues = 4;
  struct One {
    double fused, nj, nt;
    const FormCost* fc;
  };
  std::vector<One> cs;
  bool pairs = false;
  double seq = 0.0, work = 0.0, forked = 0.0;
  for (size_t i = 0; i < cells.size(); ++i) {
    const Cell& c = cells[i];
    const PairRule r = pair_rule(c, c.fwd(), nphi[i], c.nb, phi[i] == u[i], true);
    const FormCost* fc = form_cost(c.geom.n1, true);
    if (!fc || r.fused_ns == 0.0) return false;
    const double nj = (double)c.nsrc * c.nb, nt = (double)c.nk * nphi[i];
    pairs = pairs || r.pairs;
    seq += nj * r.ns;
    work += nj * nt * fc->wg[fc->per_cu - 1] * 1e3 / fc->per_cu / num_cus;
    cs.push_back(One{nj * r.fused_ns, nj, nt, fc});
  }
  std::sort(cs.begin(), cs.end(), [](const One& a, const One& b) { return a.fused > b.fused; });
  for (size_t i = 0; i < cs.size(); i += kQueues) {
    const int beside = (int)std::min<size_t>(kQueues, cs.size() - i);
    double most = 0.0;
    for (int k = 0; k < beside; ++k) {
      const One& o = cs[i + k];
      const int stack = std::min(o.fc->per_cu, std::max(1, beside - 1));
      most = std::max(most, o.nt > num_cus ? o.fused : o.nj * o.fc->wg[stack - 1] * 1e3);
    }
    forked += most;
  }
  return pairs && 1.15 * seq < std::max(forked, work);
}

template <typename TW, typename TM>
fock_status pairs_blocks(int nr, int np, int nt, int nj, int ns, const PairStage<TW>& stage, const cx<TM>* M,
                         const Mirror<TM>& mr, c128* out, double scale, bool accumulate, int rows, long njmax,
                         cx<TW>* W, void* run, c128* mir, c64* mcomp, hipStream_t st) {
  constexpr bool F32 = sizeof(TM) == 4;
  const bool two = mr.dst != nullptr;
  fock_status s;
  hipError_t e;
  WsumArgs<TW, TM> wa{};
  wa.W = W;
  wa.M = M;
  wa.F = mr.F;
  wa.out = out;
  wa.mir = two ? mir : nullptr;
  wa.mcomp = two && F32 ? mcomp : nullptr;
  wa.ns = ns;
  wa.nsrc = nj;
  wa.nr = nr;
  wa.np = np;
  wa.group = pair_group(rows, nr);
  wa.accumulate = accumulate ? 1 : 0;
  wa.scale = scale;
  auto block = [&](int t0, int ntb, int j0, int njb, bool tri, bool first, bool last, bool mfirst) -> fock_status {
    wa.t0 = t0;
    wa.nt = ntb;
    wa.j0 = j0;
    wa.nj = njb;
    wa.tri = tri ? 1 : 0;
    wa.jb0 = j0 % ns;
    wa.first = first ? 1 : 0;
    wa.last = last ? 1 : 0;
    wa.mfirst = mfirst ? 1 : 0;
    // the sums kept between the blocks of a row, indexed by target
    wa.comp = F32 ? (c64*)run - (long)t0 * nr : nullptr;
    wa.run = F32 ? nullptr : (c128*)run - (long)t0 * nr;
    if ((e = stage(PairBlock{t0, ntb, j0, njb, tri ? 1 : 0, pair_count(ntb, njb, tri)}, W)) != hipSuccess)
      return hip_fail(e, "pair kernel");
    if ((e = launch_wsum<TW, TM>(wa, st)) != hipSuccess) return hip_fail(e, "pair sums");
    return FOCK_OK;
  };
  for (int t0 = 0; t0 < nt; t0 += rows) {
    const int ntb = std::min(rows, nt - t0);
    const int jend = mr.tri ? t0 : nj;
    for (int j0 = 0; j0 < jend;) {
      int j1 = (int)std::min<long>(jend, j0 + njmax);
      if (F32 && !two && j1 < jend) {
        // whole FP32 partial sums per block: a target's sum does not depend on the blocks
        const int b = j1 % ns;
        j1 -= b % 16;
        if (j1 <= j0) j1 = j0 + std::min(16, ns - j0 % ns);
      }
      const bool first = j0 == 0, last = !mr.tri && j1 == jend;
      if ((s = block(t0, ntb, j0, j1 - j0, false, first, last, !mr.tri && t0 == 0)) != FOCK_OK) return s;
      j0 = j1;
    }
    if (mr.tri && (s = block(t0, ntb, t0, ntb, true, t0 == 0, true, true)) != FOCK_OK) return s;
  }
  if (two && (e = launch_mirror_add(mr.dst, mir, wa.mcomp, mr.scale, mr.scale_im, mr.accumulate ? 1 : 0, nj, nr, rows,
                                    wa.group, mr.tri ? 1 : 0, np, st)) != hipSuccess)
    return hip_fail(e, "mirror sums");
  return FOCK_OK;
}

PairsLayout pairs_layout(int nr, int nt, int nj, int ns, size_t fb, size_t budget, bool sums32, bool two, bool tri) {
  PairsLayout l;
  pairs_block_shape(nt, nj, ns, nr, fb, budget, sums32 && !two, tri, &l.rows, &l.njmax);
  const int group = pair_group(l.rows, nr);
  l.groups = (l.rows + group - 1) / group;
  auto piece = [&](size_t bytes) {
    const size_t at = l.end;
    l.end = (at + bytes + 255) & ~size_t(255);
    l.largest = std::max(l.largest, bytes);
    return at;
  };
  piece((size_t)l.rows * l.njmax * fb);
  if (tri ? nt > l.rows : nj > l.njmax) l.run = piece((size_t)l.rows * nr * (sums32 ? sizeof(c64) : sizeof(c128)));
  if (two) l.mir = piece((size_t)l.groups * nj * nr * sizeof(c128));
  if (two && sums32) l.mcomp = piece((size_t)l.groups * nj * nr * sizeof(c64));
  return l;
}

bool Plan::pairs_ready(int nr, int nt, int nj, int ns, size_t fb, bool sums32, bool two, bool tri) const {
  PairsLayout l;
  return !g_capturing || pairs_fit(nr, nt, nj, ns, fb, pair_batch, sums32, two, tri, &l, pscratch.bytes);
}

template <typename TW, typename TM>
fock_status Plan::run_pairs(int nr, int np, int nt, int nj, int ns, const PairStage<TW>& stage, const cx<TM>* M, c128* out,
                            double scale, bool accumulate, const Mirror<TM>& mr, size_t batch, hipStream_t st, bool others) {
  constexpr bool F32 = sizeof(TM) == 4;
  const size_t fb = (size_t)nr * sizeof(cx<TW>);
  const bool two = mr.dst != nullptr;
  // sums of this precision at 16^3 and 20^3 may run on several streams at once
  if (prec == FOCK_FP64_FUSED) PlanCall::order();
  fock_status s;
  PairsLayout l;
  // under capture in what is there, if that is possible
  const bool there = g_capturing && pairs_fit(nr, nt, nj, ns, fb, batch, F32, two, mr.tri, &l, pscratch.bytes);
  if (there) pscratch.hold();
  for (; !there; batch /= 2) {
    if (!pairs_fit(nr, nt, nj, ns, fb, batch, F32, two, mr.tri, &l))
      return fail(FOCK_ERR_NOMEM, "pair scratch: %zu bytes exceed the plan workspace cap of %zu bytes", l.largest,
                  workspace_cap);
    s = pscratch.ensure(l.end, 0, "pair scratch");
    if (s == FOCK_OK) break;
    // other forms are faster than small batches, where there are any
    if (batch <= (others ? size_t(64) << 20 : fb)) return s;
  }
  g_last_error.clear();  // a smaller batch after a failed allocation is no failure
  char* base = (char*)pscratch.ptr;
  return pairs_blocks<TW, TM>(nr, np, nt, nj, ns, stage, M, mr, out, scale, accumulate, l.rows, l.njmax, (cx<TW>*)base,
                              base + l.run, (c128*)(base + l.mir), (c64*)(base + l.mcomp), st);
}

template <typename T>
PairStage<T> cube_stage(int n, int num_cus, const PairSet& ps, const cx<T>* X, int nx, const cx<T>* P, int ns,
                        const T* Kt, hipStream_t st) {
  PairArgs<T> pa{};
  pa.X = X;
  pa.P = P;
  pa.Kt = Kt;
  pa.qidx = ps.qidx;
  pa.nx = nx;
  pa.ns = ns;
  pa.nsk = ps.nsk;
  return [=](const PairBlock& b, cx<T>* W) {
    PairArgs<T> q = pa;
    q.b = b;
    q.W = W;
    return launch_pair_w<T>(n, q, num_cus, st);
  };
}

template <typename T>
PairStage<T> plane_stage(const Geom& g, int num_cus, const PairSet& ps, const c128* X, int nx, const c128* P, int ns,
                         const double* K, hipStream_t st) {
  PlaneArgs<T> pa{};
  pa.X = X;
  pa.P = P;
  pa.K = K;
  pa.qidx = ps.qidx;
  pa.nx = nx;
  pa.ns = ns;
  pa.nsk = ps.nsk;
  pa.n1 = g.n1;
  const int n2 = g.n2, n3 = g.n3;
  return [=](const PairBlock& b, cx<T>* W) {
    PlaneArgs<T> q = pa;
    q.b = b;
    q.W = W;
    return launch_pair_planes<T>(n2, n3, q, num_cus, st);
  };
}

template PairStage<float> cube_stage<float>(int, int, const PairSet&, const c64*, int, const c64*, int, const float*,
                                            hipStream_t);
template PairStage<double> cube_stage<double>(int, int, const PairSet&, const c128*, int, const c128*, int,
                                              const double*, hipStream_t);
template PairStage<float> plane_stage<float>(const Geom&, int, const PairSet&, const c128*, int, const c128*, int,
                                             const double*, hipStream_t);
template PairStage<double> plane_stage<double>(const Geom&, int, const PairSet&, const c128*, int, const c128*, int,
                                               const double*, hipStream_t);

template fock_status pairs_blocks<float, float>(int, int, int, int, int, const PairStage<float>&, const c64*,
                                                const Mirror<float>&, c128*, double, bool, int, long, c64*, void*,
                                                c128*, c64*, hipStream_t);
#define FOCKMI_RUN_PAIRS(TW, TM)                                                                                  \
  template fock_status Plan::run_pairs<TW, TM>(int, int, int, int, int, const PairStage<TW>&, const cx<TM>*, c128*,    \
                                               double, bool, const Mirror<TM>&, size_t, hipStream_t, bool);
FOCKMI_RUN_PAIRS(float, float)
FOCKMI_RUN_PAIRS(double, double)
FOCKMI_RUN_PAIRS(float, double)
#undef FOCKMI_RUN_PAIRS

}  // namespace fockmi

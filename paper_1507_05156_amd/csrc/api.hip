// C ABI of libfockmi: plans, argument checks and dispatch of the device kernels.
//
// The operator (Sec. II C, Eqs. (15)-(16)) is run through one general routine,
//   out[kt][s] = (accumulate ? out : 0) + scale * sum_{ks, b} M[ks][b] * W(P[ks][b], X[kt][s]; K_{kt-ks}),
// W(p, x; K) = (1/N_r) IDFT(K DFT(conj(p) x)). The forward operator is
// (X, P, M) = (phi, u, u) with scale = -1/N_k; the reverse-mode formulas use
// the other role assignments (see fock_vjp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <tuple>
#include <vector>
#include <cstdlib>
#include <cstdint>

#include "../../include/fockmi.h"
#include "kernels.hpp"
#include "plan.hpp"

using namespace fockmi;

namespace fockmi {

thread_local std::string g_last_error;

fock_status fail(fock_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

fock_status hip_fail(hipError_t e, const char* where) {
  return fail(FOCK_ERR_HIP, "%s: %s", where, hipGetErrorString(e));
}

bool valid_len(int n) { return n == 16 || n == 20 || n == 24 || n == 32; }

thread_local bool g_capturing = false;
static thread_local PlanCall* g_call = nullptr;

PlanCall::PlanCall(Plan* p, hipStream_t st) : p_(p), st_(st), lock_(p->calls) {
  g_capturing = stream_captures(st);
  g_call = this;
}

void PlanCall::order() {
  PlanCall* c = g_call;
  if (!c || c->ordered_ || g_capturing) return;
  c->ordered_ = true;
  if (c->p_->done_recorded) (void)hipStreamWaitEvent(c->st_, c->p_->done, 0);
}

// The record costs 2.8 us between calls that follow each other at once (fp64f apply of 16^3 / 8 k /
// 4 bands 42.2 -> 45.0 us, orthonormalisation of it 17.3 -> 20.2), nothing where a call is waited for.
PlanCall::~PlanCall() {
  if (ordered_) {
    p_->done_recorded = hipEventRecord(p_->done, st_) == hipSuccess;
    if (!p_->done_recorded) {  // a call on another stream could not wait for this one
      (void)hipGetLastError();
      (void)hipStreamSynchronize(st_);
    }
  }
  g_capturing = false;
  g_call = nullptr;
}

bool PlanCall::give_back(const DevBuf* asking) {
  if (!g_call || g_capturing) return false;
  DevBuf& b = g_call->p_->pscratch;
  if (&b == asking || !b.ptr || b.held) return false;
  b.drop();
  return true;
}

void DevBuf::hold() {
  if (ptr && g_capturing) held = true;
}

fock_status DevBuf::ensure(size_t need, size_t cap, const char* what) {
  if (need <= bytes) {
    hold();
    return FOCK_OK;
  }
  if (cap && need > cap)
    return fail(FOCK_ERR_NOMEM, "%s: %zu bytes exceed the plan workspace cap of %zu bytes", what, need, cap);
  drop();
  hipError_t e = hipMalloc(&ptr, need);
  if (e != hipSuccess && PlanCall::give_back(this)) {
    (void)hipGetLastError();
    e = hipMalloc(&ptr, need);
  }
  if (e != hipSuccess) {
    ptr = nullptr;
    (void)hipGetLastError();
    return fail(FOCK_ERR_NOMEM, "%s: hipMalloc(%zu) failed: %s", what, need, hipGetErrorString(e));
  }
  bytes = need;
  hold();
  return FOCK_OK;
}

bool stream_captures(hipStream_t st) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return cs != hipStreamCaptureStatusNone;
}

void DevBuf::drop() {
  if (ptr && held) kept.push_back(ptr);
  else if (ptr) (void)hipFree(ptr);
  ptr = nullptr;
  bytes = 0;
  held = false;
}

void DevBuf::release() {
  held = false;
  drop();
  for (void* p : kept) (void)hipFree(p);
  kept.clear();
}

fock_status Plan::check_ready(int cell) const {
  if (magic != kMagic) return fail(FOCK_ERR_STATE, "plan is not valid (destroyed or corrupt)");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != device)
    return fail(FOCK_ERR_STATE, "plan was created on device %d, current device is %d", device, dev);
  if (cell < 0 || cell >= (int)cells.size()) return fail(FOCK_ERR_ARG, "cell index %d out of range", cell);
  return FOCK_OK;
}

// ------------------------------------------------------------------ plumbing
namespace {
// the two events of a tuning measurement
struct TuneEvents {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t create() {
    hipError_t e = hipEventCreate(&e0);
    return e == hipSuccess ? hipEventCreate(&e1) : e;
  }
  ~TuneEvents() {
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  }
};
}  // namespace

fock_status Plan::run_plain(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M, int ns,
                            c128* out, double scale, bool accumulate, hipStream_t st) {
  const int nr = c.nr, nt = ps.ntk * nx, nj = ps.nsk * ns;
  const bool cube = c.Kp.ptr != nullptr;  // the field fits on a CU
  // many targets: the fused FP64 kernel, which keeps each target's sum on its CU; under capture also where
  // there is no scratch for the pair form
  if (cube && !(pair_rule(c, ps, nx, ns, X == P && P == M, false).pairs &&
                pairs_ready(nr, nt, nj, ns, nr * sizeof(c128), false, false, false))) {
    const fock_status s = run_fused64(c, ps, X, nx, P, M, ns, out, scale, accumulate, st);
    if (s != FOCK_ERR_NOMEM) return s;
    g_last_error.clear();  // no room for its sums (nothing has been launched): the pair form takes them in blocks
  }
  // The pair symmetry, where u is targets and sources over the whole mesh; not in FP32, whose
  // k-ranges give the full application's bits.
  Mirror<double> mr;
  if (split_sym && !c.f32plain && !c.ds && X == P && P == M && nx == ns && ps.ntk == c.nk && ps.nsk == c.nk &&
      ps.qidx == (const int*)c.qidx.ptr && nt > 3 * kPairTile && pairs_tri_fits(nt, ns, nr, false) &&
      pairs_ready(nr, nt, nj, ns, nr * sizeof(c128), false, true, true)) {
    mr.F = X;
    mr.dst = out;
    mr.scale = scale;
    mr.accumulate = mr.tri = true;
  }
  auto run = [&](size_t batch) -> fock_status {
    hipError_t e;
    if ((e = prof_begin(st)) != hipSuccess) return hip_fail(e, "profile event");
    auto sums = [&](const Mirror<double>& m) -> fock_status {
      if (c.f32plain)
        return run_pairs<float, double>(
            nr, 0, nt, nj, ns, plane_stage<float>(c.geom, num_cus, ps, X, nx, P, ns, (const double*)c.Kpl.ptr, st), M,
            out, scale, accumulate, m, batch, st, cube || m.dst);
      return run_pairs<double, double>(
          nr, 0, nt, nj, ns,
          cube ? cube_stage<double>(c.geom.n1, num_cus, ps, X, nx, P, ns, (const double*)c.Kp.ptr, st)
               : plane_stage<double>(c.geom, num_cus, ps, X, nx, P, ns, (const double*)c.Kpl.ptr, st),
          M, out, scale, accumulate, m, batch, st, cube || m.dst);
    };
    fock_status s = sums(mr);
    if (s == FOCK_ERR_NOMEM && mr.dst) {
      // no room for the mirror sums: every pair (nothing has been launched)
      g_last_error.clear();
      s = sums(Mirror<double>{});
    }
    if (s != FOCK_OK) prof_drop();
    if (s == FOCK_ERR_NOMEM && cube) {
      // no room for a batch (nothing has been launched): the fused kernel
      g_last_error.clear();
      return run_fused64(c, ps, X, nx, P, M, ns, out, scale, accumulate, st);
    }
    if (s != FOCK_OK) return s;
    if ((e = prof_end(st)) != hipSuccess) return hip_fail(e, "profile event");
    return FOCK_OK;
  };
  const std::string key = key_for(c, ps, nx, "plain");
  TuneEntry te;
  if (tune.get(key, &te)) return run((size_t)te.fields["batch_mb"] << 20);
  if (!tuning || accumulate || g_capturing) return run(pair_batch);
  // measure the pair-batch size (each candidate writes the same result to rounding)
  TuneEvents ev;
  hipError_t e = ev.create();
  if (e != hipSuccess) return hip_fail(e, "tuning event");
  double best = 1e300;
  int bmb = 16384;
  for (int mb : {1024, 4096, 16384}) {
    (void)hipEventRecord(ev.e0, st);
    fock_status s = run((size_t)mb << 20);
    if (s != FOCK_OK) return s;
    (void)hipEventRecord(ev.e1, st);
    if ((e = hipEventSynchronize(ev.e1)) != hipSuccess) return hip_fail(e, "tuning sync");
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, ev.e0, ev.e1);
    if (ms < best) {
      best = ms;
      bmb = mb;
    }
  }
  te.fields["batch_mb"] = bmb;
  te.fields["ms"] = best;
  tune.put(key, te);
  save_tune();
  return run((size_t)bmb << 20);
}

fock_status Plan::shadow(DevBuf& buf, const c128* src, size_t count, const char* what, hipStream_t st, int np,
                         const c64** out) {
  fock_status s = buf.ensure(count * sizeof(c64), workspace_cap, what);
  if (s != FOCK_OK) return s;
  hipError_t e = np ? launch_to_c64_paired((c64*)buf.ptr, src, (long)count, np, st)
                    : launch_to_c64((c64*)buf.ptr, src, (long)count, st);
  if (e != hipSuccess) return hip_fail(e, what);
  *out = (const c64*)buf.ptr;
  return FOCK_OK;
}

fock_status Plan::run_fused(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M, int ns,
                            c128* out, double scale, bool accumulate, hipStream_t st) {
  const int nr = c.nr;
  const c64 *Xs = nullptr, *Ps = nullptr, *Ms = nullptr;
  fock_status s;
  // the complex64 shadows, in natural order or in the pair form's
  int shadow_np = -1;
  auto shadows = [&](int np) -> fock_status {
    fock_status st2;
    if (np == shadow_np) return FOCK_OK;
    if ((st2 = shadow(shadow_p, P, (size_t)ps.nsk * ns * nr, "complex64 shadow (P)", st, np, &Ps)) != FOCK_OK) return st2;
    if (M == P) {
      Ms = Ps;
    } else if ((st2 = shadow(shadow_m, M, (size_t)ps.nsk * ns * nr, "complex64 shadow (M)", st, np, &Ms)) != FOCK_OK) {
      return st2;
    }
    const bool same_k = ps.ntk == ps.nsk && nx == ns;  // then X may share a source array's shadow
    if (same_k && X == P) {
      Xs = Ps;
    } else if (same_k && X == M) {
      Xs = Ms;
    } else if ((st2 = shadow(shadow_x, X, (size_t)ps.ntk * nx * nr, "complex64 shadow (X)", st, np, &Xs)) != FOCK_OK) {
      return st2;
    }
    shadow_np = np;
    return FOCK_OK;
  };
  const int nitems = ps.ntk * nx;
  const int n = c.geom.n1;
  // the lockstep form runs one workgroup per CU (a multiple of 8: one share per XCD)
  LockstepCfg ls{nullptr, (num_cus / 8) * 8};
  const bool has_ls = fused_has_lockstep(n) && ls.nwg >= 8;
  // the split 32^3 form runs one workgroup per CU, two per target (a multiple of 16)
  const int nwg_split = (num_cus / 16) * 16;
  const bool has_split = n == 32 && c.SD.ptr && nwg_split >= 16 && has_ls && !accumulate;
  // its pair symmetry: u as targets and sources over the whole k mesh (W of source b on
  // target a is conj of W of a on b); the mirror copies need 8 nitems nr (8 + 16 + 8) bytes
  const size_t mirror_bytes = (size_t)8 * nitems * nr * (sizeof(c64) * 2 + sizeof(c128));
  bool sym = has_split && split_sym && !c.ds && ps.ntk == c.nk && ps.nsk == c.nk &&
                   ps.qidx == (const int*)c.qidx.ptr && X == P && P == M && nx == ns && c.nk >= 3 &&
                   (!workspace_cap || mirror_bytes <= workspace_cap);
  // the two-stage pair form, with the pair symmetry when u is targets and sources over the whole mesh
  const bool pairs_tri = split_sym && !c.ds && ps.ntk == c.nk && ps.nsk == c.nk &&
                         ps.qidx == (const int*)c.qidx.ptr && X == P && P == M && nx == ns &&
                         pairs_tri_fits(nitems, ns, nr, true);
  PairRule rule = pair_rule(c, ps, nx, ns, X == P && P == M, true);
  if (n == 32) rule.tri = pairs_tri;
  auto usable = [&](int v) {
    if (n != 32) {
      // of a sum that fock_apply_noalloc shares, only the form of the rule; else the rule is a default
      if (rule.shared) return rule.pairs ? v == 3 : (v >= 0 && v < fused_variants(n));
      return (v >= 0 && v < fused_variants(n)) || (v == 3 && rule.pairs);
    }
    return v == 0 || (v == 1 && has_ls) || (v == 2 && has_split) || v == 3;
  };
  auto fallback_variant = [&](int v) {
    return usable(v) ? v : (n == 32 ? (has_ls ? 1 : 0) : (usable(3) ? 3 : 0));
  };
  // the lockstep form's k' split: the part count (dividing the source k-points,
  // at most 4) with the fewest rounds of ls.nwg workgroups, in units of a whole
  // target's sum
  int ksplit = 1;
  if (has_ls) {
    if ((s = sync.ensure(kLockstepInts * sizeof(int), workspace_cap, "lockstep counters")) != FOCK_OK) return s;
    ls.counters = (int*)sync.ptr;
    double best = 1e300;
    for (int h = 1; h <= 4; ++h) {
      if (ps.nsk % h) continue;
      const double rounds = std::ceil((double)nitems * h / ls.nwg) / h;
      if (rounds < best * (1.0 - 1e-9)) {
        best = rounds;
        ksplit = h;
      }
    }
  }
  FusedArgs a{};
  a.Kt = (const float*)c.Kt.ptr;
  a.qidx = ps.qidx;
  a.out = out;
  a.nk = ps.nsk;
  a.nx = nx;
  a.nb = ns;
  a.item0 = 0;
  a.nitems = nitems;
  a.scale = scale;
  a.accumulate = accumulate ? 1 : 0;
  a.xcd_map = xcd_map;
  a.n = n;
  a.ksplit = 1;
  a.part_out = nullptr;
  a.gate = nullptr;
  // buffers of one variant (grown on demand, kept by the plan)
  auto prepare = [&](int v) -> fock_status {
    fock_status st2;
    if ((st2 = shadows(v == 3 ? n * n : 0)) != FOCK_OK) return st2;
    a.X = Xs;
    a.P = Ps;
    a.M = Ms;
    if (v == 3) return FOCK_OK;  // run_pairs sizes its own buffers
    const int h = v == 1 ? ksplit : 1;
    if ((st2 = comp.ensure((size_t)h * nitems * nr * sizeof(c64), workspace_cap, "compensation buffer")) != FOCK_OK)
      return st2;
    if (h > 1 && (st2 = parts.ensure((size_t)(h - 1) * nitems * nr * sizeof(c128), workspace_cap, "k' part sums")) !=
                     FOCK_OK)
      return st2;
    const size_t acc_elems = fused_acc_scratch_elems(n, v == 0 ? nitems : ls.nwg);
    if (acc_elems && (st2 = accs.ensure(acc_elems * sizeof(c64), workspace_cap, "FP32 partial sums")) != FOCK_OK)
      return st2;
    if (v == 2) {
      if ((st2 = xbuf.ensure(split32_xbuf_elems(nwg_split) * sizeof(c64), workspace_cap, "exchange buffers")) !=
          FOCK_OK)
        return st2;
      if ((st2 = sflags.ensure(split32_flag_ints(nwg_split) * sizeof(int), workspace_cap, "rendezvous counters")) !=
          FOCK_OK)
        return st2;
      if ((st2 = sstatus.ensure(sizeof(int), workspace_cap, "abort word")) != FOCK_OK) return st2;
      if (sym) {
        // the mirror copies; when the device cannot hold them, the split form runs every pair
        const size_t nel = (size_t)8 * nitems * nr;
        if (mpart.ensure(nel * sizeof(c64), workspace_cap, "mirror partial sums") != FOCK_OK ||
            msum.ensure(nel * sizeof(c128), workspace_cap, "mirror FP64 sums") != FOCK_OK ||
            mcomp.ensure(nel * sizeof(c64), workspace_cap, "mirror compensation") != FOCK_OK ||
            mdone.ensure(split32_mirror_ctr_ints(nitems) * sizeof(int), workspace_cap, "mirror counters") != FOCK_OK) {
          mpart.drop();
          msum.drop();
          mcomp.drop();
          mdone.drop();
          sym = false;
          g_last_error.clear();  // the call goes on and succeeds: no failure to report
        }
      }
      if (sym) {
        if (sym_key[0] != nwg_split || sym_key[1] != c.nk || sym_key[2] != ns || sym_key[3] != split_stagger_shift) {
          std::vector<int> rank, cnt;
          split32_sym_tables(nwg_split, c.nk, ns, split_stagger_shift, &rank, &cnt);
          if ((st2 = sym_rank.ensure(rank.size() * sizeof(int), workspace_cap, "mirror push order")) != FOCK_OK)
            return st2;
          if ((st2 = sym_cnt.ensure(cnt.size() * sizeof(int), workspace_cap, "mirror push counts")) != FOCK_OK)
            return st2;
          hipError_t e2 = hipMemcpy(sym_rank.ptr, rank.data(), rank.size() * sizeof(int), hipMemcpyHostToDevice);
          if (e2 == hipSuccess)
            e2 = hipMemcpy(sym_cnt.ptr, cnt.data(), cnt.size() * sizeof(int), hipMemcpyHostToDevice);
          if (e2 != hipSuccess) return hip_fail(e2, "mirror tables");
          sym_key[0] = nwg_split;
          sym_key[1] = c.nk;
          sym_key[2] = ns;
          sym_key[3] = split_stagger_shift;
        }
        sym_rank.hold();
        sym_cnt.hold();
      }
      if (!fallbacks.ptr) {
        if ((st2 = fallbacks.ensure(sizeof(long long), workspace_cap, "fallback count")) != FOCK_OK) return st2;
        hipError_t e2 = launch_zero_ll((long long*)fallbacks.ptr, st);
        if (e2 != hipSuccess) return hip_fail(e2, "fallback count");
      }
    }
    a.comp = (c64*)comp.ptr;
    a.accs = (c64*)accs.ptr;
    a.ksplit = h;
    a.part_out = h > 1 ? (c128*)parts.ptr : nullptr;
    return FOCK_OK;
  };
  // one application in variant v
  fock_status pairs_status = FOCK_OK;
  auto launch = [&](int v) -> hipError_t {
    if (v == 3) {
      Mirror<float> mr;
      if (rule.tri) {
        mr.F = Xs;
        mr.dst = out;
        mr.scale = scale;
        mr.accumulate = true;
        mr.tri = true;
      }
      pairs_status = run_pairs<float, float>(
          nr, n * n, nitems, ps.nsk * ns, ns,
          cube_stage<float>(n, num_cus, ps, Xs, nx, Ps, ns, (const float*)c.Kp.ptr, st), Ms, out, scale, accumulate, mr, pair_batch, st);
      return hipSuccess;
    }
    if (v != 2) return launch_fused_apply(n, a, st, v, &ls);
    SplitArgs sa{};
    sa.f = a;
    sa.SD = (const float*)c.SD.ptr;
    sa.xbuf = (c64*)xbuf.ptr;
    sa.flags = (int*)sflags.ptr;
    sa.status = (int*)sstatus.ptr;
    sa.wait_ticks = split_wait_ticks;
    if (sym) {
      sa.sym = 1;
      sa.ndelta = c.nk / 2 + 1;
      sa.npush = (c.nk - 1) / 2;
      sa.stagger_shift = split_stagger_shift;
      sa.rank = (const int*)sym_rank.ptr;
      sa.mpart = (c64*)mpart.ptr;
      sa.msum = (c128*)msum.ptr;
      sa.mcomp = (c64*)mcomp.ptr;
      sa.mdone = (int*)mdone.ptr;
    }
    hipError_t e2 = launch_split32(sa, nwg_split, st);
    if (e2 != hipSuccess) return e2;
    // the mirror copies into the output (skipped when the split launch stopped)
    if (sym && (e2 = launch_split32_sym_combine(out, (const c128*)msum.ptr, (const c64*)mcomp.ptr,
                                                (const c64*)mpart.ptr, (const int*)sym_cnt.ptr, nitems, scale,
                                                (const int*)sstatus.ptr, st)) != hipSuccess)
      return e2;
    // the lockstep form behind it, run only if the split launch stopped
    FusedArgs fb = a;
    fb.gate = (const int*)sstatus.ptr;
    if ((e2 = launch_fused_apply(n, fb, st, 1, &ls)) != hipSuccess) return e2;
    if (profiling) e2 = launch_count_abort((long long*)fallbacks.ptr, (const int*)sstatus.ptr, st);
    return e2;
  };
  int variant = fallback_variant(n == 32 && split_form ? 2 : (rule.pairs ? 3 : fused_default_variant(n)));
  hipError_t e;
  const std::string key = key_for(c, ps, nx, "fused");
  TuneEntry te;
  if (tune.get(key, &te)) {
    variant = fallback_variant((int)te.fields["variant"]);
    a.xcd_map = (int)te.fields["xcd_map"];
  } else if (tuning && !accumulate && !g_capturing) {
    // measure every candidate on this call's data (each writes the same result up
    // to the grouping of its FP64 additions); the XCD map matters only for the grid form
    TuneEvents ev;
    if ((e = ev.create()) != hipSuccess) return hip_fail(e, "tuning event");
    double best = 1e300;
    int bv = 0, bx = 1;
    for (int v = 0; v < 4; ++v) {
      if (!usable(v)) continue;
      if ((s = prepare(v)) != FOCK_OK) return s;
      for (int x = 0; x < (v == 0 || (n != 32 && v < 3) ? 2 : 1); ++x) {
        a.xcd_map = v == 0 || (n != 32 && v < 3) ? x : 1;
        (void)hipEventRecord(ev.e0, st);
        if ((e = launch(v)) != hipSuccess) return hip_fail(e, "fused pair kernel");
        if (pairs_status == FOCK_ERR_NOMEM) {
          // no room for a batch (nothing has been launched): not a candidate
          g_last_error.clear();
          pairs_status = FOCK_OK;
          break;
        }
        if (pairs_status != FOCK_OK) return pairs_status;
        (void)hipEventRecord(ev.e1, st);
        if ((e = hipEventSynchronize(ev.e1)) != hipSuccess) return hip_fail(e, "tuning sync");
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, ev.e0, ev.e1);
        if (ms < best) {
          best = ms;
          bv = v;
          bx = a.xcd_map;
        }
      }
    }
    te.fields["variant"] = bv;
    te.fields["xcd_map"] = bx;
    te.fields["ms"] = best;
    tune.put(key, te);
    save_tune();
    variant = bv;
    a.xcd_map = bx;
  }
  // Under capture without scratch for the mirror sums every pair, without any for the pair form a form that
  // sums on the CU, and the pair form where only its scratch is there.
  const size_t fb = nr * sizeof(c64);
  const bool one_sided = pairs_ready(nr, nitems, ps.nsk * ns, ns, fb, true, false, false);
  if (rule.tri && !pairs_ready(nr, nitems, ps.nsk * ns, ns, fb, true, true, true)) rule.tri = false;
  if (variant == 3 && !rule.tri && !one_sided) variant = n == 32 && has_ls ? 1 : 0;
  if (variant != 3 && g_capturing && one_sided && comp.bytes < (size_t)(variant == 1 ? ksplit : 1) * nitems * fb)
    variant = 3;
  if ((s = prepare(variant)) != FOCK_OK) return s;
  if ((e = prof_begin(st)) != hipSuccess) return hip_fail(e, "profile event");
  if ((e = launch(variant)) != hipSuccess) return hip_fail(e, "fused pair kernel");
  if (pairs_status == FOCK_ERR_NOMEM) {
    // no room for a batch (nothing has been launched): the forms that sum on the CU need less
    g_last_error.clear();
    pairs_status = FOCK_OK;
    variant = n == 32 ? (has_split ? 2 : (has_ls ? 1 : 0)) : 0;
    if ((s = prepare(variant)) != FOCK_OK) return s;
    if ((e = launch(variant)) != hipSuccess) return hip_fail(e, "fused pair kernel");
  }
  if (pairs_status != FOCK_OK) return pairs_status;
  if ((e = prof_end(st)) != hipSuccess) return hip_fail(e, "profile event");
  return FOCK_OK;
}

std::string Plan::key_for(const Cell& c, const PairSet& ps, int nx, const char* what) const {
  char buf[192];
  std::snprintf(buf, sizeof(buf), "%s/%s/%s/n%dx%dx%d/nt%d/ns%d/nb%d/nx%d", arch_name().c_str(),
                prec == FOCK_FP32_COMP ? "fp32" : (c.f64f ? "fp64f" : "fp64"), what, c.geom.n1, c.geom.n2, c.geom.n3, ps.ntk, ps.nsk, c.nb,
                nx);
  return buf;
}

void Plan::save_tune() {
  if (!tune_path.empty()) (void)tune.save(tune_path);
}

fock_status Plan::general(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M, int ns,
                          c128* out, double scale, bool accumulate, hipStream_t st) {
  if (prec == FOCK_FP32_COMP && !c.f32plain) return run_fused(c, ps, X, nx, P, M, ns, out, scale, accumulate, st);
  if (c.f64f) return run_fused64(c, ps, X, nx, P, M, ns, out, scale, accumulate, st);
  return run_plain(c, ps, X, nx, P, M, ns, out, scale, accumulate, st);
}

fock_status Plan::run_fused64(Cell& c, const PairSet& ps, const c128* X, int nx, const c128* P, const c128* M,
                              int ns, c128* out, double scale, bool accumulate, hipStream_t st) {
  const int nitems = ps.ntk * nx;
  fock_status s;
  hipError_t e;
  PairRule rule = pair_rule(c, ps, nx, ns, X == P && P == M, false);
  // Under capture, the fused kernels of 16^3 and 20^3 where the plan's precision is this one: they need no
  // plan memory, so that graphs of one plan may replay on several streams at once. Elsewhere the pair form
  // if its buffers are there already.
  if (rule.pairs && g_capturing &&
      ((c.f64f && fused64_acc_scratch_elems(c.geom.n1, 1) == 0) ||
       !pairs_ready(c.nr, nitems, ps.nsk * ns, ns, c.nr * sizeof(c128), false, false, false)))
    rule.pairs = false;
  if (rule.tri && !pairs_ready(c.nr, nitems, ps.nsk * ns, ns, c.nr * sizeof(c128), false, true, true)) rule.tri = false;
  if (rule.pairs) {
    if ((e = prof_begin(st)) != hipSuccess) return hip_fail(e, "profile event");
    auto sums = [&](bool tri) -> fock_status {
      Mirror<double> mr;
      if (tri) {
        mr.F = X;
        mr.dst = out;
        mr.scale = scale;
        mr.accumulate = mr.tri = true;
      }
      return run_pairs<double, double>(
          c.nr, 0, nitems, ps.nsk * ns, ns,
          cube_stage<double>(c.geom.n1, num_cus, ps, X, nx, P, ns, (const double*)c.Kp.ptr, st), M, out, scale,
          accumulate, mr, pair_batch, st);
    };
    s = sums(rule.tri);
    if (s == FOCK_ERR_NOMEM && rule.tri) s = sums(false);
    if (s == FOCK_OK) {
      g_last_error.clear();
      if ((e = prof_end(st)) != hipSuccess) return hip_fail(e, "profile event");
      return FOCK_OK;
    }
    prof_drop();
    if (s != FOCK_ERR_NOMEM) return s;
    g_last_error.clear();  // no room for a batch (nothing has been launched): the fused kernel needs less
  }
  const size_t acc_elems = fused64_acc_scratch_elems(c.geom.n1, nitems);
  if (acc_elems && (s = accs.ensure(acc_elems * sizeof(c128), workspace_cap, "FP64 sums")) != FOCK_OK) return s;
  Fused64Args a{};
  a.X = X;
  a.P = P;
  a.M = M;
  a.Kt = (const double*)c.Kp.ptr;
  a.qidx = ps.qidx;
  a.out = out;
  a.accs = (c128*)accs.ptr;
  a.nk = ps.nsk;
  a.nx = nx;
  a.nb = ns;
  a.item0 = 0;
  a.nitems = nitems;
  a.scale = scale;
  a.accumulate = accumulate ? 1 : 0;
  a.xcd_map = xcd_map;
  if ((e = prof_begin(st)) != hipSuccess) return hip_fail(e, "profile event");
  if ((e = launch_fused64_apply(c.geom.n1, a, st)) != hipSuccess) return hip_fail(e, "fused FP64 pair kernel");
  if ((e = prof_end(st)) != hipSuccess) return hip_fail(e, "profile event");
  return FOCK_OK;
}

fock_status Plan::two_sided(Cell& c, const c128* X, int nx, const c128* us, double scale, c128* out, const c128* F,
                            double mre, double mim, bool maccumulate, c128* gu, hipStream_t st, bool* done) {
  const PairSet ps = c.fwd();
  const int nr = c.nr, nt = ps.ntk * nx, nj = ps.nsk * c.nb, n = c.geom.n1;
  const bool f32 = prec == FOCK_FP32_COMP;
  const bool planes = f32 ? c.f32plain : c.Kp.ptr == nullptr;
  *done = false;
  if (f32 && !planes && n == 32 && split_form) return FOCK_OK;
  if (!planes && n <= 24) {
    // against the faster form of each side; the mirror sums add about a twentieth
    const PairRule a = pair_rule(c, ps, nx, c.nb, false, f32), b = pair_rule(c, c.rev(), c.nb, nx, false, f32);
    if (a.pairs_ns == 0.0 || b.pairs_ns == 0.0) return FOCK_OK;  // no room for a batch
    const double two = 1.05 * a.pairs_ns * nj;
    const double one = std::min(a.fused_ns, a.pairs_ns) * nj + std::min(b.fused_ns, b.pairs_ns) * nt;
    if (two > one) return FOCK_OK;
  }
  // under capture as in run_fused64
  if (g_capturing && ((c.f64f && fused64_acc_scratch_elems(n, 1) == 0) ||
                      !pairs_ready(nr, nt, nj, c.nb, (size_t)nr * (f32 ? sizeof(c64) : sizeof(c128)), f32 && !planes,
                                   true, false)))
    return FOCK_OK;
  fock_status s;
  hipError_t e;
  if ((e = prof_begin(st)) != hipSuccess) return hip_fail(e, "profile event");
  if (f32 && !planes) {
    const c64 *Xs = nullptr, *Ps = nullptr, *Fs = nullptr;
    if ((s = shadow(shadow_p, us, (size_t)nj * nr, "complex64 shadow (P)", st, n * n, &Ps)) != FOCK_OK) return s;
    if ((s = shadow(shadow_x, X, (size_t)nt * nr, "complex64 shadow (X)", st, n * n, &Xs)) != FOCK_OK) return s;
    if ((s = shadow(shadow_m, F, (size_t)nt * nr, "complex64 shadow (M)", st, n * n, &Fs)) != FOCK_OK) return s;
    Mirror<float> mr{Fs, gu, mre, mim, maccumulate, false};
    s = run_pairs<float, float>(nr, n * n, nt, nj, c.nb,
                                cube_stage<float>(n, num_cus, ps, Xs, nx, Ps, c.nb, (const float*)c.Kp.ptr, st), Ps, out,
                                scale, false, mr, pair_batch, st);
  } else {
    Mirror<double> mr{F, gu, mre, mim, maccumulate, false};
    if (f32)
      s = run_pairs<float, double>(
          nr, 0, nt, nj, c.nb, plane_stage<float>(c.geom, num_cus, ps, X, nx, us, c.nb, (const double*)c.Kpl.ptr, st), us,
          out, scale, false, mr, pair_batch, st);
    else
      s = run_pairs<double, double>(
          nr, 0, nt, nj, c.nb,
          planes ? plane_stage<double>(c.geom, num_cus, ps, X, nx, us, c.nb, (const double*)c.Kpl.ptr, st)
                 : cube_stage<double>(n, num_cus, ps, X, nx, us, c.nb, (const double*)c.Kp.ptr, st),
          us, out, scale, false, mr, pair_batch, st);
  }
  if (s != FOCK_OK) prof_drop();
  if (s == FOCK_ERR_NOMEM) {
    // no room for the batch or the mirror sums (nothing has been launched): two separate sums
    g_last_error.clear();
    return FOCK_OK;
  }
  if (s != FOCK_OK) return s;
  if ((e = prof_end(st)) != hipSuccess) return hip_fail(e, "profile event");
  *done = true;
  return FOCK_OK;
}

fock_status Plan::sources(Cell& c, const c128* arr, int nper, DevBuf& buf, hipStream_t st, const c128** out) {
  if (!c.ds) {
    *out = arr;
    return FOCK_OK;
  }
  const size_t block = (size_t)nper * c.nr;  // elements of one k-point's fields
  fock_status s = buf.ensure((size_t)c.nsrc * block * sizeof(c128), workspace_cap, "source sub-mesh orbitals");
  if (s != FOCK_OK) return s;
  for (int i = 0; i < c.nsrc; ++i) {
    hipError_t e = hipMemcpyAsync((c128*)buf.ptr + (size_t)i * block, arr + (size_t)c.src[i] * block,
                                  block * sizeof(c128), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "gather source orbitals");
  }
  *out = (const c128*)buf.ptr;
  return FOCK_OK;
}

fock_status Plan::apply_krange(Cell& c, const c128* u, int k0, int nkout, const c128* phi, int nphi, c128* out,
                               hipStream_t st) {
  const c128* us = nullptr;
  fock_status s = sources(c, u, c.nb, srcbuf, st, &us);
  if (s != FOCK_OK) return s;
  PairSet ps = c.fwd();  // the targets k0 .. k0 + nkout - 1: rows k0.. of the (target, source) table
  ps.ntk = nkout;
  ps.qidx += (size_t)k0 * ps.nsk;
  return general(c, ps, phi, nphi, us, us, c.nb, out, -1.0 / c.nsrc, false, st);
}

fock_status Plan::apply_op(Cell& c, const c128* u, const c128* phi, int nphi, c128* out, hipStream_t st) {
  const c128* us = nullptr;
  fock_status s = sources(c, u, c.nb, srcbuf, st, &us);
  if (s != FOCK_OK) return s;
  return general(c, c.fwd(), phi, nphi, us, us, c.nb, out, -1.0 / c.nsrc, false, st);
}

}  // namespace fockmi

// ====================================================================== ABI
extern "C" {

const char* fock_last_error(void) { return fockmi::g_last_error.c_str(); }

fock_status fock_plan_create(const fock_cell_desc* cells, int ncells, fock_prec prec, const char* tune_cache_json,
                             fockmi_plan* out) {
  g_last_error.clear();
  if (!out) return fail(FOCK_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (!cells || ncells < 1) return fail(FOCK_ERR_ARG, "need at least one cell");
  if (prec != FOCK_FP64 && prec != FOCK_FP32_COMP && prec != FOCK_FP64_FUSED)
    return fail(FOCK_ERR_ARG, "unknown precision %d", (int)prec);
  for (int ci = 0; ci < ncells; ++ci) {
    const fock_cell_desc& d = cells[ci];
    for (int dd = 0; dd < 3; ++dd)
      if (!valid_len(d.n[dd]))
        return fail(FOCK_ERR_SIZE, "cell %d: grid length %d not in {16, 20, 24, 32}", ci, d.n[dd]);
    if (d.nk < 1 || d.nb < 1) return fail(FOCK_ERR_ARG, "cell %d: nk and nb must be >= 1", ci);
    if (!d.kpts) return fail(FOCK_ERR_ARG, "cell %d: kpts is NULL", ci);
    if (!(d.omega > 0.0) || !std::isfinite(d.omega)) return fail(FOCK_ERR_ARG, "cell %d: omega must be > 0", ci);
    if (!(d.gs > 0.0)) return fail(FOCK_ERR_ARG, "cell %d: gs must be > 0", ci);
    if ((long)d.nk * d.nk > 65535L * 64) return fail(FOCK_ERR_ARG, "cell %d: too many k-points", ci);
    if (d.nsrc < 0 || d.nsrc > d.nk) return fail(FOCK_ERR_ARG, "cell %d: nsrc = %d outside 0..nk", ci, d.nsrc);
    if (d.nsrc > 0 && d.src) {
      std::vector<char> used(d.nk, 0);
      for (int i = 0; i < d.nsrc; ++i) {
        const int k = d.src[i];
        if (k < 0 || k >= d.nk) return fail(FOCK_ERR_ARG, "cell %d: source index %d out of range", ci, k);
        if (used[k]) return fail(FOCK_ERR_ARG, "cell %d: source index %d repeated", ci, k);
        used[k] = 1;
      }
    }
  }
  Plan* p = new Plan();
  p->prec = prec;
  if (hipGetDevice(&p->device) != hipSuccess) {
    delete p;
    return fail(FOCK_ERR_HIP, "hipGetDevice failed");
  }
  if (noalloc_setup(p->device) != FOCK_OK) {
    std::string msg = g_last_error;
    delete p;
    g_last_error = msg;
    return FOCK_ERR_HIP;
  }
  if (tune_cache_json) {
    p->tune_path = tune_cache_json;
    p->tuning = true;
    (void)p->tune.load(p->tune_path);
  }
  if (const char* g = std::getenv("FOCKMI_GRAPH")) p->use_graph = std::atoi(g) != 0;
  if (const char* g = std::getenv("FOCKMI_SPLIT_WAIT_TICKS")) {
    p->split_wait_ticks = std::atol(g);
    p->split_form = 1;  // a plan that sets the split form's wait limit runs the split form
  }
  if (const char* g = std::getenv("FOCKMI_SPLIT_SYM")) p->split_sym = std::atoi(g);
  if (const char* g = std::getenv("FOCKMI_SPLIT_STAGGER_SHIFT")) p->split_stagger_shift = std::min(std::max(std::atoi(g), 0), 30);
  {
    hipDeviceProp_t prop;
    p->num_cus = hipGetDeviceProperties(&prop, p->device) == hipSuccess ? prop.multiProcessorCount : 256;
  }
  fock_status s = FOCK_OK;
  if (hipError_t e = hipEventCreateWithFlags(&p->done, hipEventDisableTiming); e != hipSuccess) {
    p->done = nullptr;
    s = hip_fail(e, "plan event");
  }
  for (int ci = 0; ci < ncells && s == FOCK_OK; ++ci) {
    p->cells.emplace_back();
    s = p->init_cell(p->cells.back(), cells[ci], ci);
  }
  if (s != FOCK_OK) {
    std::string msg = g_last_error;
    p->destroy();
    delete p;
    g_last_error = msg;
    return s;
  }
  *out = reinterpret_cast<fockmi_plan>(p);
  return FOCK_OK;
}

fock_status fock_plan_destroy(fockmi_plan plan) {
  if (!plan) return FOCK_OK;
  Plan* p = reinterpret_cast<Plan*>(plan);
  if (p->magic != Plan::kMagic) return fail(FOCK_ERR_STATE, "plan is not valid (destroyed or corrupt)");
  p->destroy();
  delete p;
  return FOCK_OK;
}

fock_status fock_apply(fockmi_plan plan, int cell, const void* u_occ, const void* phi, int nphi, void* vphi,
                       void* stream) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  fock_status s = p->check_ready(cell);
  if (s != FOCK_OK) return s;
  Cell& c = p->cells[cell];
  if (!u_occ || !phi || !vphi) return fail(FOCK_ERR_ARG, "NULL device pointer");
  if (!aligned16(u_occ) || !aligned16(phi) || !aligned16(vphi))
    return fail(FOCK_ERR_ARG, "device pointers must be 16-byte aligned");
  if (nphi < 1) return fail(FOCK_ERR_ARG, "nphi must be >= 1");
  const size_t bu = (size_t)c.nk * c.nb * c.nr * sizeof(c128);
  const size_t bp = (size_t)c.nk * nphi * c.nr * sizeof(c128);
  if (overlap(vphi, bp, u_occ, bu) || overlap(vphi, bp, phi, bp))
    return fail(FOCK_ERR_ARG, "vphi overlaps an input array");
  PlanCall use(p, (hipStream_t)stream);
  return p->apply_op(c, (const c128*)u_occ, (const c128*)phi, nphi, (c128*)vphi, (hipStream_t)stream);
}

fock_status fock_apply_krange(fockmi_plan plan, int cell, const void* u_occ, int k0, int nk_out, const void* phi,
                              int nphi, void* vphi, void* stream) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  fock_status s = p->check_ready(cell);
  if (s != FOCK_OK) return s;
  Cell& c = p->cells[cell];
  if (!u_occ || !phi || !vphi) return fail(FOCK_ERR_ARG, "NULL device pointer");
  if (!aligned16(u_occ) || !aligned16(phi) || !aligned16(vphi))
    return fail(FOCK_ERR_ARG, "device pointers must be 16-byte aligned");
  if (nphi < 1) return fail(FOCK_ERR_ARG, "nphi must be >= 1");
  if (k0 < 0 || nk_out < 1 || k0 + nk_out > c.nk)
    return fail(FOCK_ERR_ARG, "k-range [%d, %d) outside the cell's %d k-points", k0, k0 + nk_out, c.nk);
  const size_t bu = (size_t)c.nk * c.nb * c.nr * sizeof(c128);
  const size_t bp = (size_t)nk_out * nphi * c.nr * sizeof(c128);
  if (overlap(vphi, bp, u_occ, bu) || overlap(vphi, bp, phi, bp))
    return fail(FOCK_ERR_ARG, "vphi overlaps an input array");
  PlanCall use(p, (hipStream_t)stream);
  return p->apply_krange(c, (const c128*)u_occ, k0, nk_out, (const c128*)phi, nphi, (c128*)vphi,
                         (hipStream_t)stream);
}

fock_status fock_energy(fockmi_plan plan, int cell, const void* u_occ, double* ex_re, double* ex_im, void* stream) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  fock_status s = p->check_ready(cell);
  if (s != FOCK_OK) return s;
  Cell& c = p->cells[cell];
  if (!u_occ) return fail(FOCK_ERR_ARG, "NULL device pointer");
  if (!aligned16(u_occ)) return fail(FOCK_ERR_ARG, "device pointers must be 16-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  PlanCall use(p, st);
  const size_t count = (size_t)c.nk * c.nb * c.nr;
  if ((s = p->vu.ensure(count * sizeof(c128), p->workspace_cap, "energy work array")) != FOCK_OK) return s;
  if ((s = p->apply_op(c, (const c128*)u_occ, (const c128*)u_occ, c.nb, (c128*)p->vu.ptr, st)) != FOCK_OK) return s;
  double re = 0, im = 0;
  if ((s = p->dot((const c128*)u_occ, (const c128*)p->vu.ptr, count, st, &re, &im)) != FOCK_OK) return s;
  const double w = (c.gs / 2.0) / c.nk * c.vol / c.nr;
  if (ex_re) *ex_re = w * re;
  if (ex_im) *ex_im = w * im;
  return FOCK_OK;
}

fock_status fock_energy_vjp(fockmi_plan plan, int cell, const void* u_occ, double g_e, void* g_u_occ, void* stream) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  fock_status s = p->check_ready(cell);
  if (s != FOCK_OK) return s;
  Cell& c = p->cells[cell];
  if (!u_occ || !g_u_occ) return fail(FOCK_ERR_ARG, "NULL device pointer");
  if (!aligned16(u_occ) || !aligned16(g_u_occ)) return fail(FOCK_ERR_ARG, "device pointers must be 16-byte aligned");
  if (!std::isfinite(g_e)) return fail(FOCK_ERR_ARG, "g_e is not finite");
  const size_t bu = (size_t)c.nk * c.nb * c.nr * sizeof(c128);
  if (overlap(g_u_occ, bu, u_occ, bu)) return fail(FOCK_ERR_ARG, "g_u_occ overlaps u_occ");
  hipStream_t st = (hipStream_t)stream;
  PlanCall use(p, st);
  const c128* U = (const c128*)u_occ;
  c128* GU = (c128*)g_u_occ;
  // E_x = w sum conj(u) V_x[u] u, w = (g_s/2)(1/N_k)(Omega/N_r). u enters as the
  // target (conj(u) and u outside the pair sum) and as the source orbitals; the
  // target occurrences give 2 w V_x u, the source occurrences the source-side
  // adjoint with cotangent w u, which equals 2 w V_x u when every k-point is a source.
  const double cw = g_e * (c.gs / 2.0) / c.nk * c.vol / c.nr;
  const c128* Us = nullptr;
  if ((s = p->sources(c, U, c.nb, p->srcbuf, st, &Us)) != FOCK_OK) return s;
  if (!c.ds) return p->general(c, c.fwd(), U, c.nb, Us, Us, c.nb, GU, -4.0 * cw / c.nsrc, false, st);
  if ((s = p->general(c, c.fwd(), U, c.nb, Us, Us, c.nb, GU, -2.0 * cw / c.nsrc, false, st)) != FOCK_OK) return s;
  // source side: -(1/|S|) sum_{k,i} 2 (w u_ik) W_{k'-k}(conj(u_ik) u_jk') for k' in S
  const size_t block = (size_t)c.nb * c.nr;
  if ((s = p->srcout.ensure((size_t)c.nsrc * block * sizeof(c128), p->workspace_cap, "source gradient")) != FOCK_OK)
    return s;
  c128* gs = (c128*)p->srcout.ptr;
  if ((s = p->general(c, c.rev(), Us, c.nb, U, U, c.nb, gs, -2.0 * cw / c.nsrc, false, st)) != FOCK_OK) return s;
  for (int i = 0; i < c.nsrc; ++i) {
    hipError_t e = launch_scale_add(GU + (size_t)c.src[i] * block, gs + (size_t)i * block, 1.0, 0.0, (long)block, st);
    if (e != hipSuccess) return hip_fail(e, "add source gradient");
  }
  return FOCK_OK;
}

fock_status fock_vjp(fockmi_plan plan, int cell, const void* u_occ, const void* phi, int nphi, const void* g_vphi,
                     void* g_u_occ, void* g_phi, void* stream) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  fock_status s = p->check_ready(cell);
  if (s != FOCK_OK) return s;
  Cell& c = p->cells[cell];
  if (!u_occ || !phi || !g_vphi) return fail(FOCK_ERR_ARG, "NULL device pointer");
  if (!aligned16(u_occ) || !aligned16(phi) || !aligned16(g_vphi) || (g_u_occ && !aligned16(g_u_occ)) ||
      (g_phi && !aligned16(g_phi)))
    return fail(FOCK_ERR_ARG, "device pointers must be 16-byte aligned");
  if (nphi < 1) return fail(FOCK_ERR_ARG, "nphi must be >= 1");
  const size_t bu = (size_t)c.nk * c.nb * c.nr * sizeof(c128);
  const size_t bp = (size_t)c.nk * nphi * c.nr * sizeof(c128);
  if (g_u_occ && (overlap(g_u_occ, bu, u_occ, bu) || overlap(g_u_occ, bu, phi, bp) || overlap(g_u_occ, bu, g_vphi, bp)))
    return fail(FOCK_ERR_ARG, "g_u_occ overlaps an input array");
  if (g_phi && (overlap(g_phi, bp, u_occ, bu) || overlap(g_phi, bp, phi, bp) || overlap(g_phi, bp, g_vphi, bp) ||
                (g_u_occ && overlap(g_phi, bp, g_u_occ, bu))))
    return fail(FOCK_ERR_ARG, "g_phi overlaps another array");
  hipStream_t st = (hipStream_t)stream;
  PlanCall use(p, st);
  const double scale = -1.0 / c.nsrc;
  const c128* U = (const c128*)u_occ;
  const c128* F = (const c128*)phi;
  const c128* G = (const c128*)g_vphi;
  const c128* Us = nullptr;
  if ((s = p->sources(c, U, c.nb, p->srcbuf, st, &Us)) != FOCK_OK) return s;
  c128* gu = (c128*)g_u_occ;
  if (g_u_occ && c.ds) {
    const size_t block = (size_t)c.nb * c.nr;
    if ((s = p->srcout.ensure((size_t)c.nsrc * block * sizeof(c128), p->workspace_cap, "source gradient")) != FOCK_OK)
      return s;
    gu = (c128*)p->srcout.ptr;
  }
  // the pairs of g_phi = V_x[u] g give the third family below as well: W of (g_ik, u_jk')
  // in that order is the conjugate of W of (u_jk', g_ik)
  bool shared = false;
  if (g_phi && g_u_occ &&
      (s = p->two_sided(c, G, nphi, Us, scale, (c128*)g_phi, F, scale, 0.0, false, gu, st, &shared)) != FOCK_OK)
    return s;
  if (g_phi && !shared) {
    if ((s = p->general(c, c.fwd(), G, nphi, Us, Us, c.nb, (c128*)g_phi, scale, false, st)) != FOCK_OK) return s;
  }
  if (g_u_occ) {
    // targets u at the source k-points k', sources (phi or g) at every k, kernel K_{k'-k}
    hipError_t e;
    if ((s = p->general(c, c.rev(), Us, c.nb, F, G, nphi, gu, scale, shared, st)) != FOCK_OK) return s;
    if (!shared && (s = p->general(c, c.rev(), Us, c.nb, G, F, nphi, gu, scale, true, st)) != FOCK_OK) return s;
    if (c.ds) {
      // orbitals off the sub-mesh carry no gradient; scatter the sub-mesh rows
      const size_t block = (size_t)c.nb * c.nr;
      if ((e = launch_zero((c128*)g_u_occ, (long)c.nk * block, st)) != hipSuccess) return hip_fail(e, "clear gradient");
      for (int i = 0; i < c.nsrc; ++i) {
        if ((e = hipMemcpyAsync((c128*)g_u_occ + (size_t)c.src[i] * block, gu + (size_t)i * block,
                                block * sizeof(c128), hipMemcpyDeviceToDevice, st)) != hipSuccess)
          return hip_fail(e, "scatter gradient");
      }
    }
  }
  return FOCK_OK;
}

fock_status fock_profile_enable(fockmi_plan plan, int enable) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  if (p->magic != Plan::kMagic) return fail(FOCK_ERR_STATE, "plan is not valid (destroyed or corrupt)");
  std::lock_guard<std::mutex> lock(p->calls);
  p->profiling = enable != 0;
  return FOCK_OK;
}

fock_status fock_profile_fallbacks(fockmi_plan plan, long long* count, int reset) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  if (p->magic != Plan::kMagic) return fail(FOCK_ERR_STATE, "plan is not valid (destroyed or corrupt)");
  std::lock_guard<std::mutex> lock(p->calls);
  long long n = 0;
  hipError_t e;
  if (p->fallbacks.ptr) {
    if ((e = hipDeviceSynchronize()) != hipSuccess) return hip_fail(e, "sync");
    if ((e = hipMemcpy(&n, p->fallbacks.ptr, sizeof(n), hipMemcpyDeviceToHost)) != hipSuccess)
      return hip_fail(e, "read fallback count");
    if (reset) {
      if ((e = launch_zero_ll((long long*)p->fallbacks.ptr, nullptr)) != hipSuccess) return hip_fail(e, "reset");
      if ((e = hipDeviceSynchronize()) != hipSuccess) return hip_fail(e, "sync");
    }
  }
  if (count) *count = n;
  return FOCK_OK;
}

fock_status fock_profile_read(fockmi_plan plan, double* kernel_ms, long long* launches, int reset) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  if (p->magic != Plan::kMagic) return fail(FOCK_ERR_STATE, "plan is not valid (destroyed or corrupt)");
  std::lock_guard<std::mutex> lock(p->calls);
  fock_status s = p->prof_collect();
  if (s != FOCK_OK) return s;
  if (kernel_ms) *kernel_ms = p->prof_ms;
  if (launches) *launches = p->prof_launches;
  if (reset) {
    p->prof_ms = 0.0;
    p->prof_launches = 0;
  }
  return FOCK_OK;
}

}  // extern "C"

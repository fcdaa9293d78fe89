// fock_apply_noalloc: the FP32-form application of the exchange operator for
// callers that cannot allocate device memory (code under HIP graph capture,
// tight serving loops, harnesses that forbid allocation).
//
// Every scratch buffer of the call (the complex64 shadows of the orbitals and
// targets, the Neumaier compensation field and, for 32^3 cells, the FP32 band
// sums) is carved out of one file-scope device array, `scratch`, of
// kNoAllocBytes. Each GPU holds its own copy of the array until the process
// ends; its device address is looked up once per device at plan creation
// (noalloc_setup) and kept per device. Host code never passes the array's name
// to a kernel: in host code that name is only a stand-in for the symbol.
//
// For grid lengths up to 24 the call runs what fock_apply runs (the grid form of the
// fused kernel, one workgroup per target, or for small sums the two-stage pair form,
// by the same rule), so that for those cells the two calls give the same bits; at
// 32^3 it runs the grid form. Every call on a GPU shares that GPU's
// array and leaves its contents behind; calls that overlap on one GPU race.
// The fused kernel writes every compensation and band-sum element before it
// reads it, so nothing needs clearing between calls.
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/fockmi.h"
#include "plan.hpp"

using namespace fockmi;

namespace fockmi {

extern thread_local std::string g_last_error;

constexpr int kNoAllocMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kNoAllocMaxDevices] = {};
}  // namespace

// scratch layout (256-byte aligned pieces): source shadow [nsrc][nb][N_r], target shadow
// [nk][nphi][N_r] unless phi is u_occ, compensation [nk][nphi][N_r], FP32 band sums
// [nk * nphi][N_r] where the kernel keeps them in global memory
struct NoAllocLayout {
  size_t x, c, a, end;
};
static NoAllocLayout noalloc_layout(const Cell& c, const PairSet& ps, int nx, int ns, bool x_is_u) {
  auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t nitems = (size_t)(ps.ntk_all ? ps.ntk_all : ps.ntk) * nx;
  NoAllocLayout l;
  l.x = up((size_t)ps.nsk * ns * c.nr * sizeof(c64));
  l.c = l.x + (x_is_u ? 0 : up(nitems * c.nr * sizeof(c64)));
  l.a = l.c + up(nitems * c.nr * sizeof(c64));
  l.end = l.a + up(fused_acc_scratch_elems(c.geom.n1, (int)nitems) * sizeof(c64));
  return l;
}

size_t noalloc_bytes(const Cell& c, const PairSet& ps, int nx, int ns, bool x_is_u) {
  return noalloc_layout(c, ps, nx, ns, x_is_u).end;
}

// Looks up this device's copy of `scratch` (the device must be current). Called
// by fock_plan_create; idempotent per device.
fock_status noalloc_setup(int device) {
  if (device < 0 || device >= kNoAllocMaxDevices) return FOCK_OK;  // the allocation-free call reports it
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (g_noalloc_ptr[device]) return FOCK_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    (void)hipGetLastError();
    return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "scratch array address");
  }
  g_noalloc_ptr[device] = ptr;
  return FOCK_OK;
}

}  // namespace fockmi

extern "C" fock_status fock_apply_noalloc(fockmi_plan plan, int cell, const void* u_occ, const void* phi, int nphi,
                                          void* vphi, void* stream) {
  g_last_error.clear();
  if (!plan) return fail(FOCK_ERR_ARG, "plan is NULL");
  Plan* p = reinterpret_cast<Plan*>(plan);
  fock_status s = p->check_ready(cell);
  if (s != FOCK_OK) return s;
  if (p->prec != FOCK_FP32_COMP) return fail(FOCK_ERR_ARG, "fock_apply_noalloc needs a FOCK_FP32_COMP plan");
  Cell& c = p->cells[cell];
  if (c.f32plain) return fail(FOCK_ERR_SIZE, "fock_apply_noalloc needs a cubic grid");
  if (!u_occ || !phi || !vphi) return fail(FOCK_ERR_ARG, "NULL device pointer");
  if (!aligned16(u_occ) || !aligned16(phi) || !aligned16(vphi))
    return fail(FOCK_ERR_ARG, "device pointers must be 16-byte aligned");
  if (nphi < 1) return fail(FOCK_ERR_ARG, "nphi must be >= 1");
  const size_t bu = (size_t)c.nk * c.nb * c.nr * sizeof(c128);
  const size_t bp = (size_t)c.nk * nphi * c.nr * sizeof(c128);
  if (overlap(vphi, bp, u_occ, bu) || overlap(vphi, bp, phi, bp))
    return fail(FOCK_ERR_ARG, "vphi overlaps an input array");
  void* base = (p->device >= 0 && p->device < kNoAllocMaxDevices) ? g_noalloc_ptr[p->device] : nullptr;
  if (!base) return fail(FOCK_ERR_STATE, "the scratch array of device %d was not set up", p->device);

  const PairSet ps = c.fwd();
  const int nitems = ps.ntk * nphi;
  const bool x_is_u = phi == u_occ && nphi == c.nb && !c.ds;
  const size_t blk = (size_t)c.nb * c.nr;  // elements of one source k-point
  const NoAllocLayout lay = noalloc_layout(c, ps, nphi, c.nb, x_is_u);
  const size_t o_u = 0, o_x = lay.x, o_c = lay.c, o_a = lay.a, need = lay.end;
  if (need > kNoAllocBytes)
    return fail(FOCK_ERR_SIZE, "fock_apply_noalloc: this cell needs %zu bytes of scratch, above the fixed %zu bytes",
                need, kNoAllocBytes);
  char* sp = (char*)base;
  c64* su = (c64*)(sp + o_u);
  c64* sx = x_is_u ? su : (c64*)(sp + o_x);
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  const bool pairs = c.geom.n1 <= 24 && p->pair_rule(c, ps, nphi, c.nb, x_is_u, true).pairs;
  const int np = c.geom.n2 * c.geom.n3;
  auto convert = [&](c64* dst, const c128* src, long count) {
    return pairs ? launch_to_c64_paired(dst, src, count, np, st) : launch_to_c64(dst, src, count, st);
  };
  // shadows: the source k-points' orbitals (gathered from S when down-sampled), then the targets
  const c128* U = (const c128*)u_occ;
  if (!c.ds) {
    if ((e = convert(su, U, (long)ps.nsk * (long)blk)) != hipSuccess) return hip_fail(e, "complex64 shadow (u)");
  } else {
    for (int i = 0; i < ps.nsk; ++i)
      if ((e = convert(su + (size_t)i * blk, U + (size_t)c.src[i] * blk, (long)blk)) != hipSuccess)
        return hip_fail(e, "complex64 shadow (u)");
  }
  if (!x_is_u && (e = convert(sx, (const c128*)phi, (long)nitems * c.nr)) != hipSuccess)
    return hip_fail(e, "complex64 shadow (phi)");
  if (pairs) {
    // the sums kept between blocks take the compensation's place, the batch what is left
    const size_t fb = (size_t)c.nr * sizeof(c64);
    int rows = 0;
    long njmax = 0;
    pairs_block_shape(nitems, ps.nsk * c.nb, c.nb, c.nr, fb, kNoAllocBytes - o_a, true, false, &rows, &njmax);
    return pairs_blocks<float, float>(
        c.nr, np, nitems, ps.nsk * c.nb, c.nb,
        cube_stage<float>(c.geom.n1, p->num_cus, ps, sx, nphi, su, c.nb, (const float*)c.Kp.ptr, st), su,
        Mirror<float>{}, (c128*)vphi, -1.0 / c.nsrc, false, rows, njmax, (c64*)(sp + o_a), sp + o_c, nullptr, nullptr,
        st);
  }
  FusedArgs a{};
  a.X = sx;
  a.P = su;
  a.M = su;
  a.Kt = (const float*)c.Kt.ptr;
  a.qidx = ps.qidx;
  a.out = (c128*)vphi;
  a.comp = (c64*)(sp + o_c);
  a.accs = (c64*)(sp + o_a);
  a.nk = ps.nsk;
  a.nx = nphi;
  a.nb = c.nb;
  a.item0 = 0;
  a.nitems = nitems;
  a.scale = -1.0 / c.nsrc;
  a.accumulate = 0;
  a.xcd_map = 1;
  a.n = c.geom.n1;
  a.ksplit = 1;
  a.part_out = nullptr;
  if ((e = launch_fused_apply(c.geom.n1, a, st, 0, nullptr)) != hipSuccess) return hip_fail(e, "fused pair kernel");
  return FOCK_OK;
}

// Fused FP64 pair kernel: every step of Eq. (15) for one pair in complex128,
// without leaving the CU, for cubic grids of length 16, 20 and 24.
//
// The structure is the FP32 form's: one workgroup of N*N threads owns one
// target field X[kt][s] and runs over all sources (k', j); each thread holds
// one line of the field in registers (x phase: along n1 at fixed (m2, m3);
// y phase: along n2 at fixed (l1, m3); z phase: along n3 at fixed (l1, l2),
// where the kernel multiplies), and LDS carries only the transposes. What
// differs is the arithmetic and where the sum lives:
//   * every product, transform and sum is FP64;
//   * the sum over all (k', j) is one FP64 accumulator per element, in
//     registers for N = 16 and 20, and for N = 24 (a line of 24 complex128
//     values already takes 96 of the 168 VGPRs a 9-wave workgroup may use) in
//     registers, LDS and a per-workgroup global buffer;
//   * out = scale * sum (+ out) is written once, at the end.
// A complex128 field of 24^3 does not fit in LDS, so at N = 24 each transpose
// runs in three rounds over a third of the field: rounds of whole waves (of two,
// 288 threads each, one wave took both branches) that leave half of the LDS to
// the sum. Bound by latency: one workgroup per CU, whose waves wait for each
// other at 28 barriers per pair. 64 k-points of 16 bands, phi apart from u:
// 156 ms in two rounds with 4 elements of the sum in LDS and loads in fours,
// 131 ms in three rounds with 9 (146 with 4).
#include "pairs_dev.hpp"

namespace fockmi {

template <int N>
constexpr bool f64_acc_in_regs() {
  return N <= 20;
}

// Where the FP64 accumulator is a global buffer (24^3), its first elements of
// each thread's line live in registers and the next ones in LDS (thread-private
// slots beside the transpose array), which takes their read-modify-write off
// device memory (64 k-points of 16 bands: 146 ms with 4 in LDS, 131 with the 9
// that fit; 6 or 8 in registers spill, 134 and 142 ms).
template <int N>
constexpr int f64_acc_regs() {
  return f64_acc_in_regs<N>() ? 0 : 4;
}
template <int N>
constexpr int f64_acc_lds() {
  return f64_acc_in_regs<N>() ? 0 : 9;
}

// the target held in registers for the whole work item (see the FP32 kernel):
// at 16^3 two 256-thread workgroups per CU leave room for it
template <int N>
constexpr bool f64_x_in_regs() {
  return N == 16;
}

bool fused64_supported(int n) { return n == 16 || n == 20 || n == 24; }

size_t fused64_acc_scratch_elems(int n, int nslots) {
  return (fused64_supported(n) && n > 20) ? (size_t)nslots * n * n * n : 0;
}

namespace {

template <int N>
__device__ __forceinline__ void f64_item(const Fused64Args& a, int item, int acc_slot, c128* __restrict__ lds,
                                         c128* __restrict__ lds_acc) {
  constexpr int NTI = N * N;
  constexpr int NR = N * N * N;
  constexpr bool ACCREG = f64_acc_in_regs<N>();
  constexpr bool XREG = f64_x_in_regs<N>();
  constexpr int AR = f64_acc_regs<N>(), AL = f64_acc_lds<N>();  // accumulator elements in registers, in LDS
  // loads issued together and consumed after the last of them is in flight: pair-product operands,
  // table values, multipliers (and the sum). From 4 of each: 45.1 -> 43.8 ms at 20^3
  // and 14.2 -> 13.8 ms at 16^3 (64 k-points of 16 bands); 138.7 -> 130.9 ms at 24^3, where 12 + 24
  // beats 8 + 12 and 24 + 24 spills (191 ms).
  constexpr int GP = N / 2, G = N == 24 ? 6 : 4;
  static_assert(N % 2 == 0 && N % G == 0, "load groups must tile the line");

  const int t = threadIdx.x;
  const CubeTransform<N, double, false> cube(t);
  const int kt = item / a.nx;
  const int s = item % a.nx;
  // global byte offsets: x-phase element (m1, m2 = chi, m3 = clo) at voff + m1 * N*N*16;
  // table and accumulator buffer are value-major: (v, t) at (v * NTI + t) * size
  const unsigned voff = (unsigned)((cube.chi * N + cube.clo) * 16);
  const unsigned voff_t16 = (unsigned)(t * 16);
  constexpr unsigned FB = NR * 16u;

  const rsrc_t rX = make_rsrc(a.X + ((long)kt * a.nx + s) * NR, FB);
  const rsrc_t rOut = make_rsrc(a.out + ((long)kt * a.nx + s) * NR, FB);
  const rsrc_t rAcc = make_rsrc(ACCREG ? a.out : a.accs + (long)acc_slot * NR, ACCREG ? 0u : FB);

  c128 acc[ACCREG ? N : 1];
  c128 accr[AR > 0 ? AR : 1];
  c128 xr[XREG ? N : 1];
  if constexpr (XREG) static_for<N>([&](auto m1) { xr[m1] = ld_c128(rX, voff, (unsigned)(decltype(m1)::value * NTI * 16)); });
  if constexpr (ACCREG) {
#pragma unroll
    for (int m1 = 0; m1 < N; ++m1) acc[m1] = c128{0.0, 0.0};
  }

  for (int ks = 0; ks < a.nk; ++ks) {
    const int qi = __builtin_amdgcn_readfirstlane(a.qidx[kt * a.nk + ks]);
    const rsrc_t rK = make_rsrc(a.Kt + (long)qi * NR, NR * 8u);
    for (int j = 0; j < a.nb; ++j) {
      const rsrc_t rP = make_rsrc(a.P + ((long)ks * a.nb + j) * NR, FB);
      const rsrc_t rM = make_rsrc(a.M + ((long)ks * a.nb + j) * NR, FB);
      c128 v[N];
      static_for<N / GP>([&](auto cc) {
        constexpr int C0 = decltype(cc)::value * GP;
        c128 p[GP], x[GP];
        static_for<GP>([&](auto q) {
          const unsigned so = (unsigned)((C0 + decltype(q)::value) * NTI * 16);
          p[q] = ld_c128(rP, voff, so);
          if constexpr (XREG) x[q] = xr[C0 + decltype(q)::value];
          else x[q] = ld_c128(rX, voff, so);
        });
        __builtin_amdgcn_sched_barrier(0);
        static_for<GP>([&](auto q) { v[C0 + decltype(q)::value] = cmulc(p[q], x[q]); });
      });
      cube.forward(v, lds);
      // table values, two to a 16-byte load
      {
        c128 kv[N / 2];
        static_for<N / 2>([&](auto q) { kv[q] = ld_c128(rK, voff_t16, (unsigned)(decltype(q)::value * NTI * 16)); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<N / 2>([&](auto q) {
          constexpr int I = 2 * decltype(q)::value;
          v[I] = cscale(v[I], kv[q].re);
          v[I + 1] = cscale(v[I + 1], kv[q].im);
        });
      }
      cube.inverse(v, lds);

      // multiply-accumulate into the FP64 sum over all (k', j)
      if constexpr (ACCREG) {
        static_for<N / G>([&](auto cc) {
          constexpr int C0 = decltype(cc)::value * G;
          c128 mv[G];
          static_for<G>([&](auto q) { mv[q] = ld_c128(rM, voff, (unsigned)((C0 + decltype(q)::value) * NTI * 16)); });
          __builtin_amdgcn_sched_barrier(0);
          static_for<G>([&](auto q) {
            constexpr int m1 = C0 + decltype(q)::value;
            acc[m1] = cmac(acc[m1], mv[q], v[m1]);
          });
        });
      } else {
        // the position of the pair in the (k', j) loop is uniform: one branch per pair
        const bool first = ks == 0 && j == 0;
        // in groups of GA elements, every load of a group issued before any of its stores: the
        // compiler cannot tell the accumulator's stores from the multiplier's loads, so one
        // element at a time would cost two memory round trips each
        auto mac = [&](auto load_acc) {
          constexpr bool LOAD = decltype(load_acc)::value;
          constexpr int GA = G;
          static_for<N / GA>([&](auto gg) {
            constexpr int C0 = decltype(gg)::value * GA;
            c128 mv[GA], av[GA];
            static_for<GA>([&](auto q) {
              constexpr int m1 = C0 + decltype(q)::value;
              mv[decltype(q)::value] = ld_c128(rM, voff, (unsigned)(m1 * NTI * 16));
              if constexpr (LOAD && m1 >= AR + AL) av[decltype(q)::value] = ld_c128(rAcc, voff_t16, (unsigned)(m1 * NTI * 16));
            });
            __builtin_amdgcn_sched_barrier(0);
            static_for<GA>([&](auto q) {
              constexpr int m1 = C0 + decltype(q)::value;
              const unsigned so = (unsigned)(m1 * NTI * 16);
              c128 tot = cmul(mv[decltype(q)::value], v[m1]);
              if constexpr (m1 < AR) {
                accr[m1] = LOAD ? accr[m1] + tot : tot;
              } else if constexpr (m1 < AR + AL) {
                c128& slot = lds_acc[(m1 - AR) * NTI + t];
                slot = LOAD ? slot + tot : tot;
              } else {
                if constexpr (LOAD) tot = av[decltype(q)::value] + tot;
                st_c128(tot, rAcc, voff_t16, so);
              }
            });
          });
        };
        if (first) mac(std::false_type{});
        else mac(std::true_type{});
      }
    }
  }
  // out = scale * sum (+ out)
#pragma unroll
  for (int m1 = 0; m1 < N; ++m1) {
    const unsigned so = (unsigned)(m1 * NTI * 16);
    c128 sum;
    if constexpr (ACCREG) sum = acc[m1];
    else if (m1 < AR) sum = accr[m1 < AR ? m1 : 0];
    else if (m1 < AR + AL) sum = lds_acc[(m1 - AR) * NTI + t];
    else sum = ld_c128(rAcc, voff_t16, so);
    c128 o = cscale(sum, a.scale);
    if (a.accumulate) o = ld_c128(rOut, voff, so) + o;
    st_c128(o, rOut, voff, so);
  }
}

template <int N>
__global__ void __launch_bounds__(N * N) fused64_apply_kernel(Fused64Args a) {
  __shared__ c128 lds[CubeTransform<N, double, false>::kLdsElems];
  __shared__ c128 lds_acc[f64_acc_lds<N>() > 0 ? f64_acc_lds<N>() * N * N : 1];
  static_assert((CubeTransform<N, double, false>::kLdsElems + f64_acc_lds<N>() * N * N) * 16 <= 160 * 1024, "LDS of the fused FP64 kernel");
  int b = blockIdx.x;
  if (a.xcd_map) {
    // workgroups go round-robin over the 8 XCDs; give each XCD a contiguous run of targets
    const int nwg = gridDim.x;
    const int q = nwg / 8, rem = nwg % 8;
    const int x = b % 8, r = b / 8;
    b = x * q + (x < rem ? x : rem) + r;
  }
  f64_item<N>(a, a.item0 + b, blockIdx.x, lds, lds_acc);
}

template <int N>
hipError_t launch64(const Fused64Args& a, hipStream_t st) {
  hipLaunchKernelGGL(fused64_apply_kernel<N>, dim3(a.nitems), dim3(N * N), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fused64_apply(int n, const Fused64Args& a, hipStream_t st) {
  switch (n) {
    case 16: return launch64<16>(a, st);
    case 20: return launch64<20>(a, st);
    case 24: return launch64<24>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fockmi

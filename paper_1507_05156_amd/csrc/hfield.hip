// h x for whole FP64 fields on cubic grids of length 16, 20 and 24 in one kernel:
//   out = (base ? base : 0) + c (T[a] x + v_loc x + alpha V_x x), acc = acc_src + out
// with V_x x given. One workgroup per field, the field's transform on the CU as in the pair
// kernel; T[a] multiplies |k + G + a|^2 / 2 in the z phase.
//
// Bound: by launches where fields are few, by HBM where they are many (x, V_x x and the running
// sums are read once and written once). As a copy, six FFT passes, the multiply, the combination
// and the sum it took 10 launches and 12 passes. Four Taylor steps of 16^3 / 8 k / 4 bands with the
// gradient by the pulse amplitude (64 applications of h): 3.1 ms of kernels before, 0.7 ms here.
#include "pairs_dev.hpp"
#include "prop.hpp"

namespace fockmi {

namespace {

template <int N>
__global__ void __launch_bounds__(N * N) h_cube_kernel(HCubeArgs a) {
  constexpr int NTI = N * N;
  constexpr int NR = N * N * N;
  constexpr int G = N == 24 ? 2 : 4;
  static_assert(N % G == 0, "load groups must tile the line");
  __shared__ c128 lds[CubeTransform<N, double>::kLdsElems];
  const CubeTransform<N, double> cube(threadIdx.x);
  const int f = blockIdx.x, k = f / a.nf;
  const unsigned voff = (unsigned)((cube.chi * N + cube.clo) * 16);
  const rsrc_t rx = make_rsrc(a.x + (long)f * NR, NR * 16u);
  c128 v[N];
  static_for<N>([&](auto m) { v[m] = ld_c128(rx, voff, (unsigned)(decltype(m)::value * NTI * 16)); });
  cube.forward(v, lds);
  auto freq = [](int j) { return (double)(j < (N + 1) / 2 ? j : j - N); };
  const double f1 = freq(cube.chi), f2 = freq(cube.clo);
  double p[3];
  for (int d = 0; d < 3; ++d) p[d] = a.kpts[3 * k + d] + a.a[d] + f1 * a.g.B[0][d] + f2 * a.g.B[1][d];
  static_for<N>([&](auto l) {
    constexpr int L = decltype(l)::value;
    constexpr double f3 = L < (N + 1) / 2 ? L : L - N;
    const double q0 = p[0] + f3 * a.g.B[2][0], q1 = p[1] + f3 * a.g.B[2][1], q2 = p[2] + f3 * a.g.B[2][2];
    v[L] = cscale(v[L], 0.5 / NR * (q0 * q0 + q1 * q1 + q2 * q2));
  });
  cube.inverse(v, lds);
  // an absent operand is an empty buffer, whose loads give zero
  const unsigned voff8 = voff / 2;
  auto field = [&](const c128* p) { return make_rsrc(p ? p + (long)f * NR : nullptr, p ? NR * 16u : 0u); };
  const rsrc_t rw = field(a.vx), rb = field(a.base), rs = field(a.acc_src), ro = field(a.out), ra = field(a.acc);
  const rsrc_t rv = make_rsrc(a.vloc, a.vloc ? NR * 8u : 0u);
  static_for<N / G>([&](auto gg) {
    constexpr int C0 = decltype(gg)::value * G;
    c128 x[G], w[G], b[G], s[G];
    double vl[G];
    static_for<G>([&](auto q) {
      constexpr int I = decltype(q)::value;
      constexpr unsigned so = (unsigned)((C0 + I) * NTI * 16);
      vl[I] = ld_f64(rv, voff8, so / 2);
      x[I] = ld_c128(rx, voff, so);
      w[I] = ld_c128(rw, voff, so);
      b[I] = ld_c128(rb, voff, so);
      s[I] = ld_c128(rs, voff, so);
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<G>([&](auto q) {
      constexpr int I = decltype(q)::value;
      constexpr unsigned so = (unsigned)((C0 + I) * NTI * 16);
      c128 h = v[C0 + I];
      h = c128{h.re + vl[I] * x[I].re, h.im + vl[I] * x[I].im};
      h = c128{h.re + a.alpha * w[I].re, h.im + a.alpha * w[I].im};
      const c128 r{b[I].re + (a.cre * h.re - a.cim * h.im), b[I].im + (a.cre * h.im + a.cim * h.re)};
      st_c128(r, ro, voff, so);
      st_c128(c128{s[I].re + r.re, s[I].im + r.im}, ra, voff, so);
    });
  });
}

}  // namespace

bool h_cube_supported(const Geom& g) {
  return g.n1 == g.n2 && g.n2 == g.n3 && (g.n1 == 16 || g.n1 == 20 || g.n1 == 24);
}

hipError_t launch_h_cube(const HCubeArgs& a, int nk, hipStream_t st) {
  const dim3 grid((unsigned)(nk * a.nf));
  switch (a.g.n1) {
    case 16: hipLaunchKernelGGL(h_cube_kernel<16>, grid, dim3(256), 0, st, a); break;
    case 20: hipLaunchKernelGGL(h_cube_kernel<20>, grid, dim3(400), 0, st, a); break;
    case 24: hipLaunchKernelGGL(h_cube_kernel<24>, grid, dim3(576), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace fockmi

// Stage 1 of the two-stage pair form (pairs.hpp) where a pair's field does not fit on a CU
// (32^3 in FP64) or the grid is not cubic: W of one pair per workgroup in three passes over
// the pair's slot of the batch.
//
//   A  planes m1: rho = conj(P) X along m2, DFT along m2, transpose in LDS, DFT along m3;
//      stored as [m1][l3][l2], so that the lanes' l2 stay contiguous;
//   B  lines along m1 at fixed (l3, l2): DFT, kernel multiply (table in the same order),
//      inverse DFT, in place;
//   C  planes m1: inverse DFT along l3, transpose, inverse DFT along l2, stored as W.
//
// One workgroup runs the three passes of a pair back to back, so the slot is read again while
// it is still near: at 32^3 in FP64 the 256 pairs in flight take 128 MiB, half the Infinity
// Cache, and only the operands' first reads and the last store have to reach HBM.
//
// Bound: the slot's five passes over memory beyond L2 (A writes, B reads and writes, C reads
// and writes: 2.5 MiB per pair of 32^3 in FP64), at 5.3 TB/s over the kernel; without pass A,
// B or C (timing copies) it takes 56%, 67% or 70% of its time. 32^3 / 8 k / 16 bands in FP64:
// 32.1 ms per application with one kernel and one pass over HBM per step (21 passes per pair),
// 5.3 ms in this form (4.45 ms here, half of it the pair symmetry); adjoint of 16 x 20 x 24 /
// 12 k / 6 bands 7.5 -> 2.1 ms. Loading the pair product's operands in groups of 4 instead of
// 8, workgroups of 4 waves, two to a CU, and a plain last store were no faster.
#include "pairs_dev.hpp"
#include "plane_lds.hpp"

namespace fockmi {

namespace {

// u[m3] of lane l2 <- v[l2] of lane m3, within each plane of the wave; the buffer is the
// wave's own, LDS runs a wave's accesses in order, and one component at a time halves it
template <int N2, int N3, typename T, bool FWD, int NA, int NB>
__device__ __forceinline__ void plane_transpose(T* buf, int pl, int idx, cx<T> (&a)[NA], cx<T> (&b)[NB]) {
  using S = PlaneShape<N2, N3>;
  // forward: a = lines along l2 held by lane m3, b = lines along m3 held by lane l2; inverse: the reverse
  T* col = buf + S::col(pl, idx);  // lane m3: element l2 at l2 * ROW
  T* row = buf + S::row(pl, idx);  // lane l2: element m3 at m3
  const bool wr = pl < S::PL && idx < (FWD ? N3 : N2);
  static_for<2>([&](auto comp) {
    constexpr bool RE = decltype(comp)::value == 0;
    if (wr) {
      static_for<NA>([&](auto i) {
        constexpr int I = decltype(i)::value;
        if constexpr (FWD) col[I * S::ROW] = RE ? a[I].re : a[I].im;
        else row[I] = RE ? a[I].re : a[I].im;
      });
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    static_for<NB>([&](auto i) {
      constexpr int I = decltype(i)::value;
      T x;
      if constexpr (FWD) x = row[I];
      else x = col[I * S::ROW];
      if constexpr (RE) b[I].re = x;
      else b[I].im = x;
    });
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  });
}

template <int N1, typename T>
__device__ __forceinline__ void line_pass(cx<T>* w, const double* __restrict__ K, int np) {
  for (int pos = threadIdx.x; pos < np; pos += 64 * kPlaneWaves) {
    cx<T> v[N1];
    static_for<N1>([&](auto i) { v[i] = w[decltype(i)::value * np + pos]; });
    fft<N1, -1>(v);
    static_for<N1>([&](auto i) { v[i] = cscale(v[i], (T)K[decltype(i)::value * np + pos]); });
    fft<N1, +1>(v);
    static_for<N1>([&](auto i) { w[decltype(i)::value * np + pos] = v[i]; });
  }
}

template <int N2, int N3, typename T>
__global__ void __launch_bounds__(64 * kPlaneWaves) __attribute__((amdgpu_waves_per_eu(2)))
pair_planes_kernel(PlaneArgs<T> a) {
  using S = PlaneShape<N2, N3>;
  __shared__ T lds[kPlaneWaves * S::WORDS];
  static_assert(sizeof(lds) <= 160 * 1024, "LDS of the plane passes");
  constexpr int NP = N2 * N3;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pl = lane / S::L, idx = lane % S::L;
  T* buf = lds + wv * S::WORDS;
  const int nr = a.n1 * NP;
  PairWalk walk(a.b);
  if (!walk.start()) return;
  for (;;) {
    const int gt = a.b.t0 + walk.ti, gj = a.b.j0 + walk.j;
    const int qi = ld_uniform(a.qidx + (long)(gt / a.nx) * a.nsk + gj / a.ns);
    const c128* X = a.X + (long)gt * nr;
    const c128* P = a.P + (long)gj * nr;
    cx<T>* w = a.W + ((long)walk.j * a.b.nt + walk.ti) * nr;
    for (int m0 = wv * S::PL; m0 < a.n1; m0 += kPlaneWaves * S::PL) {
      const int m1 = m0 + pl;
      const bool on = pl < S::PL && m1 < a.n1;
      cx<T> v[N2], u[N3];
      static_for<N2>([&](auto i) { v[i] = cx<T>{0, 0}; });
      if (on && idx < N3) {
        const int o = m1 * NP + idx;
        static_for<(N2 + 7) / 8>([&](auto g) {
          constexpr int C0 = decltype(g)::value * 8, CN = N2 - C0 < 8 ? N2 - C0 : 8;
          c128 p[CN], x[CN];
          static_for<CN>([&](auto i) {
            p[i] = P[o + (C0 + decltype(i)::value) * N3];
            x[i] = X[o + (C0 + decltype(i)::value) * N3];
          });
          static_for<CN>([&](auto i) {
            v[C0 + decltype(i)::value] = cmulc(cx<T>{(T)p[i].re, (T)p[i].im}, cx<T>{(T)x[i].re, (T)x[i].im});
          });
        });
      }
      fft<N2, -1>(v);
      plane_transpose<N2, N3, T, true>(buf, pl, idx, v, u);
      fft<N3, -1>(u);
      if (on && idx < N2) static_for<N3>([&](auto i) { w[m1 * NP + decltype(i)::value * N2 + idx] = u[i]; });
    }
    __syncthreads();
    const double* K = a.K + (long)qi * nr;
    switch (a.n1) {
      case 16: line_pass<16>(w, K, NP); break;
      case 20: line_pass<20>(w, K, NP); break;
      case 24: line_pass<24>(w, K, NP); break;
      default: line_pass<32>(w, K, NP); break;
    }
    __syncthreads();
    for (int m0 = wv * S::PL; m0 < a.n1; m0 += kPlaneWaves * S::PL) {
      const int m1 = m0 + pl;
      const bool on = pl < S::PL && m1 < a.n1;
      cx<T> u[N3], v[N2];
      static_for<N3>([&](auto i) { u[i] = cx<T>{0, 0}; });
      if (on && idx < N2) static_for<N3>([&](auto i) { u[i] = w[m1 * NP + decltype(i)::value * N2 + idx]; });
      fft<N3, +1>(u);
      plane_transpose<N2, N3, T, false>(buf, pl, idx, u, v);
      fft<N2, +1>(v);
      // every lane of a plane has read its line (the transpose's reads) before the plane is rewritten
      if (on && idx < N3) static_for<N2>([&](auto i) { st_w(w + m1 * NP + decltype(i)::value * N3 + idx, v[i]); });
    }
    if (!walk.next()) return;
  }
}

template <int N2, int N3, typename T>
hipError_t launch_nn(const PlaneArgs<T>& a, int num_cus, hipStream_t st) {
  // workgroups of a CU: what the LDS holds, at most two (two waves per SIMD each)
  using S = PlaneShape<N2, N3>;
  const long per = (a.b.npairs + 7) / 8;
  const long slots = (long)(num_cus / 8) * (kPlaneWaves * S::WORDS * sizeof(T) * 2 <= 160 * 1024 && sizeof(T) == 4 ? 2 : 1);
  const int g = (int)(per < slots ? per : slots);
  hipLaunchKernelGGL((pair_planes_kernel<N2, N3, T>), dim3(8 * g), dim3(64 * kPlaneWaves), 0, st, a);
  return hipGetLastError();
}

template <int N2, typename T>
hipError_t launch_n2(int n3, const PlaneArgs<T>& a, int num_cus, hipStream_t st) {
  switch (n3) {
    case 16: return launch_nn<N2, 16>(a, num_cus, st);
    case 20: return launch_nn<N2, 20>(a, num_cus, st);
    case 24: return launch_nn<N2, 24>(a, num_cus, st);
    case 32: return launch_nn<N2, 32>(a, num_cus, st);
    default: return hipErrorInvalidValue;
  }
}

// Kp[q][l1][l3][l2] = K[q][l1][l2][l3]
__global__ void __launch_bounds__(256) plane_table_kernel(double* __restrict__ Kp, const double* __restrict__ K,
                                                          long count, int n2, int n3) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long)gridDim.x * 256) {
    const int l2 = (int)(i % n2);
    const long r = i / n2;
    const int l3 = (int)(r % n3);
    Kp[i] = K[(r / n3 * n2 + l2) * n3 + l3];
  }
}

}  // namespace

template <typename T>
hipError_t launch_pair_planes(int n2, int n3, const PlaneArgs<T>& a, int num_cus, hipStream_t st) {
  if (a.n1 != 16 && a.n1 != 20 && a.n1 != 24 && a.n1 != 32) return hipErrorInvalidValue;
  switch (n2) {
    case 16: return launch_n2<16>(n3, a, num_cus, st);
    case 20: return launch_n2<20>(n3, a, num_cus, st);
    case 24: return launch_n2<24>(n3, a, num_cus, st);
    case 32: return launch_n2<32>(n3, a, num_cus, st);
    default: return hipErrorInvalidValue;
  }
}
template hipError_t launch_pair_planes<float>(int, int, const PlaneArgs<float>&, int, hipStream_t);
template hipError_t launch_pair_planes<double>(int, int, const PlaneArgs<double>&, int, hipStream_t);

hipError_t launch_plane_table(double* Kp, const double* K, int nq, const Geom& g, hipStream_t st) {
  const long count = (long)nq * g.n1 * g.n2 * g.n3;
  long b = (count + 255) / 256;
  if (b > 65536) b = 65536;
  hipLaunchKernelGGL(plane_table_kernel, dim3((unsigned)b), dim3(256), 0, st, Kp, K, count, g.n2, g.n3);
  return hipGetLastError();
}

}  // namespace fockmi

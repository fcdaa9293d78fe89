// Two-stage pair form: W of every pair of a block through a batch buffer, then the sums.
//
//   stage 1 (pair_w_kernel)  one pair per workgroup pass: rho = conj(P_j) X_i, forward 3D
//                            FFT, kernel multiply, inverse FFT, W_ji stored to the batch;
//   stage 2 (wsum_kernel)    out_i += sum_j M_j W_ji, and for a two-sided block also
//                            mir_j += sum_i F_i conj(W_ji), both from one read of W.
//
// Stage 2 with both sides is what the two-stage form is for. The pair (j, i) with targets
// and sources exchanged has the density conj(rho) and the table of -q on the reflected
// grid, K_{-q}(-G) = K_q(G) (Nyquist planes are averaged over both signs), so its W is
// conj(W_ji): with u as targets and sources one transform serves two rows of the result,
// and no sum crosses workgroups while a pair is transformed.
//
// Bound: stage 1 at 32^3 by its transforms and their transposes (17 us of the 30 us a CU
// takes per pair; the rest is the operands' loads and the drain of the W stores, which one
// field per CU cannot overlap), stage 2 by the one read of W. 32^3 / 216 k / 16 bands, FP32:
// 1,732 ms per application with every pair of k-points pushed between CU pairs (split32.hip),
// 1,270 ms in this form with plain W accesses, 1,142 ms with non-temporal ones, 1,088 ms with
// the next pair's first operands loaded before the stores, 1,076 ms with every access of stage 1
// 16 bytes wide (stage 1 at 24^3 in FP32: 50.8 -> 45.1 ns per pair). One of eight k-point shards
// of it (one-sided sums): 284.6 -> 235 ms.
#include "pairs_dev.hpp"

namespace fockmi {

namespace {

// Every access moves 16 bytes per lane: 8-byte ones take as many cycles of the L1 for half the
// data, and the kernel's operands, tables and W (900 KiB per pair of 32^3 in FP32) are what the
// transforms do not hide. points 2h and 2h + 1 of a line along n1:
template <int NTI>
__device__ __forceinline__ void ld_two(rsrc_t r, unsigned t, int h, cx<float>* v) {
  typedef float v4 __attribute__((ext_vector_type(4)));
  const v4 q = __builtin_bit_cast(v4, __builtin_amdgcn_raw_buffer_load_b128(r, t * 16u, (unsigned)(h * NTI * 16), 0));
  v[0] = {q.x, q.y};
  v[1] = {q.z, q.w};
}
template <int NTI>
__device__ __forceinline__ void ld_two(rsrc_t r, unsigned t, int h, cx<double>* v) {
  v[0] = ld_c128(r, t * 16u, (unsigned)(2 * h * NTI * 16));
  v[1] = ld_c128(r, t * 16u, (unsigned)((2 * h + 1) * NTI * 16));
}
template <int NTI>
__device__ __forceinline__ void st_two(cx<float>* w, unsigned t, int h, const cx<float>* v) {
  typedef float v4 __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(v4{v[0].re, v[0].im, v[1].re, v[1].im}, (v4*)((char*)w + h * (NTI * 16) + t * 16u));
}
template <int NTI>
__device__ __forceinline__ void st_two(cx<double>* w, unsigned t, int h, const cx<double>* v) {
  st_w((cx<double>*)((char*)w + 2 * h * (NTI * 16) + t * 16u), v[0]);
  st_w((cx<double>*)((char*)w + (2 * h + 1) * (NTI * 16) + t * 16u), v[1]);
}
// 16 bytes of table values of the thread
template <int NTI>
__device__ __forceinline__ void ld_tab(rsrc_t r, unsigned t, int g, float* k) {
  typedef float v4 __attribute__((ext_vector_type(4)));
  const v4 q = __builtin_bit_cast(v4, __builtin_amdgcn_raw_buffer_load_b128(r, t * 16u, (unsigned)(g * NTI * 16), 0));
  k[0] = q.x, k[1] = q.y, k[2] = q.z, k[3] = q.w;
}
template <int NTI>
__device__ __forceinline__ void ld_tab(rsrc_t r, unsigned t, int g, double* k) {
  const cx<double> q = ld_c128(r, t * 16u, (unsigned)(g * NTI * 16));
  k[0] = q.re, k[1] = q.im;
}

// elements whose loads are in flight together: operands of the pair product, kernel values
// (24^3 FP64, with transposes in two rounds: groups of 4 took 120 ns per pair, of 12 115 ns; 24
// kernel values at once spill)
template <int N, typename T>
constexpr int pw_grp_px() { return 12; }
// elements of the next pair's operands loaded before the current pair's W is stored (at 32^3
// what the registers hold beside the line: 6; 1 ahead 1,114 ms, 6 ahead 1,088 ms)
template <int N, typename T>
constexpr int pw_ahead() { return sizeof(T) == 8 ? (N == 24 ? 2 : 4) : (N == 32 ? 6 : 8); }
template <int N, typename T>
constexpr int pw_grp_k() { return sizeof(T) == 8 ? 12 : (N <= 24 ? N : 8); }

template <int N, typename T, int WPE>
__global__ void __launch_bounds__(N * N) __attribute__((amdgpu_waves_per_eu(WPE))) pair_w_kernel(PairArgs<T> a) {
  constexpr int NTI = N * N;
  constexpr int NR = N * N * N;
  __shared__ cx<T> lds[CubeTransform<N, T>::kLdsElems];
  static_assert(sizeof(lds) <= 160 * 1024, "LDS of the pair kernel");

  const int t = threadIdx.x;
  const CubeTransform<N, T> cube(t);
  const unsigned pos = (unsigned)(cube.chi * N + cube.clo);
  constexpr unsigned FB = (unsigned)(NR * sizeof(cx<T>));

  PairWalk walk(a.b);
  if (!walk.start()) return;
  auto res_x = [&] { return make_rsrc(a.X + (long)(a.b.t0 + walk.ti) * NR, FB); };
  auto res_p = [&] { return make_rsrc(a.P + (long)(a.b.j0 + walk.j) * NR, FB); };
  // The first PF operands of a pair are loaded before the previous pair's W is stored: a
  // wait for a load also waits for every store issued before it.
  constexpr int PF = pw_ahead<N, T>();
  cx<T> fp[PF], fx[PF];
  auto fetch = [&] {
    const rsrc_t rX = res_x(), rP = res_p();
    static_for<PF / 2>([&](auto e) {
      constexpr int H = decltype(e)::value;
      ld_two<NTI>(rP, pos, H, fp + 2 * H);
      ld_two<NTI>(rX, pos, H, fx + 2 * H);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  fetch();
  for (;;) {
    const int gt = a.b.t0 + walk.ti, gj = a.b.j0 + walk.j;
    const int qi = ld_uniform(a.qidx + (long)(gt / a.nx) * a.nsk + gj / a.ns);
    const rsrc_t rX = res_x(), rP = res_p();
    const rsrc_t rK = make_rsrc(a.Kt + (long)qi * NR, NR * (unsigned)sizeof(T));
    cx<T> v[N];
    constexpr int G = pw_grp_px<N, T>(), NG = (N - PF + G - 1) / G;
    if constexpr (NG == 0) static_for<PF>([&](auto e) { v[decltype(e)::value] = cmulc(fp[e], fx[e]); });
    static_for<NG>([&](auto cc) {
      constexpr int C0 = PF + decltype(cc)::value * G, CN = (N - C0 < G) ? N - C0 : G;
      cx<T> p[CN], xx[CN];
      static_assert(PF % 2 == 0 && CN % 2 == 0, "points go in twos");
      static_for<CN / 2>([&](auto e) {
        constexpr int H = decltype(e)::value;
        ld_two<NTI>(rP, pos, C0 / 2 + H, p + 2 * H);
        ld_two<NTI>(rX, pos, C0 / 2 + H, xx + 2 * H);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(cc)::value == 0) static_for<PF>([&](auto e) { v[decltype(e)::value] = cmulc(fp[e], fx[e]); });
      static_for<CN>([&](auto e) { v[C0 + decltype(e)::value] = cmulc(p[e], xx[e]); });
    });
    cube.forward(v, lds);
    static_for<(N + pw_grp_k<N, T>() - 1) / pw_grp_k<N, T>()>([&](auto cc) {
      constexpr int G = pw_grp_k<N, T>(), C0 = decltype(cc)::value * G, CN = (N - C0 < G) ? N - C0 : G;
      T kv[CN];
      constexpr int V = 16 / (int)sizeof(T);
      static_assert(C0 % V == 0 && CN % V == 0, "table values go 16 bytes at a time");
      static_for<CN / V>([&](auto e) { ld_tab<NTI>(rK, (unsigned)t, C0 / V + decltype(e)::value, kv + V * decltype(e)::value); });
      __builtin_amdgcn_sched_barrier(0);
      static_for<CN>([&](auto e) { v[C0 + decltype(e)::value] = cscale(v[C0 + decltype(e)::value], kv[e]); });
    });
    cube.inverse(v, lds);
    cx<T>* w = a.W + ((long)walk.j * a.b.nt + walk.ti) * NR;
    const bool more = walk.next();
    if (more) fetch();
    static_for<N / 2>([&](auto h) { st_two<NTI>(w, pos, decltype(h)::value, v + 2 * decltype(h)::value); });
    if (!more) return;
  }
}

// s + c += x with the rounding error carried in c (no contraction: see fused.hip)
__device__ __forceinline__ void fold(double& s, double& c, double x) {
#pragma clang fp contract(off)
  const double t = s + x;
  if (fabs(s) >= fabs(x)) c += (s - t) + x;
  else c += (x - t) + s;
  s = t;
}

// conj(w) * f added to acc
template <typename T>
__device__ __forceinline__ cx<T> cmac_conj(cx<T> acc, cx<T> w, cx<T> f) {
  return {fmadd(w.im, f.im, fmadd(w.re, f.re, acc.re)), fmadd(-w.im, f.re, fmadd(w.re, f.im, acc.im))};
}

// Stage 2. One wave holds TI targets on 64 grid points and streams the sources; the
// NW waves of a workgroup hold NW such tiles on the same points, so the mirror sums of NW * TI
// targets meet in LDS and go to memory once per source. TI is a whole pair tile where that
// fills the device, and 2 for rows of few targets, whose waves then load a batch of NW sources
// ahead: 32 fields of 16^3 in FP64 33 -> 18 us one-sided, 41 -> 23 us two-sided.
template <typename TW, typename T, int TI, int NW, bool TWO>
__global__ void __launch_bounds__(64 * NW) wsum_kernel(WsumArgs<TW, T> a) {
  static_assert(kPairTile % TI == 0, "a wave's targets lie in one pair tile");
  constexpr bool AHEAD = TI < kPairTile;  // the batch's loads issued together
  constexpr bool F32 = sizeof(T) == 4;
  __shared__ cx<T> part[TWO ? NW * NW * 64 : 1];  // [source of the batch][wave][lane]
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = blockIdx.x * 64 + lane;
  const int tile = blockIdx.y * NW + w;
  const int left = a.nt - tile * TI;
  const int n = left < 0 ? 0 : (left < TI ? left : TI);
  const long nr = a.nr;
  const long tg0 = (long)(a.t0 + tile * TI);  // first target of this wave
  const int rn = natural_index(r, a.np);      // where the outputs hold this point

  cx<T> f[TWO ? TI : 1];
  cx<T> acc[TI];
  c128 s[F32 ? TI : 1];
  cx<float> c[F32 ? TI : 1];
  static_for<TI>([&](auto i) {
    constexpr int I = decltype(i)::value;
    acc[I] = cx<T>{0, 0};
    if constexpr (TWO) f[I] = I < n ? a.F[(tg0 + I) * nr + r] : cx<T>{0, 0};
    if constexpr (F32) {
      s[I] = (I < n && (!a.first || a.accumulate)) ? a.out[(tg0 + I) * nr + rn] : c128{0.0, 0.0};
      c[I] = (I < n && !a.first) ? a.comp[(tg0 + I) * nr + r] : cx<float>{0.0f, 0.0f};
    } else {
      if (I < n && !a.first) acc[I] = a.run[(tg0 + I) * nr + r];
    }
  });
  int jb = a.jb0;  // band of the current source within its k-point
  const cx<TW>* wp = a.W + (long)tile * TI * nr + r;
  const int pt = tile * TI / kPairTile;  // the pair tile
  for (int j0 = 0; j0 < a.nj; j0 += NW) {
    const int j1 = j0 + NW < a.nj ? j0 + NW : a.nj;
    cx<TW> wq[AHEAD ? NW : 1][TI];
    cx<T> mq[AHEAD ? NW : 1];
    if constexpr (AHEAD) {
      if (n > 0) {
        // past the last source the last one again, not used
        static_for<NW>([&](auto q) {
          constexpr int Q = decltype(q)::value;
          const int j = j0 + Q < a.nj ? j0 + Q : a.nj - 1;
          const cx<TW>* wj = wp + (long)j * a.nt * nr;
          mq[Q] = a.M[(long)(a.j0 + j) * nr + r];
          static_for<TI>([&](auto i) { wq[Q][decltype(i)::value] = ld_w(wj + (decltype(i)::value < n ? decltype(i)::value : 0) * nr); });
        });
      }
    }
    auto source = [&](int j, auto qq) {
      constexpr int Q = decltype(qq)::value;
      const int jt = j / kPairTile;
      const bool on = n > 0 && (!a.tri || pt >= jt);
      const bool mir = TWO && on && (!a.tri || pt > jt);
      cx<T> ms{0, 0};
      if (on) {
        const cx<TW>* wj = wp + (long)j * a.nt * nr;
        const cx<T> m = AHEAD ? mq[Q] : a.M[(long)(a.j0 + j) * nr + r];
        cx<T> wv[TI];
        static_for<TI>([&](auto i) {
          constexpr int I = decltype(i)::value;
          if (I < n) {
            const cx<TW> q = AHEAD ? wq[Q][I] : ld_w(wj + I * nr);
            wv[I] = cx<T>{(T)q.re, (T)q.im};
          } else {
            wv[I] = cx<T>{0, 0};
          }
        });
        static_for<TI>([&](auto i) { acc[decltype(i)::value] = cmac(acc[decltype(i)::value], m, wv[decltype(i)::value]); });
        if constexpr (TWO) {
          if (mir) static_for<TI>([&](auto i) { ms = cmac_conj(ms, wv[decltype(i)::value], f[decltype(i)::value]); });
        }
      }
      if constexpr (TWO) part[((j - j0) * NW + w) * 64 + lane] = ms;
      ++jb;
      if constexpr (F32) {
        // the FP32 sum covers at most 16 sources of one k-point, then goes into the
        // compensated FP64 sum
        const bool endk = jb == a.ns;
        if (endk || (jb & 15) == 0 || j == a.nj - 1) {
          static_for<TI>([&](auto i) {
            constexpr int I = decltype(i)::value;
            double cr = c[I].re, ci = c[I].im;
            fold(s[I].re, cr, a.scale * (double)acc[I].re);
            fold(s[I].im, ci, a.scale * (double)acc[I].im);
            c[I] = cx<float>{(float)cr, (float)ci};
            acc[I] = cx<T>{0, 0};
          });
        }
      }
      if (jb == a.ns) jb = 0;
    };
    if constexpr (AHEAD) {
      static_for<NW>([&](auto q) {
        if (j0 + decltype(q)::value < j1) source(j0 + decltype(q)::value, q);
      });
    } else {
      for (int j = j0; j < j1; ++j) source(j, std::integral_constant<int, 0>{});
    }
    if constexpr (TWO) {
      __syncthreads();
      if (j0 + w < j1) {
        // the groups of NW tiles keep mirror sums of their own
        const long o = ((long)blockIdx.y * a.nsrc + a.j0 + j0 + w) * nr + r;
        double re = 0.0, im = 0.0;
        static_for<NW>([&](auto k) {
          const cx<T> v = part[(w * NW + decltype(k)::value) * 64 + lane];
          re += (double)v.re;
          im += (double)v.im;
        });
        c128 ms = a.mfirst ? c128{0.0, 0.0} : a.mir[o];
        if constexpr (F32) {
          const cx<float> mc = a.mfirst ? cx<float>{0.0f, 0.0f} : a.mcomp[o];
          double cr = mc.re, ci = mc.im;
          fold(ms.re, cr, re);
          fold(ms.im, ci, im);
          a.mcomp[o] = cx<float>{(float)cr, (float)ci};
        } else {
          ms.re += re;
          ms.im += im;
        }
        a.mir[o] = ms;
      }
      __syncthreads();
    }
  }
  static_for<TI>([&](auto i) {
    constexpr int I = decltype(i)::value;
    if (I < n) {
      const long o = (tg0 + I) * nr + r, on = (tg0 + I) * nr + rn;
      if constexpr (F32) {
        a.out[on] = a.last ? c128{s[I].re + (double)c[I].re, s[I].im + (double)c[I].im} : s[I];
        if (!a.last) a.comp[o] = c[I];
      } else if (a.last) {
        c128 v = cscale(acc[I], a.scale);
        if (a.accumulate) v = a.out[on] + v;
        a.out[on] = v;
      } else {
        a.run[o] = acc[I];
      }
    }
  });
}

// dst[j] = (accumulate ? dst[j] : 0) + (sre + i sim) * sum over the groups g of mir[g][j] + mcomp[g][j],
// groups in order. Of a symmetric sum in rows of `rows` fields, the fields of the last row
// have the groups of that row only.
template <bool F32>
__global__ void __launch_bounds__(256) mirror_add_kernel(c128* __restrict__ dst, const c128* __restrict__ mir,
                                                         const cx<float>* __restrict__ mcomp, double sre, double sim,
                                                         int accumulate, int nsrc, int nr, int rows, int group,
                                                         int tri, int np) {
  const long count = (long)nsrc * nr;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long)gridDim.x * 256) {
    int in_row = rows;
    if (tri) {
      const int row0 = (int)(i / nr) / rows * rows;
      in_row = nsrc - row0 < rows ? nsrc - row0 : rows;
    }
    const int ng = (in_row + group - 1) / group;
    const long o = np ? i / nr * nr + natural_index((int)(i % nr), np) : i;
    c128 d = accumulate ? dst[o] : c128{0.0, 0.0};
    for (int g = 0; g < ng; ++g) {
      c128 m = mir[g * count + i];
      if constexpr (F32) {
        m.re += (double)mcomp[g * count + i].re;
        m.im += (double)mcomp[g * count + i].im;
      }
      d.re += sre * m.re - sim * m.im;
      d.im += sre * m.im + sim * m.re;
    }
    dst[o] = d;
  }
}

template <int N, typename T, int WPE>
hipError_t launch_pw(const PairArgs<T>& a, int slots, hipStream_t st) {
  const long per = (a.b.npairs + 7) / 8;
  const int g = (int)(per < slots / 8 ? per : slots / 8);
  hipLaunchKernelGGL((pair_w_kernel<N, T, WPE>), dim3(8 * g), dim3(N * N), 0, st, a);
  return hipGetLastError();
}

template <typename T>
int phases(int n) {
  switch (n) {
    case 16: return pw_nph<16, T>();
    case 20: return pw_nph<20, T>();
    case 24: return pw_nph<24, T>();
    default: return pw_nph<32, T>();
  }
}

}  // namespace

int pair_phases(int n, bool f64) { return f64 ? phases<double>(n) : phases<float>(n); }

template <>
int pair_w_slots<float>(int n, int num_cus) {
  const int c = (num_cus / 8) * 8;
  return n == 16 ? 4 * c : (n == 20 ? 2 * c : c);
}
template <>
int pair_w_slots<double>(int n, int num_cus) {
  const int c = (num_cus / 8) * 8;
  return n == 16 ? 2 * c : c;
}

template <>
hipError_t launch_pair_w<float>(int n, const PairArgs<float>& a, int num_cus, hipStream_t st) {
  const int slots = pair_w_slots<float>(n, num_cus);
  switch (n) {
    case 16: return launch_pw<16, float, 4>(a, slots, st);
    case 20: return launch_pw<20, float, 4>(a, slots, st);
    case 24: return launch_pw<24, float, 3>(a, slots, st);
    case 32: return launch_pw<32, float, 4>(a, slots, st);
    default: return hipErrorInvalidValue;
  }
}
template <>
hipError_t launch_pair_w<double>(int n, const PairArgs<double>& a, int num_cus, hipStream_t st) {
  const int slots = pair_w_slots<double>(n, num_cus);
  switch (n) {
    case 16: return launch_pw<16, double, 2>(a, slots, st);
    case 20: return launch_pw<20, double, 2>(a, slots, st);
    case 24: return launch_pw<24, double, 3>(a, slots, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename TW, typename TM, int TI>
static hipError_t wsum_ti(const WsumArgs<TW, TM>& a, hipStream_t st) {
  constexpr int NW = kPairGroup / kPairTile;
  const int tiles = (a.nt + TI - 1) / TI;
  const dim3 grid((unsigned)(a.nr / 64), (unsigned)((tiles + NW - 1) / NW));
  if (a.mir)
    hipLaunchKernelGGL((wsum_kernel<TW, TM, TI, NW, true>), grid, dim3(64 * NW), 0, st, a);
  else
    hipLaunchKernelGGL((wsum_kernel<TW, TM, TI, NW, false>), grid, dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

template <typename TW, typename TM>
hipError_t launch_wsum(const WsumArgs<TW, TM>& a, hipStream_t st) {
  if (a.nr % 64 != 0) return hipErrorInvalidValue;
  return a.group == kPairGroup ? wsum_ti<TW, TM, kPairTile>(a, st) : wsum_ti<TW, TM, kPairFew>(a, st);
}
template hipError_t launch_wsum<float, float>(const WsumArgs<float, float>&, hipStream_t);
template hipError_t launch_wsum<double, double>(const WsumArgs<double, double>&, hipStream_t);
template hipError_t launch_wsum<float, double>(const WsumArgs<float, double>&, hipStream_t);

hipError_t launch_mirror_add(c128* dst, const c128* mir, const c64* mcomp, double sre, double sim, int accumulate, int nsrc,
                             int nr, int rows, int group, int tri, int np, hipStream_t st) {
  long g = ((long)nsrc * nr + 255) / 256;
  if (g > 65536) g = 65536;
  if (mcomp)
    hipLaunchKernelGGL(mirror_add_kernel<true>, dim3((unsigned)g), dim3(256), 0, st, dst, mir, mcomp, sre, sim, accumulate,
                       nsrc, nr, rows, group, tri, np);
  else
    hipLaunchKernelGGL(mirror_add_kernel<false>, dim3((unsigned)g), dim3(256), 0, st, dst, mir, mcomp, sre, sim,
                       accumulate, nsrc, nr, rows, group, tri, np);
  return hipGetLastError();
}

}  // namespace fockmi

// 3D FFTs of whole complex128 fields through HBM, one pass per axis (the kinetic operator,
// the preconditioner and the gradient by the vector potential).
//
// Each pass gives one thread one grid line, transformed in registers.
// Lines along n1 and n2 are strided, so neighbouring lanes take neighbouring
// lines and every load is coalesced; lines along n3 are contiguous and are
// staged through LDS so that the global loads stay coalesced.
#include "kernels.hpp"

namespace fockmi {

namespace {

// one thread per line of length N with element stride `inner`; lines are
// enumerated (outer, inner) with base = outer * N * inner + inner_index
template <int N, int SIGN, typename T>
__global__ void __launch_bounds__(64) fft_strided_kernel(cx<T>* __restrict__ data, long nlines, int inner, long field_lines,
                                   long field_elems) {
  const long L = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (L >= nlines) return;
  const long f = L / field_lines;
  const long li = L % field_lines;
  const long base = f * field_elems + (li / inner) * (long)N * inner + (li % inner);
  cx<T> v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = data[base + (long)i * inner];
  fft<N, SIGN>(v);
#pragma unroll
  for (int i = 0; i < N; ++i) data[base + (long)i * inner] = v[i];
}

constexpr int kContigLines = 64;

template <int N, int SIGN, typename T>
__global__ void __launch_bounds__(kContigLines) fft_contig_kernel(cx<T>* __restrict__ data, long nlines) {
  __shared__ cx<T> tile[kContigLines * (N + 1)];
  const long line0 = (long)blockIdx.x * kContigLines;
  const int tid = threadIdx.x;
  const long avail = nlines - line0;
  const int nl = avail < kContigLines ? (int)avail : kContigLines;
  cx<T>* gbase = data + line0 * N;
  for (int idx = tid; idx < nl * N; idx += kContigLines) {
    const int ln = idx / N, pos = idx % N;
    tile[ln * (N + 1) + pos] = gbase[idx];
  }
  __syncthreads();
  if (tid < nl) {
    cx<T> v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = tile[tid * (N + 1) + i];
    fft<N, SIGN>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) tile[tid * (N + 1) + i] = v[i];
  }
  __syncthreads();
  for (int idx = tid; idx < nl * N; idx += kContigLines) {
    const int ln = idx / N, pos = idx % N;
    gbase[idx] = tile[ln * (N + 1) + pos];
  }
}

template <int N, int SIGN, typename T>
hipError_t strided_pass(cx<T>* data, int nfields, int inner, long field_lines, long field_elems, hipStream_t st) {
  const long nlines = (long)nfields * field_lines;
  const int bs = 64;
  hipLaunchKernelGGL((fft_strided_kernel<N, SIGN, T>), dim3((unsigned)((nlines + bs - 1) / bs)), dim3(bs), 0, st,
                     data, nlines, inner, field_lines, field_elems);
  return hipGetLastError();
}

template <int SIGN, typename T>
hipError_t strided_dispatch(int n, cx<T>* data, int nfields, int inner, long field_lines, long field_elems,
                            hipStream_t st) {
  switch (n) {
    case 16: return strided_pass<16, SIGN, T>(data, nfields, inner, field_lines, field_elems, st);
    case 20: return strided_pass<20, SIGN, T>(data, nfields, inner, field_lines, field_elems, st);
    case 24: return strided_pass<24, SIGN, T>(data, nfields, inner, field_lines, field_elems, st);
    case 32: return strided_pass<32, SIGN, T>(data, nfields, inner, field_lines, field_elems, st);
    default: return hipErrorInvalidValue;
  }
}

template <int N, int SIGN, typename T>
hipError_t contig_pass(cx<T>* data, long nlines, hipStream_t st) {
  hipLaunchKernelGGL((fft_contig_kernel<N, SIGN, T>), dim3((unsigned)((nlines + kContigLines - 1) / kContigLines)),
                     dim3(kContigLines), 0, st, data, nlines);
  return hipGetLastError();
}

template <int SIGN, typename T>
hipError_t contig_dispatch(int n, cx<T>* data, long nlines, hipStream_t st) {
  switch (n) {
    case 16: return contig_pass<16, SIGN, T>(data, nlines, st);
    case 20: return contig_pass<20, SIGN, T>(data, nlines, st);
    case 24: return contig_pass<24, SIGN, T>(data, nlines, st);
    case 32: return contig_pass<32, SIGN, T>(data, nlines, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

template <typename T>
hipError_t launch_fft3_plain(cx<T>* data, int nfields, const Geom& g, int sign, hipStream_t st) {
  const long fe = (long)g.n1 * g.n2 * g.n3;
  hipError_t e = hipSuccess;
  // axis 1 (stride n2*n3): lines (m2, m3); axis 2 (stride n3): lines (m1, m3); axis 3 contiguous
  auto ax1 = [&](int s) {
    return s < 0 ? strided_dispatch<-1, T>(g.n1, data, nfields, g.n2 * g.n3, (long)g.n2 * g.n3, fe, st)
                 : strided_dispatch<+1, T>(g.n1, data, nfields, g.n2 * g.n3, (long)g.n2 * g.n3, fe, st);
  };
  auto ax2 = [&](int s) {
    return s < 0 ? strided_dispatch<-1, T>(g.n2, data, nfields, g.n3, (long)g.n1 * g.n3, fe, st)
                 : strided_dispatch<+1, T>(g.n2, data, nfields, g.n3, (long)g.n1 * g.n3, fe, st);
  };
  auto ax3 = [&](int s) {
    const long nl = (long)nfields * g.n1 * g.n2;
    return s < 0 ? contig_dispatch<-1, T>(g.n3, data, nl, st) : contig_dispatch<+1, T>(g.n3, data, nl, st);
  };
  if (sign < 0) {
    if ((e = ax1(-1)) != hipSuccess) return e;
    if ((e = ax2(-1)) != hipSuccess) return e;
    return ax3(-1);
  }
  if ((e = ax3(+1)) != hipSuccess) return e;
  if ((e = ax2(+1)) != hipSuccess) return e;
  return ax1(+1);
}

template hipError_t launch_fft3_plain<double>(cx<double>*, int, const Geom&, int, hipStream_t);

}  // namespace fockmi

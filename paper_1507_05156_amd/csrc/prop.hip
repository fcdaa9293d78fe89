// Device kernels of the propagator and orthonormalisation (FP64).
//
// Kinetic operator of the velocity-gauge Hamiltonian (Eq. (2)) on the periodic
// parts: T[a] u = IDFT( |k + G_l + a|^2 / 2 * DFT u ) / N_r with G_l in FFT
// order (l = -n/2 on the Nyquist slot) and a = A/c.
#include "kernels.hpp"
#include "prop.hpp"

namespace fockmi {

namespace {

__device__ __forceinline__ void gvec(const Geom& g, long l, double kx, double ky, double kz, double a0, double a1,
                                     double a2, double p[3]) {
  const int j3 = (int)(l % g.n3);
  const int j2 = (int)((l / g.n3) % g.n2);
  const int j1 = (int)(l / ((long)g.n2 * g.n3));
  const double l1 = j1 < (g.n1 + 1) / 2 ? j1 : j1 - g.n1;
  const double l2 = j2 < (g.n2 + 1) / 2 ? j2 : j2 - g.n2;
  const double l3 = j3 < (g.n3 + 1) / 2 ? j3 : j3 - g.n3;
  p[0] = kx + a0 + l1 * g.B[0][0] + l2 * g.B[1][0] + l3 * g.B[2][0];
  p[1] = ky + a1 + l1 * g.B[0][1] + l2 * g.B[1][1] + l3 * g.B[2][1];
  p[2] = kz + a2 + l1 * g.B[0][2] + l2 * g.B[1][2] + l3 * g.B[2][2];
}

// F[k][f][l] *= scale * |k + G_l + a|^2 / 2
__global__ void kinetic_mul_kernel(c128* __restrict__ F, const double* __restrict__ kpts, int nf, Geom g,
                                   double a0, double a1, double a2, double scale) {
  const long nr = (long)g.n1 * g.n2 * g.n3;
  const long l = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int field = blockIdx.y;  // k * nf + f
  if (l >= nr) return;
  const int k = field / nf;
  double p[3];
  gvec(g, l, kpts[3 * k], kpts[3 * k + 1], kpts[3 * k + 2], a0, a1, a2, p);
  const double e = scale * 0.5 * (p[0] * p[0] + p[1] * p[1] + p[2] * p[2]);
  c128 v = F[(long)field * nr + l];
  v.re *= e;
  v.im *= e;
  F[(long)field * nr + l] = v;
}

// F[k][f][l] *= scale / (1 + |k + G_l + a|^2 / (2 e0)): the kinetic preconditioner
// of the block eigensolver, damping the plane waves far above the energy e0
__global__ void precond_mul_kernel(c128* __restrict__ F, const double* __restrict__ kpts, int nf, Geom g, double a0,
                                   double a1, double a2, double e0, double scale) {
  const long nr = (long)g.n1 * g.n2 * g.n3;
  const long l = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int field = blockIdx.y;
  if (l >= nr) return;
  const int k = field / nf;
  double p[3];
  gvec(g, l, kpts[3 * k], kpts[3 * k + 1], kpts[3 * k + 2], a0, a1, a2, p);
  const double f = scale / (1.0 + 0.5 * (p[0] * p[0] + p[1] * p[1] + p[2] * p[2]) / e0);
  c128 v = F[(long)field * nr + l];
  v.re *= f;
  v.im *= f;
  F[(long)field * nr + l] = v;
}

// out = (base ? base : 0) + c * (kin + vloc .* x + alpha * vx)
__global__ void hcombine_kernel(c128* __restrict__ out, const c128* __restrict__ base, const c128* __restrict__ kin,
                                const c128* __restrict__ x, const c128* __restrict__ vx,
                                const double* __restrict__ vloc, double alpha, double cre, double cim, long count,
                                int nr) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long)gridDim.x * blockDim.x) {
    c128 h = kin[i];
    if (vloc) {
      const double v = vloc[i % nr];
      const c128 xi = x[i];
      h.re += v * xi.re;
      h.im += v * xi.im;
    }
    if (vx) {
      const c128 w = vx[i];
      h.re += alpha * w.re;
      h.im += alpha * w.im;
    }
    c128 o = base ? base[i] : c128{0.0, 0.0};
    o.re += cre * h.re - cim * h.im;
    o.im += cre * h.im + cim * h.re;
    out[i] = o;
  }
}

constexpr int kRedThreads = 256;

template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* sh) {
  for (int q = 0; q < NV; ++q) sh[q * kRedThreads + threadIdx.x] = v[q];
  __syncthreads();
  for (int w = kRedThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int q = 0; q < NV; ++q) sh[q * kRedThreads + threadIdx.x] += sh[q * kRedThreads + threadIdx.x + w];
    __syncthreads();
  }
  for (int q = 0; q < NV; ++q) v[q] = sh[q * kRedThreads];
}

// out[f] = sum_r |psi[f][r]|^2, one block per field, fixed order
__global__ void __launch_bounds__(kRedThreads) norms_kernel(double* __restrict__ out, const c128* __restrict__ psi,
                                                            int nr) {
  __shared__ double sh[kRedThreads];
  const c128* p = psi + (long)blockIdx.x * nr;
  double v[1] = {0.0};
  for (int i = threadIdx.x; i < nr; i += kRedThreads) v[0] += p[i].re * p[i].re + p[i].im * p[i].im;
  block_sum<1>(v, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = v[0];
}

// partial[b][0..5] = sum over a grid-stride slice of conj(L) * (k+G+a)_d * F for d = 0, 1, 2 (re, im)
__global__ void __launch_bounds__(kRedThreads) agrad_partial_kernel(double* __restrict__ partial,
                                                                    const c128* __restrict__ L,
                                                                    const c128* __restrict__ F,
                                                                    const double* __restrict__ kpts, int nf,
                                                                    Geom g, double a0, double a1, double a2,
                                                                    long count) {
  __shared__ double sh[6 * kRedThreads];
  const long nr = (long)g.n1 * g.n2 * g.n3;
  double v[6] = {0, 0, 0, 0, 0, 0};
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long)gridDim.x * blockDim.x) {
    const long field = i / nr;
    const long l = i % nr;
    const int k = (int)(field / nf);
    double p[3];
    gvec(g, l, kpts[3 * k], kpts[3 * k + 1], kpts[3 * k + 2], a0, a1, a2, p);
    const c128 x = L[i], y = F[i];
    const double re = x.re * y.re + x.im * y.im;  // conj(x) * y
    const double im = x.re * y.im - x.im * y.re;
    for (int d = 0; d < 3; ++d) {
      v[2 * d] += p[d] * re;
      v[2 * d + 1] += p[d] * im;
    }
  }
  block_sum<6>(v, sh);
  if (threadIdx.x == 0)
    for (int q = 0; q < 6; ++q) partial[6 * blockIdx.x + q] = v[q];
}

__global__ void __launch_bounds__(kRedThreads) sum_rows_kernel(double* __restrict__ out,
                                                               const double* __restrict__ partial, int nrows,
                                                               int width) {
  __shared__ double sh[kRedThreads];
  for (int q = 0; q < width; ++q) {
    double v[1] = {0.0};
    for (int i = threadIdx.x; i < nrows; i += kRedThreads) v[0] += partial[(long)i * width + q];
    block_sum<1>(v, sh);
    if (threadIdx.x == 0) out[q] = v[0];
    __syncthreads();
  }
}

// Gram-Schmidt through the Gram matrix, for up to kGramBands fields per k-point: with
// G_ij = w <v_i, v_j> = (L L^H)_ij the orthonormal fields are q_j = sum_{i <= j} conj(L^-1)_ji v_i,
// the result of Gram-Schmidt in band order. One read of the fields for G, one read and one
// write for the product; modified Gram-Schmidt passes over them nb^2 times from one
// workgroup per k. 32^3 / 216 k / 16 bands, a copy of the fields (0.8 ms) included: 11.3 -> 1.9 ms;
// error against a double Gram-Schmidt in 64 bits 1.1e-16 -> 1.9e-16; against one in 80 bits, both
// routes' arithmetic on the host with 16 random fields of 32,768 points, 1.6e-16 -> 1.0e-16.
//
// The error of this route grows with the square of the fields' condition number, that of
// modified Gram-Schmidt with the number itself: a k-point whose scaled Gram matrix is not
// close enough to diagonal (trace of its inverse above 1.5 nb), or whose factorisation fails
// (dependent or vanishing fields, infinities, NaN), is left to modified Gram-Schmidt
// (bad[k] = 1).
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kGramWaves = 4;

// part[k][chunk] = 16 x 16 complex partial sums of conj(v_i) v_j over the points of a chunk, on
// the matrix cores: lane l holds field l mod 16 at the four points 4 (l / 16) .. + 3 of a run of
// 16, and each 16x16x4 product sums one point of every lane group
__global__ void __launch_bounds__(64 * kGramWaves) gram16_kernel(double* __restrict__ part,
                                                                 const c128* __restrict__ psi, int nb, int nr,
                                                                 int len) {
  __shared__ double sh[kGramWaves - 1][2 * kGramBands * kGramBands];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int band = lane & 15, grp = lane >> 4;
  const int k = blockIdx.y, chunk = blockIdx.x;
  const c128* v = psi + ((long)k * nb + (band < nb ? band : 0)) * nr;
  const int r1 = (chunk + 1) * len < nr ? (chunk + 1) * len : nr;
  // sums of their own per point of the run: the rounding of a sum grows with its length
  v4d ar[4], ai[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) ar[q] = ai[q] = v4d{0, 0, 0, 0};
  for (int r0 = chunk * len + 16 * wv; r0 < r1; r0 += 16 * kGramWaves) {
    c128 x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = v[r0 + 4 * grp + q];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double re = band < nb ? x[q].re : 0.0, im = band < nb ? x[q].im : 0.0;
      ar[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(re, re, ar[q], 0, 0, 0);
      ar[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(im, im, ar[q], 0, 0, 0);
      ai[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(re, im, ai[q], 0, 0, 0);
      ai[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-im, re, ai[q], 0, 0, 0);
    }
  }
  const v4d gre = (ar[0] + ar[1]) + (ar[2] + ar[3]), gim = (ai[0] + ai[1]) + (ai[2] + ai[3]);
  // lane l, register q: row l / 16 + 4 q, column l mod 16; waves added in order
  if (wv > 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sh[wv - 1][2 * ((grp + 4 * q) * kGramBands + band)] = gre[q];
      sh[wv - 1][2 * ((grp + 4 * q) * kGramBands + band) + 1] = gim[q];
    }
  }
  __syncthreads();
  if (wv == 0) {
    double* o = part + ((long)k * gridDim.x + chunk) * (2 * kGramBands * kGramBands);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = 2 * ((grp + 4 * q) * kGramBands + band);
      double re = gre[q], im = gim[q];
      for (int u = 0; u < kGramWaves - 1; ++u) {
        re += sh[u][e];
        im += sh[u][e + 1];
      }
      o[e] = re;
      o[e + 1] = im;
    }
  }
}

// s + c += x, the rounding error of the addition carried in c
__device__ __forceinline__ void two_sum_add(double& s, double& c, double x) {
#pragma clang fp contract(off)
  const double t = s + x, b = t - s;
  c += (s - (t - b)) + (x - b);
  s = t;
}

// Of G = w * sum of the chunks: T[k][j][j] = (L^-1)_jj and, for i < j, T[k][j][i] =
// conj(L^-1)_ji / (L^-1)_jj, so that q_j = T_jj (v_j + sum T_ji v_i); bad[k]
constexpr int kFactorParts = 4;
__global__ void __launch_bounds__(kFactorParts * kGramBands * kGramBands) gram_factor_kernel(c128* __restrict__ T, int* __restrict__ bad,
                                                         const double* __restrict__ part, int nchunk, int nb,
                                                         double w) {
  constexpr int N = kGramBands;
  __shared__ c128 g[N][N + 1], li[N][N + 1];
  __shared__ double d[N], inv[N], q[N], dg[N];
  __shared__ int fail;
  const int t = threadIdx.x;
  const long k = blockIdx.x;
  const double* p = part + k * nchunk * (2 * N * N);
  // the chunks' sums with the error of each addition carried along, a quarter of the chunks on each
  // part of the workgroup. 32^3 / 1 k / 4 bands: 147 us with one wave for all of it (128 chunks in
  // series), 31 us so
  __shared__ double sh[kFactorParts - 1][N * N][4];
  const int e0 = t % (N * N), pt = t / (N * N);
  double re = 0.0, im = 0.0, cre = 0.0, cim = 0.0;
  if (e0 / N < nb && e0 % N < nb) {
    for (int c = pt; c < nchunk; c += kFactorParts) {
      const c128 z = *(const c128*)(p + (long)c * (2 * N * N) + 2 * e0);
      two_sum_add(re, cre, z.re);
      two_sum_add(im, cim, z.im);
    }
  }
  if (pt > 0) {
    double* o = sh[pt - 1][e0];
    o[0] = re;
    o[1] = cre;
    o[2] = im;
    o[3] = cim;
  }
  __syncthreads();
  if (pt == 0) {
    for (int u = 0; u < kFactorParts - 1; ++u) {
      const double* o = sh[u][e0];
      two_sum_add(re, cre, o[0]);
      cre += o[1];
      two_sum_add(im, cim, o[2]);
      cim += o[3];
    }
    g[e0 / N][e0 % N] = c128{w * (re + cre), w * (im + cim)};
    li[e0 / N][e0 % N] = c128{0.0, 0.0};
  }
  if (t == 0) fail = 0;
  __syncthreads();
  if (t < nb) {
    q[t] = g[t][t].re;
    d[t] = 1.0 / sqrt(q[t]);
    if (!(q[t] > 0.0) || !(q[t] < 1e300) || !(d[t] < 1e150)) fail = 1;
  }
  __syncthreads();
  if (const int e = t; e < N * N) {
    const int i = e / N, j = e % N;
    if (i < nb && j < nb) g[i][j] = i == j ? c128{1.0, 0.0} : cscale(g[i][j], d[i] * d[j]);
  }
  __syncthreads();
  // Cholesky of the scaled matrix, row t of the factor on thread t; L overwrites the lower part
  for (int j = 0; j < nb; ++j) {
    if (t == j) {
      double s = 1.0;
      for (int c = 0; c < j; ++c) s -= g[j][c].re * g[j][c].re + g[j][c].im * g[j][c].im;
      if (!(s > 0.0)) fail = 1;
      inv[j] = 1.0 / sqrt(s);
      dg[j] = 1.0 / sqrt(q[j] * s);  // the factor of q_j, rounded as few times as a norm's
    }
    __syncthreads();
    if (t > j && t < nb) {
      c128 s = g[t][j];
      for (int c = 0; c < j; ++c) {
        const c128 z = cmulc(g[j][c], g[t][c]);
        s = s - z;
      }
      g[t][j] = cscale(s, inv[j]);
    }
    __syncthreads();
  }
  // column t of L^-1
  double tr = 0.0;
  if (t < nb) {
    for (int i = t; i < nb; ++i) {
      c128 s = i == t ? c128{1.0, 0.0} : c128{0.0, 0.0};
      for (int c = t; c < i; ++c) s = s - cmul(g[i][c], li[c][t]);
      li[i][t] = cscale(s, inv[i]);
      tr += li[i][t].re * li[i][t].re + li[i][t].im * li[i][t].im;
    }
  }
  __shared__ double trs[N];
  if (t < N) trs[t] = t < nb ? tr : 0.0;
  __syncthreads();
  if (t == 0) {
    double s = 0.0;
    for (int i = 0; i < nb; ++i) s += trs[i];
    if (!(s <= 1.5 * nb)) fail = 1;
    bad[k] = fail;
  }
  if (const int e = t; e < N * N) {
    const int j = e / N, i = e % N;
    const c128 z = li[j][i];
    c128 o{0.0, 0.0};
    if (j < nb && i < j) {
      const double f = d[i] / (inv[j] * d[j]);
      o = c128{z.re * f, -z.im * f};
    } else if (j < nb && i == j) {
      o.re = dg[j];
    }
    T[k * N * N + e] = o;
  }
}

// q_j = T_jj (v_j + sum_{i < j} T_ji v_i) in place, one point per thread
template <int NB>
__global__ void __launch_bounds__(256) gram_apply_kernel(c128* __restrict__ psi, const c128* __restrict__ T,
                                                         const int* __restrict__ bad, int nb, int nr) {
  const long k = blockIdx.y;
  if (bad[k]) return;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= nr) return;
  c128* v = psi + k * nb * nr + r;
  const c128* t = T + k * kGramBands * kGramBands;
  c128 x[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) x[i] = i < nb ? v[(long)i * nr] : c128{0.0, 0.0};
#pragma unroll
  for (int j = NB - 1; j >= 0; --j) {
    if (j >= nb) continue;
    // the corrections first, v_j last: its digits are rounded once
    c128 s{0.0, 0.0};
#pragma unroll
    for (int i = 0; i < j; ++i) s = cmac(s, t[j * kGramBands + i], x[i]);
    v[(long)j * nr] = cscale(x[j] + s, t[j * kGramBands + j].re);
  }
}

// Modified Gram-Schmidt of the nb fields of one k-point (one workgroup per k), cell inner
// product w * sum conj(a) b; bad (may be NULL): only the k-points with bad[k] != 0
constexpr int kMgsThreads = 1024;
__global__ void __launch_bounds__(kMgsThreads) mgs_kernel(c128* __restrict__ psi, int nb, int nr, double w,
                                                          const int* __restrict__ bad) {
  if (bad && !bad[blockIdx.x]) return;
  __shared__ double sh[2 * kMgsThreads];
  c128* base = psi + (long)blockIdx.x * nb * nr;
  const int t = threadIdx.x;
  for (int b = 0; b < nb; ++b) {
    c128* vb = base + (long)b * nr;
    for (int c = 0; c < b; ++c) {
      const c128* vc = base + (long)c * nr;
      double re = 0.0, im = 0.0;
      for (int i = t; i < nr; i += kMgsThreads) {
        const c128 x = vc[i], y = vb[i];
        re += x.re * y.re + x.im * y.im;
        im += x.re * y.im - x.im * y.re;
      }
      sh[t] = re;
      sh[kMgsThreads + t] = im;
      __syncthreads();
      for (int s = kMgsThreads / 2; s > 0; s >>= 1) {
        if (t < s) {
          sh[t] += sh[t + s];
          sh[kMgsThreads + t] += sh[kMgsThreads + t + s];
        }
        __syncthreads();
      }
      const double pr = w * sh[0], pi = w * sh[kMgsThreads];
      __syncthreads();
      for (int i = t; i < nr; i += kMgsThreads) {
        const c128 x = vc[i];
        c128 y = vb[i];
        y.re -= pr * x.re - pi * x.im;
        y.im -= pr * x.im + pi * x.re;
        vb[i] = y;
      }
      __syncthreads();
    }
    double s2 = 0.0;
    for (int i = t; i < nr; i += kMgsThreads) s2 += vb[i].re * vb[i].re + vb[i].im * vb[i].im;
    sh[t] = s2;
    __syncthreads();
    for (int s = kMgsThreads / 2; s > 0; s >>= 1) {
      if (t < s) sh[t] += sh[t + s];
      __syncthreads();
    }
    const double inv = 1.0 / sqrt(w * sh[0]);
    __syncthreads();
    for (int i = t; i < nr; i += kMgsThreads) {
      c128 y = vb[i];
      y.re *= inv;
      y.im *= inv;
      vb[i] = y;
    }
    __syncthreads();
  }
}

unsigned grid_for(long count, int bs) {
  long g = (count + bs - 1) / bs;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (unsigned)g;
}

}  // namespace

hipError_t launch_kinetic_mul(c128* F, const double* kpts, int nk, int nf, const Geom& g, const double a[3],
                              double scale, hipStream_t st) {
  const long nr = (long)g.n1 * g.n2 * g.n3;
  dim3 grid((unsigned)((nr + 255) / 256), (unsigned)(nk * nf));
  hipLaunchKernelGGL(kinetic_mul_kernel, grid, dim3(256), 0, st, F, kpts, nf, g, a[0], a[1], a[2], scale);
  return hipGetLastError();
}

hipError_t launch_precond_mul(c128* F, const double* kpts, int nk, int nf, const Geom& g, const double a[3],
                              double e0, double scale, hipStream_t st) {
  const long nr = (long)g.n1 * g.n2 * g.n3;
  dim3 grid((unsigned)((nr + 255) / 256), (unsigned)(nk * nf));
  hipLaunchKernelGGL(precond_mul_kernel, grid, dim3(256), 0, st, F, kpts, nf, g, a[0], a[1], a[2], e0, scale);
  return hipGetLastError();
}

hipError_t launch_hcombine(c128* out, const c128* base, const c128* kin, const c128* x, const c128* vx,
                           const double* vloc, double alpha, double cre, double cim, long count, int nr,
                           hipStream_t st) {
  hipLaunchKernelGGL(hcombine_kernel, dim3(grid_for(count, 256)), dim3(256), 0, st, out, base, kin, x, vx, vloc,
                     alpha, cre, cim, count, nr);
  return hipGetLastError();
}

hipError_t launch_norms(double* out, const c128* psi, int nfields, int nr, hipStream_t st) {
  hipLaunchKernelGGL(norms_kernel, dim3(nfields), dim3(kRedThreads), 0, st, out, psi, nr);
  return hipGetLastError();
}

hipError_t launch_agrad(double* out6, double* partial, int nblk, const c128* L, const c128* F, const double* kpts,
                        int nf, const Geom& g, const double a[3], long count, hipStream_t st) {
  hipLaunchKernelGGL(agrad_partial_kernel, dim3(nblk), dim3(kRedThreads), 0, st, partial, L, F, kpts, nf, g, a[0],
                     a[1], a[2], count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sum_rows_kernel, dim3(1), dim3(kRedThreads), 0, st, out6, partial, nblk, 6);
  return hipGetLastError();
}

hipError_t launch_mgs(c128* psi, int nk, int nb, int nr, double w, hipStream_t st) {
  hipLaunchKernelGGL(mgs_kernel, dim3(nk), dim3(kMgsThreads), 0, st, psi, nb, nr, w, nullptr);
  return hipGetLastError();
}

// chunks of a k-point's points: about 8,192 workgroups in all, at least 256 points each
static int gram_chunks(int nk, int nr) {
  const int most = nr / 256 > 0 ? nr / 256 : 1, want = (8192 + nk - 1) / nk;
  return want < most ? want : most;
}

size_t gram_work_bytes(int nk, int nr) {
  constexpr size_t mat = kGramBands * kGramBands * sizeof(c128);
  return (size_t)nk * ((gram_chunks(nk, nr) + 1) * mat + sizeof(int));
}

// The faster route by measured costs in us, 1 to 6 bands of 16^3 to 32^3 on 1 to 384 k-points.
// Modified Gram-Schmidt keeps one CU per k-point busy (4 us and two passes per band, 5 passes per
// pair of bands) until its traffic reaches 5 TB/s; the Gram matrix costs 4 launches, the
// event that orders the use of its scratch (3 us) and, per point,
// what 16 fields cost on the matrix cores plus the bands' passes. 20^3 / 20 k / 1 band: 12 us
// against 24; 16^3 / 8 k: 2 bands 16 against 21, 4 bands 41 against 22; 32^3 / 384 k: 2 bands 507
// against 817, 4 bands 1,624 against 1,139.
bool gram_pays(int nk, int nb, int nr) {
  const double x = nr / 32768.0, pairs = 0.5 * nb * (nb - 1), points = (double)nk * nr;
  const double alone = (nb * (4.0 + 16.0 * x) + pairs * 20.0 * x) * (1.0 + (nk < 256 ? nk / 256.0 : 1.0));
  const double bytes = (3.0 * nb + 5.0 * pairs) * 16.0 * points;
  const double mgs = alone > bytes / 5e6 ? alone : bytes / 5e6;
  return 23.0 + points * (38.0 + 12.7 * nb) * 1e-6 < mgs;
}

hipError_t launch_gram_schmidt(c128* psi, int nk, int nb, int nr, double w, void* work, hipStream_t st) {
  if (nb > kGramBands || nr % 64 != 0) return hipErrorInvalidValue;
  const int want = gram_chunks(nk, nr);
  const int len = ((nr + want - 1) / want + 63) / 64 * 64, nchunk = (nr + len - 1) / len;
  double* part = (double*)work;
  c128* T = (c128*)(part + (size_t)nk * nchunk * 2 * kGramBands * kGramBands);
  int* bad = (int*)(T + (size_t)nk * kGramBands * kGramBands);
  hipError_t e;
  hipLaunchKernelGGL(gram16_kernel, dim3(nchunk, nk), dim3(64 * kGramWaves), 0, st, part, psi, nb, nr, len);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(gram_factor_kernel, dim3(nk), dim3(kFactorParts * kGramBands * kGramBands), 0, st, T, bad, part, nchunk, nb, w);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const dim3 grid((nr + 255) / 256, nk);
  if (nb <= 4) hipLaunchKernelGGL(gram_apply_kernel<4>, grid, dim3(256), 0, st, psi, T, bad, nb, nr);
  else if (nb <= 8) hipLaunchKernelGGL(gram_apply_kernel<8>, grid, dim3(256), 0, st, psi, T, bad, nb, nr);
  else hipLaunchKernelGGL(gram_apply_kernel<kGramBands>, grid, dim3(256), 0, st, psi, T, bad, nb, nr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(mgs_kernel, dim3(nk), dim3(kMgsThreads), 0, st, psi, nb, nr, w, bad);
  return hipGetLastError();
}

}  // namespace fockmi

// Device helpers of the two-stage pair form's kernels (pairs.hip, planes.hip).
#pragma once

#include "fused_common.hpp"
#include "pairs.hpp"

namespace fockmi {

// rounds of a transpose through LDS and the LDS elements they need
template <int N, int NPH>
constexpr int pw_lds_elems() {
  constexpr int H = N / NPH;
  return NPH == 1 ? N * N * (N + 1) : (N * N * H > H * N * (N + 1) ? N * N * H : H * N * (N + 1));
}

// Rounds per transpose where a field does not fit in LDS: three at 24^3 in FP64, whose rounds are
// whole waves (two rounds of 288 threads are not) and of which two fit side by side; two at 32^3
// in FP32 (four, two side by side, spill: 27 of the 216 k-points of 16 bands 233 -> 269 ms).
template <int N, typename T>
constexpr int pw_nph() {
  return (long)N * N * (N + 1) * (long)sizeof(cx<T>) <= 160L * 1024 ? 1 : (N % 3 == 0 ? 3 : 2);
}

// 3D transform of one field of N^3 values by N * N threads, one line per thread in registers
// (fft_reg.hpp); LDS carries the transposes (see fused.hip). x phase: the line along n1 at
// (m2, m3) = (chi, clo); z phase: the line along n3 at (l1, l2) = (chi, clo).
// TWOBUF: rounds go through two buffers in turn, over all transposes of a field: the threads of a
// round read while those of the next one write, and one barrier per round covers both (a buffer
// is written again only after the barrier that its readers have passed). Pairs of 24^3 in FP64,
// 64 k-points of 16 bands: 78.1 ms in two rounds, 77.7 in three, 70.5 in three with two buffers.
template <int N, typename T, bool TWOBUF = (pw_nph<N, T>() > 2)>
struct CubeTransform {
  static constexpr int NPH = pw_nph<N, T>();
  static constexpr int E = (int)sizeof(cx<T>);
  static constexpr int NTI = N * N;
  static constexpr int H = N / NPH;
  static constexpr int TPG = NTI / NPH;
  static constexpr int NBK = N / NPH;
  static constexpr bool XY_WAVES = TPG % 64 == 0;
  static constexpr bool YZ_WAVES = XY_WAVES && (NBK * H) % 64 == 0;
  static constexpr int kRound = pw_lds_elems<N, NPH>();  // elements of one round
  static constexpr int kLdsElems = TWOBUF ? 2 * kRound : kRound;
  // with one round both transposes use one array and every phase writes back to the slots it
  // read, so each transpose needs one barrier
  static constexpr bool INPLACE = NPH == 1;
  static constexpr unsigned SX = INPLACE ? (unsigned)(N * (N + 1) * E) : (unsigned)(N * H * E);
  static constexpr unsigned SY = INPLACE ? (unsigned)((N + 1) * E) : (unsigned)(H * E);
  static constexpr int L1S = (int)((65535u / SX) + 1) < N ? (int)((65535u / SX) + 1) : N;
  int grp, gyz, chi, clo;
  unsigned lx0, ly0, lyz0, lz0;  // LDS byte offsets of the thread's elements in the transposes

  __device__ __forceinline__ explicit CubeTransform(int t) {
    grp = (NPH == 1) ? 0 : (XY_WAVES ? __builtin_amdgcn_readfirstlane(t / TPG) : t / TPG);
    const int tl = t % TPG;
    const int hl = tl % H;
    clo = hl + H * grp;
    chi = tl / H;
    gyz = (NPH == 1) ? 0 : (YZ_WAVES ? __builtin_amdgcn_readfirstlane(chi / NBK) : chi / NBK);
    const int lrow = chi % NBK;
    lx0 = INPLACE ? (unsigned)((chi * (N + 1) + hl) * E) : (unsigned)((chi * H + hl) * E);
    ly0 = INPLACE ? (unsigned)((chi * N * (N + 1) + hl) * E) : (unsigned)((chi * N * H + hl) * E);
    lyz0 = (unsigned)((lrow * N * (N + 1) + clo) * E);
    lz0 = (unsigned)((lrow * N + clo) * (N + 1) * E);
  }

  // byte offset of round r of the four transposes of a field
  static constexpr unsigned buf(int r) { return TWOBUF && r % 2 ? (unsigned)(kRound * E) : 0u; }
  static_assert(!TWOBUF || NPH > 1, "one round has one buffer");

  // v: the x-phase line in, the transformed z-phase line out
  __device__ __forceinline__ void forward(cx<T> (&v)[N], cx<T>* lds) const {
    fft<N, -1>(v);
    // x -> y
#pragma unroll
    for (int g = 0; g < NPH; ++g) {
      if (grp == g) {
        const unsigned b0 = opaque(lx0 + buf(g)), b1 = opaque(lx0 + buf(g) + L1S * SX);
        static_for<N>([&](auto l1) {
          constexpr int L = decltype(l1)::value;
          if constexpr (L < L1S) lds_at<L * SX>(lds, b0) = v[L];
          else lds_at<(L - L1S) * SX>(lds, b1) = v[L];
        });
      }
      __syncthreads();
      if (grp == g) {
        const unsigned b = opaque(ly0 + buf(g));
        static_for<N>([&](auto m2) { v[m2] = lds_at<decltype(m2)::value * SY>(lds, b); });
      }
      if constexpr (!INPLACE && !TWOBUF) __syncthreads();
    }
    fft<N, -1>(v);
    // y -> z
#pragma unroll
    for (int g = 0; g < NPH; ++g) {
      if (gyz == g) {
        const unsigned b = opaque(lyz0 + buf(NPH + g));
        static_for<N>([&](auto l2) { lds_at<decltype(l2)::value * (N + 1) * E>(lds, b) = v[l2]; });
      }
      __syncthreads();
      if (gyz == g) {
        const unsigned b = opaque(lz0 + buf(NPH + g));
        static_for<N>([&](auto m3) { v[m3] = lds_at<decltype(m3)::value * E>(lds, b); });
      }
      if constexpr (!INPLACE && !TWOBUF) __syncthreads();
    }
    fft<N, -1>(v);
  }

  // v: the z-phase line in, the (unnormalised) x-phase line out
  __device__ __forceinline__ void inverse(cx<T> (&v)[N], cx<T>* lds) const {
    fft<N, +1>(v);
    // z -> y
#pragma unroll
    for (int g = 0; g < NPH; ++g) {
      if (gyz == g) {
        const unsigned b = opaque(lz0 + buf(2 * NPH + g));
        static_for<N>([&](auto m3) { lds_at<decltype(m3)::value * E>(lds, b) = v[m3]; });
      }
      __syncthreads();
      if (gyz == g) {
        const unsigned b = opaque(lyz0 + buf(2 * NPH + g));
        static_for<N>([&](auto l2) { v[l2] = lds_at<decltype(l2)::value * (N + 1) * E>(lds, b); });
      }
      if constexpr (!INPLACE && !TWOBUF) __syncthreads();
    }
    fft<N, +1>(v);
    // y -> x
#pragma unroll
    for (int g = 0; g < NPH; ++g) {
      if (grp == g) {
        const unsigned b = opaque(ly0 + buf(3 * NPH + g));
        static_for<N>([&](auto m2) { lds_at<decltype(m2)::value * SY>(lds, b) = v[m2]; });
      }
      __syncthreads();
      if (grp == g) {
        const unsigned b0 = opaque(lx0 + buf(3 * NPH + g)), b1 = opaque(lx0 + buf(3 * NPH + g) + L1S * SX);
        static_for<N>([&](auto l1) {
          constexpr int L = decltype(l1)::value;
          if constexpr (L < L1S) v[L] = lds_at<L * SX>(lds, b0);
          else v[L] = lds_at<(L - L1S) * SX>(lds, b1);
        });
      }
      if constexpr (!INPLACE && !TWOBUF) __syncthreads();
    }
    fft<N, +1>(v);
  }
};

// a uniform load through the scalar cache: a vector load here would wait for the W stores
// in flight, like every load that is waited for behind them
__device__ __forceinline__ int ld_uniform(const int* p) {
  return *(const __attribute__((address_space(4))) int*)(uintptr_t)p;
}

// W is written once and read once, much later: the non-temporal hint keeps it from pushing
// the operands out of L2 (an XCD's 32 CUs write 8 MiB of W per pair round, twice its L2)
template <typename T>
__device__ __forceinline__ void st_w(cx<T>* p, cx<T> v) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store((v2){v.re, v.im}, (v2*)p);
}
template <typename T>
__device__ __forceinline__ cx<T> ld_w(const cx<T>* p) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  const v2 v = __builtin_nontemporal_load((const v2*)p);
  return {v.x, v.y};
}

// natural index of element i of a field in the paired order (np = n2 * n3; 0: natural order)
__device__ __forceinline__ int natural_index(int i, int np) {
  if (np == 0) return i;
  const int h = i / (2 * np), e = i - h * 2 * np;
  return (2 * h + (e & 1)) * np + (e >> 1);
}

// The pairs of a block in order: target tiles of kPairTile, for each tile its sources, for
// each source the tile's targets. XCD x (workgroups b = x mod 8) walks a contiguous eighth of
// them, so that the tile's targets, the current sources and the kernel table meet in its L2.
struct PairWalk {
  int nt, nj, tri;
  long q, q1;
  long tile_q0 = 0, tile_q1 = 0;  // pairs of the current tile
  int tile = 0, tw = 0;           // the tile and its targets
  int ti = 0, j = 0;              // target and source of the current pair within the block
  __device__ __forceinline__ explicit PairWalk(const PairBlock& b) : nt(b.nt), nj(b.nj), tri(b.tri) {
    const int x = blockIdx.x & 7;
    q = b.npairs * x / 8 + (blockIdx.x >> 3);
    q1 = b.npairs * (x + 1) / 8;
  }
  __device__ __forceinline__ void enter(int t) {
    tile = t;
    tw = nt - t * kPairTile < kPairTile ? nt - t * kPairTile : kPairTile;
    const int njt = tri ? (nj < (t + 1) * kPairTile ? nj : (t + 1) * kPairTile) : nj;
    tile_q1 = tile_q0 + (long)tw * njt;
  }
  __device__ __forceinline__ void locate() {
    while (q >= tile_q1) {
      tile_q0 = tile_q1;
      enter(tile + 1);
    }
    const int rem = (int)(q - tile_q0);
    j = __builtin_amdgcn_readfirstlane(rem / tw);
    ti = __builtin_amdgcn_readfirstlane(tile * kPairTile + rem % tw);
  }
  // false: this workgroup has no pair
  __device__ __forceinline__ bool start() {
    if (q >= q1) return false;
    enter(0);
    locate();
    return true;
  }
  __device__ __forceinline__ bool next() {
    q += gridDim.x >> 3;
    if (q >= q1) return false;
    locate();
    return true;
  }
};

}  // namespace fockmi

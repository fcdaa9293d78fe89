// Launchers of the two-stage pair form (pairs.hip).
#pragma once

#include "kernels.hpp"

namespace fockmi {

constexpr int kPairTile = 8;   // targets of one tile: the targets one wave of stage 2 holds
constexpr int kPairGroup = 64;  // targets of one workgroup of stage 2: those whose mirror sums meet there
constexpr int kPairFew = 2;     // targets of a wave of stage 2 in rows too short to fill the device
// the group of rows of `rows` targets: 8 waves of whole tiles where these make 2,048 waves (8 per CU)
inline int pair_group(int rows, int nr) {
  return (long)(nr / 64) * ((rows + kPairTile - 1) / kPairTile) < 2048 ? kPairGroup / kPairTile * kPairFew : kPairGroup;
}

// A block of pairs: nt targets from t0 on (index kt * nx + s) against nj sources from j0 on
// (index ks * ns + band). With tri, targets and sources are the same fields (t0 == j0,
// nt == nj) and only the pairs whose target tile is not below the source tile are run.
// W of pair (t, j) is field j * nt + t of the batch. In FP32 the one-CU kernel's fields (X, P,
// W, and with them M and F of stage 2) hold the points m1 = 2h, 2h + 1 side by side, element
// (h, m2, m3, b) at ((h * n2 + m2) * n3 + m3) * 2 + b, so that a lane moves 16 bytes at a time;
// elsewhere they are in natural order.
struct PairBlock {
  int t0, nt, j0, nj, tri;
  long npairs;      // pairs the block runs
};
template <typename T>
struct PairArgs {
  const cx<T>* X;   // targets [ntk][nx][nr]
  const cx<T>* P;   // sources [nsk][ns][nr], conjugated in the density
  const T* Kt;      // [nq][nr] kernel tables in the pair kernel's order, 1/N_r folded
  const int* qidx;  // [ntk][nsk]
  cx<T>* W;
  int nx, ns, nsk;
  PairBlock b;
};
// The same block for the plane passes (planes.hip): inputs in complex128, rounded to T as they
// are read, and tables [nq][l1][l3][l2] in FP64.
template <typename T>
struct PlaneArgs {
  const c128* X;
  const c128* P;
  const double* K;
  const int* qidx;
  cx<T>* W;
  int nx, ns, nsk, n1;
  PairBlock b;
};
template <typename T>
hipError_t launch_pair_planes(int n2, int n3, const PlaneArgs<T>& a, int num_cus, hipStream_t st);
hipError_t launch_plane_table(double* Kp, const double* K, int nq, const Geom& g, hipStream_t st);

inline long pair_count(int nt, int nj, bool tri) {
  if (!tri) return (long)nt * nj;
  long n = 0;
  for (int t = 0; t < nt; t += kPairTile) {
    const int w = nt - t < kPairTile ? nt - t : kPairTile, m = t + kPairTile < nj ? t + kPairTile : nj;
    n += (long)w * m;
  }
  return n;
}
// workgroups that run at once on num_cus CUs
template <typename T>
int pair_w_slots(int n, int num_cus);
// n: cubic grid length, {16, 20, 24, 32} in FP32, {16, 20, 24} in FP64
template <typename T>
hipError_t launch_pair_w(int n, const PairArgs<T>& a, int num_cus, hipStream_t st);

// The sums over one block. out: the targets' sums; mir (NULL: one-sided): the sources' sums
// of F_t conj(W), unscaled, over the pairs of different tiles when tri. TM float: FP32 products and
// partial sums, compensated FP64 sums; double: FP64 throughout (W widened).
template <typename TW, typename TM>
struct WsumArgs {
  const cx<TW>* W;
  const cx<TM>* M;  // [sources][nr]
  const cx<TM>* F;  // [targets][nr]
  c128* out;        // [targets][nr]
  cx<float>* comp;  // FP32: compensation of out between the blocks of one target
  c128* run;        // FP64: the unscaled sum between the blocks of one target
  c128* mir;        // [groups of the row][nsrc][nr]
  cx<float>* mcomp; // FP32: compensation of mir
  int t0, nt, j0, nj, ns, tri;
  int nsrc;         // all sources
  int jb0;          // band index of source j0 within its k-point
  int group;        // pair_group of the rows
  int nr;
  int np;           // n2 * n3 when the fields are in the paired order (out is natural), else 0
  int first, last;  // first / last block of these targets
  int mfirst;       // first block of these sources' mirror sums
  int accumulate;   // add to the existing out
  double scale;
};
template <typename TW, typename TM>
hipError_t launch_wsum(const WsumArgs<TW, TM>& a, hipStream_t st);
// dst = (accumulate ? dst : 0) + (sre + i sim) * sum over the groups of (mir + mcomp); mcomp may be NULL
hipError_t launch_mirror_add(c128* dst, const c128* mir, const c64* mcomp, double sre, double sim, int accumulate, int nsrc,
                             int nr, int rows, int group, int tri, int np, hipStream_t st);

}  // namespace fockmi

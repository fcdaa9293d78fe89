// Device helpers of the two-stage pair form's kernels (pairs.hip, planes.hip).
#pragma once

#include "fused_common.hpp"
#include "pairs.hpp"

namespace fockmi {

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

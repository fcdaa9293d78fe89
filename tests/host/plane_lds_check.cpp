// Every LDS element that a lane of the plane passes reads or writes lies in its wave's own buffer,
// for every plane shape: prints "n2 n3 planes outside" per shape, `outside` the accesses beyond it.
#include <cstdio>

#include "plane_lds.hpp"

template <int N2, int N3>
void check() {
  using S = fockmi::PlaneShape<N2, N3>;
  int outside = 0;
  for (int lane = 0; lane < 64; ++lane) {
    const int pl = lane / S::L, idx = lane % S::L;
    for (int i = 0; i < N2; ++i) {
      const int e = S::col(pl, idx) + i * S::ROW;
      outside += e < 0 || e >= S::WORDS;
    }
    for (int i = 0; i < N3; ++i) {
      const int e = S::row(pl, idx) + i;
      outside += e < 0 || e >= S::WORDS;
    }
  }
  std::printf("%d %d %d %d\n", N2, N3, S::PL, outside);
}

template <int N2>
void shapes() {
  check<N2, 16>();
  check<N2, 20>();
  check<N2, 24>();
  check<N2, 32>();
}

int main() {
  shapes<16>();
  shapes<20>();
  shapes<24>();
  shapes<32>();
}

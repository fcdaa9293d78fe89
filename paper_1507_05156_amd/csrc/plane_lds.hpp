// LDS layout of the plane passes' transposes (planes.hip); host code too, so that the reads of
// every lane can be checked against the buffer.
#pragma once

namespace fockmi {

constexpr int kPlaneWaves = 8;

// One wave holds PL planes of N2 x N3 values, lane `lane` the line idx = lane % L of plane
// pl = lane / L. With L = 20 or 24 the last lanes have no plane (pl == PL).
template <int N2, int N3>
struct PlaneShape {
  static constexpr int L = N2 > N3 ? N2 : N3;  // lanes of one plane
  static constexpr int PL = 64 / L;            // planes of one wave
  static constexpr int ROW = N3 + 1;           // padded row of the transpose
  static constexpr int WORDS = PL * N2 * ROW;  // values of one wave's transpose buffer (one component at a time)
  // first element of a lane's column (stride ROW, N2 of them) and of its row (N3 of them). Lanes
  // without a line or a plane read where another lane reads; nothing uses what they read.
  static constexpr int base(int pl) { return (pl < PL ? pl : 0) * N2 * ROW; }
  static constexpr int col(int pl, int idx) { return base(pl) + (idx < N3 ? idx : 0); }
  static constexpr int row(int pl, int idx) { return base(pl) + (idx < N2 ? idx : 0) * ROW; }
};

}  // namespace fockmi

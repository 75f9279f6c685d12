// Which loads a thread of the single-step H_K^(0) stencil issues: it owns the four x2 rows y0 .. y0 + 3 at x3
// site i3 of each plane (host and device code, so that the ranges can be checked without a device).
#pragma once

#if defined(__HIP__) || defined(__HIPCC__)
#define QF_HD __host__ __device__ __forceinline__
#else
#define QF_HD inline
#endif

namespace qf {

constexpr int ST_RPT = 4;     // x2 rows per thread

struct StencilRows {
  bool rin[ST_RPT];   // the row is a lattice row (and i3 a lattice site): loaded, updated and stored
  bool up, dn;        // load row y0 - 1, row y0 + ST_RPT
  bool xe;            // load the x3 neighbour outside the wave: i3 - 1 for lane 0, i3 + 1 for lane 63
};

// The rows above and below are loaded only beside a lattice row.  (Tiles are 16 rows, so a thread's rows may
// lie past the lattice with the row above them past it too.)
QF_HD StencilRows stencil_rows(int N, int y0, int i3, int lane) {
  StencilRows s;
  const bool xin = i3 < N;
  for (int r = 0; r < ST_RPT; ++r) s.rin[r] = xin && y0 + r < N;
  s.up = s.rin[0] && y0 > 0;
  s.dn = xin && y0 + ST_RPT < N;
  s.xe = (lane == 0 && xin && i3 > 0) || (lane == 63 && i3 + 1 < N);
  return s;
}

}  // namespace qf

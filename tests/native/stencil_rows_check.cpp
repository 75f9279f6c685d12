// The single-step stencil's loads over every lattice size, tile and lane: all inside the lattice, and every
// neighbour that an updated site needs from memory is loaded.
#include <cstdio>

#include "stencil_rows.h"

int main() {
  constexpr int TX = 64, TY = 16;     // the tile
  long long checks = 0, failures = 0;
  auto check = [&](bool ok, const char *what, int N, int y0, int i3) {
    ++checks;
    if (!ok && failures++ < 5) std::printf("FAIL %s: N %d, rows from %d, site %d\n", what, N, y0, i3);
  };
  for (int N = 8; N <= 512; N += 2)
    for (int y0 = 0; y0 < (N + TY - 1) / TY * TY; y0 += qf::ST_RPT)
      for (int i3 = 0; i3 < (N + TX - 1) / TX * TX; ++i3) {
        const int lane = i3 % TX;
        const qf::StencilRows s = qf::stencil_rows(N, y0, i3, lane);
        const bool xin = i3 < N;
        for (int r = 0; r < qf::ST_RPT; ++r) check(s.rin[r] == (xin && y0 + r < N), "row", N, y0, i3);
        check(!s.up || (xin && y0 - 1 >= 0 && y0 - 1 < N), "row above in the lattice", N, y0, i3);
        check(!s.dn || (xin && y0 + qf::ST_RPT < N), "row below in the lattice", N, y0, i3);
        check(s.up || !(s.rin[0] && y0 > 0), "row above loaded", N, y0, i3);
        check(s.dn || !(s.rin[qf::ST_RPT - 1] && y0 + qf::ST_RPT < N), "row below loaded", N, y0, i3);
        const int nb = lane == 0 ? i3 - 1 : i3 + 1;
        check(!s.xe || ((lane == 0 || lane == 63) && nb >= 0 && nb < N), "site beside in the lattice", N, y0, i3);
        check(s.xe || !(xin && (lane == 0 || lane == 63) && nb >= 0 && nb < N), "site beside loaded", N, y0, i3);
      }
  std::printf("%lld checks, %lld failures\n", checks, failures);
  return failures != 0;
}

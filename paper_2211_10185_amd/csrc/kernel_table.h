// Tables of the transform-pass kernels (host code).
#pragma once

#include <cstddef>

namespace qf {

// Kernels of one split-x2 variant (x2 = n1 x N/n1, plane groups of xi, pencil tiles of pencil_tt x3
// columns); pencil is null where the variant does not exist, and a slab entry where the variant has
// no use for that kind.  plane_edges: chunks start and end with plane passes (M_SPLIT) instead of
// slab passes.
enum { SLAB_REAL = 0, SLAB_COMPLEX = 1, SLAB_EDGE = 2, SLAB_AB = 3, SLAB_KINDS = 4 };
constexpr int SPLIT_VARIANTS = 5;
struct SplitKernels {
  const void *slab[SLAB_KINDS];
  const void *pencil;
  size_t slab_lds, pencil_lds;
  int slab_nt[SLAB_KINDS], pencil_nt, n1, xi, pencil_tt;
  bool plane_edges;
};

// Kernels of the FP64 energy measurement of one lattice size (slab: by state precision); pencil is null
// where the size has none.  tps, pps: tiles of one state.
struct MeasKernels {
  const void *slab[2];
  const void *pencil;
  size_t slab_lds, pencil_lds;
  int slab_nt, pencil_nt, tps, pps;
};

// Transform-pass kernels instantiated for one lattice size (index 0: complex64,
// 1: complex128); plane entries are null where an N^2 plane does not fit LDS.
struct FftKernels {
  const void *plane[2];
  const void *row[2];
  const void *col[2];
  size_t plane_lds[2], row_lds[2], col_lds[2];
  int plane_nt;
  SplitKernels split[2][SPLIT_VARIANTS];   // two-pass split-x2 schedule: precision, variant
  MeasKernels meas;
};

// visit(kernel, its dynamic LDS bytes) for every kernel of a size; stops at the first result other than
// `ok` and returns it.
template <class R, class Visit> R for_each_kernel(const FftKernels &k, R ok, Visit visit) {
  R r = ok;
  auto one = [&](const void *f, size_t lds) {
    if (f && r == ok) r = visit(f, lds);
  };
  for (int w = 0; w < 2; ++w) {
    one(k.plane[w], k.plane_lds[w]);
    one(k.row[w], k.row_lds[w]);
    one(k.col[w], k.col_lds[w]);
    for (const SplitKernels &s : k.split[w]) {
      one(s.pencil, s.pencil_lds);
      for (const void *f : s.slab) one(f, s.slab_lds);
    }
    one(k.meas.slab[w], k.meas.slab_lds);
  }
  one(k.meas.pencil, k.meas.pencil_lds);
  return r;
}

}  // namespace qf

// for_each_kernel visits every kernel pointer of a size's table with its own LDS size, and stops at a failure.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>

#include "kernel_table.h"

int main() {
  using namespace qf;
  std::map<const void *, size_t> want;
  uintptr_t next = 0x1000;
  auto kernel = [&](size_t lds) { const void *f = (const void *)next; next += 16; want[f] = lds; return f; };
  FftKernels k;
  std::memset(&k, 0, sizeof(k));
  size_t lds = 100;
  for (int w = 0; w < 2; ++w) {
    k.plane[w] = kernel(k.plane_lds[w] = ++lds);
    k.row[w] = kernel(k.row_lds[w] = ++lds);
    k.col[w] = kernel(k.col_lds[w] = ++lds);
    for (SplitKernels &s : k.split[w]) {
      s.slab_lds = ++lds;
      for (const void *&f : s.slab) f = kernel(s.slab_lds);
      s.pencil = kernel(s.pencil_lds = ++lds);
    }
  }
  k.meas.slab_lds = ++lds;
  for (const void *&f : k.meas.slab) f = kernel(k.meas.slab_lds);
  k.meas.pencil = kernel(k.meas.pencil_lds = ++lds);

  int failures = 0;
  std::map<const void *, size_t> got;
  if (for_each_kernel(k, 0, [&](const void *f, size_t l) { got[f] = l; return 0; }) != 0) ++failures;
  if (got != want) { ++failures; std::printf("FAIL visited %zu of %zu kernels\n", got.size(), want.size()); }
  // nothing after a failure
  int calls = 0;
  if (for_each_kernel(k, 0, [&](const void *, size_t) { return ++calls == 3 ? 9 : 0; }) != 9 || calls != 3) ++failures;
  // absent kernels
  std::memset(&k, 0, sizeof(k));
  for_each_kernel(k, 0, [&](const void *, size_t) { ++failures; return 0; });
  std::printf("%zu kernels, %d failures\n", want.size(), failures);
  return failures != 0;
}

// Instantiations of the split-x2 passes (slab and pencil kernels), some sizes and one precision per
// compilation (the build compiles this file once per QF_SPLIT_PART value).
#include "split_passes.h"

#if QF_SPLIT_PART == 0
#define QF_T float
#define QF_SIZES(X) X(32) X(36) X(40) X(48) X(50) X(54) X(60) X(64) X(72) X(80) X(90)
#elif QF_SPLIT_PART == 1
#define QF_T float
#define QF_SIZES(X) X(96) X(100) X(108) X(120)
#elif QF_SPLIT_PART == 2
#define QF_T float
#define QF_SIZES(X) X(128) X(144) X(150) X(160)
#elif QF_SPLIT_PART == 3
#define QF_T float
#define QF_SIZES(X) X(162) X(180) X(192) X(200)
#elif QF_SPLIT_PART == 4
#define QF_T float
#define QF_SIZES(X) X(216) X(240) X(250) X(256)
#elif QF_SPLIT_PART == 5
#define QF_T double
#define QF_SIZES(X) X(32) X(36) X(40) X(48) X(50) X(54) X(60) X(64) X(72) X(80)
#elif QF_SPLIT_PART == 6
#define QF_T double
#define QF_SIZES(X) X(90) X(96) X(100) X(108) X(120) X(128) X(144) X(150)
#else
#define QF_T double
#define QF_SIZES(X) X(160) X(162) X(180) X(192) X(200) X(216) X(240) X(250) X(256)
#endif

#define QF_CAT2(a, b) a##b
#define QF_CAT(a, b) QF_CAT2(a, b)

namespace qf {

#define REG_SPLIT(n)          \
  register_split<QF_T, n>(t); \
  if constexpr (sizeof(QF_T) == 8) register_meas<n>(t);
void QF_CAT(register_split_part, QF_SPLIT_PART)(FftKernels *t) { QF_SIZES(REG_SPLIT) }

}  // namespace qf

// Two-level axis lengths 36..128: (n1, n2) for the x/y passes, (z1, z2) for
// the z pass.  Splits near the square root keep a thread's serial code short;
// the z pass then splits level B over (component, k1) threads (z pass in us:
// 100 = 25 x 4 22.0, 10 x 10 17.5; 128 = 32 x 4 29.1, 8 x 16 26.0;
// 64 = 16 x 4 8.2, 8 x 8 7.5; 96 = 24 x 4, 12 x 8 and 8 x 12 within 2%).
#include "kernels.hpp"

namespace cbs {
const SizeOps* sizes_mid(int* count) {
  static const SizeOps table[] = {
    CBS_SIZE_XYZ(36, 6, 6, 6, 6),     CBS_SIZE_XYZ(40, 8, 5, 8, 5),
    CBS_SIZE_XYZ(48, 8, 6, 8, 6),     CBS_SIZE_XYZ(64, 8, 8, 8, 8),
    CBS_SIZE_XYZ(96, 12, 8, 24, 4),   CBS_SIZE_XYZ(100, 10, 10, 10, 10),
    CBS_SIZE_XYZ(128, 16, 8, 8, 16)};
  *count = int(sizeof(table) / sizeof(table[0]));
  return table;
}
}  // namespace cbs

// Axis lengths 2..32.  Primes and lengths below 9 are a single register codelet
// (n = n x 1); the others are split in two levels.  A grid this small holds few
// waves per SIMD, so a pass lasts as long as one thread's serial code: splitting
// a DFT-32 into 8 x 4 spreads it over eight times the threads (32^3 iteration
// 24.8 -> 16.5 us, 27^3 24.4 -> 17.1, 24^3 20.1 -> 15.1, 16^3 16.5 -> 14.4;
// below 9 points there is nothing to gain: 8 = 4 x 2 13.2 us against 13.0).
#include "kernels.hpp"

namespace cbs {
#define S1(n) CBS_SIZE_XYZ(n, n, 1, n, 1)
#define S2(n, a, b) CBS_SIZE_XYZ(n, a, b, a, b)
const SizeOps* sizes_small(int* count) {
  static const SizeOps table[] = {
    S1(2),  S1(3),  S1(4),  S1(5),  S1(6),  S1(7),  S1(8),  S1(11), S1(13), S1(29),
    S2(9, 3, 3),  S2(10, 5, 2), S2(12, 4, 3), S2(14, 7, 2), S2(15, 5, 3), S2(16, 4, 4),
    S2(18, 6, 3), S2(20, 5, 4), S2(24, 6, 4), S2(25, 5, 5), S2(27, 9, 3), S2(32, 8, 4)};
  *count = int(sizeof(table) / sizeof(table[0]));
  return table;
}
}  // namespace cbs

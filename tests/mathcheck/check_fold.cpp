// The event kernel's 48-bit digit columns (device_common.hpp: fold_carry, fold_row3) on the
// host: kFoldEvents largest digits between two carries, over several stretches, against the
// same sums in 128-bit integers.  Prints the number of sums that differ.
#include <cstdio>
#include <initializer_list>

#include "integrands.hpp"

typedef __int128 i128;

int main() {
  int bad = 0, n = 0;
  const long long ones = static_cast<long long>(vg::kMask48);
  const long long digits[] = {0, 1, ones, ones - 1, -ones, -1, 0xffff00000000ll, 0x800000000000ll};
  for (long long lo : digits)
    for (long long hi : digits)
      for (int last : {0, 1, 64, static_cast<int>(vg::kFoldEvents)})
        for (int stretches = 0; stretches <= 5; ++stretches) {
          // columns as the LDS atomics leave them: sums modulo 2^64
          unsigned long long u[3] = {0, 0, 0};
          long long c[3] = {0, 0, 0};
          i128 want = 0;
          for (int s = 0; s <= stretches; ++s) {
            const long long ev = s < stretches ? static_cast<long long>(vg::kFoldEvents) : last;
            u[0] = static_cast<unsigned long long>(c[0]) + static_cast<unsigned long long>(lo) * ev;
            u[1] = static_cast<unsigned long long>(c[1]) + static_cast<unsigned long long>(hi) * ev;
            c[0] = static_cast<long long>(u[0]);
            c[1] = static_cast<long long>(u[1]);
            want += (static_cast<i128>(hi) * (i128(1) << 48) + lo) * ev;
            if (s < stretches) vg::fold_carry(c, 1);
          }
          long long r[3];
          vg::fold_row3(c[0], c[1], r, 1);
          const i128 got = (static_cast<i128>(r[2]) << 64) + (static_cast<i128>(r[1]) << 32) + r[0] +
                           static_cast<i128>(c[2]) * (i128(1) << 48) * (i128(1) << 48);
          ++n;
          if (got != want) ++bad;
        }
  std::printf("{\"sums\": %d, \"bad\": %d}\n", n, bad);
  return 0;
}

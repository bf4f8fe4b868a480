// CPU check of the pass plan of every row length: factor_radices accepts
// exactly the lengths made of 2, 3 and 5, its radices are ones the kernels
// have, largest first, and multiply to the length; the magic numbers of
// fastdiv divide every index the kernels form exactly.
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "sht_internal.h"

using namespace sht;

int main() {
  int fail = 0, lengths = 0;
  for (int I = 1; I <= SHT_MAX_I; ++I) {
    int x = I, rad[SHT_MAX_RADICES], n = 0;
    for (int p : {2, 3, 5})
      while (x % p == 0) x /= p;
    const bool ok = factor_radices(I, rad, &n);
    if (ok != (x == 1)) ++fail;
    if (!ok) continue;
    ++lengths;
    int prod = 1;
    for (int q = 0; q < n; ++q) {
      const int r = rad[q];
      bool known = false;
      for (int k : {2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16}) known = known || r == k;
      if (!known || (q > 0 && r > rad[q - 1])) ++fail;
      prod *= r;
      // divisors: butterflies per sequence and products of earlier radices
      for (int d : {I / r, prod / r}) {
        if (d < 2) continue;
        const uint32_t magic = 0xFFFFFFFFu / (uint32_t)d + 1u;
        for (uint32_t j = 0; j < 8192; ++j)
          if ((uint32_t)(((uint64_t)j * magic) >> 32) != j / (uint32_t)d) ++fail;
      }
    }
    if (prod != I || n > SHT_MAX_RADICES) ++fail;
  }
  std::printf("radix_check: %d lengths, %d failures\n", lengths, fail);
  return fail ? 1 : 0;
}

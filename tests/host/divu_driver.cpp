// Host driver for the launch-time division of the HIP path: checks DivU
// against the machine's division and prints the number of quotients compared.
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include "../../paper_2607_06519_amd/csrc/divu.h"

int main() {
  const uint32_t top = 0x7FFFFFFFu;
  unsigned long long n_checked = 0;
  auto check = [&](uint32_t n, uint32_t d) {
    fdkv::DivU q;
    q.set(d);
    ++n_checked;
    if (q.div(n) != n / d) {
      printf("wrong: %u / %u\n", n, d);
      return false;
    }
    return true;
  };
  uint64_t r = 88172645463325252ull;
  auto rnd = [&]() { return r ^= r << 13, r ^= r >> 7, r ^= r << 17, (uint32_t)(r >> 33); };
  for (uint32_t i = 0; i < 400000; ++i) {
    // small divisors, those around every power of two, and random ones
    uint32_t d = i < 4096 ? i + 1 : (1u << (i % 31)) + rnd() % 3 - 1;
    if (i % 3 == 0 && i >= 4096) d = rnd() >> (i % 31);
    if (d < 1 || d > top) d = 1;
    const uint32_t m = rnd() % (top / d + 1);
    for (uint32_t n : {0u, d - 1, d, m * d, m * d ? m * d - 1 : 0u, top, top - top % d, top - top % d ? top - top % d - 1 : 0u, rnd()})
      if (n <= top && !check(n, d)) return 1;
  }
  printf("%llu\n", n_checked);
  return 0;
}

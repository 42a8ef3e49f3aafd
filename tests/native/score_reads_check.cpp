// The vector reads of a select pass stay inside the score array's allocation,
// for every array length and every lane of its grid, whole vectors or not.
#include <cstdint>
#include <cstdio>

#include "../../paper_2410_22697_amd/csrc/launch_rules.hpp"

int main() {
  int past = 0, wrong = 0;
  for (int64_t n = 1; n < 3000; ++n)
    for (int64_t q = 0; q < n / 4 + 600; ++q) {
      const int64_t at = ms::score_vector(q, n);
      past += at < 0 || (at + 1) * 16 > ms::score_bytes(n);
      wrong += q < n / 4 && at != q;  // whole vectors are their own
    }
  std::printf("past %d wrong %d\n", past, wrong);
  return past || wrong;
}

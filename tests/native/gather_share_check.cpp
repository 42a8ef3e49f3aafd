// How many of the launched blocks move HBM rows beside a miss gather: a rule of
// the step's own two lists.
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "../../paper_2410_22697_amd/csrc/launch_rules.hpp"

int main() {
  int bad = 0;
  const uint64_t rows[] = {0, 1, 2, 50, 1000, 37000, 160000, 1300000};
  for (uint64_t blocks : {1ull, 95ull, 96ull, 97ull, 512ull, 4096ull})
    for (uint64_t hbm : rows)
      for (uint64_t host : rows) {
        const uint64_t s = ms::hbm_share(hbm, host, blocks);
        bad += s < 1 || s > blocks;
        // nothing comes over the link: the whole grid
        bad += host == 0 && s != blocks;
        // 16 blocks for each HBM row per host row, 96 at least
        if (host > 0) bad += s < blocks && (s < 96 || s < 16 * hbm / host);
        // more HBM rows never get fewer blocks, more host rows never more
        bad += ms::hbm_share(2 * hbm, host, blocks) < s;
        bad += host > 0 && ms::hbm_share(hbm, 2 * host, blocks) > s;
      }
  // few misses among many rows: the link is done before a small share would be
  bad += ms::hbm_share(160000, 100, 4096) != 4096;
  std::printf("wrong %d\n", bad);
  return bad != 0;
}

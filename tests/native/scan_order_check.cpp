// The dispatch of single-pass scans that run at once, on a model of the chip:
// 8 XCDs of 32 CUs that hold 32 waves each; block i of a launch goes to XCD
// i % 8, each XCD starts a launch's blocks in order, and a block ends once
// every tile before its own has started (its sum is then published, or comes).
// Which launch an XCD serves first is chosen against the scans: XCD x prefers
// launch x % launches. With the library's rule for taking tiles every mix
// ends; in block order alone two scans larger than the chip never do.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../paper_2410_22697_amd/csrc/launch_rules.hpp"

namespace {
constexpr int kXcds = 8, kCus = 32, kCuWaves = 32;

struct Scan {
  int64_t tiles;
  int threads;
  bool tickets;
};

struct Block {
  int launch, xcd, cu;
  int64_t tile;
};

// true if every block of every launch ends
bool ends(const std::vector<Scan>& scans) {
  const int n = (int)scans.size();
  std::vector<std::vector<int64_t>> next(n, std::vector<int64_t>(kXcds));  // next block of a launch on an XCD
  std::vector<std::vector<char>> started(n);
  std::vector<int64_t> taken(n, 0), first(n, 0);  // tickets handed out; first tile not started
  std::vector<std::vector<int>> used(kXcds, std::vector<int>(kCus, 0));
  std::vector<Block> live;
  for (int l = 0; l < n; ++l) {
    started[l].assign(scans[l].tiles, 0);
    for (int x = 0; x < kXcds; ++x) next[l][x] = x;
  }
  for (;;) {
    bool moved = false;
    for (int x = 0; x < kXcds; ++x)
      for (int j = 0; j < n; ++j) {
        const int l = (x + j) % n;
        const int waves = scans[l].threads / 64;
        bool placed = true;
        while (placed && next[l][x] < scans[l].tiles) {
          placed = false;
          for (int c = 0; c < kCus && !placed; ++c)
            if (used[x][c] + waves <= kCuWaves) {
              const int64_t tile = scans[l].tickets ? taken[l]++ : next[l][x];
              used[x][c] += waves;
              live.push_back({l, x, c, tile});
              started[l][tile] = 1;
              next[l][x] += kXcds;
              placed = moved = true;
            }
        }
      }
    for (int l = 0; l < n; ++l)
      while (first[l] < scans[l].tiles && started[l][first[l]]) ++first[l];
    std::vector<Block> rest;
    for (const Block& b : live)
      if (first[b.launch] >= b.tile) {  // every tile before it has started
        used[b.xcd][b.cu] -= scans[b.launch].threads / 64;
        moved = true;
      } else {
        rest.push_back(b);
      }
    live.swap(rest);
    bool left = !live.empty();
    for (int l = 0; l < n; ++l) left = left || first[l] < scans[l].tiles;
    if (!left) return true;
    if (!moved) return false;
  }
}
}  // namespace

int main() {
  int bad = 0, mixes = 0;
  const int64_t sizes[] = {1, 8, 64, 160, 168, 169, 336, 337, 672, 673, 2000, 6000};
  const int threads[] = {256, 512, 1024};
  std::vector<Scan> all;
  const int64_t four = ms::ordered_scan_waves(0), eight = ms::ordered_scan_waves(8);
  auto scan = [](int64_t tiles, int nt, int64_t ordered) {
    return Scan{tiles, nt, ms::scan_takes_tickets(tiles, nt, ordered)};
  };
  for (int64_t t : sizes)
    for (int nt : threads) all.push_back(scan(t, nt, four));
  // two scans of each pair of sizes, and two of each at once (4 hardware queues)
  for (const Scan& a : all)
    for (const Scan& b : all) {
      bad += !ends({a, b});
      bad += !ends({a, b, a, b}) + !ends({a, a, a, b});
      mixes += 3;
    }
  // four largest scans in block order of each block size, in every mix
  std::vector<Scan> most;
  for (int nt : threads) {
    int64_t t = 1;
    while (!ms::scan_takes_tickets(t + 1, nt, four)) ++t;
    most.push_back(scan(t, nt, four));
  }
  for (int i = 0; i < 81; ++i) {
    bad += !ends({most[i % 3], most[i / 3 % 3], most[i / 9 % 3], most[i / 27]});
    ++mixes;
  }
  // eight hardware queues
  for (int64_t t : sizes)
    for (int nt : threads) {
      bad += !ends(std::vector<Scan>(8, scan(t, nt, eight)));
      ++mixes;
    }
  // the model sees what the tickets are for: scans in block order that are
  // larger than the chip hold each other out, and four that are above the line
  const bool stuck = !ends({{2000, 1024, false}, {2000, 1024, false}}) && !ends({{6000, 256, false}, {2000, 512, false}}) &&
                     !ends(std::vector<Scan>(4, {1000, 512, false}));
  std::printf("mixes %d stuck %d seen %d\n", mixes, bad, (int)stuck);
  return bad || !stuck;
}

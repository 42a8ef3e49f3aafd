// launch_rules.hpp - rules that shape launches and their reads, in plain C++ so
// that they are also built and checked without a GPU (constexpr ones run in
// kernels too).
#pragma once

#include <cstdint>

namespace ms {

// How the blocks of a single-pass scan take their tiles. A tile waits for the
// tiles before it. In block order it could wait for ever if other launches kept
// those off the chip for good, which only other scans can do, as their blocks
// wait too. Each XCD starts a launch's blocks in order, so the XCD that the
// first missing tile of scan A needs holds no waiting block of A: the others
// have to fill it alone. Scans of at most ordered_scan_waves waves therefore
// keep block order: three of them leave every XCD (32 CUs of 32 waves; those of
// a kernel whose registers leave room for half as many count twice) the 16 waves
// of the largest block, and HIP runs a process's streams on 4 hardware queues
// (more, if GPU_MAX_HW_QUEUES asks for them: the limit falls with their number).
// Larger scans take tickets: a block takes the next tile when it starts, so
// every tile before a waiting one belongs to a running block, whatever else
// runs. Tickets cost a launch a round trip before its first load and are handed
// out one after the other (k_frontier, 282 tiles: 19.0 -> 20.5 us; k_round_evict,
// 845 tiles: 39 -> 49), which is why they are not used everywhere. (Several
// processes on one card add up their queues; the wait is bounded too.)
constexpr int64_t kXcdWaves = 32 * 32, kXcds = 8;
inline int64_t ordered_scan_waves(int queues) {
  return kXcds * (kXcdWaves - 16) / ((queues > 4 ? queues : 4) - 1);
}
inline bool scan_takes_tickets(int64_t tiles, int threads, int64_t ordered_waves) {
  return (tiles + kXcds - 1) / kXcds * kXcds * (threads / 64) > ordered_waves;
}

// A round's select passes read the n scores in 16-byte vectors: vector q of the
// grid, or vector 0 past the whole ones (those lanes read their last scores one
// by one and drop the vector). The array therefore has room for one vector,
// also where it holds fewer than four scores.
constexpr int64_t score_vector(int64_t q, int64_t n) { return q < n / 4 ? q : 0; }
inline int64_t score_bytes(int64_t n) { return n < 4 ? 16 : n * 4; }

// Blocks that move a step's HBM rows beside its miss gather, of the `blocks`
// launched: the rows have the link's time to move in, so they take few blocks
// and leave the chip to the next step's sampling (and the memory system to the
// link). A block moves a row about 1/8 as fast as the whole link does, so 16
// blocks for each HBM row per host row need half the link's time. Eight
// look-ahead steps on the 111M-node share (9 HBM rows per host row), us per pass
// by blocks: 4096 2990, 512 2960, 256 2865, 128 2765, 64 2765, 32 2783; on the
// 2.45M-node graph 4096 5330, 128 5292, 32 5290; a step waited for on the
// 111M-node share 4096 557, by this rule 548. Least share and factor: 32 and 4,
// 96 and 16, 256 and 64: 16 steps with a round on the 170K-node graph 5242, 4937,
// 4932; eight on the 111M-node share 2762, 2776, 2952, on the 2.45M-node graph
// 5303, 5305, 5324. By the step's own lists: few misses
// (the link is done early) get the whole grid (190K HBM rows, 880 host rows: 126
// us a step, 153 with the share of a step of 7 and 1).
constexpr uint64_t kMinHbmShare = 96;
constexpr uint64_t hbm_share(uint64_t n_hbm, uint64_t n_host, uint64_t blocks) {
  if (n_host == 0) return blocks;
  const uint64_t want = 16 * n_hbm / n_host;
  const uint64_t share = want > kMinHbmShare ? want : kMinHbmShare;
  return share < blocks ? share : blocks;
}

}  // namespace ms

// sample_kernels.hpp - fanout sampling, frontier dedup and relabel (one hop
// of the NeighborSampler of Algorithm 2, DGL block convention).
#pragma once

#include "common.hpp"

namespace ms {

constexpr int kScanNT = 1024;       // threads per scan block
constexpr int kScanItems = 4;       // items per thread
constexpr int kScanTile = kScanNT * kScanItems;

__device__ __forceinline__ int64_t size_of(const int64_t* p, int64_t c) { return p ? *p : c; }

// Single-pass scan by decoupled look-back: tile b publishes its aggregate,
// then its inclusive prefix once the tiles before it are known. flags[b] =
// tag << 32 | value, tag = 2 * epoch (aggregate) or 2 * epoch + 1 (inclusive
// prefix); the epoch differs for every launch, so flags are never cleared.
// A wait ends if every tile before the waiting one gets a block: see scan_tile.
// It is bounded all the same: past the limit the step is flagged (status bit
// 8) and the tile goes on with the values it has.
constexpr int kLookbackSpins = 1 << 20;

// The tile of this block of a scan: its index, or with TICKETS (launches that
// scan_takes_tickets names) the next ticket. The last block to take one puts
// the counter back to zero for the next scan of the same stream. Whole block,
// before a check that makes the block leave.
template <bool TICKETS>
__device__ __forceinline__ int64_t scan_tile(uint32_t* ticket) {
  if constexpr (!TICKETS) return (int64_t)blockIdx.x;
  __shared__ uint32_t tile;
  if (threadIdx.x == 0) {
    const uint32_t t = atomicAdd(ticket, 1u);
    tile = t;
    if (t == gridDim.x - 1) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return (int64_t)(uint32_t)wave_uniform((int32_t)tile);
}

__device__ __forceinline__ uint32_t lookback_exclusive(uint64_t* flags, int64_t b, uint32_t agg, uint32_t epoch,
                                                       int32_t* status, uint32_t* excl_lds) {
  const uint32_t t_agg = 2u * epoch, t_inc = 2u * epoch + 1u;
  if (wave_id() == 0) {
    const int lane = lane_id();
    if (lane == 0)
      __hip_atomic_store(&flags[b], ((uint64_t)(b == 0 ? t_inc : t_agg) << 32) | agg, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    uint32_t excl = 0;
    int64_t p = b - 1;  // the window is tiles p - 63 .. p, lane l on tile p - l
    int spins = 0;
    while (p >= 0) {
      const int64_t i = p - lane;
      // before tile 0: an inclusive prefix of zero
      const uint64_t f = i >= 0 ? __hip_atomic_load(&flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                : ((uint64_t)t_inc << 32);
      const uint32_t tag = (uint32_t)(f >> 32);
      const uint64_t ready = ballot(tag == t_agg || tag == t_inc);
      const uint64_t inc = ballot(tag == t_inc);
      // lanes 0..k must be ready, k = the nearest inclusive prefix (or the window)
      const int k = inc ? __ffsll((unsigned long long)inc) - 1 : MS_WAVE - 1;
      const uint64_t need = k == MS_WAVE - 1 ? ~0ull : ((2ull << k) - 1);
      if ((ready & need) == need) {
        excl += wave_sum(lane <= k ? (uint32_t)f : 0u);
        if (inc) break;
        p -= MS_WAVE;
        continue;
      }
      if (++spins > kLookbackSpins) {
        if (lane == 0) atomicOr(status, 8);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    if (lane == 0) {
      if (b > 0)
        __hip_atomic_store(&flags[b], ((uint64_t)t_inc << 32) | (excl + agg), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      *excl_lds = excl;
    }
  }
  __syncthreads();
  return *excl_lds;
}

// A frontier row as the sampler takes it, read in one 16-byte load: the node,
// its row length and where its row starts in the CSR (a row is shorter than
// 2^32 entries).
typedef uint32_t v4r __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4r row_record(int32_t v, int64_t start, int64_t d) {
  return v4r{(uint32_t)v, (uint32_t)d, (uint32_t)start, (uint32_t)((uint64_t)start >> 32)};
}

// -------------------------------------------------------------- hop 1's rows
// The seed batch is hop 1's frontier. Block b: the rows of tile b get
// min(deg, fo) positions; the tile's exclusive prefix comes from the
// single-pass scan, and bptr[0..n0] gets the offsets. Rows longer than big_min
// go to the front of big_rows (one global atomic per block). With
// small_end > 0 the other rows go to its back, the r-th listed one at
// big_rows[small_end - 1 - r]: with n0 <= small_end rows the two parts never
// meet, and the one-wave-per-row sampler then finds a row for each of its
// first n0 waves. Every load of a thread is issued before the first is used.
// Each seed is checked (a local id, not repeated: the first to set its bit in
// `seen` keeps it) and placed: F_0 = seeds, pos_of[seed] = its position, its
// row record, n_0 = n0. A bad seed sets the step's status, which every later
// kernel checks first.
template <bool TICKETS>
__global__ __launch_bounds__(kScanNT) void k_seed_rows(const int64_t* __restrict__ csr_indptr,
                                                       const int32_t* __restrict__ seeds, int32_t n0, int32_t L,
                                                       int32_t* __restrict__ nodes, StepSizes* sz, int32_t fo,
                                                       int32_t* __restrict__ bptr, uint64_t* flags, uint32_t epoch,
                                                       int32_t* __restrict__ pos_of, uint32_t* __restrict__ seen,
                                                       v4r* __restrict__ rec, int32_t* __restrict__ big_rows,
                                                       int64_t big_min, int64_t small_end, int32_t* next_sizes,
                                                       uint32_t* ticket) {
  const int64_t tile = scan_tile<TICKETS>(ticket);
  __shared__ int32_t lds[kScanNT / MS_WAVE + 1];
  __shared__ int32_t big_lds[kScanTile];  // long rows from the front, the others from the back
  __shared__ int32_t big_n, small_n;
  __shared__ unsigned long long big_base, small_base;
  __shared__ uint32_t excl_lds;
  // (the step's sizes are clear here: no status to check)
  const int64_t n = n0;
  if (tile == 0 && threadIdx.x == 0) sz->n[0] = n;
  if (tile == 0 && next_sizes && threadIdx.x < sizeof(StepSizes) / 4) next_sizes[threadIdx.x] = 0;
  const int64_t base = tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
  if (threadIdx.x == 0) big_n = small_n = 0;
  __syncthreads();
  int32_t c[kScanItems] = {};
  int32_t s = 0;
  if (tile * kScanTile < n) {
    int32_t v[kScanItems];
    int64_t lo[kScanItems], hi[kScanItems];
#pragma unroll
    for (int it = 0; it < kScanItems; ++it) v[it] = seeds[base + it < n ? base + it : n - 1];
#pragma unroll
    for (int it = 0; it < kScanItems; ++it) pin(v[it]);
    // the marks (an atomic each, whose old word says whether the seed is a
    // repeat) and the row extents in one round, no result used before all are
    // under way; lanes without a seed, and bad ones, mark nothing and load an
    // in-range row
    uint32_t was[kScanItems];
    bool ok[kScanItems];
#pragma unroll
    for (int it = 0; it < kScanItems; ++it) {
      ok[it] = v[it] >= 0 && v[it] < L;
      const int32_t x = ok[it] ? v[it] : 0;
      was[it] = 0u;
      if (ok[it] && base + it < n) was[it] = atomicOr(&seen[x >> 5], 1u << (x & 31));
      lo[it] = csr_indptr[x];
      hi[it] = csr_indptr[x + 1];
    }
#pragma unroll
    for (int it = 0; it < kScanItems; ++it) pin(was[it]);
#pragma unroll
    for (int it = 0; it < kScanItems; ++it) {
      pin(lo[it]);
      pin(hi[it]);
    }
#pragma unroll
    for (int it = 0; it < kScanItems; ++it) {
      const int64_t i = base + it;
      if (i < n) {
        if (!ok[it]) {
          atomicOr(&sz->status, 1);
          continue;
        }
        if ((was[it] >> (v[it] & 31)) & 1u) atomicOr(&sz->status, 2);
        pos_of[v[it]] = (int32_t)i;
        nodes[i] = v[it];
        const int64_t d = hi[it] - lo[it];
        rec[i] = row_record(v[it], lo[it], d);
        c[it] = d < fo ? (int32_t)d : fo;
        s += c[it];
        if (d > big_min)
          big_lds[atomicAdd(&big_n, 1)] = (int32_t)i;
        else if (small_end)
          big_lds[kScanTile - 1 - atomicAdd(&small_n, 1)] = (int32_t)i;
      }
    }
  }
  int32_t tot;
  const int32_t ex = block_exclusive_scan<kScanNT>(s, lds, &tot);  // (its barriers complete the big_lds appends)
  const uint32_t before = lookback_exclusive(flags, tile, (uint32_t)tot, epoch, &sz->status, &excl_lds);
  int64_t run = (int64_t)before + ex;
#pragma unroll
  for (int it = 0; it < kScanItems; ++it) {
    const int64_t i = base + it;
    if (i < n) {
      run += c[it];
      bptr[i + 1] = (int32_t)run;
    }
  }
  if (threadIdx.x == 0) {
    if (tile == 0) bptr[0] = 0;
    if (tile == gridDim.x - 1) sz->e[0] = (int64_t)before + tot;
    big_base = big_n ? atomicAdd((unsigned long long*)&sz->n_big[0], (unsigned long long)big_n) : 0ull;
    small_base = small_n ? atomicAdd((unsigned long long*)&sz->n_small[0], (unsigned long long)small_n) : 0ull;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < big_n; j += kScanNT) big_rows[big_base + j] = big_lds[j];
  for (int j = threadIdx.x; j < small_n; j += kScanNT)
    big_rows[small_end - 1 - (int64_t)(small_base + j)] = big_lds[kScanTile - 1 - j];
}

// --------------------------------------------------------------- sampler
// One wavefront per frontier node. Rows with d <= fanout are copied. For
// longer rows the choice is the fanout positions of smallest (key, j), written
// in ascending j:
//   - rows of up to 256 positions: every key is in the wave's registers (one
//     Philox block a lane), and choose_quads takes the smallest;
//   - longer rows, fanouts up to 56: a threshold pass draws every key (lane q of
//     an iteration draws one Philox block = keys of positions 4q..4q+3, a quad)
//     and keeps, in ascending q, the quads with a key < tau; choose_quads then
//     chooses among their keys;
//   - longer rows, larger fanouts: the pass keeps the (key, j) pairs with
//     key < tau, and select_emit finds the fanout-th smallest key T by a bitwise
//     search over ballots (from below tau's top bit); ties at T are taken in
//     list order (= ascending j).
// tau is set so that about fanout + 3*sqrt(fanout) + 3 keys survive, and is
// bisected if fewer than fanout or more than the list holds survive (rare).
// The chosen ids are marked in the sampled-id bitmap as they are written. Rows
// longer than big_min (listed as the frontier's rows were written) are taken
// first. Where the frontier is small, so that its few longest rows bound the
// hop's time, each of them gets a whole block: its waves filter consecutive
// quarters of the row with the same tau, and the four lists, concatenated in
// order, are the row's list. Otherwise (many rows keep the chip busy) each gets
// one wave, ahead of the shorter rows. Other rows get one wave each.
constexpr int kSampleWaves = 4;  // k_sample_blocks: waves per block (a long row's quarters)
constexpr int kRowWaves = 2;     // k_sample_waves: waves per workgroup (one row each)
constexpr int kCandSlots = 5;                   // candidates per lane in the selection
constexpr int kCandCap = kCandSlots * MS_WAVE;  // candidates per wave (LDS): 320, so the
                                                // largest fanout (256) keeps 64 of slack for ties
constexpr int64_t kBigRow = 2048;
constexpr int64_t kBigBlocks = 2048;  // blocks that walk the big list (8 per CU)
constexpr int64_t kBlockRowsMax = 65536;  // frontiers up to this size sample long rows by blocks
// Waves of k_sample_waves at most: enough for the frontiers that occur, where a
// grid for the bound would dispatch many waves that find no row. Look-ahead
// steps, us per pass by this limit: eight on the 111M-node share 32K 2879, 64K
// 2761, 128K 2750, the whole bound 2780; four bf16 ones of 4096 seeds on the
// 2.45M-node graph 128K 7555-7650, the whole bound (1.4M) 7750-7810.
constexpr int64_t kRowWavesMax = 131072;
constexpr int kTauIters = 64;         // threshold passes: x4 growth (<= 16) then bisection (<= 33)

struct SampleArgs {
  const int32_t* csr_indices;
  const v4r* rec;           // row records of the frontier
  StepSizes* sz;
  const int32_t* bptr;
  int32_t* out;
  int32_t hop;  // 1-based
  int32_t fo;
  uint32_t t;
  uint32_t key0, key1;
  double mu32;              // (fo + 3 sqrt(fo) + 3) * 2^32
  int64_t big_min;          // rows longer than this are listed in big_rows
  const int32_t* big_rows;  // appended by k_seed_rows and k_frontier
  int64_t n_bound;          // bound of the frontier's rows
  int64_t row_waves;        // k_sample_waves: small_end of the row list (the other rows' part ends there)
  int64_t big_blocks;       // k_sample_blocks: blocks [0, big_blocks) walk the big list, one row per
                            // block; the rest take all other rows, one per wave
  uint32_t* bits;           // sampled-id bitmap: this block's copy is (block % copies)
  int64_t copy_words;       // words from one copy to the next
  uint32_t copies;          // a power of two
  int32_t* err;             // threshold search could not isolate a candidate set
  int32_t tau_iters;        // threshold passes allowed per row (kTauIters)
  uint64_t* flags;          // tile states of the frontier scan that follows: cleared here
  int64_t n_flags;
};

// The copy of the sampled-id bitmap that this block marks. Atomics on one
// 128-byte line go through one after another (about 100 M/s), and a small id
// space has few lines: 11.4K marks on the 8 lines of 7.8K ids took 14 of a
// launch's 16.5 us. So small spaces have kSmallCopies copies, which the dedup
// scan ors together.
constexpr uint32_t kSmallCopies = 8;
__device__ __forceinline__ uint32_t* mark_bits(const SampleArgs& a) {
  return a.bits + (int64_t)(blockIdx.x & (a.copies - 1)) * a.copy_words;
}

__device__ __forceinline__ void clear_flags(const SampleArgs& a) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_flags;
       i += (int64_t)gridDim.x * blockDim.x)
    a.flags[i] = 0ull;
}

// A row record, the same in every lane, in scalar registers.
struct Row {
  int32_t v;
  uint32_t d;
  int64_t start;
  __device__ __forceinline__ Row(const v4r* rec, int64_t row) {
    const v4r r = rec[row];
    set(r);
  }
  __device__ __forceinline__ explicit Row(const v4r& r) { set(r); }
  __device__ __forceinline__ void set(const v4r& r) {
    v = wave_uniform((int32_t)r.x);
    d = (uint32_t)wave_uniform((int32_t)r.y);
    start = (int64_t)(((uint64_t)(uint32_t)wave_uniform((int32_t)r.w) << 32) | (uint32_t)wave_uniform((int32_t)r.z));
  }
};

// Philox4x32-10 with counter (q, v, t, hop) for every q of one row. Words 1-3
// of the counter are the same across the row, so round 1's product of word 2
// (t) and round 2's product of word 0 (which round 1 builds from t, v and the
// key only) are computed once per row; the other rounds are the published
// block function unchanged.
struct PhiloxRow {
  uint32_t x1, y1;      // words 0 and 1 after round 1
  uint32_t a2hi, a2lo;  // round 2's 64-bit product of word 0
  uint32_t hop, k0, k1;
  __device__ __forceinline__ PhiloxRow(uint32_t v, uint32_t t, uint32_t hop_, uint32_t key0, uint32_t key1)
      : hop(hop_), k0(key0), k1(key1) {
    const uint64_t b1 = (uint64_t)0xCD9E8D57u * t;
    x1 = (uint32_t)(b1 >> 32) ^ v ^ key0;
    y1 = (uint32_t)b1;
    const uint64_t a2 = (uint64_t)0xD2511F53u * x1;
    a2hi = (uint32_t)(a2 >> 32);
    a2lo = (uint32_t)a2;
  }
  // the block of counter q, given round 1's product of word 0, a1 = M0 * q
  // (a lane's consecutive iterations add M0 * 64 to it instead of
  // multiplying again)
  __device__ __forceinline__ uint4 from_a1(uint64_t a1) const {
    const uint32_t z1 = (uint32_t)(a1 >> 32) ^ hop ^ k1, w1 = (uint32_t)a1;
    uint32_t r0 = k0 + 0x9E3779B9u, r1 = k1 + 0xBB67AE85u;  // round 2's key
    const uint64_t b2 = (uint64_t)0xCD9E8D57u * z1;
    uint4 c = make_uint4((uint32_t)(b2 >> 32) ^ y1 ^ r0, (uint32_t)b2, a2hi ^ w1 ^ r1, a2lo);
#pragma unroll
    for (int r = 2; r < 10; ++r) {
      r0 += 0x9E3779B9u;
      r1 += 0xBB67AE85u;
      const uint64_t a = (uint64_t)0xD2511F53u * c.x;
      const uint64_t b = (uint64_t)0xCD9E8D57u * c.z;
      c = make_uint4(xor3_key((uint32_t)(b >> 32), c.y, r0), (uint32_t)b, xor3_key((uint32_t)(a >> 32), c.w, r1),
                     (uint32_t)a);
    }
    return c;
  }
};

__device__ __forceinline__ uint64_t first_tau(double mu32, int64_t d) {
  const double t = mu32 / (double)d + 1.0;
  return t >= 4294967296.0 ? (1ull << 32) : (uint64_t)t;
}

// Threshold bookkeeping: returns true when the count is acceptable, else
// moves tau (bisection once both sides are known).
struct TauSearch {
  uint64_t lo = 0, hi = (1ull << 32) + 1, tau;
  __device__ bool step(int cnt, int fo, int cap, bool* fail) {
    const uint64_t full = 1ull << 32;
    if (cnt >= fo && cnt <= cap) return true;
    if (cnt < fo) {
      lo = tau;
      tau = (hi > full) ? (tau * 4 > full ? full : tau * 4) : (lo + hi) / 2;
    } else {
      hi = tau;
      tau = (lo + hi) / 2;
    }
    if (hi <= full && hi - lo <= 1) *fail = true;
    return false;
  }
};

__device__ __forceinline__ void emit_id(int32_t* __restrict__ out, int p, int32_t u, uint32_t* __restrict__ bits) {
  out[p] = u;
  // a no-return atomic OR, with no read before it (of the word, or of the
  // frontier): a read would put a second dependent load on the row's last
  // steps. Ids already in the frontier are marked too; the dedup scan drops them.
  atomicOr(&bits[u >> 5], 1u << (u & 31));
}

// Selection among cnt <= kCandCap candidates held in LDS in ascending j
// (list[i] = key << 32 | j); writes the fo chosen neighbours to out in
// ascending j. One wavefront; element i sits in slot i / 64 of lane i % 64.
__device__ __forceinline__ void select_emit(const uint64_t* list, int cnt, int fo, uint64_t tau,
                                            const int32_t* __restrict__ nb, int32_t* __restrict__ out,
                                            uint32_t* __restrict__ bits) {
  const int lane = lane_id();
  const int S = (cnt + MS_WAVE - 1) / MS_WAVE;  // 1..kCandSlots
  uint32_t key[kCandSlots], pos[kCandSlots];
  bool valid[kCandSlots];
#pragma unroll
  for (int s = 0; s < kCandSlots; ++s) {
    const int idx = s * MS_WAVE + lane;
    valid[s] = s < S && idx < cnt;
    const uint64_t e = valid[s] ? list[idx] : 0ull;
    key[s] = (uint32_t)(e >> 32);
    pos[s] = (uint32_t)e;
  }
  // T = largest x with count(key < x) < fo; every key is below tau
  uint32_t T = 0;
  const uint64_t tm1 = tau - 1;
  const int top = tm1 == 0 ? 0 : 63 - __clzll(tm1);
  for (int b = top; b >= 0; --b) {
    const uint32_t trial = T | (1u << b);
    int c = __popcll(ballot(valid[0] && key[0] < trial));
    // unrolled with static indices (a loop to S would index the arrays
    // dynamically); S is the same in every lane
#pragma unroll
    for (int s = 1; s < kCandSlots; ++s)
      if (s < S) c += __popcll(ballot(valid[s] && key[s] < trial));
    if (c < fo) T = trial;
  }
  int n_lt = 0;
  uint64_t lt[kCandSlots], eq[kCandSlots];
#pragma unroll
  for (int s = 0; s < kCandSlots; ++s) {
    lt[s] = ballot(valid[s] && key[s] < T);
    eq[s] = ballot(valid[s] && key[s] == T);
    n_lt += __popcll(lt[s]);
  }
  const int need = fo - n_lt;
  int eq_before = 0;  // ties in earlier slots (all lanes)
  int p_before = 0;   // selected in earlier slots
#pragma unroll
  for (int s = 0; s < kCandSlots; ++s) {
    const bool is_lt = (lt[s] >> lane) & 1ull, is_eq = (eq[s] >> lane) & 1ull;
    const bool sel = is_lt || (is_eq && eq_before + lanes_below(eq[s]) < need);
    const uint64_t sm = ballot(sel);
    if (sel) emit_id(out, p_before + lanes_below(sm), nb[pos[s]], bits);
    p_before += __popcll(sm);
    eq_before += __popcll(eq[s]);
  }
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Appends to c (at cnt, in ascending j) the candidates (key << 32 | j) among
// the four keys of block q = q0 + lane whose key is <= tm1, stopping at
// kCandCap entries but counting them all. Every lane's four positions exist;
// mn is the smallest of the lane's four keys.
// A row's ~fanout + 3 sqrt(fanout) + 3 candidates are spread over its
// iterations, so an iteration with a candidate usually has one, or a few in
// different lanes: when no lane has two, a lane's candidate is its smallest
// key and its list index the running count plus the candidate lanes below it.
__device__ __forceinline__ void take_block(uint4 k4, uint32_t mn, uint32_t q, uint32_t tm1, uint64_t* c, int& cnt) {
  pin(k4.x);
  pin(k4.y);
  pin(k4.z);
  pin(k4.w);
  const uint64_t m0 = ballot(k4.x <= tm1), m1 = ballot(k4.y <= tm1), m2 = ballot(k4.z <= tm1),
                 m3 = ballot(k4.w <= tm1);
  const uint64_t any = m0 | m1 | m2 | m3;
  if (!any) return;
  const uint64_t bit = 1ull << lane_id();
  const int n_any = __popcll(any);
  if (__popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3) == n_any) {  // one per candidate lane
    if (any & bit) {
      const uint32_t s = (m0 & bit) ? 0u : (m1 & bit) ? 1u : (m2 & bit) ? 2u : 3u;
      const int p = cnt + lanes_below(any);
      if (p < kCandCap) c[p] = ((uint64_t)mn << 32) | (4 * q + s);
    }
    cnt += n_any;
    return;
  }
  // lower lanes first, then s within the lane
  int p = cnt + lanes_below(m0) + lanes_below(m1) + lanes_below(m2) + lanes_below(m3);
  const uint64_t m[4] = {m0, m1, m2, m3};
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if (m[s] & bit) {
      if (p < kCandCap) c[p] = ((uint64_t)word_of(k4, s) << 32) | (4 * q + s);
      ++p;
    }
  cnt += __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
}

__device__ __forceinline__ uint32_t min4(const uint4& w) { return min(min(w.x, w.y), min(w.z, w.w)); }

// Filters 4-position groups [g0, g1) of a row of d positions: appends to c, in
// ascending j, the candidates (key << 32 | j) whose key is <= tm1 (below tau),
// stopping at kCandCap entries but counting them all. One wavefront.
// The usual iteration of a long row has no key below tau, which one test on
// the smallest of each lane's four keys settles. (Two or four Philox blocks
// per lane in flight were measured slower: the loop is bound by VALU issue,
// not by the latency of its dependent multiplies.)
__device__ __forceinline__ int filter_groups(const PhiloxRow& ph, uint32_t g0, uint32_t g1, uint32_t d32,
                                             uint32_t tm1, uint64_t* c) {
  const int lane = lane_id();
  int cnt = 0;
  const uint32_t gf = min(g1, d32 / 4);  // groups below gf are whole
  uint64_t a1 = (uint64_t)0xD2511F53u * (g0 + lane);
  for (uint32_t q0 = g0; q0 < g1; q0 += MS_WAVE, a1 += (uint64_t)0xD2511F53u * MS_WAVE) {
    const uint32_t q = q0 + lane;
    const uint4 wv = ph.from_a1(a1);
    if (q0 + MS_WAVE <= gf) {  // every position of this iteration exists
      const uint32_t mn = min4(wv);
      if (!ballot(mn <= tm1)) continue;
      take_block(wv, mn, q, tm1, c, cnt);
      continue;
    }
    const bool in = q < g1;
    const uint64_t m0 = ballot(in && 4 * q < d32 && wv.x <= tm1);
    const uint64_t m1 = ballot(in && 4 * q + 1 < d32 && wv.y <= tm1);
    const uint64_t m2 = ballot(in && 4 * q + 2 < d32 && wv.z <= tm1);
    const uint64_t m3 = ballot(in && 4 * q + 3 < d32 && wv.w <= tm1);
    if (!(m0 | m1 | m2 | m3)) continue;
    int p = cnt + lanes_below(m0) + lanes_below(m1) + lanes_below(m2) + lanes_below(m3);
    const uint64_t bit = 1ull << lane;
    const uint64_t m[4] = {m0, m1, m2, m3};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (m[s] & bit) {
        if (p < kCandCap) c[p] = ((uint64_t)word_of(wv, s) << 32) | (4 * q + s);
        ++p;
      }
    cnt += __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
  }
  return cnt;
}

// ---- rows of quads: the choice among whole Philox blocks
// A quad is one Philox block: the keys of positions 4q..4q+3. The usual fanouts
// keep few candidates per row, each in a quad of its own, so the filter keeps
// whole quads (no compaction of the single keys: an iteration with a candidate
// costs ~6 vector instructions more than one without, 17 when the candidates
// were picked apart), and the choice is made among the quads' keys in
// registers, one quad per lane and slot.
constexpr uint32_t kShortRow = 4 * MS_WAVE;  // a row of one iteration: its quads never leave the registers

template <int QS>
struct QuadList {
  static constexpr int kCap = QS * MS_WAVE;
  uint4 k[kCap];
  uint32_t q[kCap];
};

// Quads slots a fanout needs so that first thresholds (mu survivors expected)
// hardly ever overflow them: five standard deviations of room; 0: the list of
// single keys.
inline int quad_slots(double mu) {
  const double most = mu + 5.0 * sqrt(mu);
  return most <= MS_WAVE ? 1 : most <= 2 * MS_WAVE ? 2 : 0;
}

// Filters groups [g0, g1) of a row of d positions: appends to l, in ascending
// q, the quads with a key <= tm1 (keys of positions past the row's end count as
// the largest key; the choice drops them), storing at most kCap of them but
// counting them all. One wavefront.
template <int QS>
__device__ __forceinline__ int filter_quads(const PhiloxRow& ph, uint32_t g0, uint32_t g1, uint32_t d32, uint32_t tm1,
                                            QuadList<QS>& l) {
  const int lane = lane_id();
  int n = 0;
  const uint32_t gf = min(g1, d32 / 4);  // groups below gf are whole
  uint64_t a1 = (uint64_t)0xD2511F53u * (g0 + lane);
  for (uint32_t q0 = g0; q0 < g1; q0 += MS_WAVE, a1 += (uint64_t)0xD2511F53u * MS_WAVE) {
    const uint32_t q = q0 + lane;
    uint4 k = ph.from_a1(a1);
    bool has;
    if (q0 + MS_WAVE <= gf) {  // every position of this iteration exists
      has = min4(k) <= tm1;
    } else {
      k.y = 4 * q + 1 < d32 ? k.y : ~0u;
      k.z = 4 * q + 2 < d32 ? k.z : ~0u;
      k.w = 4 * q + 3 < d32 ? k.w : ~0u;
      has = q < g1 && min4(k) <= tm1;
    }
    const uint64_t m = ballot(has);
    if (!m) continue;
    const int p = n + lanes_below(m);
    if (has && p < QuadList<QS>::kCap) {
      l.k[p] = k;
      l.q[p] = q;
    }
    n += __popcll(m);
  }
  return n;
}

// The quads of a lane, as the choice reads them: the keys of positions that do
// not count (past the row's end, above tm1, no quad) are set to the largest
// key, and `valid` has a bit for each that does.
template <int QS>
struct LaneQuads {
  uint4 k[QS];
  uint32_t q[QS];
  uint32_t valid[QS];
  int total;  // valid keys of the wave

  __device__ __forceinline__ void set(int s, bool in, uint4 k4, uint32_t q_, uint32_t d32, uint32_t tm1) {
    q[s] = q_;
    const bool v0 = in && 4 * q_ < d32 && k4.x <= tm1, v1 = in && 4 * q_ + 1 < d32 && k4.y <= tm1;
    const bool v2 = in && 4 * q_ + 2 < d32 && k4.z <= tm1, v3 = in && 4 * q_ + 3 < d32 && k4.w <= tm1;
    k[s] = make_uint4(v0 ? k4.x : ~0u, v1 ? k4.y : ~0u, v2 ? k4.z : ~0u, v3 ? k4.w : ~0u);
    valid[s] = (v0 ? 1u : 0u) | (v1 ? 2u : 0u) | (v2 ? 4u : 0u) | (v3 ? 8u : 0u);
    total += __popcll(ballot(v0)) + __popcll(ballot(v1)) + __popcll(ballot(v2)) + __popcll(ballot(v3));
  }
  __device__ __forceinline__ void read(const QuadList<QS>& l, int n, uint32_t d32, uint32_t tm1) {
    total = 0;
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const int i = s * MS_WAVE + lane_id();
      const bool in = i < n;
      set(s, in, in ? l.k[i] : make_uint4(~0u, ~0u, ~0u, ~0u), in ? l.q[i] : 0u, d32, tm1);
    }
  }
  __device__ __forceinline__ int below(uint32_t x) const {
    int c = 0;
#pragma unroll
    for (int s = 0; s < QS; ++s)
      c += __popcll(ballot(k[s].x < x)) + __popcll(ballot(k[s].y < x)) + __popcll(ballot(k[s].z < x)) +
           __popcll(ballot(k[s].w < x));
    return c;
  }
};

// Chooses the fo smallest (key, j) of total >= fo valid keys, all <= tm1, and
// writes their neighbours to out in ascending j. A bisection looks for a bound
// below which exactly fo keys lie (with n keys about log2(n) + 1 steps: the
// bound only has to fall between the fo-th key and the next), and ends at the
// fo-th key itself where ties leave no such bound; the ties are then taken in
// ascending j.
template <int QS>
__device__ __forceinline__ void choose_quads(const LaneQuads<QS>& c, int fo, uint32_t tm1,
                                             const int32_t* __restrict__ nb, int32_t* __restrict__ out,
                                             uint32_t* __restrict__ bits) {
  uint32_t sel[QS];
  bool exact = c.total == fo;
  uint32_t lo = 0, hi = tm1, x = 0;
  if (!exact) {
    while (lo < hi) {  // fewer than fo keys below lo, more than fo at or below hi
      x = lo + ((hi - lo) >> 1) + 1;
      const int n = c.below(x);
      if (n == fo) {
        exact = true;
        break;
      }
      if (n < fo)
        lo = x;
      else
        hi = x - 1;
    }
    if (!exact) x = lo;
#pragma unroll
    for (int s = 0; s < QS; ++s)
      sel[s] = (c.k[s].x < x ? 1u : 0u) | (c.k[s].y < x ? 2u : 0u) | (c.k[s].z < x ? 4u : 0u) | (c.k[s].w < x ? 8u : 0u);
  } else {
#pragma unroll
    for (int s = 0; s < QS; ++s) sel[s] = c.valid[s];
  }
  if (!exact) {
    int need = fo - c.below(x);
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const uint32_t eq = c.valid[s] & ((c.k[s].x == x ? 1u : 0u) | (c.k[s].y == x ? 2u : 0u) |
                                        (c.k[s].z == x ? 4u : 0u) | (c.k[s].w == x ? 8u : 0u));
      const uint64_t m0 = ballot(eq & 1u), m1 = ballot(eq & 2u), m2 = ballot(eq & 4u), m3 = ballot(eq & 8u);
      int r = lanes_below(m0) + lanes_below(m1) + lanes_below(m2) + lanes_below(m3);
#pragma unroll
      for (int y = 0; y < 4; ++y)
        if (eq & (1u << y)) {
          if (r < need) sel[s] |= 1u << y;
          ++r;
        }
      need -= __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
    }
  }
  int before = 0;
#pragma unroll
  for (int s = 0; s < QS; ++s) {
    const uint64_t m0 = ballot(sel[s] & 1u), m1 = ballot(sel[s] & 2u), m2 = ballot(sel[s] & 4u),
                   m3 = ballot(sel[s] & 8u);
    int p = before + lanes_below(m0) + lanes_below(m1) + lanes_below(m2) + lanes_below(m3);
    for (uint32_t y = sel[s]; y; y &= y - 1, ++p) emit_id(out, p, nb[4 * c.q[s] + __ffs(y) - 1], bits);
    before += __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
  }
}

// LDS of one wave's row.
template <int QS>
struct WaveList {
  QuadList<QS> l;
};
template <>
struct WaveList<0> {
  uint64_t c[kCandCap];
};

// One row by one wavefront: its record r, its offset in the output at. QS:
// quad slots per lane (0: the list of single keys).
template <int QS>
__device__ __forceinline__ void sample_row_wave(const SampleArgs& a, const Row& r, int64_t at, WaveList<QS>& w) {
  const int lane = lane_id();
  const int32_t fo = a.fo;
  const uint32_t d = r.d;
  int32_t* out = a.out + at;
  const int32_t* nb = a.csr_indices + r.start;
  if (d <= (uint32_t)fo) {
    for (uint32_t j = lane; j < d; j += MS_WAVE) emit_id(out, (int)j, nb[j], mark_bits(a));
    return;
  }
  const PhiloxRow ph((uint32_t)r.v, a.t, (uint32_t)a.hop, a.key0, a.key1);
  if (d <= kShortRow && a.tau_iters > 0) {
    // every key of the row is in the wave's registers: no threshold needed
    LaneQuads<1> c;
    c.total = 0;
    c.set(0, true, ph.from_a1((uint64_t)0xD2511F53u * (uint32_t)lane), (uint32_t)lane, d, ~0u);
    choose_quads<1>(c, fo, ~0u, nb, out, mark_bits(a));
    return;
  }
  TauSearch ts;
  ts.tau = first_tau(a.mu32, (int64_t)d);
  bool fail = false;
  for (int iter = 0; iter < a.tau_iters && !fail; ++iter) {
    const uint32_t tm1 = (uint32_t)(ts.tau - 1);
    if constexpr (QS > 0) {
      const int n = filter_quads<QS>(ph, 0, (d + 3) / 4, d, tm1, w.l);
      LaneQuads<QS> c;
      c.total = INT32_MAX;  // more quads than the list holds
      if (n <= QuadList<QS>::kCap) {
        wave_lds_sync();
        c.read(w.l, n, d, tm1);
      }
      if (ts.step(c.total, fo, 4 * QuadList<QS>::kCap, &fail)) {
        choose_quads<QS>(c, fo, tm1, nb, out, mark_bits(a));
        return;
      }
      wave_lds_sync();  // the next pass rewrites the list
    } else {
      const int cnt = filter_groups(ph, 0, (d + 3) / 4, d, tm1, w.c);
      if (ts.step(cnt, fo, kCandCap, &fail)) {
        wave_lds_sync();
        select_emit(w.c, cnt, fo, ts.tau, nb, out, mark_bits(a));
        return;
      }
    }
  }
  if (lane == 0) atomicOr(a.err, 4);
}

// Large frontiers (many rows keep the chip busy): every row one per wave, the
// long ones (the front of the row list) dispatched first, then the others (its
// back). Wave w takes rows w, w + waves, ... of that order: the host bounds the
// grid, as most waves of a grid for the frontier's bound (the size is known on
// the device only) would find no row.
// Workgroups of two waves: a workgroup holds its LDS until its last wave
// ends, and rows of a power-law frontier end at very different times, so
// smaller workgroups keep more waves resident (hop 3 on the papers-sized
// share: 212 us with four waves per workgroup, 199 us with two).
template <int QS>
__global__ __launch_bounds__(kRowWaves* MS_WAVE) void k_sample_waves(SampleArgs a) {
  __shared__ WaveList<QS> list[kRowWaves];
  const int wave = wave_uniform(wave_id());
  const int32_t status = a.sz->status;
  const int64_t nbig = a.sz->n_big[a.hop - 1], n = a.sz->n[a.hop - 1];
  if (status) return;
  clear_flags(a);
  for (int64_t w = (int64_t)blockIdx.x * kRowWaves + wave; w < n; w += (int64_t)gridDim.x * kRowWaves) {
    const int64_t row = wave_uniform((int32_t)a.big_rows[w < nbig ? w : a.row_waves - 1 - (w - nbig)]);
    sample_row_wave<QS>(a, Row(a.rec, row), wave_uniform(a.bptr[row]), list[wave]);
  }
}

// Small frontiers: the long rows one per block, the blocks walking the big
// list; every other row one per wave.
template <int QS>
__global__ __launch_bounds__(kSampleWaves* MS_WAVE) void k_sample_blocks(SampleArgs a) {
  __shared__ WaveList<QS> list[kSampleWaves];
  const int lane = lane_id(), wave = wave_uniform(wave_id());
  const int32_t fo = a.fo;
  if ((int64_t)blockIdx.x >= a.big_blocks) {
    // a row per wave: the step's state and the row's record in one round of
    // loads (rows past the frontier's end have stale records, which are read
    // and dropped)
    const int64_t row = (int64_t)(blockIdx.x - a.big_blocks) * kSampleWaves + wave;
    const int64_t at_row = min(row, a.n_bound - 1);
    const int32_t status = a.sz->status;
    const int64_t n = a.sz->n[a.hop - 1];
    v4r rc = {0, 0, 0, 0};
    int32_t at = 0;
    if (at_row >= 0) {
      rc = a.rec[at_row];
      at = a.bptr[at_row];
    }
    pin(rc);
    pin(at);
    if (status) return;
    clear_flags(a);
    const Row r(rc);
    // rows longer than big_min are taken by the big list
    if (row < n && (int64_t)r.d <= a.big_min) sample_row_wave<QS>(a, r, wave_uniform(at), list[wave]);
    return;
  }
  if (a.sz->status) return;
  clear_flags(a);
  __shared__ WaveList<QS> merged;
  __shared__ int counts[kSampleWaves];
  // long rows, one per block at a time
  const int64_t n_big = a.sz->n_big[a.hop - 1];
  for (int64_t b = blockIdx.x; b < n_big; b += a.big_blocks) {
    const int64_t row = wave_uniform((int32_t)a.big_rows[b]);
    const Row r(a.rec, row);
    const uint32_t d = r.d;  // > big_min >= fo
    int32_t* out = a.out + a.bptr[row];
    const int32_t* nb = a.csr_indices + r.start;
    const PhiloxRow ph((uint32_t)r.v, a.t, (uint32_t)a.hop, a.key0, a.key1);
    // this wave's quarter of the row's groups, in whole wave iterations
    const uint32_t groups = (d + 3) / 4;
    const uint32_t per = (groups + kSampleWaves * MS_WAVE - 1) / (kSampleWaves * MS_WAVE) * MS_WAVE;
    const uint32_t g0 = min(groups, (uint32_t)wave * per), g1 = min(groups, g0 + per);
    TauSearch ts;
    ts.tau = first_tau(a.mu32, (int64_t)d);
    bool fail = false, ok = false;
    for (int iter = 0; iter < a.tau_iters && !ok && !fail; ++iter) {
      const uint32_t tm1 = (uint32_t)(ts.tau - 1);
      int cnt;
      if constexpr (QS > 0)
        cnt = filter_quads<QS>(ph, g0, g1, d, tm1, list[wave].l);
      else
        cnt = filter_groups(ph, g0, g1, d, tm1, list[wave].c);
      if (lane == 0) counts[wave] = cnt;
      __syncthreads();
      int total = 0, before = 0;
      for (int x = 0; x < kSampleWaves; ++x) {
        if (x == wave) before = total;
        total += counts[x];
      }
      // every wave takes the same decision from the same counts; the four
      // lists, in order, are the row's list in ascending j
      if constexpr (QS > 0) {
        constexpr int cap = QuadList<QS>::kCap;
        LaneQuads<QS> c;
        c.total = INT32_MAX;
        if (total <= cap) {
          for (int i = lane; i < cnt; i += MS_WAVE) {
            merged.l.k[before + i] = list[wave].l.k[i];
            merged.l.q[before + i] = list[wave].l.q[i];
          }
          __syncthreads();
          c.read(merged.l, total, d, tm1);
        }
        ok = ts.step(c.total, fo, 4 * cap, &fail);
        if (ok && wave == 0) choose_quads<QS>(c, fo, tm1, nb, out, mark_bits(a));
      } else {
        ok = ts.step(total, fo, kCandCap, &fail);
        if (ok) {
          for (int i = lane; i < cnt; i += MS_WAVE) merged.c[before + i] = list[wave].c[i];
          __syncthreads();
          if (wave == 0) select_emit(merged.c, total, fo, ts.tau, nb, out, mark_bits(a));
        }
      }
      __syncthreads();  // the lists and counts are rewritten by the next pass or row
    }
    if (!ok) {
      if (threadIdx.x == 0) atomicOr(a.err, 4);
      return;  // every wave of the block leaves together
    }
  }
}

// ------------------------------------------------------------ dedup/relabel
// One launch after each hop's sampling: the frontier F_k, and the rows that
// the next hop samples for.
// New nodes in ascending id: F[n_{k-1} + rank] = u, pos_of[u] = that position,
// u the rank-th sampled id not in the frontier (bits & ~seen, the copies of
// bits ored together). `bits` is
// cleared for the next hop; the new nodes join `seen`, which the last hop
// clears for the next step. The new nodes below L (local ids) are the prefix
// at id L: the thread whose words hold id L writes that count (the last tile,
// if every id is below L). (Both bitmaps hold W + 4 words, the last four
// always zero.) For every row of F_k (unless the hop is the last) also its
// record, its offset bptr (prefix of min(deg, fo)) and its place in the row
// list, as in k_seed_rows.
// Tiles: first the rows of F_{k-1}, whose records are there (NT * kFrItems per
// tile), then TW words of the bitmap per tile. A tile publishes its new nodes
// and its sampled positions in one 64-bit word (state << 62 | positions << 31
// | nodes, both below 2^31; the sampling launch before this one cleared it)
// and takes the sums of the tiles before it by look-back, NT tiles at a time.
// A tile's set bits are first spread into LDS, so that consecutive threads
// take consecutive new nodes whatever the bitmap's density: their loads
// (ascending ids) and stores are then coalesced. With one thread walking its
// words instead, a dense bitmap kept one block busy with scattered stores:
// 107K ids, 26K-33K new nodes, 28-34 us a hop, and 9 us for the next hop's
// rows in a launch of their own; 6.5-7.9 us for both here. Of a launch on a
// small frontier (6.2 us) most is the chain of dependent steps: loads,
// look-back, loads.
// Waves per SIMD that the kernel's registers leave room for, by its rows per
// thread (kFrItems).
constexpr int frontier_waves(int items) { return items > 4 ? 4 : 8; }

struct FrontierArgs {
  uint32_t* bits;      // COPIES copies of the sampled-id bitmap
  int64_t copy_words;  // words from one copy to the next
  uint32_t* seen;
  int64_t W;
  int32_t L;
  StepSizes* sz;
  int32_t hop;  // 1-based: the hop just sampled
  uint64_t* flags;
  uint32_t* ticket;  // scan_tile's counter (TICKETS)
  int64_t old_tiles;
  int64_t n_bound;  // bound of n_{hop-1}
  int32_t* nodes;
  int32_t* pos_of;
  // rows of the next hop (not for the last one)
  const int64_t* csr_indptr;
  v4r* rec;
  int32_t fo;
  int32_t* bptr;
  int32_t* big_rows;
  int64_t big_min;
  int64_t small_end;
};

__device__ __forceinline__ uint64_t fr_state(uint32_t st, uint32_t n, uint32_t e) {
  return ((uint64_t)st << 62) | ((uint64_t)e << 31) | n;
}

struct FrSums {
  uint32_t n, e;
};

// Publishes tile b's sums (state 1), waits for the sums of the tiles before it
// and publishes the inclusive ones (state 2). Whole block; the wait is bounded
// as in lookback_exclusive.
template <int NT>
__device__ __forceinline__ FrSums fr_lookback(uint64_t* flags, int64_t b, uint32_t n, uint32_t e, int32_t* status) {
  constexpr int NW = NT / MS_WAVE;
  __shared__ uint32_t w_n[NW], w_e[NW];
  __shared__ int32_t w_st[NW];  // 0: not ready, 1: all aggregates, 2: ends at an inclusive sum
  const int lane = lane_id(), wave = wave_id();
  if (threadIdx.x == 0)
    __hip_atomic_store(&flags[b], fr_state(b == 0 ? 2u : 1u, n, e), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  FrSums x = {0, 0};
  int64_t p = b - 1;  // thread t reads tile p - t
  int spins = 0;
  while (p >= 0) {
    const int64_t i = p - (int64_t)threadIdx.x;
    // before tile 0: an inclusive sum of nothing
    const uint64_t f = i >= 0 ? __hip_atomic_load(&flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                              : fr_state(2u, 0, 0);
    const uint32_t st = (uint32_t)(f >> 62);
    const uint64_t ready = ballot(st != 0), inc = ballot(st == 2u);
    // lanes 0..k count, k = the nearest inclusive sum (or the wave's last tile)
    const int k = inc ? __ffsll((unsigned long long)inc) - 1 : MS_WAVE - 1;
    const uint64_t need = k == MS_WAVE - 1 ? ~0ull : ((2ull << k) - 1);
    const bool ok = (ready & need) == need;
    const uint32_t sn = wave_sum(lane <= k ? (uint32_t)f & 0x7FFFFFFFu : 0u);
    const uint32_t se = wave_sum(lane <= k ? (uint32_t)(f >> 31) & 0x7FFFFFFFu : 0u);
    if (lane == 0) {
      w_n[wave] = sn;
      w_e[wave] = se;
      w_st[wave] = !ok ? 0 : inc ? 2 : 1;
    }
    __syncthreads();
    uint32_t an = 0, ae = 0;
    int st_all = 1;
    for (int w = 0; w < NW && st_all == 1; ++w) {
      st_all = w_st[w];
      if (st_all) {
        an += w_n[w];
        ae += w_e[w];
      }
    }
    __syncthreads();
    if (st_all) {
      x.n += an;
      x.e += ae;
      if (st_all == 2) break;
      p -= NT;
      continue;
    }
    if (++spins > kLookbackSpins) {
      if (threadIdx.x == 0) atomicOr(status, 8);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  if (threadIdx.x == 0 && b > 0)
    __hip_atomic_store(&flags[b], fr_state(2u, x.n + n, x.e + e), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return x;
}

template <int NT, int TW, int kFrItems, bool LAST, int COPIES, bool TICKETS>
__global__ __launch_bounds__(NT, frontier_waves(kFrItems)) void k_frontier(FrontierArgs a) {
  constexpr int kFrNT = NT, kFrWaves = NT / MS_WAVE, kFrChunk = NT * kFrItems;
  constexpr int WPT = TW > NT ? TW / NT : 1;  // words per thread (of the first TW / WPT threads)
  static_assert(WPT == 1 || (WPT == 4 && COPIES == 1), "one word or one 16-byte vector");
  static_assert(kFrItems * kFrWaves <= MS_WAVE, "the waves' sums are scanned by one wave");
  __shared__ int32_t lds[kFrWaves + 1];
  __shared__ int32_t list[kFrChunk];
  __shared__ int32_t wsum[kFrItems * kFrWaves + 1];
  __shared__ int32_t red[2][kFrWaves];
  __shared__ int32_t big_n, small_n;
  __shared__ unsigned long long base_of[2];
  const int lane = lane_id(), wave = wave_id();
  // the step's status and sizes, and the tile's words or row lengths, in one
  // round of loads; with tickets the sizes come under the ticket's round trip,
  // and the kernel's arguments before it
  if constexpr (TICKETS)
    asm volatile("" ::"s"(a.bits), "s"(a.seen), "s"(a.W), "s"(a.L), "s"(a.hop), "s"(a.old_tiles), "s"(a.n_bound),
                 "s"(a.rec), "s"(a.flags), "s"(a.csr_indptr), "s"(a.bptr), "s"(a.nodes), "s"(a.ticket), "s"(a.fo));
  int32_t status = a.sz->status;
  int64_t n_prev = a.sz->n[a.hop - 1];
  const int64_t tile = scan_tile<TICKETS>(a.ticket);
  if constexpr (TICKETS) {
    pin(status);
    pin(n_prev);
  }
  const bool old = tile < a.old_tiles;
  const int64_t row0 = tile * kFrChunk;             // of a tile of old rows
  const int64_t word0 = (tile - a.old_tiles) * TW;  // of a bitmap tile
  const int64_t i0w = word0 + (int64_t)threadIdx.x * WPT;          // this thread's first word
  const bool words = !old && (int)threadIdx.x * WPT < TW && i0w < a.W;
  uint32_t w[WPT], sn[WPT];
  uint32_t d[kFrItems] = {};
#pragma unroll
  for (int x = 0; x < WPT; ++x) w[x] = sn[x] = 0u;
  if (words) {
    if (WPT == 4) {  // (i0w is a multiple of four: aligned, and the padding words cover the last ones)
      const uint4 b4 = *reinterpret_cast<const uint4*>(a.bits + i0w), s4 = *reinterpret_cast<const uint4*>(a.seen + i0w);
      const uint32_t bb[4] = {b4.x, b4.y, b4.z, b4.w}, ss[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
      for (int x = 0; x < WPT; ++x) {
        w[x] = bb[x];
        sn[x] = ss[x];
      }
    } else {
      uint32_t b[COPIES];
#pragma unroll
      for (int x = 0; x < COPIES; ++x) b[x] = a.bits[x * a.copy_words + i0w];
      sn[0] = a.seen[i0w];
#pragma unroll
      for (int x = 0; x < COPIES; ++x) w[0] |= b[x];
    }
  }
  if (!LAST && old) {
#pragma unroll
    for (int it = 0; it < kFrItems; ++it) d[it] = a.rec[min(row0 + it * kFrNT + threadIdx.x, a.n_bound - 1)].y;
  }
#pragma unroll
  for (int x = 0; x < WPT; ++x) {
    pin(w[x]);
    pin(sn[x]);
  }
  if (!LAST) {
#pragma unroll
    for (int it = 0; it < kFrItems; ++it) pin(d[it]);
  }
  if (status) return;
  int32_t ex = 0, tot = 0, below = -1;
  if (old) {
    tot = (int32_t)min(max(n_prev - row0, (int64_t)0), (int64_t)kFrChunk);
  } else {
    int32_t mine = 0;
#pragma unroll
    for (int x = 0; x < WPT; ++x) {
      const uint32_t b = w[x];
      w[x] = b & ~sn[x];
      mine += __popc(w[x]);
      if (b) {
#pragma unroll
        for (int y = 0; y < COPIES; ++y) a.bits[y * a.copy_words + i0w + x] = 0u;
      }
      if (LAST) {
        if (sn[x]) a.seen[i0w + x] = 0u;
      } else if (w[x]) {
        a.seen[i0w + x] = sn[x] | w[x];
      }
    }
    ex = block_exclusive_scan<kFrNT>(mine, lds, &tot);
    const int64_t wL = (int64_t)(a.L >> 5);
    if (words && wL < a.W && wL >= i0w && wL < i0w + WPT) {
      below = ex;
#pragma unroll
      for (int x = 0; x < WPT; ++x) {
        if (i0w + x < wL) below += __popc(w[x]);
        else if (i0w + x == wL) below += __popc(w[x] & ((1u << (a.L & 31)) - 1u));
      }
    }
  }
  const int64_t id0 = word0 << 5;
  int32_t u[kFrItems] = {};
  int64_t lo[kFrItems] = {}, hi[kFrItems] = {};
  // items c0 + it * kFrNT + thread of the tile: their nodes and row lengths
  auto load = [&](int32_t c0) {
    const int32_t m = min(tot - c0, kFrChunk);
    if (old) return;  // (one chunk: its row lengths were loaded above)
    __syncthreads();
    int32_t o = ex;
#pragma unroll
    for (int x = 0; x < WPT; ++x)
      for (uint32_t y = w[x]; y; y &= y - 1) {
        if (o >= c0 && o < c0 + kFrChunk) list[o - c0] = (int32_t)((threadIdx.x * WPT + x) * 32 + __ffs(y) - 1);
        ++o;
      }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kFrItems; ++it) {
      const int32_t j = it * kFrNT + threadIdx.x;
      u[it] = (int32_t)id0 + list[j < m ? j : 0];
    }
    if (LAST) return;
#pragma unroll
    for (int it = 0; it < kFrItems; ++it)
      if (it * kFrNT < m) {  // the same in every lane
        lo[it] = a.csr_indptr[u[it]];
        hi[it] = a.csr_indptr[u[it] + 1];
      }
#pragma unroll
    for (int it = 0; it < kFrItems; ++it) {
      pin(lo[it]);
      pin(hi[it]);
      d[it] = (uint32_t)(hi[it] - lo[it]);
    }
  };
  // the tile's sampled positions and long rows
  int32_t sum_e = 0, n_big = 0;
  if (!LAST) {
    for (int32_t c0 = 0; c0 < tot; c0 += kFrChunk) {
      load(c0);
#pragma unroll
      for (int it = 0; it < kFrItems; ++it)
        if (c0 + it * kFrNT + (int32_t)threadIdx.x < tot) {
          sum_e += d[it] < (uint32_t)a.fo ? (int32_t)d[it] : a.fo;
          n_big += (int64_t)d[it] > a.big_min;
        }
    }
    sum_e = wave_sum(sum_e);
    n_big = wave_sum(n_big);
    if (lane == 0) {
      red[0][wave] = sum_e;
      red[1][wave] = n_big;
    }
    if (threadIdx.x == 0) big_n = small_n = 0;
    __syncthreads();
    sum_e = n_big = 0;
    for (int x = 0; x < kFrWaves; ++x) {
      sum_e += red[0][x];
      n_big += red[1][x];
    }
    // (issued before the look-back, whose wait covers their latency)
    if (threadIdx.x == 0) {
      base_of[0] = n_big ? atomicAdd((unsigned long long*)&a.sz->n_big[a.hop], (unsigned long long)n_big) : 0ull;
      base_of[1] = a.small_end && tot > n_big
                       ? atomicAdd((unsigned long long*)&a.sz->n_small[a.hop], (unsigned long long)(tot - n_big))
                       : 0ull;
    }
  }
  const FrSums before = fr_lookback<NT>(a.flags, tile, old ? 0u : (uint32_t)tot, (uint32_t)sum_e, &a.sz->status);
  if (below >= 0) a.sz->n_local_new[a.hop - 1] = (int64_t)before.n + below;
  if (threadIdx.x == 0) {
    if (tile == gridDim.x - 1) {
      a.sz->n[a.hop] = n_prev + before.n + (old ? 0 : tot);
      if (!LAST) a.sz->e[a.hop] = (int64_t)before.e + sum_e;
      if ((int64_t)(a.L >> 5) >= a.W) a.sz->n_local_new[a.hop - 1] = (int64_t)before.n + tot;  // every id is below L
    }
    if (!LAST && tile == 0) a.bptr[0] = 0;
  }
  const int64_t i0 = old ? row0 : n_prev + before.n;  // frontier row of item 0
  __syncthreads();  // (base_of)
  int64_t run = before.e;
  for (int32_t c0 = 0; c0 < tot; c0 += kFrChunk) {
    if (LAST || tot > kFrChunk) load(c0);  // (a tile of one chunk still holds it)
    int32_t c[kFrItems], inc[kFrItems];
    if (!LAST) {
      __syncthreads();
#pragma unroll
      for (int it = 0; it < kFrItems; ++it) {
        const bool in = c0 + it * kFrNT + (int32_t)threadIdx.x < tot;
        c[it] = !in ? 0 : d[it] < (uint32_t)a.fo ? (int32_t)d[it] : a.fo;
        inc[it] = 0;
        if (c0 + it * kFrNT < tot) inc[it] = wave_inclusive_scan(c[it]);  // (the same in every lane)
        if (lane == MS_WAVE - 1) wsum[it * kFrWaves + wave] = inc[it];
      }
      __syncthreads();
      if (wave == 0) {
        const int32_t x = lane < kFrItems * kFrWaves ? wsum[lane] : 0;
        const int32_t y = wave_inclusive_scan(x);
        if (lane < kFrItems * kFrWaves) wsum[lane] = y - x;
        if (lane == kFrItems * kFrWaves - 1) wsum[kFrItems * kFrWaves] = y;
      }
      __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < kFrItems; ++it) {
      const int32_t j = c0 + it * kFrNT + (int32_t)threadIdx.x;
      const bool in = j < tot;
      const int64_t i = i0 + j;
      if (c0 + it * kFrNT >= tot) break;
      if (in && !old) {
        a.nodes[i] = u[it];
        a.pos_of[u[it]] = (int32_t)i;
        if (!LAST) a.rec[i] = row_record(u[it], lo[it], d[it]);
      }
      if (!LAST) {
        if (in) a.bptr[i + 1] = (int32_t)(run + wsum[it * kFrWaves + wave] + inc[it]);
        const bool big = in && (int64_t)d[it] > a.big_min, small = in && !big && a.small_end;
        const uint64_t mb = ballot(big), ms = ballot(small);
        if (mb) {
          int32_t at = 0;
          if (lane == 0) at = atomicAdd(&big_n, __popcll(mb));
          at = __shfl(at, 0, MS_WAVE);
          if (big) a.big_rows[base_of[0] + at + lanes_below(mb)] = (int32_t)i;
        }
        if (ms) {
          int32_t at = 0;
          if (lane == 0) at = atomicAdd(&small_n, __popcll(ms));
          at = __shfl(at, 0, MS_WAVE);
          if (small) a.big_rows[a.small_end - 1 - (int64_t)(base_of[1] + at + lanes_below(ms))] = (int32_t)i;
        }
      }
    }
    if (!LAST) run += wsum[kFrItems * kFrWaves];
  }
}

// Sampled ids to their frontier positions: NT threads x kRelItems ids per
// block and pass, block b of the hop's nblocks striding over them; every load
// of a thread is issued before the first is used (the first pass's together
// with the hop's size: the array holds e_bound ids), and lanes past the end
// store nothing.
constexpr int kRelItems = 4;
template <int NT>
__device__ __forceinline__ void relabel_hop(int32_t* __restrict__ ids, const StepSizes* sz, int hop, int64_t e_bound,
                                            const int32_t* __restrict__ pos_of, int64_t b, int64_t nblocks) {
  const int32_t status = sz->status;
  const int64_t e = sz->e[hop - 1];
  for (int64_t b0 = b * NT * kRelItems; b0 < e_bound; b0 += nblocks * NT * kRelItems) {
    int32_t u[kRelItems], p[kRelItems];
#pragma unroll
    for (int it = 0; it < kRelItems; ++it) u[it] = ids[min(b0 + (int64_t)it * NT + threadIdx.x, e_bound - 1)];
#pragma unroll
    for (int it = 0; it < kRelItems; ++it) pin(u[it]);
    if (status || b0 >= e) return;
#pragma unroll
    for (int it = 0; it < kRelItems; ++it) {
      const int64_t i = b0 + (int64_t)it * NT + threadIdx.x;
      p[it] = pos_of[i < e ? u[it] : 0];
    }
#pragma unroll
    for (int it = 0; it < kRelItems; ++it) pin(p[it]);
#pragma unroll
    for (int it = 0; it < kRelItems; ++it) {
      const int64_t i = b0 + (int64_t)it * NT + threadIdx.x;
      if (i < e) ids[i] = p[it];
    }
  }
}

}  // namespace ms

// common.hpp - device utilities for libmassive (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define MS_WAVE 64

namespace ms {

__device__ __forceinline__ int lane_id() { return threadIdx.x & (MS_WAVE - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x / MS_WAVE; }

// number of set bits of `mask` in lanes below this one
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// A value the caller knows to be the same in every lane of the wave, moved to
// a scalar register, so that branches on it are scalar and loads through it
// are scalar loads.
__device__ __forceinline__ int32_t wave_uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t wave_uniform(int64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)x);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// x of the lane that a data-parallel-primitive control names, 0 in the lanes
// that it leaves out (and in rows outside the row mask).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}

// Inclusive prefix sum over the 64 lanes of a wave. 32-bit sums go through DPP
// moves (shifts within a row of 16 lanes, then the last lane of each row
// broadcast to the rows after it), which a following add takes in a few
// cycles; a shuffle goes through the LDS unit, and a chain of six cost ~0.25 us
// in the latency-bound kernels that scan.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
  if constexpr (sizeof(T) == 4) {
    uint32_t v = (uint32_t)x;
    v += dpp<0x111, 0xF>(v);  // row_shr:1
    v += dpp<0x112, 0xF>(v);  // row_shr:2
    v += dpp<0x114, 0xF>(v);  // row_shr:4
    v += dpp<0x118, 0xF>(v);  // row_shr:8
    v += dpp<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return (T)v;
  }
  const int lane = lane_id();
#pragma unroll
  for (int o = 1; o < MS_WAVE; o <<= 1) {
    T y = __shfl_up(x, o, MS_WAVE);
    if (lane >= o) x += y;
  }
  return x;
}

// Keeps a loaded value where it is: an empty asm that reads and writes it.
// Loads whose values are only used under a per-lane condition are otherwise
// sunk by the compiler into that condition, each behind its own wait, so the
// loads of a thread would be issued one at a time.
template <typename T>
__device__ __forceinline__ void pin(T& x) {
  asm volatile("" : "+v"(x));
}

// Sum over the wave's lanes, the same in every lane.
template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
  if constexpr (sizeof(T) == 4) return (T)__builtin_amdgcn_readlane((int)wave_inclusive_scan(x), MS_WAVE - 1);
#pragma unroll
  for (int o = MS_WAVE / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, MS_WAVE);
  return x;
}

// Exclusive prefix sum over a block of NT threads; lds needs NT/64 + 1 slots.
// Returns this thread's exclusive prefix; *total gets the block sum.
template <int NT, typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* lds, T* total) {
  constexpr int NW = NT / MS_WAVE;
  const int lane = lane_id(), wave = wave_id();
  T x = wave_inclusive_scan(v);
  if (lane == MS_WAVE - 1) lds[wave] = x;
  __syncthreads();
  if (wave == 0) {
    T w = lane < NW ? lds[lane] : T(0);
    T wi = wave_inclusive_scan(w);
    if (lane < NW) lds[lane] = wi - w;
    if (lane == NW - 1) lds[NW] = wi;
  }
  __syncthreads();
  T res = lds[wave] + x - v;
  *total = lds[NW];
  __syncthreads();
  return res;
}

// a ^ b ^ key in one instruction: gfx950's three-input bitwise operation
// (truth table 0x96 = XOR of all three); key is wave-uniform (an SGPR, the
// one scalar operand the instruction may take).
__device__ __forceinline__ uint32_t xor3_key(uint32_t a, uint32_t b, uint32_t key) {
  uint32_t r;
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(key));
  return r;
}

__device__ __forceinline__ uint32_t word_of(const uint4& w, int s) {
  return s == 0 ? w.x : (s == 1 ? w.y : (s == 2 ? w.z : w.w));
}

// Device-side sizes of the current step (one struct in HBM per context).
struct StepSizes {
  int64_t n[9];      // frontier sizes n_0..n_K
  int64_t e[8];      // sampled edges per hop
  int64_t local, hits, misses;
  int64_t n_hbm, n_miss;  // lengths of the two gather lists
  int64_t n_big[8];       // rows longer than the big-row threshold, per hop
  int64_t n_small[8];     // the other rows, when they are listed too (one-wave-per-row sampler)
  int64_t n_local_new[8]; // new frontier nodes below L (local), per hop
  int64_t n_pending;      // hits on slots still refilling (read over the host link)
  int32_t status;    // != 0: invalid seeds; later kernels of the step skip
  int32_t blocks_done;  // blocks of the step's miss gather that have finished
};

// Eviction-round device scalars.
struct RoundState {
  int64_t nE, nC;          // |E|, |C|
  int64_t k;               // k' = min(|E|, |C|)
  int64_t need;            // ties at the threshold still to take
  uint32_t prefix, pmask;  // radix-select prefix of the threshold key (S_A word)
  uint32_t prefix_lo, pmask_lo;  // ... and of its rank word (scores by global id)
  int64_t n_lt;            // candidates strictly before the threshold
  int64_t nE_sel, k_sel;   // |E| and k' when k' < |E| (E must be narrowed), else 0
  int32_t done, pad;       // blocks of the current select pass that have added their bins
};

// Totals over the context's life (device side).
struct Counters {
  int64_t rounds;          // rounds that evicted at least one slot
  int64_t evicted;         // slots evicted (= rows refilled)
  int32_t bad;             // some round produced inconsistent indices (never expected)
  int32_t pad;
  int64_t refilled;        // rows the refill copied over the host link (slots
                           // written through by a miss gather are not copied)
};

}  // namespace ms

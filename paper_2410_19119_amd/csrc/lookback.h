// Prefix sums across the workgroups of one launch (single-pass scan with
// decoupled look-back, Merrill and Garland 2016): every workgroup publishes
// its tile's total, reads the totals of the tiles before it until it meets one
// whose inclusive prefix is known, and publishes its own.
//
// Tiles are taken from a counter, so a tile's predecessors have all been
// started, and none of them waits before it has published its total: every
// wait ends. A published word carries value and state together, is written
// and read by relaxed atomics at device scope (coherent across the XCDs'
// L2s), and names the launch it belongs to, so that one zeroed array serves
// all launches of a call without being cleared in between.
#pragma once

#include "lp_device.h"

namespace lp {

// [31:0] value, [34:33] 1 = tile total, 2 = inclusive prefix, [63:35] launch
struct LookArgs {
  uint64_t* words;
  uint32_t* ticket;  // zero between launches
  uint32_t launch;   // >= 1, a new one for every launch that uses `words`
};

constexpr uint32_t kLookTotal = 1, kLookPrefix = 2;

__device__ __forceinline__ uint64_t look_word(uint32_t launch, uint32_t state, uint32_t v) {
  return ((uint64_t)(launch & 0x1FFFFFFFu) << 35) | ((uint64_t)state << 33) | v;
}
__device__ __forceinline__ void look_put(uint64_t* p, uint64_t w) {
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t look_get(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// State of a word of this launch, 0 when it has not been published yet.
__device__ __forceinline__ uint32_t look_state(uint64_t w, uint32_t launch) {
  return (uint32_t)(w >> 35) == (launch & 0x1FFFFFFFu) ? (uint32_t)(w >> 33) & 3u : 0u;
}

// The workgroup's tile among `tiles` (called by exactly that many workgroups
// of the launch); `sm` is one word of LDS. The last one resets the counter.
__device__ __forceinline__ uint32_t look_ticket(const LookArgs& a, uint32_t tiles, uint32_t* sm) {
  if (threadIdx.x == 0) {
    const uint32_t t = atomicAdd(a.ticket, 1u);
    if (t + 1 == tiles) __hip_atomic_store(a.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *sm = t;
  }
  __syncthreads();
  return *sm;
}

// Predecessors a lane reads at a time: a wavefront then moves on by 256 tiles
// per round trip to memory, which is what a launch of many small tiles waits
// for.
constexpr int kLookPer = 4;

// Which of a lane's kLookPer predecessors (nearest first, states st) count
// towards its sum, and what the wavefront learns: the lane whose predecessors
// end the walk (-1: none), or that one of those needed is still open.
struct LookStep {
  int use;   // this lane adds its first `use` words
  int stop;  // lane that ends the walk, -1: go on
  bool wait;
};
__device__ __forceinline__ LookStep look_step(const uint32_t (&st)[kLookPer]) {
  int use = kLookPer;
  bool known = false, open = false;
#pragma unroll
  for (int k = 0; k < kLookPer; ++k) {
    if (known || open) continue;
    if (st[k] == 0) open = true;
    else if (st[k] == kLookPrefix) {
      known = true;
      use = k + 1;
    }
  }
  const uint64_t mk = __ballot(known), mo = __ballot(open);
  LookStep r;
  r.stop = mk ? __ffsll((unsigned long long)mk) - 1 : -1;
  const uint64_t upto = r.stop < 0 || r.stop == kWave - 1 ? ~0ull : (1ull << (r.stop + 1)) - 1ull;
  r.wait = (mo & upto) != 0;
  r.use = r.stop >= 0 && lane_id() > r.stop ? 0 : use;
  return r;
}

// Sum of the tiles before `tile`, publishing this tile's total and prefix;
// called by one whole wavefront.
__device__ __forceinline__ uint32_t look_sum(const LookArgs& a, uint32_t tile, uint32_t total) {
  const int lane = lane_id();
  if (lane == 0) look_put(&a.words[tile], look_word(a.launch, tile ? kLookTotal : kLookPrefix, total));
  uint32_t sum = 0;
  for (int64_t at = (int64_t)tile - 1; at >= 0;) {
    uint64_t w[kLookPer];
    uint32_t st[kLookPer];
#pragma unroll
    for (int k = 0; k < kLookPer; ++k) {
      const int64_t t = at - lane * kLookPer - k;
      w[k] = t >= 0 ? look_get(&a.words[t]) : look_word(a.launch, kLookPrefix, 0);
    }
#pragma unroll
    for (int k = 0; k < kLookPer; ++k) st[k] = look_state(w[k], a.launch);
    const LookStep ls = look_step(st);
    if (ls.wait) {
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    uint32_t v = 0;
#pragma unroll
    for (int k = 0; k < kLookPer; ++k)
      if (k < ls.use) v += (uint32_t)w[k];
    sum += wave_reduce_add<uint32_t>(v);
    if (ls.stop >= 0) break;
    at -= kWave * kLookPer;
  }
  if (lane == 0 && tile) look_put(&a.words[tile], look_word(a.launch, kLookPrefix, sum + total));
  return sum;
}

// Segmented: the running 64-bit sum that reaches `tile` from the tiles before
// it, given whether a segment starts in this tile and the sum after its last
// start (the whole tile's if none). Two words per tile hold the halves.
__device__ __forceinline__ int64_t look_seg_sum(const LookArgs& a, uint32_t tile, uint32_t seg, int64_t tail) {
  const int lane = lane_id();
  const uint32_t mine = tile == 0 || seg ? kLookPrefix : kLookTotal;
  if (lane < 2)
    look_put(&a.words[2 * (uint64_t)tile + lane],
             look_word(a.launch, mine, (uint32_t)((uint64_t)tail >> (32 * lane))));
  uint64_t sum = 0;
  for (int64_t at = (int64_t)tile - 1; at >= 0;) {
    uint64_t lo[kLookPer], hi[kLookPer];
    uint32_t st[kLookPer];
#pragma unroll
    for (int k = 0; k < kLookPer; ++k) {
      const int64_t t = at - lane * kLookPer - k;
      lo[k] = hi[k] = look_word(a.launch, kLookPrefix, 0);
      if (t >= 0) {
        lo[k] = look_get(&a.words[2 * t]);
        hi[k] = look_get(&a.words[2 * t + 1]);
      }
    }
#pragma unroll
    for (int k = 0; k < kLookPer; ++k) {  // both halves of the same publication
      const uint32_t sl = look_state(lo[k], a.launch), sh = look_state(hi[k], a.launch);
      st[k] = sl == sh ? sl : 0u;
    }
    const LookStep ls = look_step(st);
    if (ls.wait) {
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    uint64_t v = 0;
#pragma unroll
    for (int k = 0; k < kLookPer; ++k)
      if (k < ls.use) v += (hi[k] << 32) | (lo[k] & 0xFFFFFFFFull);
    sum += wave_reduce_add<uint64_t>(v);
    if (ls.stop >= 0) break;
    at -= kWave * kLookPer;
  }
  if (mine == kLookTotal && lane < 2)
    look_put(&a.words[2 * (uint64_t)tile + lane],
             look_word(a.launch, kLookPrefix, (uint32_t)((sum + (uint64_t)tail) >> (32 * lane))));
  return (int64_t)sum;
}

}  // namespace lp

// Host-side launchers of the device-wide primitives (prims.hip) and the
// scratch-memory helper used by every entry point.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "lp_common.h"

namespace lp {

// Reports a failed HIP call on stderr when LPGPU_DEBUG is set in the
// environment, then maps it to a status code.
lp_status hip_fail(hipError_t e, const char* what, const char* file, int line);

// Clears a pending error left by earlier runtime calls of the caller, so that
// launch checks only see this library's errors.
inline void clear_error() { (void)hipGetLastError(); }

// The library's device-memory cache (one per device). A block released on
// stream s is kept and handed out again: to work on s at once (stream order
// puts the new use after the old one), to another stream once the event
// recorded at the release has completed. Steady-state calls therefore make no
// HIP allocation and never wait for the allocator. cache_alloc returns
// nullptr when the device is out of memory even after the cache was emptied.
void* cache_alloc(size_t bytes, hipStream_t s);
void cache_free(void* p, hipStream_t s);
// Frees every cached block (also of handle_alloc) of every device (waits for each device first).
void cache_trim_all();
// Buffers of handles that are not ordered with a stream (lp_compress,
// lp_graph_from_csr) and of their plans, on the current device. A block is
// given back once the device is idle and up to kHandlePool bytes of them are
// kept per device for later handles, blocks of at most half of that each:
// mapping and unmapping such memory costs more than the work on it
// (compressing an R-MAT graph of 2.4e8 entries takes 1.5 ms on the device; a
// pass that mapped and unmapped its 0.6 GB took 2.9 to 16.7 ms).
constexpr size_t kHandlePool = (size_t)2 << 30;
void* handle_alloc(size_t bytes);
void handle_free(void* p);  // the device that p is on has no work left that uses p
// The caller's allocator for all later cache_alloc calls (nullptr: the cache).
lp_status set_allocator(const lp_allocator* a);
// Bytes of the current device handed out and kept by the cache, and bytes
// handed out by the caller's allocator (all devices).
void memory_info(uint64_t* live, uint64_t* cached, uint64_t* external);

// Stream-ordered scratch allocations from the cache, released (on the same
// stream) when the object goes out of scope. A failed allocation sets
// `failed`.
class Scratch {
 public:
  explicit Scratch(hipStream_t s) : stream_(s) {}
  ~Scratch() {
    for (void* p : ptrs_) cache_free(p, stream_);
  }
  template <typename T>
  T* alloc(size_t count) {
    const size_t bytes = (count ? count : 1) * sizeof(T);
    void* p = cache_alloc(bytes, stream_);
    if (!p) {
      (void)hip_fail(hipErrorOutOfMemory, "cache_alloc", __FILE__, __LINE__);
      failed = true;
      return nullptr;
    }
    ptrs_.push_back(p);
    return static_cast<T*>(p);
  }
  hipStream_t stream() const { return stream_; }
  bool failed = false;

 private:
  hipStream_t stream_;
  std::vector<void*> ptrs_;
};

// Exclusive prefix sum of in[0..n) into out[0..n); *total_dev (if not null)
// receives the sum of all n inputs. out may alias in.
lp_status scan_exclusive_u64(const uint64_t* in, uint64_t* out, int64_t n, uint64_t* total_dev,
                             Scratch& sc);
lp_status scan_exclusive_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total_dev,
                             Scratch& sc);

// Stable LSD radix sort of (key, val) pairs, at most max_n of them (their
// number is *count_dev), on key bits [0, bits). The pairs start in buffers 0;
// which of the two buffer sets holds the result is known on the device only
// (*sel), since passes whose digit is the same in all keys are left out.
struct SortedPairs {
  uint64_t* k[2] = {nullptr, nullptr};
  uint32_t* v[2] = {nullptr, nullptr};
  const uint32_t* sel = nullptr;
};
struct SortPlan;
class PairSorter {
 public:
  // Device memory of one sorter from `sc`; `zero` words of it, starting at
  // zero_base(), must be cleared before the first sort (zeroed by the caller
  // together with its own).
  lp_status init(uint64_t* keys_a, uint32_t* vals_a, uint64_t* keys_b, uint32_t* vals_b, int64_t max_n, int bits,
                 Scratch& sc);
  uint32_t* zero_base() const { return zero_; }
  int64_t zero_words() const { return zero_words_; }
  // One sort of the pairs in buffers 0 on the scratch stream of init.
  lp_status sort(const uint32_t* count_dev);
  const SortedPairs& out() const { return out_; }

 private:
  SortedPairs out_;
  SortPlan* plan_ = nullptr;
  uint64_t* words_ = nullptr;
  uint32_t* zero_ = nullptr;
  int64_t zero_words_ = 0, max_n_ = 0;
  int passes_ = 0, which_ = 0;
  uint32_t launch_ = 0;
  hipStream_t stream_ = nullptr;
};

// Clears n 32-bit words (a kernel, so that it can be captured).
lp_status zero_u32(uint32_t* p, int64_t n, hipStream_t s);

#define last_error() ::lp::hip_fail(hipGetLastError(), "kernel launch", __FILE__, __LINE__)

// Workgroups for `items` of which one takes per_block. Only kernels that loop
// may be given a cap: most of the lists that a kernel walks with one item per
// thread reach the number of vertices, 2^31 - 1.
inline unsigned grid_for(int64_t items, int per_block, unsigned cap = 0x7FFFFFFF) {
  int64_t b = (items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > (int64_t)cap) b = cap;
  return (unsigned)b;
}

#define LP_CHECK_HIP(call)                                            \
  do {                                                                \
    hipError_t e_ = (call);                                           \
    if (e_ != hipSuccess) {                                           \
      (void)hipGetLastError();                                        \
      return ::lp::hip_fail(e_, #call, __FILE__, __LINE__);           \
    }                                                                 \
  } while (0)

#define LP_CHECK(st)                  \
  do {                                \
    lp_status s_ = (st);              \
    if (s_ != LP_OK) return s_;       \
  } while (0)

#define LP_CHECK_LAUNCH() LP_CHECK(last_error())

// One workgroup of `threads` per item of [0, count): launch(first, grid) starts
// the workgroups of items first .. first + grid - 1. One launch unless count *
// threads reaches 2^32 threads, which HIP does not launch at once.
template <typename L>
lp_status launch_sliced(int64_t count, int threads, L&& launch) {
  const int64_t most = 0xFFFFFFFFll / threads;
  for (int64_t first = 0; first < count; first += most) {
    launch(first, dim3((unsigned)(count - first < most ? count - first : most)));
    LP_CHECK_LAUNCH();
  }
  return LP_OK;
}

}  // namespace lp

#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <unordered_map>
#include <utility>
#include <vector>

// Device-wide primitives written for wave64 / gfx950: reduce-then-scan prefix
// sums and a stable LSD radix sort of (key, value) pairs with 8-bit digits.
// The LP acceptance step and contraction use them.
#include "lookback.h"
#include "lp_device.h"
#include "prims.h"

namespace lp {

lp_status hip_fail(hipError_t e, const char* what, const char* file, int line) {
  if (e == hipSuccess) return LP_OK;
  static const bool debug = getenv("LPGPU_DEBUG") != nullptr;
  if (debug) fprintf(stderr, "[lpgpu] %s failed at %s:%d: %s\n", what, file, line, hipGetErrorString(e));
  return e == hipErrorOutOfMemory ? LP_ENOMEM : LP_EDEVICE;
}

// ----------------------------------------------------------- memory cache --
namespace {

struct CBlock {
  void* p;
  hipStream_t s;   // stream of the release
  hipEvent_t ev;   // recorded on s at the release
};

struct DevCache {
  std::mutex mu;
  std::multimap<size_t, CBlock> free_;    // by size
  std::unordered_map<void*, size_t> live;  // handed-out blocks
  std::vector<hipEvent_t> spare;           // events of reused blocks
  size_t cached = 0, limit = 0, live_bytes = 0;
};

constexpr int kCacheDevices = 64;

DevCache* cache_of(int* dev_out) {
  static DevCache caches[kCacheDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kCacheDevices) {
    clear_error();
    return nullptr;
  }
  if (dev_out) *dev_out = dev;
  return &caches[dev];
}

// LPGPU_CACHE_LOG set: every HIP allocation and release of the cache is
// reported on stderr.
bool cache_log() {
  static const bool on = getenv("LPGPU_CACHE_LOG") != nullptr;
  return on;
}

// Sizes are rounded up to eight classes per power of two (at least 512
// bytes), so a block serves later requests of the same class.
size_t size_class(size_t b) {
  if (b <= 512) return 512;
  const int e = 63 - __builtin_clzll((unsigned long long)(b - 1));  // 2^e < b <= 2^(e+1)
  const size_t step = (size_t)1 << (e - 3);
  return (b + step - 1) / step * step;
}

// Frees cached blocks (largest first) whose release has completed until at
// most `keep` bytes stay cached. Caller holds c.mu.
void trim_locked(DevCache& c, size_t keep) {
  for (auto it = c.free_.end(); c.cached > keep && it != c.free_.begin();) {
    --it;
    if (hipEventQuery(it->second.ev) != hipSuccess) continue;
    if (cache_log()) fprintf(stderr, "[lpgpu-cache] hipFree %zu (cached %zu)\n", it->first, c.cached);
    (void)hipFree(it->second.p);
    (void)hipEventDestroy(it->second.ev);
    c.cached -= it->first;
    it = c.free_.erase(it);
  }
  clear_error();
}

// Buffers of handles (handle_alloc): idle blocks by size, and the device and
// size of every block handed out.
struct HandlePool {
  std::mutex mu;
  std::multimap<size_t, void*> idle[kCacheDevices];
  std::unordered_map<void*, std::pair<size_t, int>> live;
  size_t cached[kCacheDevices] = {};
};

HandlePool& handle_pool() {
  static HandlePool* const pool = new HandlePool();  // outlives every handle
  return *pool;
}

// Frees idle handle blocks of a device (largest first) until at most `keep`
// bytes of them are left. Caller holds the pool's lock.
void handle_trim_locked(HandlePool& hp, int dev, size_t keep) {
  auto& f = hp.idle[dev];
  while (hp.cached[dev] > keep && !f.empty()) {
    auto it = std::prev(f.end());
    (void)hipFree(it->second);
    hp.cached[dev] -= it->first;
    f.erase(it);
  }
  clear_error();
}

// Frees every idle handle block of the current device; false if there was none.
bool handle_trim_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kCacheDevices) {
    clear_error();
    return false;
  }
  HandlePool& hp = handle_pool();
  std::lock_guard<std::mutex> lock(hp.mu);
  const bool any = hp.cached[dev] > 0;
  handle_trim_locked(hp, dev, 0);
  return any;
}

// The caller's allocator (lp_set_allocator): when set, every scratch block
// and every buffer of a handle made inside a call comes from it. Blocks keep
// the allocator that made them, so switching allocators never mixes them up.
// The caller's functions are called without any lock of the library held.
struct ExtBlock {
  size_t bytes;
  lp_allocator a;
};
std::mutex g_ext_mu;
lp_allocator g_ext{};
bool g_ext_on = false;
std::unordered_map<void*, ExtBlock> g_ext_live;
uint64_t g_ext_bytes = 0;

}  // namespace

void* cache_alloc(size_t bytes, hipStream_t s) {
  lp_allocator a{};
  bool ext = false;
  {
    std::lock_guard<std::mutex> lock(g_ext_mu);
    ext = g_ext_on;
    a = g_ext;
  }
  if (ext) {
    void* p = a.alloc(bytes ? bytes : 1, (void*)s, a.ctx);
    // out of memory: what freed handles left behind is the device's, not this allocator's
    if (!p && handle_trim_device()) p = a.alloc(bytes ? bytes : 1, (void*)s, a.ctx);
    if (!p) return nullptr;
    std::lock_guard<std::mutex> lock(g_ext_mu);
    g_ext_live[p] = ExtBlock{bytes, a};
    g_ext_bytes += bytes;
    return p;
  }
  DevCache* c = cache_of(nullptr);
  if (!c) return nullptr;
  const size_t need = size_class(bytes);
  std::lock_guard<std::mutex> lock(c->mu);
  if (!c->limit) {
    size_t fr = 0, tot = 0;
    if (hipMemGetInfo(&fr, &tot) != hipSuccess) tot = 0;
    clear_error();
    // keep up to half of the device: the working set of one call (a
    // contraction of 4e9 edges takes two record buffers of 33 GB) must stay
    // cached between calls, or every call pays for mapping it again
    c->limit = std::max<size_t>(tot / 2, (size_t)2 << 30);
  }
  for (auto it = c->free_.lower_bound(need); it != c->free_.end() && it->first <= need + need / 4; ++it) {
    CBlock& b = it->second;
    const bool done = hipEventQuery(b.ev) == hipSuccess;
    clear_error();
    if (!done && b.s != s) continue;
    // on the releasing stream the wait is implied by stream order; it is
    // enqueued anyway so that a recycled stream handle stays safe
    if (!done && hipStreamWaitEvent(s, b.ev, 0) != hipSuccess) {
      clear_error();
      continue;
    }
    void* p = b.p;
    c->spare.push_back(b.ev);
    c->cached -= it->first;
    c->live[p] = it->first;
    c->live_bytes += it->first;
    c->free_.erase(it);
    return p;
  }
  void* p = nullptr;
  if (hipMalloc(&p, need) != hipSuccess) {
    clear_error();
    // out of memory: wait for the device, empty the cache, try once more
    if (cache_log()) fprintf(stderr, "[lpgpu-cache] out of memory for %zu bytes: emptying %zu cached\n", need, c->cached);
    (void)hipDeviceSynchronize();
    trim_locked(*c, 0);
    (void)handle_trim_device();
    if (hipMalloc(&p, need) != hipSuccess) {
      clear_error();
      return nullptr;
    }
  }
  if (cache_log()) fprintf(stderr, "[lpgpu-cache] hipMalloc %zu (cached %zu)\n", need, c->cached);
  c->live[p] = need;
  c->live_bytes += need;
  return p;
}

void cache_free(void* p, hipStream_t s) {
  if (!p) return;
  {
    ExtBlock b{};
    bool ext = false;
    {
      std::lock_guard<std::mutex> lock(g_ext_mu);
      auto it = g_ext_live.find(p);
      if (it != g_ext_live.end()) {
        b = it->second;
        ext = true;
        g_ext_bytes -= b.bytes;
        g_ext_live.erase(it);
      }
    }
    if (ext) {
      b.a.free(p, (void*)s, b.a.ctx);
      return;
    }
  }
  DevCache* c = cache_of(nullptr);
  if (!c) return;
  std::lock_guard<std::mutex> lock(c->mu);
  auto lv = c->live.find(p);
  if (lv == c->live.end()) return;  // not a cache block
  const size_t size = lv->second;
  c->live.erase(lv);
  c->live_bytes -= size;
  hipEvent_t ev = nullptr;
  if (!c->spare.empty()) {
    ev = c->spare.back();
    c->spare.pop_back();
  } else if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
    clear_error();
    (void)hipStreamSynchronize(s);  // no event: release synchronously
    (void)hipFree(p);
    clear_error();
    return;
  }
  if (hipEventRecord(ev, s) != hipSuccess) {
    clear_error();
    c->spare.push_back(ev);
    (void)hipStreamSynchronize(s);
    (void)hipFree(p);
    clear_error();
    return;
  }
  c->free_.insert({size, CBlock{p, s, ev}});
  c->cached += size;
  if (c->cached > c->limit) trim_locked(*c, c->limit);
}

void* handle_alloc(size_t bytes) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kCacheDevices) {
    clear_error();
    return nullptr;
  }
  HandlePool& hp = handle_pool();
  const size_t need = bytes > kHandlePool / 2 ? bytes : size_class(bytes);
  std::lock_guard<std::mutex> lock(hp.mu);
  auto& f = hp.idle[dev];
  void* p = nullptr;
  size_t size = need;
  const auto it = f.lower_bound(need);
  if (it != f.end() && it->first <= need + need / 4) {
    p = it->second;
    size = it->first;
    hp.cached[dev] -= size;
    f.erase(it);
  } else if (hipMalloc(&p, need) != hipSuccess) {
    clear_error();
    handle_trim_locked(hp, dev, 0);
    if (hipMalloc(&p, need) != hipSuccess) {
      clear_error();
      return nullptr;
    }
  }
  hp.live[p] = {size, dev};
  return p;
}

void handle_free(void* p) {
  if (!p) return;
  HandlePool& hp = handle_pool();
  std::lock_guard<std::mutex> lock(hp.mu);
  const auto lv = hp.live.find(p);
  if (lv == hp.live.end()) return;
  const size_t size = lv->second.first;
  const int dev = lv->second.second;
  hp.live.erase(lv);
  if (size > kHandlePool / 2) {
    (void)hipFree(p);
    clear_error();
    return;
  }
  handle_trim_locked(hp, dev, kHandlePool - size);
  hp.idle[dev].insert({size, p});
  hp.cached[dev] += size;
}

lp_status set_allocator(const lp_allocator* a) {
  if (a && (!a->alloc || !a->free)) return LP_EINVAL;
  std::lock_guard<std::mutex> lock(g_ext_mu);
  g_ext_on = a != nullptr;
  g_ext = a ? *a : lp_allocator{};
  return LP_OK;
}

void memory_info(uint64_t* live, uint64_t* cached, uint64_t* external) {
  DevCache* c = cache_of(nullptr);
  uint64_t l = 0, k = 0, e = 0;
  if (c) {
    std::lock_guard<std::mutex> lock(c->mu);
    l = c->live_bytes;
    k = c->cached;
  }
  int dev = 0;
  if (c && hipGetDevice(&dev) == hipSuccess) {
    HandlePool& hp = handle_pool();
    std::lock_guard<std::mutex> lock(hp.mu);
    k += hp.cached[dev];
  }
  {
    std::lock_guard<std::mutex> lock(g_ext_mu);
    e = g_ext_bytes;
  }
  if (live) *live = l;
  if (cached) *cached = k;
  if (external) *external = e;
}

void cache_trim_all() {
  int cur = 0;
  if (hipGetDevice(&cur) != hipSuccess) {
    clear_error();
    return;
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess) ndev = 0;
  clear_error();
  for (int d = 0; d < ndev && d < kCacheDevices; ++d) {
    if (hipSetDevice(d) != hipSuccess) {
      clear_error();
      continue;
    }
    DevCache* c = cache_of(nullptr);
    if (!c) continue;
    {
      HandlePool& hp = handle_pool();
      std::lock_guard<std::mutex> lock(hp.mu);
      handle_trim_locked(hp, d, 0);
    }
    std::lock_guard<std::mutex> lock(c->mu);
    if (c->free_.empty()) continue;
    (void)hipDeviceSynchronize();
    trim_locked(*c, 0);
  }
  (void)hipSetDevice(cur);
  clear_error();
}

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

template <typename T>
__device__ __forceinline__ T shfl_up_any(T x, int d) {
  static_assert(sizeof(T) % 4 == 0, "word-sized types only");
  union U {
    T t;
    uint32_t w[sizeof(T) / 4];
  } a, b;
  a.t = x;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) b.w[i] = __shfl_up(a.w[i], d, kWave);
  return b.t;
}

// In-order (non-commutative safe) block inclusive scan of one value per thread.
template <typename T, typename Op>
__device__ __forceinline__ T block_scan_incl(T x, T* sm, T* total) {
  const int lane = lane_id();
  const int w = threadIdx.x / kWave;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T y = shfl_up_any(x, d);
    if (lane >= d) x = Op::op(y, x);
  }
  if (lane == kWave - 1) sm[w] = x;
  __syncthreads();
  T pre = Op::id();
  T tot = Op::id();
#pragma unroll
  for (int i = 0; i < kScanThreads / kWave; ++i) {
    if (i < w) pre = Op::op(pre, sm[i]);
    tot = Op::op(tot, sm[i]);
  }
  __syncthreads();
  *total = tot;
  return Op::op(pre, x);
}

template <typename T>
struct SumOp {
  __device__ static T id() { return T(0); }
  __device__ static T op(T a, T b) { return a + b; }
};

// ---- plain sums --------------------------------------------------------
template <typename T>
struct LoadArr {
  const T* in;
  __device__ T operator()(int64_t i) const { return in[i]; }
};

template <typename T, typename Op, typename Load>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(Load load, int64_t n, T* aggs) {
  __shared__ T sm[kScanThreads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T acc = Op::id();
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i < n) acc = Op::op(acc, load(base + i));
  T tot;
  (void)block_scan_incl<T, Op>(acc, sm, &tot);
  if (threadIdx.x == 0) aggs[blockIdx.x] = tot;
}

// Exclusive sum scan of one tile with a carry-in from block_off.
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_excl_down(const T* in, T* out, int64_t n,
                                                                 const T* block_off, T* total_dev) {
  __shared__ T sm[kScanThreads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T x[kScanItems];
  T acc = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    x[i] = (base + i < n) ? in[base + i] : T(0);
    acc += x[i];
  }
  T tot;
  T incl = block_scan_incl<T, SumOp<T>>(acc, sm, &tot);
  T run = incl - acc + (block_off ? block_off[blockIdx.x] : T(0));
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) out[base + i] = run;
    run += x[i];
  }
  if (total_dev && block_off == nullptr && threadIdx.x == 0) *total_dev = tot;
}

template <typename T>
lp_status scan_exclusive_t(const T* in, T* out, int64_t n, T* total_dev, Scratch& sc) {
  hipStream_t s = sc.stream();
  if (n <= 0) {
    if (total_dev) LP_CHECK_HIP(hipMemsetAsync(total_dev, 0, sizeof(T), s));
    return LP_OK;
  }
  int64_t nb = (n + kScanTile - 1) / kScanTile;
  if (nb == 1) {
    hipLaunchKernelGGL(k_scan_excl_down<T>, dim3(1), dim3(kScanThreads), 0, s, in, out, n, (const T*)nullptr,
                       total_dev);
    LP_CHECK_LAUNCH();
    return LP_OK;
  }
  T* aggs = sc.alloc<T>(nb);
  if (!aggs) return LP_ENOMEM;
  hipLaunchKernelGGL((k_scan_reduce<T, SumOp<T>, LoadArr<T>>), dim3((unsigned)nb), dim3(kScanThreads), 0, s,
                     LoadArr<T>{in}, n, aggs);
  LP_CHECK_LAUNCH();
  LP_CHECK(scan_exclusive_t<T>(aggs, aggs, nb, total_dev, sc));
  hipLaunchKernelGGL(k_scan_excl_down<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, out, n,
                     (const T*)aggs, (T*)nullptr);
  LP_CHECK_LAUNCH();
  return LP_OK;
}

// ---- radix sort ----------------------------------------------------------
// One histogram launch counts the digits of all passes, then every pass is one
// launch: a workgroup ranks its tile's pairs by digit (per wavefront, in
// order), learns each digit's position from the tiles before it by look-back
// (lookback.h), gathers the pairs by digit in LDS and writes them out in runs.
// Each pair is read and written once per pass. A pass in which all keys share
// the digit (the high gain bits of proposals, mostly) is left out. Every
// workgroup of a pass derives the digits' positions from the counts itself:
// having the last workgroup of the histogram do it once took two device-wide
// fences, 9 to 24 us per sort. 9e6 pairs take 45 us a pass (4.8 TB/s), 16384
// pairs 7 us.
constexpr int kRsThreads = 256;
// Pairs per thread: tiles of 2048 pairs keep more workgroups busy on few
// pairs, tiles of 4096 halve the look-back of many (the acceptance of a round of
// RGG-2D graphs with one and the other: 20,001 vertices 47 and 56 us, 1,048,576
// 129 and 133, 2,000,001 183 and 177, 4,000,001 273 and 255).
constexpr int kRsItemsFew = 8, kRsItemsMany = 16;
constexpr int64_t kRsFew = 1 << 20;  // most pairs sorted in small tiles
constexpr int kRsBack = 4;           // predecessors read at a time in a look-back
constexpr int kRsBins = 256;
constexpr int kRsPasses = 8;
constexpr int kRsHistGrid = 1024;  // most workgroups of the histogram launch
constexpr int kRsHistUnroll = 4;   // keys in flight per thread
constexpr int kRsHistRun = kRsThreads * kRsHistUnroll;

}  // namespace

struct SortPlan {
  uint32_t hist[2][kRsPasses][kRsBins];  // digit counts of this sort and (zero) of the next one
  uint32_t src[kRsPasses + 1];           // buffer set a pass reads (and the result's)
  uint32_t ticket;
};

namespace {

// Digit counts of all passes; clears the counts of the next sort.
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const uint64_t* __restrict__ keys, const uint32_t* count_dev,
                                                        int passes, SortPlan* plan, int which) {
  __shared__ uint32_t h[kRsPasses][kRsBins];
  const int t = threadIdx.x;
  if (blockIdx.x == 0)
    for (int p = 0; p < passes; ++p) plan->hist[which ^ 1][p][t] = 0;
  for (int p = 0; p < passes; ++p) h[p][t] = 0;
  __syncthreads();
  const int64_t n = *count_dev;
  for (int64_t j0 = (int64_t)blockIdx.x * kRsHistRun; j0 < n; j0 += (int64_t)gridDim.x * kRsHistRun) {
    uint64_t k[kRsHistUnroll];
#pragma unroll
    for (int i = 0; i < kRsHistUnroll; ++i) {
      const int64_t j = j0 + i * kRsThreads + t;
      k[i] = j < n ? keys[j] : 0;
    }
    for (int p = 0; p < passes; ++p) {
#pragma unroll
      for (int i = 0; i < kRsHistUnroll; ++i) {
        if (j0 + i * kRsThreads + t >= n) continue;
        const uint32_t dg = (uint32_t)(k[i] >> (8 * p)) & (kRsBins - 1);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)dg);
        const uint64_t act = __ballot(1), same = __ballot(dg == d0);
        if (same == act) {  // one digit in the whole wavefront: one addition
          if (lane_id() == __ffsll((unsigned long long)act) - 1) atomicAdd(&h[p][d0], (uint32_t)__popcll(act));
        } else {
          atomicAdd(&h[p][dg], 1u);
        }
      }
    }
  }
  __syncthreads();
  for (int p = 0; p < passes; ++p)
    if (h[p][t]) atomicAdd(&plan->hist[which][p][t], h[p][t]);
}

template <int kRsItems>
__global__ __launch_bounds__(kRsThreads) void k_rs_pass(SortedPairs b, const uint32_t* count_dev, SortPlan* plan,
                                                        int which, int pass, LookArgs look) {
  constexpr int kW = kRsThreads / kWave;
  constexpr int kRsTile = kRsThreads * kRsItems;
  __shared__ __align__(16) uint64_t stage[kRsTile];
  __shared__ uint32_t wcnt[kW][kRsBins];
  __shared__ uint32_t dstart[kRsBins];  // first place of every digit in the tile
  __shared__ uint32_t gbase[kRsBins];   // its first position in the output, minus dstart
  __shared__ int32_t scan[kW];
  __shared__ uint32_t tsm;
  const int64_t n = *count_dev;
  const uint32_t tiles = (uint32_t)((n + kRsTile - 1) / kRsTile);
  if (blockIdx.x >= tiles) return;
  const int t = threadIdx.x, w = t / kWave, lane = lane_id();
  const uint32_t src = plan->src[pass];
  const uint32_t all = plan->hist[which][pass][t];  // pairs of digit t
  const bool skip = __syncthreads_or((int64_t)all == n);
  if (blockIdx.x == 0 && t == 0) plan->src[pass + 1] = skip ? src : src ^ 1u;
  if (skip) return;
  const uint32_t tile = look_ticket(look, tiles, &tsm);
  const uint64_t* kin = b.k[src];
  const uint32_t* vin = b.v[src];
  uint64_t* kout = b.k[src ^ 1u];
  uint32_t* vout = b.v[src ^ 1u];
  // wavefront w holds the tile's pairs [w * 64 * kRsItems, ...), item by item
  const int64_t base = (int64_t)tile * kRsTile + (int64_t)w * kWave * kRsItems;
  uint64_t key[kRsItems];
  uint32_t val[kRsItems];
#pragma unroll
  for (int i = 0; i < kRsItems; ++i) {
    const int64_t j = base + i * kWave + lane;
    key[i] = j < n ? kin[j] : 0;
    val[i] = j < n ? vin[j] : 0;
  }
  for (int k = 0; k < kW; ++k) wcnt[k][t] = 0;
  __syncthreads();
  // rank among the wavefront's earlier pairs of the same digit
  const uint64_t lt = lanemask_lt();
  uint32_t rank[kRsItems];
#pragma unroll
  for (int i = 0; i < kRsItems; ++i) {
    const bool valid = base + i * kWave + lane < n;
    const uint32_t d = (uint32_t)(key[i] >> (8 * pass)) & (kRsBins - 1);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint64_t m = __ballot((d >> q) & 1u);
      peers &= ((d >> q) & 1u) ? m : ~m;
    }
    const uint32_t r = (uint32_t)__popcll(peers & lt), cnt = (uint32_t)__popcll(peers);
    uint32_t before = 0;
    if (valid) before = wcnt[w][d];
    wave_sync_lds();
    if (valid && r + 1 == cnt) wcnt[w][d] = before + cnt;
    wave_sync_lds();
    rank[i] = before + r;
  }
  __syncthreads();
  // thread t: digit t. Its count per wavefront becomes the wavefront's offset
  uint32_t cnt = 0;
#pragma unroll
  for (int k = 0; k < kW; ++k) {
    const uint32_t c = wcnt[k][t];
    wcnt[k][t] = cnt;
    cnt += c;
  }
  uint64_t* words = look.words + (uint64_t)tile * kRsBins + t;
  look_put(words, look_word(look.launch, tile ? kLookTotal : kLookPrefix, cnt));
  int32_t tot;
  const uint32_t ds = (uint32_t)block_incl_scan_add<kRsThreads, int32_t>((int32_t)cnt, scan, &tot) - cnt;
  dstart[t] = ds;
  const uint32_t first = (uint32_t)block_incl_scan_add<kRsThreads, int32_t>((int32_t)all, scan, &tot) - all;
  __syncthreads();
  uint32_t place[kRsItems];
#pragma unroll
  for (int i = 0; i < kRsItems; ++i) {
    const uint32_t d = (uint32_t)(key[i] >> (8 * pass)) & (kRsBins - 1);
    place[i] = dstart[d] + wcnt[w][d] + rank[i];
    if (base + i * kWave + lane < n) stage[place[i]] = key[i];
  }
  uint32_t before = 0;
  for (int64_t q = (int64_t)tile - 1; q >= 0;) {
    uint64_t wd[kRsBack];
#pragma unroll
    for (int k = 0; k < kRsBack; ++k)
      wd[k] = q >= k ? look_get(look.words + (uint64_t)(q - k) * kRsBins + t) : look_word(look.launch, kLookPrefix, 0);
    bool known = false, open = false;
#pragma unroll
    for (int k = 0; k < kRsBack; ++k) {
      if (known || open) continue;
      const uint32_t st = look_state(wd[k], look.launch);
      if (st == 0) {
        open = true;
      } else {
        before += (uint32_t)wd[k];
        known = st == kLookPrefix;
        --q;
      }
    }
    if (known) break;
    if (open) __builtin_amdgcn_s_sleep(1);
  }
  if (tile) look_put(words, look_word(look.launch, kLookPrefix, before + cnt));
  gbase[t] = first + before - ds;
  __syncthreads();
  const uint32_t have = (uint32_t)min((int64_t)kRsTile, n - (int64_t)tile * kRsTile);
  uint32_t dst[kRsItems];
#pragma unroll
  for (int i = 0; i < kRsItems; ++i) {
    const uint32_t j = i * kRsThreads + t;
    dst[i] = 0;
    if (j < have) {
      const uint64_t k = stage[j];
      dst[i] = gbase[(uint32_t)(k >> (8 * pass)) & (kRsBins - 1)] + j;
      kout[dst[i]] = k;
    }
  }
  __syncthreads();
  uint32_t* vstage = (uint32_t*)stage;
#pragma unroll
  for (int i = 0; i < kRsItems; ++i)
    if (base + i * kWave + lane < n) vstage[place[i]] = val[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kRsItems; ++i) {
    const uint32_t j = i * kRsThreads + t;
    if (j < have) vout[dst[i]] = vstage[j];
  }
}

__global__ void k_zero_words(uint32_t* p, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (((uintptr_t)p & 15u) == 0) {
    for (int64_t i = i0; i < n / 4; i += stride) ((uint4*)p)[i] = make_uint4(0, 0, 0, 0);
    if (i0 < n % 4) p[n / 4 * 4 + i0] = 0;
  } else {
    for (int64_t i = i0; i < n; i += stride) p[i] = 0;
  }
}

}  // namespace

lp_status scan_exclusive_u64(const uint64_t* in, uint64_t* out, int64_t n, uint64_t* total_dev, Scratch& sc) {
  return scan_exclusive_t<uint64_t>(in, out, n, total_dev, sc);
}

lp_status scan_exclusive_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total_dev, Scratch& sc) {
  return scan_exclusive_t<uint32_t>(in, out, n, total_dev, sc);
}

lp_status zero_u32(uint32_t* p, int64_t n, hipStream_t s) {
  if (n <= 0) return LP_OK;
  hipLaunchKernelGGL(k_zero_words, dim3(grid_for(n, 1024, 2048)), dim3(256), 0, s, p, n);
  return last_error();
}

lp_status PairSorter::init(uint64_t* keys_a, uint32_t* vals_a, uint64_t* keys_b, uint32_t* vals_b, int64_t max_n,
                           int bits, Scratch& sc) {
  if (max_n > 0xFFFFFFFFll || bits > 8 * kRsPasses) return LP_EUNSUPPORTED;
  stream_ = sc.stream();
  max_n_ = max_n;
  passes_ = bits > 0 ? (bits + 7) / 8 : 0;
  const int per_tile = kRsThreads * (max_n <= kRsFew ? kRsItemsFew : kRsItemsMany);
  const int64_t tiles = (max_n + per_tile - 1) / per_tile;
  static_assert(sizeof(SortPlan) % 8 == 0, "the words follow the plan");
  const size_t plan_words = sizeof(SortPlan) / 4;
  zero_words_ = (int64_t)plan_words + (passes_ ? 2 * tiles * kRsBins : 0);
  zero_ = sc.alloc<uint32_t>((size_t)zero_words_);
  if (!zero_) return LP_ENOMEM;
  plan_ = (SortPlan*)zero_;
  words_ = (uint64_t*)(zero_ + plan_words);
  out_.k[0] = keys_a;
  out_.k[1] = keys_b;
  out_.v[0] = vals_a;
  out_.v[1] = vals_b;
  out_.sel = &plan_->src[passes_];
  return LP_OK;
}

lp_status PairSorter::sort(const uint32_t* count_dev) {
  if (max_n_ <= 0 || passes_ == 0) return LP_OK;
  const bool few = max_n_ <= kRsFew;
  const int per_tile = kRsThreads * (few ? kRsItemsFew : kRsItemsMany);
  const unsigned tiles = (unsigned)((max_n_ + per_tile - 1) / per_tile);
  hipLaunchKernelGGL(k_rs_hist, dim3(grid_for(max_n_, kRsHistRun, kRsHistGrid)), dim3(kRsThreads), 0, stream_, out_.k[0],
                     count_dev, passes_, plan_, which_);
  LP_CHECK_LAUNCH();
  for (int p = 0; p < passes_; ++p) {
    hipLaunchKernelGGL(few ? k_rs_pass<kRsItemsFew> : k_rs_pass<kRsItemsMany>, dim3(tiles), dim3(kRsThreads), 0, stream_, out_, count_dev, plan_, which_, p,
                       LookArgs{words_, &plan_->ticket, ++launch_});
    LP_CHECK_LAUNCH();
  }
  which_ ^= 1;
  return LP_OK;
}

}  // namespace lp

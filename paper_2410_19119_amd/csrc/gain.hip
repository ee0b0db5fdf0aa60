// Sparse gain table (Section V of the paper; layout in gain.h), the public
// lp_gain_table handle, and the table-driven selection step that lp_refine
// uses instead of re-rating every neighbourhood in each round.
#include <algorithm>

#include "decode.h"
#include "gain.h"

namespace lp {

lp_status plan_degrees(const lp_graph* g, const int32_t** deg, const int4** lane, int32_t* nlane,
                       const int32_t** longer, int32_t* nlong, uint64_t* long_edges, hipStream_t s);

namespace {

constexpr int kGtLaneMax = 16;  // vertices up to this degree are filled / selected by one lane
// A wavefront takes a longer neighbourhood, which uses the device best as long
// as no neighbourhood lasts much longer than the others (RGG-3D of 20,001
// vertices, degree 1000, k = 3000: build, 2 % moves and queries 1.33 ms, with a
// workgroup for each 1.68). One of more than this degree and more than twice
// the mean of the longer ones gets a workgroup (R-MAT, 30,001 vertices, degree
// 64, k = 64: 0.33 ms, with wavefronts for all 0.39).
constexpr int kGtWaveMax = 512;
constexpr int kGtThreads = 256; // threads of such a workgroup
constexpr int kGtCounters = 8;
constexpr int kGtWaves = 4;     // wavefronts per 256-thread workgroup
constexpr int32_t kGtEmpty = -1;

template <typename V>
struct GtView {
  int32_t n, k;
  const uint64_t* off;
  int32_t* key;
  V* val;
  uint32_t* flag;
  int32_t* list;
  uint32_t* cnt;
};

template <typename V>
GtView<V> view_of(const GainTable& t) {
  return GtView<V>{t.g->n, t.k, t.off, t.key, (V*)t.val, t.flag, t.list, t.cnt};
}

// Home slot of block b in a hash slice of L = 2^s slots (the top s bits of a
// multiplicative hash).
__device__ __forceinline__ uint32_t gt_hash(int32_t b, uint32_t L) {
  return ((uint32_t)b * 0x9E3779B1u) >> (33u - (uint32_t)__ffs(L));
}

__device__ __forceinline__ void gt_atomic_add(int32_t* p, int32_t w) { atomicAdd(p, w); }
__device__ __forceinline__ void gt_atomic_add(int64_t* p, int64_t w) {
  atomicAdd((unsigned long long*)p, (unsigned long long)w);
}

// A vertex's slice. Slices of k slots are dense rows: hash slices are shorter.
struct GtSlice {
  uint64_t base;
  uint32_t L;
};

template <typename V>
__device__ __forceinline__ GtSlice gt_slice(const GtView<V>& t, int32_t u) {
  const uint64_t base = t.off[u];
  return GtSlice{base, (uint32_t)(t.off[u + 1] - base)};
}

template <typename V>
__device__ __forceinline__ bool gt_dense(const GtView<V>& t, const GtSlice& sl) {
  return sl.L == (uint32_t)t.k;
}

// Slot of block b in a hash slice, inserting it if `insert`; -1 if absent (or,
// when inserting, if the slice has no free slot left). h is b's home slot and
// kk what it held.
template <typename V>
__device__ __forceinline__ int64_t gt_slot(const GtView<V>& t, const GtSlice& sl, int32_t b, uint32_t h, int32_t kk,
                                           bool insert) {
  for (uint32_t p = 0; p < sl.L; ++p) {
    const uint64_t s = sl.base + h;
    if (p) kk = t.key[s];
    if (kk == b) return (int64_t)s;
    if (kk == kGtEmpty) {
      if (!insert) return -1;
      const int32_t old = atomicCAS(&t.key[s], kGtEmpty, b);
      if (old == kGtEmpty || old == b) return (int64_t)s;
    }
    h = (h + 1) & (sl.L - 1);
  }
  return -1;
}

template <typename V>
__device__ __forceinline__ bool gt_add(const GtView<V>& t, const GtSlice& sl, int32_t b, V w) {
  int64_t s;
  if (gt_dense(t, sl)) {
    s = (int64_t)(sl.base + (uint32_t)b);
  } else {
    const uint32_t h = gt_hash(b, sl.L);
    s = gt_slot(t, sl, b, h, t.key[sl.base + h], true);
    if (s < 0) return false;
  }
  gt_atomic_add(&t.val[s], w);
  return true;
}

// The home slot's key and value are read together.
template <typename V>
__device__ __forceinline__ V gt_get(const GtView<V>& t, int32_t u, int32_t b) {
  const GtSlice sl = gt_slice(t, u);
  if (sl.L == 0) return (V)0;
  if (gt_dense(t, sl)) return t.val[sl.base + (uint32_t)b];
  const uint32_t h = gt_hash(b, sl.L);
  const int32_t kk = t.key[sl.base + h];
  const V x = t.val[sl.base + h];
  if (kk == b) return x;
  const int64_t s = gt_slot(t, sl, b, h, kk, false);
  return s < 0 ? (V)0 : t.val[s];
}

// Every neighbour (v, w) of u, for one group of NT threads: chunk c of a
// chunked neighbourhood, or all of it (c < 0). Plain graphs are cut into the
// same 1000-edge pieces above the chunking threshold. f(v, w, pre(v)) is
// called by one thread per neighbour; pre only loads, so that the loads of
// several neighbours are in flight at a time.
template <int NT, typename P, typename F>
__device__ __forceinline__ void group_visit(const GraphView& g, int32_t u, uint32_t deg, int32_t c,
                                            DecodeSmem<NT>& dsm, P&& pre, F&& f) {
  const int tid = group_tid<NT>();
  if (g.offs && g.intervals) {
    // interval-coded: every thread walks a chunk's interval neighbours and
    // keeps its own, one of every NT; the others are decoded by the group (a
    // single lane walked whole chunks: 748,287 R-MAT vertices with weights,
    // k = 8, build, 2 % moves and queries 8.0 ms, now 1.2)
    const Nbh h = nbh_locate(g, u, deg);
    const uint32_t c0 = c < 0 ? 0u : (uint32_t)c, c1 = c < 0 ? h.nchunks : (uint32_t)c + 1;
    for (uint32_t ch = c0; ch < c1; ++ch) {
      const uint32_t first = ch * LP_CHUNK_LEN;
      const uint32_t cnt = h.nchunks > 1 ? min((uint32_t)LP_CHUNK_LEN, deg - first) : deg;
      LaneDec d;
      d.init(g, u, nbh_chunk_pos(g, h, ch));
      uint32_t L = 0;
      int32_t mv = u, mw = 0;
      bool have = false;
      for (; L < cnt && (d.rem > 0 || d.kleft > 0); ++L) {
        int32_t v, w;
        d.next(v, w);
        if (L % NT == (uint32_t)tid) {
          mv = v;
          mw = w;
          have = true;
        }
        if (L % NT == NT - 1) {
          f(mv, mw, pre(mv));
          have = false;
        }
      }
      if (have) f(mv, mw, pre(mv));
      if (L < cnt) {
        uint64_t pos = d.c.pos;
        int32_t pv = 0, pw = d.w;
        using Q = decltype(pre(0));
        (void)group_decode<NT>(g.bytes, pos, u, cnt - L, g.weighted, true, pv, pw, dsm, pre,
                               [&](uint32_t, int32_t v, int32_t w, const Q& q) { f(v, w, q); }, true);
      }
    }
  } else if (g.offs) {
    const Nbh h = nbh_locate(g, u, deg);
    const uint32_t c0 = c < 0 ? 0u : (uint32_t)c, c1 = c < 0 ? h.nchunks : (uint32_t)c + 1;
    for (uint32_t ch = c0; ch < c1; ++ch) {
      uint64_t pos = nbh_chunk_pos(g, h, ch);
      const uint32_t first = ch * LP_CHUNK_LEN;
      const uint32_t cnt = h.nchunks > 1 ? min((uint32_t)LP_CHUNK_LEN, deg - first) : deg;
      int32_t pv = 0, pw = 0;
      using Q = decltype(pre(0));
      (void)group_decode<NT>(g.bytes, pos, u, cnt, g.weighted, true, pv, pw, dsm, pre,
                             [&](uint32_t, int32_t v, int32_t w, const Q& q) { f(v, w, q); });
    }
  } else {
    const uint64_t e0 = g.xadj[u];
    uint32_t lo = 0, hi = deg;
    if (c >= 0) {
      lo = (uint32_t)c * LP_CHUNK_LEN;
      hi = min(deg, lo + (uint32_t)LP_CHUNK_LEN);
    }
    for (uint32_t e = lo + (uint32_t)tid; e < hi; e += 4 * NT) {
      int32_t v[4], w[4];
      decltype(pre(0)) q[4];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint64_t x = e0 + (e + k * NT < hi ? e + k * NT : e);
        v[k] = g.adjncy[x];
        w[k] = g.adjwgt ? g.adjwgt[x] : 1;
      }
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) q[k] = pre(v[k]);
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k)
        if (e + k * NT < hi) f(v[k], w[k], q[k]);
    }
  }
}

// Every neighbour of a short neighbourhood, for one lane.
template <typename F>
__device__ __forceinline__ void lane_visit(const GraphView& g, int32_t u, uint32_t deg, F&& f) {
  if (g.offs) {
    lane_decode(g, u, deg, [&](uint32_t, int32_t v, int32_t w) { f(v, w); });
  } else {
    const uint64_t e0 = g.xadj[u];
    for (uint32_t e = 0; e < deg; ++e) f(g.adjncy[e0 + e], g.adjwgt ? g.adjwgt[e0 + e] : 1);
  }
}

// Slice length and kind of every vertex: none for isolated vertices, a dense
// row of k when pow2(2 deg) >= k, else pow2(2 deg) hash slots. Also clears the
// flags and the counters.
__global__ void k_gt_len(const int32_t* deg, int32_t n, int32_t k, uint64_t* len, uint32_t* flag, uint32_t* cnt) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t d = (uint64_t)deg[u];
    uint64_t L = 0;
    if (d > 0) {
      L = 2;
      while (L < 2 * d) L <<= 1;
      if (L >= (uint64_t)k) L = (uint64_t)k;
    }
    len[u] = L;
    flag[u] = 0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) len[n] = 0;
  if (blockIdx.x == 0 && threadIdx.x < kGtCounters) cnt[threadIdx.x] = 0;
}

template <typename V>
__global__ void k_gt_clear(int32_t* key, V* val, uint64_t m) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
    key[i] = kGtEmpty;
    val[i] = 0;
  }
}

__global__ void k_gt_zero(uint32_t* a, int64_t m) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
    a[i] = 0;
}

// One lane per short neighbourhood: the edges' blocks are gathered together,
// equal ones summed in registers, and each block placed at its slot by the
// lane alone (a mask of the taken slots stands for the probing), so a slice
// costs one plain store per distinct block and array. Bound by the gathers;
// inserting edge by edge with a compare-and-swap and an add, each waiting for
// the one before, took 345 us for 2,000,003 R-MAT vertices, 88 us now.
template <bool COMP, bool ITV, typename V>
__global__ __launch_bounds__(256) void k_gt_fill_lane(GraphView g, const int4* list, int32_t cnt,
                                                      const int32_t* blocks, GtView<V> t) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= cnt) return;
  const int4 v4 = list[i];
  const int32_t u = v4.x, d = v4.y;
  const uint64_t pos = (uint64_t)(uint32_t)v4.z | ((uint64_t)(uint32_t)v4.w << 32);
  int32_t lab[kGtLaneMax], wt[kGtLaneMax];
  LaneDec dec;
  VarCursor cur;
  if constexpr (ITV) dec.init(g, u, pos);
  else if constexpr (COMP) cur.seek(g.bytes, pos);
  int32_t v = 0, w = 0;
#pragma unroll
  for (int k = 0; k < kGtLaneMax; ++k) {
    lab[k] = -1;
    wt[k] = 0;
    if (k < d) {
      if constexpr (ITV) {
        dec.next(v, w);
      } else if constexpr (COMP) {
        const uint32_t code = cur.next();
        v = (k == 0) ? u + unzigzag32(code) : v + (int32_t)code;
        if (g.weighted) w = (k == 0 ? 0 : w) + unzigzag32(cur.next());
        else w = 1;
      } else {
        v = g.adjncy[pos + k];
        w = g.adjwgt ? g.adjwgt[pos + k] : 1;
      }
      lab[k] = blocks[v];
      wt[k] = w;
    }
  }
  const GtSlice sl = gt_slice(t, u);
  const bool dn = gt_dense(t, sl);
  uint32_t taken = 0;  // a hash slice here has at most 32 slots
#pragma unroll
  for (int k = 0; k < kGtLaneMax; ++k) {
    const int32_t c = lab[k];
    bool first = c >= 0;
#pragma unroll
    for (int j = 0; j < k; ++j) first &= lab[j] != c;
    if (!first) continue;
    V sum = 0;
#pragma unroll
    for (int j = k; j < kGtLaneMax; ++j) sum += lab[j] == c ? (V)wt[j] : (V)0;
    uint32_t h = (uint32_t)c;
    if (!dn) {
      h = gt_hash(c, sl.L);
      while ((taken >> h) & 1u) h = (h + 1) & (sl.L - 1);
      taken |= 1u << h;
      t.key[sl.base + h] = c;
    }
    t.val[sl.base + h] = sum;
  }
}
static_assert(2 * kGtLaneMax <= 32, "a lane's hash slice fits a mask of 32 slots");

// Work items of the group fill: one per vertex above kGtLaneMax, one per chunk
// above the chunking threshold. Wavefronts take the neighbourhoods up to
// wave_max (from the front of the list), workgroups the longer ones (from its
// end), chunks like the neighbourhood they are of. Every thread takes
// kGtItemRun of the listed vertices, so that two counter atomics serve that
// many per thread of a workgroup.
constexpr int kGtItemRun = 4;

__device__ __forceinline__ uint32_t gt_items_of(uint32_t d, uint32_t thr) {
  return d <= (uint32_t)kGtLaneMax ? 0u : d > thr ? (d + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN : 1u;
}

__global__ __launch_bounds__(256) void k_gt_items(const int32_t* list, const int32_t* deg, int32_t n,
                                                  uint32_t thr, int32_t wave_max, int2* items, uint64_t cap,
                                                  uint32_t* nitems) {
  __shared__ int32_t scan[256 / kWave + 1];
  __shared__ uint32_t base_sm[2];
  const int64_t b = (int64_t)blockIdx.x * (256 * kGtItemRun) + threadIdx.x;
  int2 vd[kGtItemRun];
  uint32_t cnt[2] = {0, 0}, o[2];
#pragma unroll
  for (int r = 0; r < kGtItemRun; ++r) {
    vd[r] = make_int2(0, 0);
    if (b + r * 256 < n) vd[r].x = list[b + r * 256];
  }
#pragma unroll
  for (int r = 0; r < kGtItemRun; ++r) {
    if (b + r * 256 < n) vd[r].y = deg[vd[r].x];
    cnt[vd[r].y > wave_max] += gt_items_of((uint32_t)vd[r].y, thr);
  }
  for (int x = 0; x < 2; ++x) {
    int32_t tot;
    const uint32_t incl = (uint32_t)block_incl_scan_add<256, int32_t>((int32_t)cnt[x], scan, &tot);
    if (threadIdx.x == 255) base_sm[x] = tot ? atomicAdd(nitems + x, (uint32_t)tot) : 0u;
    __syncthreads();
    o[x] = base_sm[x] + incl - cnt[x];
  }
#pragma unroll
  for (int r = 0; r < kGtItemRun; ++r) {
    const uint32_t ni = gt_items_of((uint32_t)vd[r].y, thr);
    for (uint32_t j = 0; j < ni; ++j) {
      const int2 it = make_int2(vd[r].x, ni > 1 ? (int)j : -1);
      if (vd[r].y > wave_max) items[cap - 1 - o[1]++] = it;
      else items[o[0]++] = it;
    }
  }
}

__device__ __forceinline__ void lds_add_v(int32_t* p, int32_t w) { atomicAdd(p, w); }
__device__ __forceinline__ void lds_add_v(int64_t* p, int64_t w) {
  atomicAdd((unsigned long long*)p, (unsigned long long)w);
}

// One group of NT threads (a wavefront, or a workgroup) per work item. A dense
// row of at most kGtStage blocks is summed in the group's LDS first, so that
// the edges of a vertex do not all hit the same few global addresses, and then
// stored as it is (the whole neighbourhood) or added with one global atomic
// per nonzero block (a chunk of it). What bounds a group is the chain decode,
// gather, LDS add of a window of codes: up to four gathers per thread are in
// flight, and four wavefronts share the neighbourhoods much longer than the
// others, which left a single one the last to end (2,000,003 R-MAT vertices: 648 us for all, now
// 340 + 277 us).
constexpr int kGtStage = 1024;
constexpr int kGtPerCopy = 64;  // edges per copy of a row

template <int NT, typename V>
__global__ __launch_bounds__(256) void k_gt_fill_group(GraphView g, const int32_t* deg, const int32_t* blocks,
                                                       const int2* items, uint64_t cap, const uint32_t* nitems,
                                                       GtView<V> t) {
  constexpr int G = 256 / NT;  // groups of a workgroup
  __shared__ DecodeSmem<NT> dsm[G];
  __shared__ V stage[G][kGtStage + 1];
  const int w = threadIdx.x / NT, tid = group_tid<NT>();
  const int64_t ng = (int64_t)gridDim.x * G;
  const uint32_t m = nitems[NT == kWave ? 0 : 1];
  const bool staged_k = t.k <= kGtStage;
  const int32_t ks = t.k | 1;  // a copy's stride: equal blocks of the copies lie in different banks
  const auto pre = [&](int32_t v) { return blocks[v]; };
  for (int64_t i = (int64_t)blockIdx.x * G + w; i < m; i += ng) {
    const int2 it = items[NT == kWave ? i : (int64_t)cap - 1 - i];
    const int32_t u = it.x;
    const GtSlice sl = gt_slice(t, u);
    if (staged_k && gt_dense(t, sl)) {
      const uint32_t d = (uint32_t)deg[u];
      int32_t R = 1;
      while (R < kWave && 2 * R * ks <= kGtStage && 2 * R * kGtPerCopy <= (int32_t)d) R *= 2;
      for (int32_t q = tid; q < R * ks; q += NT) stage[w][q] = 0;
      group_sync<NT>();
      V* mine = stage[w] + (tid & (R - 1)) * ks;
      group_visit<NT>(g, u, d, it.y, dsm[w], pre,
                      [&](int32_t, int32_t wt, int32_t c) { lds_add_v(&mine[c], (V)wt); });
      group_sync<NT>();
      for (int32_t q = tid; q < t.k; q += NT) {
        V a = 0;
        for (int32_t r = 0; r < R; ++r) a += stage[w][r * ks + q];
        if (it.y < 0) t.val[sl.base + q] = a;
        else if (a) gt_atomic_add(&t.val[sl.base + q], a);
      }
      group_sync<NT>();
    } else {
      group_visit<NT>(g, u, (uint32_t)deg[u], it.y, dsm[w], pre,
                      [&](int32_t, int32_t wt, int32_t c) { (void)gt_add(t, sl, c, (V)wt); });
    }
  }
}

__device__ __forceinline__ void gt_consider(const GtRound& r, int32_t c, int64_t val, int64_t wu, Cand& best) {
  if (val <= 0 || val < best.r) return;
  const Cand cd{val, tiebreak_key(r.seed, r.round, (uint32_t)c), c};
  if (cand_better(cd, best) && r.W[c] + wu <= r.cap) best = cd;
}

__device__ __forceinline__ void gt_emit(const GtRound& r, int32_t u, const Cand& best, int64_t own) {
  if (best.c >= 0 && best.r > own) {
    r.ptgt[u] = best.c;
    r.pgain[u] = best.r - own;
  } else {
    r.ptgt[u] = -1;
  }
}

// One lane per vertex: own affinity and the best feasible other block, by
// (affinity desc, tie-break key asc), as the rating step of the LP rounds.
template <typename V>
__global__ __launch_bounds__(256) void k_gt_select_lane(GtView<V> t, GtRound r, const int32_t* list, int32_t cnt) {
  if (*r.done) return;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= cnt) return;
  const int32_t u = list[i];
  const int32_t own_c = r.C[u];
  const int64_t wu = r.vwgt ? r.vwgt[u] : 1;
  const GtSlice sl = gt_slice(t, u);
  const uint64_t base = sl.base;
  const uint32_t L = sl.L;
  const bool dn = gt_dense(t, sl);
  int64_t own = 0;
  Cand best = cand_none();
  for (uint32_t q = 0; q < L; ++q) {
    const int32_t c = dn ? (int32_t)q : t.key[base + q];
    if (c == kGtEmpty) continue;
    const int64_t a = (int64_t)t.val[base + q];
    if (c == own_c) own = a;
    else gt_consider(r, c, a, wu, best);
  }
  gt_emit(r, u, best, own);
}

// One wavefront per vertex (lanes stride over the slice).
template <typename V>
__global__ __launch_bounds__(256) void k_gt_select_wave(GtView<V> t, GtRound r, const int32_t* list, int32_t cnt) {
  if (*r.done) return;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave; i < cnt; i += nw) {
    const int32_t u = list[i];
    const int32_t own_c = r.C[u];
    const int64_t wu = r.vwgt ? r.vwgt[u] : 1;
    const GtSlice sl = gt_slice(t, u);
    const uint64_t base = sl.base;
    const uint32_t L = sl.L;
    const bool dn = gt_dense(t, sl);
    int64_t own = 0;
    Cand best = cand_none();
    for (uint32_t q = (uint32_t)lane_id(); q < L; q += kWave) {
      const int32_t c = dn ? (int32_t)q : t.key[base + q];
      if (c == kGtEmpty) continue;
      const int64_t a = (int64_t)t.val[base + q];
      if (c == own_c) own = a;
      else gt_consider(r, c, a, wu, best);
    }
    best = wave_best(best);
    own = wave_reduce_add(own);
    if (lane_id() == 0) gt_emit(r, u, best, own);
  }
}

// The update of one neighbour v of a moved vertex: w(u, v) leaves block
// `from` and joins block `to` in v's slice. Both home slots are read together.
// A vertex without neighbours of its own (the graph is not symmetric, which
// nothing checks) has no slots: `from` is missing and `to` finds no place.
template <typename V>
__device__ __forceinline__ void gt_move_edge(const GtView<V>& t, int32_t v, const GtSlice& sl, int32_t from,
                                             int32_t to, int32_t wt) {
  if (gt_dense(t, sl)) {
    gt_atomic_add(&t.val[sl.base + (uint32_t)from], (V)-wt);
    gt_atomic_add(&t.val[sl.base + (uint32_t)to], (V)wt);
    return;
  }
  uint32_t hf = 0, ht = 0;
  int32_t kf = kGtEmpty, kt = kGtEmpty;
  if (sl.L) {
    hf = gt_hash(from, sl.L);
    ht = gt_hash(to, sl.L);
    kf = t.key[sl.base + hf];
    kt = t.key[sl.base + ht];
  }
  const int64_t f = gt_slot(t, sl, from, hf, kf, false);
  if (f >= 0) gt_atomic_add(&t.val[f], (V)-wt);
  else atomicAdd(&t.cnt[1], 1u);
  const int64_t s = gt_slot(t, sl, to, ht, kt, true);
  if (s >= 0) gt_atomic_add(&t.val[s], (V)wt);
  else if (atomicExch(&t.flag[v], 1u) == 0u) t.list[atomicAdd(&t.cnt[0], 1u)] = v;
}

// Work items of an update: one per move of a vertex above kGtLaneMax, one per
// chunk above the chunking threshold ({move index, chunk or -1}), listed as
// those of a fill.
__global__ __launch_bounds__(256) void k_gt_move_items(const int4* moves, const uint32_t* count, const int32_t* deg,
                                                       uint32_t thr, int32_t wave_max, int2* items, uint64_t cap,
                                                       uint32_t* nitems) {
  const int64_t m = *count;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x; b < m; b += stride) {
    const int64_t i = b + threadIdx.x;
    uint32_t ni = 0;
    bool wide = false;
    if (i < m) {
      const int4 mv = moves[i];
      if (mv.x >= 0 && mv.y != mv.z) {  // short ones: k_gt_update_lane
        const uint32_t d = (uint32_t)deg[mv.x];
        ni = gt_items_of(d, thr);
        wide = d > (uint32_t)wave_max;
      }
    }
    for (int x = 0; x < 2; ++x) {
      const uint32_t c = wide == (x == 1) ? ni : 0u;
      const uint32_t incl = wave_incl_scan_add(c);
      uint32_t base = 0;
      if (lane_id() == kWave - 1 && incl) base = atomicAdd(nitems + x, incl);
      base = __shfl(base, kWave - 1, kWave);
      for (uint32_t j = 0; j < c; ++j) {
        const uint64_t o = base + incl - c + j;
        items[x ? cap - 1 - o : o] = make_int2((int)i, ni > 1 ? (int)j : -1);
      }
    }
  }
}

// A group of NT threads per update item of a move {u, from, to}: every
// neighbour v of u (in the item's chunk) moves w(u, v) from block `from` to
// block `to` in its slice. A slice without a free slot for `to` is listed for
// a rebuild; a missing `from` entry is counted (cnt[1]; never expected). A
// chain of dependent loads (code, slice, home slots) ends in two atomics, and
// a batch has few long neighbourhoods: those get a workgroup each (40,000
// moves of 2,000,003 R-MAT vertices: 355 us with a wavefront for each, 58 + 144
// us now).
template <int NT, typename V>
__global__ __launch_bounds__(256) void k_gt_update(GraphView g, const int32_t* deg, const int4* moves,
                                                   const int2* items, uint64_t cap, const uint32_t* nitems,
                                                   GtView<V> t) {
  constexpr int G = 256 / NT;
  __shared__ DecodeSmem<NT> dsm[G];
  const int w = threadIdx.x / NT;
  const int64_t ng = (int64_t)gridDim.x * G;
  const uint32_t m = nitems[NT == kWave ? 0 : 1];
  const auto pre = [&](int32_t v) { return gt_slice(t, v); };
  for (int64_t i = (int64_t)blockIdx.x * G + w; i < m; i += ng) {
    const int2 it = items[NT == kWave ? i : (int64_t)cap - 1 - i];
    const int4 mv = moves[it.x];
    const int32_t u = mv.x, from = mv.y, to = mv.z;
    group_visit<NT>(g, u, (uint32_t)deg[u], it.y, dsm[w], pre,
                    [&](int32_t v, int32_t wt, const GtSlice& sl) { gt_move_edge(t, v, sl, from, to, wt); });
  }
}

// One lane per move of a vertex of degree <= kGtLaneMax.
template <typename V>
__global__ __launch_bounds__(256) void k_gt_update_lane(GraphView g, const int32_t* deg, const int4* moves,
                                                        const uint32_t* count, GtView<V> t) {
  const int64_t m = *count;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const int4 mv = moves[i];
    if (mv.x < 0 || mv.y == mv.z) continue;
    const uint32_t d = (uint32_t)deg[mv.x];
    if (d == 0 || d > (uint32_t)kGtLaneMax) continue;
    lane_visit(g, mv.x, d, [&](int32_t v, int32_t wt) { gt_move_edge(t, v, gt_slice(t, v), mv.y, mv.z, wt); });
  }
}

// Rebuilds the listed slices from the current blocks (a slice holds at most
// deg(v) <= L / 2 live blocks, so the rebuild always fits).
template <typename V>
__global__ __launch_bounds__(256) void k_gt_rebuild(GraphView g, const int32_t* deg, const int32_t* blocks,
                                                    GtView<V> t) {
  __shared__ DecodeSmem<kWave> dsm[kGtWaves];
  const int w = threadIdx.x / kWave;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  const uint32_t m = t.cnt[0];
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave; i < m; i += nw) {
    const int32_t v = t.list[i];
    const GtSlice sl = gt_slice(t, v);
    for (uint32_t q = (uint32_t)lane_id(); q < sl.L; q += kWave) {
      t.key[sl.base + q] = kGtEmpty;
      t.val[sl.base + q] = 0;
    }
    __threadfence();
    __builtin_amdgcn_wave_barrier();
    group_visit<kWave>(g, v, (uint32_t)deg[v], -1, dsm[w], [&](int32_t x) { return blocks[x]; },
                       [&](int32_t, int32_t wt, int32_t c) { (void)gt_add(t, sl, c, (V)wt); });
    if (lane_id() == 0) t.flag[v] = 0;
  }
}

// Ends an update: the rebuilt slices are counted (cnt[2]) and the list emptied.
__global__ void k_gt_reset_list(uint32_t* cnt) {
  cnt[2] += cnt[0];
  cnt[0] = 0;
}

template <typename V>
lp_status gt_fill(const GainTable& t, const int32_t* blocks, Scratch& sc) {
  hipStream_t s = sc.stream();
  const lp_graph* g = t.g;
  const GtView<V> v = view_of<V>(t);
  hipLaunchKernelGGL(k_gt_clear<V>, dim3(grid_for((int64_t)t.entries, 256, 65536)), dim3(256), 0, s, t.key, (V*)t.val,
                     t.entries);
  LP_CHECK_LAUNCH();
  if (t.nlane > 0) {
    auto lane = !g->compressed    ? k_gt_fill_lane<false, false, V>
                : g->intervals    ? k_gt_fill_lane<true, true, V>
                                  : k_gt_fill_lane<true, false, V>;
    hipLaunchKernelGGL(lane, dim3(grid_for(t.nlane, 256)), dim3(256), 0, s, g->view(), t.lane, t.nlane, blocks, v);
    LP_CHECK_LAUNCH();
  }
  uint32_t* nitems = t.cnt + 3;
  if (t.nlong > 0) {
    hipLaunchKernelGGL(k_gt_items, dim3(grid_for(t.nlong, 256 * kGtItemRun)), dim3(256), 0, s, t.longer, t.deg,
                       t.nlong, chunk_threshold(g->intervals), t.wave_max, t.items, t.nitems_cap, nitems);
    LP_CHECK_LAUNCH();
    hipLaunchKernelGGL((k_gt_fill_group<kGtThreads, V>), dim3(grid_for(t.nlong, 16, 4096)), dim3(256), 0, s,
                       g->view(), t.deg, blocks, t.items, t.nitems_cap, nitems, v);
    LP_CHECK_LAUNCH();
    hipLaunchKernelGGL((k_gt_fill_group<kWave, V>), dim3(grid_for(t.nlong, 256 / kWave, 16384)), dim3(256), 0, s,
                       g->view(), t.deg, blocks, t.items, t.nitems_cap, nitems, v);
  }
  return last_error();
}

template <typename V>
lp_status gt_select_t(const GainTable& t, const GtRound& r, const int32_t* lane_list, int32_t nlane,
                      const int32_t* wave_list, int32_t nwave, hipStream_t s) {
  const GtView<V> v = view_of<V>(t);
  if (nlane > 0) {
    hipLaunchKernelGGL(k_gt_select_lane<V>, dim3(grid_for(nlane, 256)), dim3(256), 0, s, v, r, lane_list, nlane);
    LP_CHECK_LAUNCH();
  }
  if (nwave > 0) {
    hipLaunchKernelGGL(k_gt_select_wave<V>, dim3(grid_for(nwave, kGtWaves, 1u << 20)), dim3(256), 0, s, v, r,
                       wave_list, nwave);
    LP_CHECK_LAUNCH();
  }
  return LP_OK;
}

template <typename V>
lp_status gt_update_t(const GainTable& t, const int4* moves, const uint32_t* count, int64_t max_moves,
                      const int32_t* blocks, hipStream_t s) {
  const GtView<V> v = view_of<V>(t);
  if (max_moves <= 0) return LP_OK;
  hipLaunchKernelGGL(k_gt_zero, dim3(1), dim3(64), 0, s, t.cnt + 3, (int64_t)2);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gt_move_items, dim3(grid_for(max_moves, 256, 16384)), dim3(256), 0, s, moves, count, t.deg,
                     chunk_threshold(t.g->intervals), t.wave_max, t.items, t.nitems_cap, t.cnt + 3);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL((k_gt_update<kGtThreads, V>), dim3(grid_for(max_moves, 16, 4096)), dim3(256), 0, s, t.g->view(),
                     t.deg, moves, t.items, t.nitems_cap, t.cnt + 3, v);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL((k_gt_update<kWave, V>), dim3(grid_for(max_moves, kGtWaves, 8192)), dim3(256), 0, s,
                     t.g->view(), t.deg, moves, t.items, t.nitems_cap, t.cnt + 3, v);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gt_update_lane<V>, dim3(grid_for(max_moves, 256, 16384)), dim3(256), 0, s, t.g->view(), t.deg,
                     moves, count, v);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gt_rebuild<V>, dim3(256), dim3(256), 0, s, t.g->view(), t.deg, blocks, v);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gt_reset_list, dim3(1), dim3(1), 0, s, t.cnt);
  return last_error();
}

}  // namespace

lp_status gt_create(const lp_graph* g, const int32_t* blocks, int32_t k, hipStream_t s, GainTable* t) {
  *t = GainTable{};
  t->g = g;
  t->k = k;
  t->wide = g->max_wdeg > 0x7FFFFFFFll;
  const int32_t n = g->n;
  uint64_t long_edges = 0;
  LP_CHECK(plan_degrees(g, &t->deg, &t->lane, &t->nlane, &t->longer, &t->nlong, &long_edges, s));
  const uint64_t twice_mean = 2 * long_edges / (uint64_t)std::max(t->nlong, 1);
  t->wave_max = (int32_t)std::min<uint64_t>(std::max<uint64_t>(kGtWaveMax, twice_mean), 0x7FFFFFFF);
  auto grab = [&](size_t bytes) {
    void* p = cache_alloc(bytes ? bytes : 1, s);
    t->bytes += bytes;
    return p;
  };
  t->off = (uint64_t*)grab(((size_t)n + 1) * 8);
  t->flag = (uint32_t*)grab((size_t)n * 4);
  t->list = (int32_t*)grab((size_t)n * 4);
  t->cnt = (uint32_t*)grab(kGtCounters * 4);
  t->nitems_cap = (uint64_t)n + g->two_m / LP_CHUNK_LEN + 1;
  t->items = (int2*)grab(t->nitems_cap * sizeof(int2));
  if (!t->off || !t->flag || !t->list || !t->cnt || !t->items) {
    gt_release(t, s);
    return LP_ENOMEM;
  }
  Scratch sc(s);
  hipLaunchKernelGGL(k_gt_len, dim3(grid_for(n, 256, 65536)), dim3(256), 0, s, t->deg, n, k, t->off,
                     t->flag, t->cnt);
  LP_CHECK_LAUNCH();
  LP_CHECK(scan_exclusive_u64(t->off, t->off, (int64_t)n + 1, nullptr, sc));
  uint64_t entries = 0;
  LP_CHECK_HIP(hipMemcpyAsync(&entries, t->off + n, 8, hipMemcpyDeviceToHost, s));
  LP_CHECK_HIP(hipStreamSynchronize(s));
  t->entries = entries;
  t->key = (int32_t*)grab(entries * 4);
  t->val = grab(entries * (t->wide ? 8 : 4));
  if (!t->key || !t->val) {
    gt_release(t, s);
    return LP_ENOMEM;
  }
  return t->wide ? gt_fill<int64_t>(*t, blocks, sc) : gt_fill<int32_t>(*t, blocks, sc);
}

void gt_release(GainTable* t, hipStream_t s) {
  for (void* p : {(void*)t->off, (void*)t->flag, (void*)t->list, (void*)t->cnt, (void*)t->key, t->val,
                  (void*)t->items})
    if (p) cache_free(p, s);
  *t = GainTable{};
}

lp_status gt_select(const GainTable& t, const GtRound& r, const int32_t* lane_list, int32_t nlane,
                    const int32_t* wave_list, int32_t nwave, hipStream_t s) {
  return t.wide ? gt_select_t<int64_t>(t, r, lane_list, nlane, wave_list, nwave, s)
                : gt_select_t<int32_t>(t, r, lane_list, nlane, wave_list, nwave, s);
}

lp_status gt_update(const GainTable& t, const int4* moves, const uint32_t* count, int64_t max_moves,
                    const int32_t* blocks, hipStream_t s) {
  return t.wide ? gt_update_t<int64_t>(t, moves, count, max_moves, blocks, s)
                : gt_update_t<int32_t>(t, moves, count, max_moves, blocks, s);
}

}  // namespace lp

// ------------------------------------------------------------ public handle --

using namespace lp;

struct lp_gain_table {
  GainTable t;
  int32_t* blocks = nullptr;  // the table's partition
  int4* moves = nullptr;      // n
  uint32_t* bad = nullptr;    // [0] argument errors of the last call, [1] move count
  hipStream_t stream = nullptr;
  int device = 0;
};

namespace lp {
namespace {

__global__ void k_gt_check_blocks(const int32_t* b, int32_t n, int32_t k, uint32_t* bad) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x)
    if ((uint32_t)b[u] >= (uint32_t)k) *bad = 1u;
}

template <typename V>
__global__ void k_gt_query(GtView<V> t, int64_t m, const int32_t* us, const int32_t* bs, int64_t* out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = us[i], b = bs[i];
    out[i] = ((uint32_t)u < (uint32_t)t.n && (uint32_t)b < (uint32_t)t.k) ? (int64_t)gt_get(t, u, b) : -1;
  }
}

// Move batches: vertices in range and distinct (flag exchange), targets in
// range; the flags are cleared again by k_gt_unflag.
__global__ void k_gt_check_moves(const int32_t* us, const int32_t* to, int64_t m, int32_t n, int32_t k, uint32_t* flag,
                                 uint32_t* bad) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = us[i];
    if ((uint32_t)u >= (uint32_t)n || (uint32_t)to[i] >= (uint32_t)k) {
      *bad = 1u;
      continue;
    }
    if (atomicExch(&flag[u], 1u) != 0u) *bad = 1u;
  }
}

__global__ void k_gt_unflag(const int32_t* us, int64_t m, int32_t n, uint32_t* flag) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
    if ((uint32_t)us[i] < (uint32_t)n) flag[us[i]] = 0u;
}

__global__ void k_gt_prep_moves(const int32_t* us, const int32_t* to, int64_t m, int32_t* blocks, int4* moves,
                                uint32_t* count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = us[i];
    moves[i] = make_int4(u, blocks[u], to[i], 0);
    blocks[u] = to[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *count = (uint32_t)m;
}

lp_status host_flag(const uint32_t* dev, hipStream_t s, uint32_t* out) {
  LP_CHECK_HIP(hipMemcpyAsync(out, dev, 4, hipMemcpyDeviceToHost, s));
  LP_CHECK_HIP(hipStreamSynchronize(s));
  return LP_OK;
}

}  // namespace
}  // namespace lp

extern "C" lp_status lp_gain_table_create(const lp_graph* g, const int32_t* blocks, int32_t k, void* stream,
                                          lp_gain_table** out) {
  clear_error();
  if (!g || !out || g->nbatch || k < 1 || (g->n > 0 && (k > g->n || !blocks))) return LP_EINVAL;
  *out = nullptr;
  hipStream_t s = (hipStream_t)stream;
  const int32_t n = g->n;
  auto* h = new lp_gain_table();
  h->stream = s;
  LP_CHECK_HIP(hipGetDevice(&h->device));
  h->blocks = (int32_t*)cache_alloc((size_t)std::max(n, 1) * 4, s);
  h->moves = (int4*)cache_alloc((size_t)std::max(n, 1) * 16, s);
  h->bad = (uint32_t*)cache_alloc(16, s);
  lp_status st = (h->blocks && h->moves && h->bad) ? LP_OK : LP_ENOMEM;
  if (!st) {
    hipLaunchKernelGGL(k_gt_zero, dim3(1), dim3(64), 0, s, h->bad, (int64_t)4);
    if (n > 0) {
      hipLaunchKernelGGL(k_gt_check_blocks, dim3(grid_for(n, 256, 65536)), dim3(256), 0, s, blocks, n, k, h->bad);
      uint32_t bad = 0;
      st = host_flag(h->bad, s, &bad);
      if (!st && bad) st = LP_EINVAL;
    }
  }
  if (!st && n > 0 && hipMemcpyAsync(h->blocks, blocks, (size_t)n * 4, hipMemcpyDeviceToDevice, s) != hipSuccess)
    st = LP_EDEVICE;
  if (!st && n > 0) st = gt_create(g, h->blocks, k, s, &h->t);
  if (!st && n == 0) {
    h->t.g = g;
    h->t.k = k;
  }
  if (st) {
    lp_gain_table_free(h);
    return st;
  }
  *out = h;
  return LP_OK;
}

extern "C" lp_status lp_gain_table_affinity(const lp_gain_table* h, int64_t count, const int32_t* vertices,
                                            const int32_t* blocks, int64_t* out, void* stream) {
  clear_error();
  if (!h || count < 0 || (count > 0 && (!vertices || !blocks || !out))) return LP_EINVAL;
  if (count == 0) return LP_OK;
  hipStream_t s = (hipStream_t)stream;
  const unsigned grid = grid_for(count, 256, 65536);
  if (h->t.g->n == 0) return LP_EINVAL;
  if (h->t.wide)
    hipLaunchKernelGGL(k_gt_query<int64_t>, dim3(grid), dim3(256), 0, s, view_of<int64_t>(h->t), count, vertices,
                       blocks, out);
  else
    hipLaunchKernelGGL(k_gt_query<int32_t>, dim3(grid), dim3(256), 0, s, view_of<int32_t>(h->t), count, vertices,
                       blocks, out);
  return last_error();
}

extern "C" lp_status lp_gain_table_move(lp_gain_table* h, int64_t count, const int32_t* vertices, const int32_t* to,
                                        void* stream) {
  clear_error();
  if (!h || count < 0 || (count > 0 && (!vertices || !to))) return LP_EINVAL;
  const int32_t n = h->t.g->n;
  if (count == 0) return LP_OK;
  if (count > n) return LP_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const unsigned grid = grid_for(count, 256, 65536);
  hipLaunchKernelGGL(k_gt_zero, dim3(1), dim3(64), 0, s, h->bad, (int64_t)1);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gt_check_moves, dim3(grid), dim3(256), 0, s, vertices, to, count, n, h->t.k, h->t.flag, h->bad);
  LP_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gt_unflag, dim3(grid), dim3(256), 0, s, vertices, count, n, h->t.flag);
  LP_CHECK_LAUNCH();
  uint32_t bad = 0;
  LP_CHECK(host_flag(h->bad, s, &bad));
  if (bad) return LP_EINVAL;
  hipLaunchKernelGGL(k_gt_prep_moves, dim3(grid), dim3(256), 0, s, vertices, to, count, h->blocks, h->moves,
                     h->bad + 1);
  LP_CHECK_LAUNCH();
  return gt_update(h->t, h->moves, h->bad + 1, count, h->blocks, s);
}

extern "C" lp_status lp_gain_table_info(const lp_gain_table* h, uint64_t* entries, uint64_t* bytes, int64_t* missing,
                                        int64_t* rebuilds) {
  clear_error();
  if (!h) return LP_EINVAL;
  if (entries) *entries = h->t.entries;
  if (bytes) *bytes = h->t.bytes;
  uint32_t c[4] = {0, 0, 0, 0};
  if ((missing || rebuilds) && h->t.cnt) {
    LP_CHECK_HIP(hipMemcpyAsync(c, h->t.cnt, sizeof(c), hipMemcpyDeviceToHost, h->stream));
    LP_CHECK_HIP(hipStreamSynchronize(h->stream));
  }
  if (missing) *missing = c[1];
  if (rebuilds) *rebuilds = c[2];
  return LP_OK;
}

extern "C" void lp_gain_table_free(lp_gain_table* h) {
  if (!h) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  (void)hipSetDevice(h->device);
  gt_release(&h->t, h->stream);
  for (void* p : {(void*)h->blocks, (void*)h->moves, (void*)h->bad})
    if (p) cache_free(p, h->stream);
  (void)hipSetDevice(cur);
  delete h;
}

// Graph handles: validation, GPU compression into the gap + VarInt format
// (Section III-A), decompression, degree extraction from the first-edge-ID
// headers, and the plain-CSR handle.
#include <string.h>

#include "decode.h"
#include "graph.h"

namespace lp {

namespace {

enum : uint32_t {
  kErrRange = 1,
  kErrSelf = 2,
  kErrWeight = 4,
  kErrOrder = 8,
  kErrVwgt = 32,
};

__device__ __forceinline__ uint32_t varint_len(uint64_t x) {
  return ((70u - (uint32_t)__clzll((long long)(x | 1u))) * 37u) >> 8;  // ceil(bits / 7) for 1..64 bits
}

__device__ __forceinline__ uint32_t varint_put(uint8_t* out, uint64_t x) {
  uint32_t k = 0;
  while (x >= 0x80) {
    out[k++] = (uint8_t)((x & 0x7F) | 0x80);
    x >>= 7;
  }
  out[k++] = (uint8_t)x;
  return k;
}

struct CsrIn {
  int32_t n;
  const uint64_t* xadj;
  const int32_t* adjncy;
  const int32_t* adjwgt;
  const int32_t* vwgt;
};

// Work is handed out along the merged sequence of vertices and adjacency
// entries: vertex u sits at key(u) = xadj[u] + u, its entries right after it,
// so a stretch of T positions holds T vertices and entries together however
// the degrees vary (hubs spread over many stretches, a run of isolated
// vertices too). blk[c] is the first vertex at or after position c * T;
// stretch c holds the vertices blk[c] .. blk[c + 1] - 1 and the entries from
// c * T - blk[c] on (the first of them may belong to vertex blk[c] - 1).

// blk[c] = the smallest u with key(u) >= c * work (c < nb), blk[nb] = n.
// xadj must be non-decreasing from 0 (a decrease sets *err and leaves blk
// incomplete).
__global__ void k_codec_blocks(const uint64_t* xadj, int64_t n, uint64_t work, int64_t nb, int64_t* blk,
                               uint32_t* err) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u <= n; u += (int64_t)gridDim.x * blockDim.x) {
    if (u > 0 && xadj[u] < xadj[u - 1]) {
      atomicOr(err, 1u);
      continue;
    }
    const uint64_t hi = xadj[u] + (uint64_t)u;
    // blocks c with key(u - 1) < c * work <= key(u) (u > 0), or c = 0
    const int64_t c0 = u ? (int64_t)((xadj[u - 1] + (uint64_t)(u - 1)) / work) + 1 : 0;
    const int64_t c1 = min((int64_t)(hi / work), nb - 1);
    for (int64_t c = c0; c <= c1; ++c) blk[c] = u;
    if (u == n) blk[nb] = n;
  }
}

// ------------------------------------------------ compression of a CSR ----
// One workgroup per stretch of kCtWork positions, kCtItems consecutive
// entries per thread, so the adjacency is read in order at full width
// whatever the degrees. Two passes: k_csr_scan checks the input and sums the
// stretch's code bytes, k_csr_encode (after a prefix sum over the stretches)
// computes the codes again, places them by a prefix sum inside the workgroup,
// gathers them in LDS and stores them as 16-byte words. What bounds it is the
// adjacency read twice and the codes written once. A wave per vertex, as
// before, kept most lanes idle on low degrees and waited on a chain of
// dependent loads per vertex: R-MAT with 2^23 vertices and 2.4e8 entries took
// 7.0 ms to check, 11.1 ms to size and 10.7 ms to encode, and takes 0.35 ms
// for the first two together and 0.65 ms for the last (0.97 GB of adjacency
// and 0.5 GB of codes: 2.3 TB/s; the instructions per entry are what is left).
constexpr int kCtThreads = 256;
constexpr int kCtItems = 8;
constexpr int kCtWork = kCtThreads * kCtItems;

// What the passes find out about the input (device memory, zeroed).
struct CsrAcc {
  uint32_t xerr;  // xadj decreases (set before the passes, which then do nothing)
  uint32_t err;
  unsigned long long wdeg, deg, vtot;
  uint64_t nbytes;
  uint32_t nsplit, pad;  // vertices whose records are split into chunks (counted by the encoder)
};

// Code length of a VarInt below 2^32, and of the 32-bit zigzag of a
// difference of two IDs or two weights (all in [0, 2^31), so it fits).
__device__ __forceinline__ uint32_t varint_len32(uint32_t x) {
  return ((38u - (uint32_t)__clz((int)(x | 1u))) * 37u) >> 8;  // ceil(bits / 7)
}
__device__ __forceinline__ uint32_t zigzag32(int32_t d) { return ((uint32_t)d << 1) ^ (uint32_t)(d >> 31); }

// The part of the merged sequence a workgroup takes, and the two vertices of
// it that may be split into chunks: the one whose entries it continues
// (kind 0) and the last one it starts (kind 1). Others have fewer entries
// than the stretch has positions.
struct CtSpan {
  int64_t v0;
  int32_t nv, ne;       // vertices started here, entries
  uint64_t e0;          // first entry
  uint64_t x[2];        // first entry of the vertex of each kind
  uint32_t chunked[2];  // it is split into chunks
  uint64_t table;       // bytes of the chunk table that follows the header of the vertex of kind 1
};
static_assert(LP_CHUNK_THRESHOLD >= kCtWork, "only the last vertex a stretch starts can be split");

__device__ __forceinline__ CtSpan ct_span(const CsrIn& g, const int64_t* blk, int64_t nb, int64_t c) {
  CtSpan sp;
  const uint64_t two_m = g.xadj[g.n];
  const int64_t v0 = blk[c], v1 = blk[c + 1];
  sp.v0 = v0;
  sp.nv = (int32_t)(v1 - v0);
  sp.e0 = (uint64_t)c * kCtWork - (uint64_t)v0;
  uint64_t e1 = c + 1 < nb ? (uint64_t)(c + 1) * kCtWork - (uint64_t)v1 : two_m;
  if (e1 > two_m) e1 = two_m;
  sp.ne = e1 > sp.e0 ? (int32_t)(e1 - sp.e0) : 0;
  sp.chunked[0] = sp.chunked[1] = 0;
  sp.x[0] = sp.x[1] = 0;
  sp.table = 0;
  if (v0 > 0) {
    sp.x[0] = g.xadj[v0 - 1];
    sp.chunked[0] = g.xadj[v0] - sp.x[0] > LP_CHUNK_THRESHOLD;
  }
  if (v1 > v0) {
    sp.x[1] = g.xadj[v1 - 1];
    const uint64_t d = g.xadj[v1] - sp.x[1];
    sp.chunked[1] = d > LP_CHUNK_THRESHOLD;
    if (sp.chunked[1]) sp.table = 4 * ((d + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN - 1);
  }
  return sp;
}

// Owner marks: own[j] = 1 + the index (in the stretch) of the vertex whose
// neighbourhood starts at entry j, 0 elsewhere. own must be zero. f(i, d) for
// every vertex i with its degree.
template <typename F>
__device__ __forceinline__ void ct_mark(const CsrIn& g, const CtSpan& sp, uint16_t* own, F&& f) {
  for (int32_t i = threadIdx.x; i < sp.nv; i += kCtThreads) {
    const uint64_t x = g.xadj[sp.v0 + i], d = g.xadj[sp.v0 + i + 1] - x;
    const uint64_t pos = x - sp.e0;
    if (d > 0 && pos < (uint64_t)sp.ne) own[pos] = (uint16_t)(i + 1);
    f(i, x, d);
  }
}

// This thread's entries j0 .. j0 + kCtItems - 1 and the one before them,
// loaded before anything is known about their vertices.
template <bool WGT>
struct CtEntries {
  int32_t v[kCtItems], w[kCtItems];
  int32_t pv, pw;

  __device__ __forceinline__ CtEntries(const CsrIn& g, const CtSpan& sp) {
    load(g.adjncy + sp.e0, sp.ne, v, 0);
    pv = before(g.adjncy + sp.e0, sp, v[kCtItems - 1]);
    pw = 0;
    if constexpr (WGT) {
      load(g.adjwgt + sp.e0, sp.ne, w, 1);
      pw = before(g.adjwgt + sp.e0, sp, w[kCtItems - 1]);
    }
  }

 private:
  struct __attribute__((packed, aligned(4))) Four {
    int32_t x[4];
  };
  static __device__ __forceinline__ void load(const int32_t* a, int32_t ne, int32_t* x, int32_t fill) {
    const int32_t j0 = (int32_t)threadIdx.x * kCtItems;
    static_assert(kCtItems == 8, "two 16-byte loads");
    if (j0 + kCtItems <= ne) {
      const Four p = *(const Four*)(a + j0), q = *(const Four*)(a + j0 + 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        x[k] = p.x[k];
        x[4 + k] = q.x[k];
      }
    } else {
#pragma unroll
      for (int k = 0; k < kCtItems; ++k) x[k] = j0 + k < ne ? a[j0 + k] : fill;
    }
  }
  // the entry before this thread's first: the lane before has it
  static __device__ __forceinline__ int32_t before(const int32_t* a, const CtSpan& sp, int32_t last) {
    const int32_t j0 = (int32_t)threadIdx.x * kCtItems;
    int32_t p = dpp_i32<0x138>(last);
    if (lane_id() == 0 && j0 < sp.ne && sp.e0 + j0 > 0) p = a[j0 - 1];
    return p;
  }
};

// f(k, own, first, start, u, v, pv, w, pw) for each of this thread's entries;
// own = 1 + index of the vertex (0: the one continued from the stretch
// before), first: it begins the neighbourhood, start: it begins a chunk, pv /
// pw the entry before (meaningless at `first`).
template <bool WGT, typename F>
__device__ __forceinline__ void ct_entries(const CtEntries<WGT>& en, const CtSpan& sp, const uint16_t* own,
                                           int32_t* scan_sm, F&& f) {
  const int32_t j0 = (int32_t)threadIdx.x * kCtItems;
  int32_t pv = en.pv, pw = en.pw;
  const uint4 ow = *(const uint4*)&own[j0];  // kCtItems == 8 marks
  uint16_t o[kCtItems];
  __builtin_memcpy(o, &ow, 16);
  int32_t top = 0;
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) top = max(top, (int32_t)o[k]);
  // exclusive prefix maximum over the threads
  const int32_t inc = wave_incl_scan_max_i32(top);
  const int wv = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) scan_sm[wv] = inc;
  __syncthreads();
  int32_t cur = dpp_i32<0x138>(inc);
  for (int k = 0; k < wv; ++k) cur = max(cur, scan_sm[k]);
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) {
    if (j0 + k >= sp.ne) continue;
    if (o[k]) cur = o[k];
    // the stretch before may end with the vertex whose first entry is this one's first
    const bool first = o[k] != 0 || (cur == 0 && sp.e0 + j0 + k == sp.x[0]);
    bool start = first;
    if (sp.chunked[0] | sp.chunked[1]) {  // uniform
      const int kind = cur == 0 ? 0 : 1;
      if (!first && sp.chunked[kind] && (kind == 0 || cur == sp.nv))
        start = (uint32_t)(sp.e0 + j0 + k - sp.x[kind]) % LP_CHUNK_LEN == 0;
    }
    f(k, (uint32_t)cur, first, start, (int32_t)(sp.v0 - 1 + cur), en.v[k], pv, en.w[k], pw);
    pv = en.v[k];
    pw = en.w[k];
  }
}

// Checks (range, self-loops, weights, order), the largest degree of the
// stretch's vertices (tdeg[c]) and weighted degree (tw[c]) and, with SIZE,
// the stretch's code bytes (tsize[c], gap-only format). Weighted degrees of
// vertices that continue into other stretches are summed in wspan[stretch
// that starts them] (zeroed). c0: the launch's first stretch (here and in the
// kernels below).
template <bool WGT, bool SIZE>
__global__ __launch_bounds__(kCtThreads) void k_csr_scan(CsrIn g, const int64_t* blk, int64_t nb, int64_t c0,
                                                         CsrAcc* acc, uint32_t* tdeg, unsigned long long* tw,
                                                         unsigned long long* wspan, uint64_t* tsize) {
  __shared__ __align__(16) uint16_t own[kCtWork];
  __shared__ unsigned long long wsum[WGT ? kCtWork + 1 : 1];
  __shared__ int32_t scan[kCtThreads / kWave];
  __shared__ uint32_t red32[kCtThreads / kWave], redl[kCtThreads / kWave];
  __shared__ unsigned long long red[kCtThreads / kWave];
  if (acc->xerr) return;
  const int64_t c = c0 + blockIdx.x;
  const CtSpan sp = ct_span(g, blk, nb, c);
  const CtEntries<WGT> en(g, sp);
  *(uint4*)&own[threadIdx.x * kCtItems] = make_uint4(0, 0, 0, 0);
  if constexpr (WGT)
    for (int32_t i = threadIdx.x; i <= sp.nv; i += kCtThreads) wsum[i] = 0;
  __syncthreads();
  uint32_t md = 0, len = 0, bad = 0;
  ct_mark(g, sp, own, [&](int32_t, uint64_t x, uint64_t d) {
    md = max(md, (uint32_t)min(d, (uint64_t)0xFFFFFFFFu));
    if constexpr (SIZE) len += varint_len(x);
  });
  __syncthreads();
  uint32_t run_own = 0;
  int64_t run = 0;
  ct_entries<WGT>(en, sp, own, scan, [&](int k, uint32_t o, bool first, bool start, int32_t u, int32_t v, int32_t pv,
                                        int32_t w, int32_t pw) {
    if ((uint32_t)v >= (uint32_t)g.n) bad |= kErrRange;
    if (v == u) bad |= kErrSelf;
    if (!first && (pv > v || (WGT && pv == v && pw > w))) bad |= kErrOrder;
    if constexpr (WGT) {
      if (w < 1) bad |= kErrWeight;
      if (k == 0) run_own = o;
      if (o != run_own) {
        atomicAdd(&wsum[run_own], (unsigned long long)run);
        run = 0;
        run_own = o;
      }
      run += w;
    }
    if constexpr (SIZE) {
      len += varint_len32(start ? zigzag32(v - u) : (uint32_t)(v - pv));
      if constexpr (WGT) len += varint_len32(zigzag32(w - (start ? 0 : pw)));
    }
  });
  unsigned long long mw = 0;
  if constexpr (WGT) {
    if (run) atomicAdd(&wsum[run_own], (unsigned long long)run);
    __syncthreads();
    for (int32_t i = threadIdx.x; i <= sp.nv; i += kCtThreads) {
      const unsigned long long s = wsum[i];
      if (i == 0) {
        if (s) {
          const int64_t u = sp.v0 - 1;
          atomicAdd(&wspan[(int64_t)((g.xadj[u] + (uint64_t)u) / kCtWork)], s);
        }
      } else if (i == sp.nv && g.xadj[sp.v0 + sp.nv] > sp.e0 + (uint64_t)sp.ne) {
        atomicAdd(&wspan[c], s);
      } else {
        mw = max(mw, s);
      }
    }
    mw = wave_reduce_max(mw);
    if (lane_id() == 0) red[threadIdx.x / kWave] = mw;
  }
  md = wave_reduce_max(md);
  if (lane_id() == 0) red32[threadIdx.x / kWave] = md;
  if (bad) atomicOr(&acc->err, bad);
  len = wave_reduce_add(len);
  if (lane_id() == 0) redl[threadIdx.x / kWave] = len;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kCtThreads / kWave; ++k) {
      md = max(md, red32[k]);
      len += redl[k];
      if constexpr (WGT) mw = max(mw, red[k]);
    }
    tdeg[c] = md;
    if constexpr (WGT) tw[c] = mw;
    if constexpr (SIZE) tsize[c] = (uint64_t)len + sp.table;
  }
}

// Maxima over the stretches: degree (0xFFFFFFFF and more count as that) and
// weighted degree, the latter also over the vertices that span several.
__global__ __launch_bounds__(256) void k_csr_max(const uint32_t* tdeg, const unsigned long long* tw,
                                                 const unsigned long long* wspan, int64_t nb, CsrAcc* acc) {
  unsigned long long mw = 0, md = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += (int64_t)gridDim.x * blockDim.x) {
    md = max(md, (unsigned long long)tdeg[i]);
    if (tw) mw = max(mw, max(tw[i], wspan[i]));
  }
  md = wave_reduce_max(md);
  mw = wave_reduce_max(mw);
  if (lane_id() == 0 && md) atomicMax(&acc->deg, md);
  if (lane_id() == 0 && mw) atomicMax(&acc->wdeg, mw);
}

// A VarInt of len <= 5 bytes (x below 2^35) into zeroed LDS at byte q: its
// dwords are shared with the codes around it, hence the ORs.
__device__ __forceinline__ void put5(uint32_t* buf, uint32_t q, uint64_t x, uint32_t len) {
  const uint32_t l = (uint32_t)x;
  const uint32_t lo = (l & 0x7Fu) | ((l << 1) & 0x7F00u) | ((l << 2) & 0x7F0000u) | ((l << 3) & 0x7F000000u) |
                      (uint32_t)(0x80808080ull >> (40u - 8u * len));
  const uint64_t y = (((uint64_t)(uint32_t)(x >> 28) << 32) | lo) << (8u * (q & 3u));
  atomicOr(&buf[q >> 2], (uint32_t)y);
  if ((q & 3u) + len > 4u) atomicOr(&buf[(q >> 2) + 1], (uint32_t)(y >> 32));
}

// Any VarInt, byte by byte.
__device__ __forceinline__ void put_any(uint32_t* buf, uint32_t q, uint64_t x) {
  for (;; ++q) {
    const uint32_t c = (uint32_t)(x & 0x7F) | (x >= 0x80 ? 0x80u : 0u);
    atomicOr(&buf[q >> 2], c << (8u * (q & 3u)));
    if (x < 0x80) return;
    x >>= 7;
  }
}

// Bytes [lo, hi) of the output from LDS (byte p at buf[p - shift], shift a
// multiple of 16): whole 16-byte words as such, the ends byte by byte (the
// neighbouring stretches write the rest of those words).
__device__ __forceinline__ void ct_flush(const uint8_t* buf, uint8_t* out, uint64_t lo, uint64_t hi, uint64_t shift) {
  for (uint64_t q = (lo & ~15ull) + 16ull * threadIdx.x; q < hi; q += 16ull * kCtThreads) {
    if (q >= lo && q + 16 <= hi) {
      *(uint4*)(out + q) = *(const uint4*)(buf + (q - shift));
    } else {
      const uint64_t a = max(q, lo), b = min(q + 16, hi);
      for (uint64_t p = a; p < b; ++p) out[p] = buf[p - shift];
    }
  }
}

// Writes the records of the stretch at tbase[c] and the record offsets of its
// vertices. Chunks after a neighbourhood's first one note their position in
// cpos[first entry / LP_CHUNK_LEN] (chunk starts are at least LP_CHUNK_LEN
// entries apart), from which k_chunk_tables fills the chunk tables of the
// vertices in split_list. WIDE: a number may take ten bytes (first-edge IDs
// of 2^35 on), otherwise five.
template <bool WGT, bool WIDE>
__global__ __launch_bounds__(kCtThreads) void k_csr_encode(CsrIn g, const int64_t* blk, int64_t nb, int64_t c0,
                                                           const uint64_t* tbase, uint64_t* offs, uint64_t* cpos,
                                                           int32_t* split_list, uint32_t* nsplit, uint8_t* out) {
  // each position takes at most one header, or one neighbour code and weight code
  constexpr uint32_t kBytes = (WGT || WIDE ? 10u : 5u) * kCtWork + 48u;
  constexpr uint32_t kWords = (kBytes + 15u) / 16u * 4u;
  __shared__ __align__(16) uint32_t buf[kWords];
  __shared__ __align__(16) uint16_t own[kCtWork];
  __shared__ uint16_t hx[kCtWork + 1];  // header bytes of the stretch's vertices before each one
  __shared__ uint16_t sx[kCtWork + 1];  // code bytes of the stretch's entries before each one
  __shared__ int32_t scan[kCtThreads / kWave];
  const int64_t c = c0 + blockIdx.x;
  const CtSpan sp = ct_span(g, blk, nb, c);
  const CtEntries<WGT> en(g, sp);
  const int32_t t0 = (int32_t)threadIdx.x * kCtItems;
  *(uint4*)&own[t0] = make_uint4(0, 0, 0, 0);
  for (uint32_t q = 4 * threadIdx.x; q < kWords; q += 4 * kCtThreads) *(uint4*)&buf[q] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  ct_mark(g, sp, own, [](int32_t, uint64_t, uint64_t) {});
  // vertices are few in most stretches: `per` consecutive ones per thread, no more than are needed
  const int32_t per = (sp.nv + kCtThreads - 1) / kCtThreads;
  const int32_t i0 = (int32_t)threadIdx.x * per;
  uint64_t hv[kCtItems];
  uint32_t hl = 0;
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) {
    if (k >= per) break;
    hv[k] = 0;
    if (i0 + k < sp.nv) {
      hv[k] = g.xadj[sp.v0 + i0 + k];
      hl += varint_len(hv[k]);
    }
  }
  __syncthreads();
  uint32_t code[kCtItems], wcode[kCtItems], ow[kCtItems], sl = 0;
  uint32_t starts = 0;
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) code[k] = wcode[k] = ow[k] = 0;
  ct_entries<WGT>(en, sp, own, scan, [&](int k, uint32_t o, bool first, bool start, int32_t u, int32_t v, int32_t pv,
                                        int32_t w, int32_t pw) {
    code[k] = start ? zigzag32(v - u) : (uint32_t)(v - pv);
    sl += varint_len32(code[k]);
    if constexpr (WGT) {
      wcode[k] = zigzag32(w - (start ? 0 : pw));
      sl += varint_len32(wcode[k]);
    }
    ow[k] = o;
    starts |= (uint32_t)(start && !first) << k;
  });
  // both prefix sums at once: at most 10 * kCtWork bytes each, 16 bits
  static_assert(10 * kCtWork < 65536, "two sums share a word");
  int32_t tot;
  const uint32_t pk = (hl << 16) | sl;
  const uint32_t ex = (uint32_t)block_incl_scan_add<kCtThreads, int32_t>((int32_t)pk, scan, &tot) - pk;
  uint32_t ho = ex >> 16, so = ex & 0xFFFFu;
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) {
    if (k >= per) break;
    if (i0 + k < sp.nv) {
      hx[i0 + k] = (uint16_t)ho;
      ho += varint_len(hv[k]);
    }
  }
  uint32_t s = so;
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) {
    if (t0 + k <= sp.ne) sx[t0 + k] = (uint16_t)s;
    if (t0 + k < sp.ne) s += varint_len32(code[k]) + (WGT ? varint_len32(wcode[k]) : 0u);
  }
  if (threadIdx.x == 0) hx[sp.nv] = (uint16_t)((uint32_t)tot >> 16);
  __syncthreads();
  const uint64_t base = tbase[c];
  const uint64_t shift = base & ~15ull;
  // codes of the split vertex started here follow its table: their bytes sit
  // in LDS as if the table took table % 16 bytes
  const uint64_t gap = sp.table, lgap = gap & ~15ull;
  const uint64_t cut = sp.nv > 0 ? base + hx[sp.nv] + sx[g.xadj[sp.v0 + sp.nv - 1] - sp.e0] : base;
  const uint32_t b0 = (uint32_t)(base - shift);
  // headers
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) {
    if (k >= per) break;
    if (i0 + k >= sp.nv) continue;
    const uint32_t q = hx[i0 + k] + sx[hv[k] - sp.e0];
    offs[sp.v0 + i0 + k] = base + q;
    if constexpr (WIDE) put_any(buf, b0 + q, hv[k]);
    else put5(buf, b0 + q, hv[k], varint_len(hv[k]));
  }
  // codes
  uint32_t hb[kCtItems];
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) hb[k] = hx[ow[k]];
#pragma unroll
  for (int k = 0; k < kCtItems; ++k) {
    if (t0 + k >= sp.ne) continue;
    const uint32_t q = hb[k] + so;
    uint32_t lq = b0 + q;
    if (gap && (int32_t)ow[k] == sp.nv) lq += (uint32_t)(gap - lgap);
    if ((starts >> k) & 1u)
      cpos[(sp.e0 + t0 + k) / LP_CHUNK_LEN] = base + q + ((int32_t)ow[k] == sp.nv ? gap : 0);
    const uint32_t l = varint_len32(code[k]);
    put5(buf, lq, code[k], l);
    so += l;
    if constexpr (WGT) {
      const uint32_t lw = varint_len32(wcode[k]);
      put5(buf, lq + l, wcode[k], lw);
      so += lw;
    }
  }
  if (gap && threadIdx.x == 0) split_list[atomicAdd(nsplit, 1u)] = (int32_t)(sp.v0 + sp.nv - 1);
  __syncthreads();
  const uint64_t end = base + ((uint32_t)tot >> 16) + ((uint32_t)tot & 0xFFFFu);
  if (gap) {
    ct_flush((const uint8_t*)buf, out, base, cut, shift);
    ct_flush((const uint8_t*)buf, out, cut + gap, end + gap, shift + lgap);
  } else {
    ct_flush((const uint8_t*)buf, out, base, end, shift);
  }
}

// The chunk tables of the listed split records (wave per record).
__global__ __launch_bounds__(256) void k_chunk_tables(CsrIn g, const int32_t* list, const uint32_t* cnt,
                                                      const uint64_t* offs, const uint64_t* cpos, uint8_t* out) {
  const uint32_t m = *cnt, nw = gridDim.x * blockDim.x / kWave;
  for (uint32_t i = (blockIdx.x * blockDim.x + threadIdx.x) / kWave; i < m; i += nw) {
    const int64_t u = list[i];
    const uint64_t x = g.xadj[u], d = g.xadj[u + 1] - x, o = offs[u];
    const uint64_t table = o + varint_len(x), nch = (d + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN;
    for (uint64_t j = 1 + (uint64_t)lane_id(); j < nch; j += kWave) {
      const uint32_t rel = (uint32_t)(cpos[(x + j * LP_CHUNK_LEN) / LP_CHUNK_LEN] - o);
      uint8_t* t = out + table + 4 * (j - 1);
      t[0] = (uint8_t)rel;
      t[1] = (uint8_t)(rel >> 8);
      t[2] = (uint8_t)(rel >> 16);
      t[3] = (uint8_t)(rel >> 24);
    }
  }
}

__global__ __launch_bounds__(256) void k_vwgt_check(const int32_t* vwgt, int32_t n, uint32_t* err,
                                                    unsigned long long* total) {
  __shared__ int64_t sm[4];
  int64_t s = 0;
  uint32_t bad = 0;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
    const int32_t w = vwgt[u];
    if (w < 1) bad = kErrVwgt;
    s += w;
  }
  s = block_reduce_add<256, int64_t>(s, sm);
  if (threadIdx.x == 0) atomicAdd(total, (unsigned long long)s);
  if (bad) atomicOr(err, bad);
}

// ------------------------------------------------- interval encoding ----
// Interval-coded records (Section III-A; layout in lp.h), one workgroup per
// stretch of the merged sequence, as above. It codes the segments (unsplit
// neighbourhoods, chunks of split ones) that start in its stretch, run by
// run; a run's entries lie one after another, kItvShare consecutive ones per
// thread at most. Whether an entry is part of an interval is decided by the
// entries next to it: it is if three in a row with consecutive IDs include
// it. An interval's last entry codes the pair, prefix maxima give every entry
// the residual and the interval neighbour before it, and prefix sums of the
// bytes per section place everything. A lane per record, as before, read the
// adjacency four times at a stride: an RGG-3D of 1e6 vertices with weights
// (2.7e7 entries) took 1.1 ms to size and 1.6 ms to encode, and one hub of
// 10^5 neighbours more than all other records; it takes 0.33 and 0.66 ms now,
// bound by instructions (the code is long: with the run's body inlined at
// every use, or sixteen entries per thread, it outgrew the instruction cache
// and took twice as long).
constexpr int kItvThreads = 512;
constexpr int kItvShare = 8;
constexpr int kItvMax = kItvThreads * kItvShare;  // most entries of a run
constexpr int kItvWork = 2048;                    // positions of a stretch: 42 KB of LDS, three workgroups a CU
static_assert(LP_ITV_CHUNK_THRESHOLD >= kItvWork && LP_ITV_CHUNK_THRESHOLD <= kItvMax &&
                  kItvWork + LP_CHUNK_LEN <= kItvMax && LP_CHUNK_THRESHOLD >= LP_ITV_CHUNK_THRESHOLD,
              "a run holds a stretch's neighbourhoods but the last, one unsplit neighbourhood, or a stretch's chunks");

struct ItvShared {
  __align__(16) uint16_t own[kItvMax + 8];  // 1 + segment that starts at the entry
  uint16_t es[kItvWork + 2];                // first entry of every segment
  uint16_t lastiv[kItvWork + 2];            // 1 + last interval neighbour up to the segment's end
  uint32_t sa[kItvWork + 2];  // bytes before the segment's first entry: pairs << 16 | interval weights
  uint32_t sb[kItvWork + 2];  // residuals << 16 | intervals (when sizing: the segment's intervals)
  uint32_t sec[kItvWork + 2];    // first section of the segment, from the run's start
  uint16_t cb[kItvThreads + 2];  // per thread: which of its entries continue a run of consecutive IDs
  int32_t scan[3][kItvThreads / kWave];
};

struct ItvRun {
  uint64_t e0;        // first entry
  int32_t m, nseg;    // entries, segments (starts in ItvShared::es)
  int64_t u;          // vertex of segment i: u + i * ustep
  int32_t ustep;
  bool hdr;           // segments are records: a first-edge header each
  bool chunk0;        // segments are chunks, the first of them the neighbourhood's first
};

__device__ __forceinline__ void put_bytes(uint8_t* out, uint64_t pos, uint32_t x) {
  while (x >= 0x80u) {
    out[pos++] = (uint8_t)(x | 0x80u);
    x >>= 7;
  }
  out[pos] = (uint8_t)x;
}

// Exclusive prefix maxima over the workgroup of three values per thread.
__device__ __forceinline__ void itv_scan_max3(int32_t (&x)[3], int32_t (*sm)[kItvThreads / kWave]) {
  int32_t inc[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) inc[q] = wave_incl_scan_max_i32(x[q]);
  const int wv = threadIdx.x / kWave;
  if (lane_id() == kWave - 1)
    for (int q = 0; q < 3; ++q) sm[q][wv] = inc[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    x[q] = dpp_i32<0x138>(inc[q]);
    for (int k = 0; k < wv; ++k) x[q] = max(x[q], sm[q][k]);
  }
  __syncthreads();
}

// Codes one run (es[0..nseg] set and visible); returns its bytes. WRITE: at
// `base`, with the record offsets (hdr) or the chunk positions (cpos, as for
// the gap format).
template <bool WGT, bool WRITE>
__device__ uint32_t itv_run(const CsrIn& g, ItvShared& sh, const ItvRun& r, uint64_t base, uint64_t* offs,
                            uint64_t* cpos, uint8_t* out) {
  const int tid = threadIdx.x;
  const int32_t per = (r.m + kItvThreads - 1) / kItvThreads;
  const int32_t j0 = tid * per;
  const int32_t* ids = g.adjncy + r.e0;
  const int32_t* wts = WGT ? g.adjwgt + r.e0 : nullptr;
  int32_t id[kItvShare], w[WGT ? kItvShare : 1];
  int32_t before = 0;
#pragma unroll
  for (int32_t k = 0; k < kItvShare; ++k) {
    id[k] = 0;
    if (k < per && j0 + k < r.m) {
      id[k] = ids[j0 + k];
      if constexpr (WGT) w[k] = wts[j0 + k];
    }
  }
  if (j0 > 0 && j0 < r.m) before = ids[j0 - 1];
  for (int32_t q = 8 * tid; q < r.m + 8; q += 8 * kItvThreads) *(uint4*)&sh.own[q] = make_uint4(0, 0, 0, 0);
  if constexpr (!WRITE)
    for (int32_t i = tid; i < r.nseg; i += kItvThreads) sh.sb[i] = 0;
  __syncthreads();
  for (int32_t i = tid; i < r.nseg; i += kItvThreads)
    if (sh.es[i + 1] > sh.es[i]) sh.own[sh.es[i]] = (uint16_t)(i + 1);
  __syncthreads();
  // runs of consecutive IDs
  uint32_t c = 0, heads = 0;
  int32_t top = 0;
#pragma unroll
  for (int32_t k = 0; k < kItvShare; ++k) {
    if (k >= per || j0 + k >= r.m) continue;
    const int32_t o = sh.own[j0 + k];
    if (o) {
      top = o;
      heads |= 1u << k;
    } else if (id[k] == (k ? id[(k + kItvShare - 1) % kItvShare] : before) + 1) {
      c |= 1u << k;
    }
  }
  sh.cb[tid + 1] = (uint16_t)c;
  if (tid == 0) sh.cb[0] = sh.cb[kItvThreads + 1] = 0;
  int32_t x3[3] = {top, 0, 0};
  itv_scan_max3(x3, sh.scan);
  const int32_t seg0 = x3[0];
  // bit k: entry k - 1 of this thread continues a run
  uint32_t win = 0;
  if (per > 0) {
    win = ((uint32_t)sh.cb[tid] >> (per - 1)) & 1u;
    win |= c << 1;
    win |= ((uint32_t)sh.cb[tid + 2] & 3u) << (per + 1);
    // with one entry per thread the second one behind is the next thread's
    if (per == 1) win = (win & 7u) | (tid + 3 <= kItvThreads + 1 ? ((uint32_t)sh.cb[tid + 3] & 1u) << 3 : 0u);
  }
  const uint32_t c0 = win, c1 = win >> 1, c2 = win >> 2, c3 = win >> 3;  // bit k: entry k - 1, k, k + 1, k + 2
  const uint32_t ivm = (c0 & c1) | (c1 & c2) | (c2 & c3);
  int32_t p3[3] = {0, 0, 0};  // 1 + last run start, last residual, last interval neighbour
#pragma unroll
  for (int32_t k = 0; k < kItvShare; ++k) {
    if (k >= per || j0 + k >= r.m) continue;
    if (!((c1 >> k) & 1u)) p3[0] = j0 + k + 1;
    if ((ivm >> k) & 1u) p3[2] = j0 + k + 1;
    else p3[1] = j0 + k + 1;
  }
  itv_scan_max3(p3, sh.scan);
  if constexpr (WGT) {
    int32_t seg = seg0, li = p3[2];
#pragma unroll
    for (int32_t k = 0; k < kItvShare; ++k) {
      if (k >= per || j0 + k >= r.m) continue;
      if ((heads >> k) & 1u) seg = sh.own[j0 + k];
      if ((ivm >> k) & 1u) li = j0 + k + 1;
      if (j0 + k + 1 == sh.es[seg]) sh.lastiv[seg - 1] = (uint16_t)li;
    }
    __syncthreads();
  }
  // the residual and the interval neighbour before this thread's entries
  const int32_t rid0 = p3[1] ? ids[p3[1] - 1] : 0;
  const int32_t rw0 = WGT && p3[1] ? wts[p3[1] - 1] : 0, iw0 = WGT && p3[2] ? wts[p3[2] - 1] : 0;
  // codes: f(k, segment, interval neighbour, pair ends here, pair start code, pair length code, code, weight code)
  auto entries = [&](auto&& f) {
    int32_t seg = seg0, rs = p3[0], rid = rid0, rw = rw0, iw = iw0;
    int32_t st = seg0 ? sh.es[seg0 - 1] : 0, u = (int32_t)(r.u + (int64_t)(seg0 - 1) * r.ustep);
    bool res = p3[1] > st, ivb = p3[2] > st;  // the segment has had a residual, an interval neighbour
#pragma unroll
    for (int32_t k = 0; k < kItvShare; ++k) {
      if (k >= per || j0 + k >= r.m) continue;
      const int32_t j = j0 + k;
      if ((heads >> k) & 1u) {
        seg = sh.own[j];
        u = (int32_t)(r.u + (int64_t)(seg - 1) * r.ustep);
        st = j;
        res = ivb = false;
      }
      if (!((c1 >> k) & 1u)) rs = j + 1;
      const bool iv = (ivm >> k) & 1u;
      uint32_t pa = 0, pb = 0, code = 0, wc = 0;
      bool end = false;
      if (iv) {
        end = !((c2 >> k) & 1u);
        const int32_t l = j + 2 - rs;
        pa = zigzag32(id[k] - (l - 1) - u);
        pb = (uint32_t)(l - 3);
        if constexpr (WGT) {
          wc = zigzag32(w[k] - (ivb ? iw : 0));
          iw = w[k];
        }
        ivb = true;
      } else {
        code = res ? (uint32_t)(id[k] - rid) : zigzag32(id[k] - u);
        if constexpr (WGT) {
          int32_t pw = rw;
          if (!res) {  // the chain goes on from the segment's interval neighbours
            const int32_t lv = sh.lastiv[seg - 1];
            pw = lv > st ? wts[lv - 1] : 0;
          }
          wc = zigzag32(w[k] - pw);
          rw = w[k];
        }
        rid = id[k];
        res = true;
      }
      f(k, seg - 1, iv, end, pa, pb, code, wc);
    }
  };
  uint32_t A = 0, B = 0;
  entries([&](int32_t, int32_t s, bool iv, bool end, uint32_t pa, uint32_t pb, uint32_t code, uint32_t wc) {
    if (iv) {
      if (end) {
        A += (varint_len32(pa) + varint_len32(pb)) << 16;
        B += 1;
        if constexpr (!WRITE) atomicAdd(&sh.sb[s], 1u);
      }
      if constexpr (WGT) A += varint_len32(wc);
    } else {
      B += (varint_len32(code) + (WGT ? varint_len32(wc) : 0u)) << 16;
    }
  });
  const int32_t sper = (r.nseg + kItvThreads - 1) / kItvThreads;
  int32_t bytes;
  if constexpr (!WRITE) {
    __syncthreads();
    uint32_t mine = (A >> 16) + (A & 0xFFFFu) + (B >> 16);
    for (int32_t i = tid; i < r.nseg; i += kItvThreads)
      mine += (r.hdr ? varint_len(r.e0 + sh.es[i]) : 0u) + varint_len32(sh.sb[i]);
    (void)block_incl_scan_add<kItvThreads, int32_t>((int32_t)mine, sh.scan[0], &bytes);
  } else {
    static_assert(10 * kItvMax < 65536, "two sums share a word");
    int32_t totA, totB;
    uint32_t ea = (uint32_t)block_incl_scan_add<kItvThreads, int32_t>((int32_t)A, sh.scan[0], &totA) - A;
    uint32_t eb = (uint32_t)block_incl_scan_add<kItvThreads, int32_t>((int32_t)B, sh.scan[1], &totB) - B;
    {
      uint32_t a = ea, b2 = eb;
      entries([&](int32_t k, int32_t s, bool iv, bool end, uint32_t pa, uint32_t pb, uint32_t code, uint32_t wc) {
        if ((heads >> k) & 1u) {
          sh.sa[s] = a;
          sh.sb[s] = b2;
        }
        if (iv) {
          if (end) {
            a += (varint_len32(pa) + varint_len32(pb)) << 16;
            b2 += 1;
          }
          if constexpr (WGT) a += varint_len32(wc);
        } else {
          b2 += (varint_len32(code) + (WGT ? varint_len32(wc) : 0u)) << 16;
        }
      });
    }
    __syncthreads();
    // a segment's section bytes and intervals: up to the next segment with entries
    auto totals = [&](int32_t s, uint32_t& da, uint32_t& db) {
      const int32_t e = sh.es[s + 1];
      const int32_t nx = e < r.m ? (int32_t)sh.own[e] - 1 : -1;
      da = (nx >= 0 ? sh.sa[nx] : (uint32_t)totA) - sh.sa[s];
      db = (nx >= 0 ? sh.sb[nx] : (uint32_t)totB) - sh.sb[s];
    };
    uint32_t mine = 0;
    for (int32_t k = 0; k < sper; ++k) {
      const int32_t i = tid * sper + k;
      if (i >= r.nseg) break;
      uint32_t da = 0, db = 0;
      if (sh.es[i + 1] > sh.es[i]) totals(i, da, db);
      mine += (r.hdr ? varint_len(r.e0 + sh.es[i]) : 0u) + varint_len32(db & 0xFFFFu) + (da >> 16) + (da & 0xFFFFu) +
              (db >> 16);
    }
    uint32_t at = (uint32_t)block_incl_scan_add<kItvThreads, int32_t>((int32_t)mine, sh.scan[2], &bytes) - mine;
    for (int32_t k = 0; k < sper; ++k) {
      const int32_t i = tid * sper + k;
      if (i >= r.nseg) break;
      uint32_t da = 0, db = 0;
      if (sh.es[i + 1] > sh.es[i]) totals(i, da, db);
      const uint32_t cnt = db & 0xFFFFu;
      uint32_t q = at;
      if (r.hdr) {
        offs[r.u + i] = base + q;
        q += varint_put(out + base + q, r.e0 + sh.es[i]);
      } else if (i > 0 || !r.chunk0) {
        // a first chunk has no entry in the table, and its place here may be
        // that of the last chunk of the vertex before
        cpos[(r.e0 + sh.es[i]) / LP_CHUNK_LEN] = base + q;
      }
      put_bytes(out, base + q, cnt);
      q += varint_len32(cnt);
      sh.sec[i] = q;
      at = q + (da >> 16) + (da & 0xFFFFu) + (db >> 16);
    }
    __syncthreads();
    int32_t last = -1;
    uint32_t da = 0, db = 0, sa = 0, sb = 0;
    uint64_t sec = 0;
    entries([&](int32_t, int32_t s, bool iv, bool end, uint32_t pa, uint32_t pb, uint32_t code, uint32_t wc) {
      if (s != last) {
        totals(s, da, db);
        sa = sh.sa[s];
        sb = sh.sb[s];
        sec = base + sh.sec[s];
        last = s;
      }
      const uint32_t a = ea - sa, b2 = eb - sb;
      if (iv) {
        if (end) {
          const uint32_t la = varint_len32(pa), lb = varint_len32(pb);
          put_bytes(out, sec + (a >> 16), pa);
          put_bytes(out, sec + (a >> 16) + la, pb);
          ea += (la + lb) << 16;
          eb += 1;
        }
        if constexpr (WGT) {
          put_bytes(out, sec + (da >> 16) + (a & 0xFFFFu), wc);
          ea += varint_len32(wc);
        }
      } else {
        const uint64_t q = sec + (da >> 16) + (da & 0xFFFFu) + (b2 >> 16);
        const uint32_t lc = varint_len32(code);
        put_bytes(out, q, code);
        if constexpr (WGT) put_bytes(out, q + lc, wc);
        eb += (lc + (WGT ? varint_len32(wc) : 0u)) << 16;
      }
    });
  }
  __syncthreads();
  return (uint32_t)bytes;
}

// WRITE == false: the code bytes of every stretch (tsize). WRITE: the records
// at tsize[c] (the stretch's first byte by then); vertices split into chunks
// are listed for k_chunk_tables.
template <bool WGT, bool WRITE>
__global__ __launch_bounds__(kItvThreads) void k_itv(CsrIn g, const int64_t* blk, int64_t nb, int64_t c0,
                                                     uint64_t* tsize, uint64_t* offs, uint64_t* cpos,
                                                     int32_t* split_list, uint32_t* nsplit, uint8_t* out) {
  __shared__ ItvShared sh;
  const int64_t c = c0 + blockIdx.x;
  const int64_t v0 = blk[c], v1 = blk[c + 1];
  const uint64_t two_m = g.xadj[g.n];
  const uint64_t e0 = (uint64_t)c * kItvWork - (uint64_t)v0;
  const uint64_t e1 = c + 1 < nb ? (uint64_t)(c + 1) * kItvWork - (uint64_t)v1 : two_m;
  const uint64_t start = WRITE ? tsize[c] : 0;
  uint64_t pos = start;
  // the last vertex started here: split into chunks, or too long to share a run
  const uint64_t xl = v1 > v0 ? g.xadj[v1 - 1] : 0, dl = v1 > v0 ? g.xadj[v1] - xl : 0;
  const bool split = dl > LP_ITV_CHUNK_THRESHOLD;
  const bool alone = !split && v1 > v0 && g.xadj[v1] - g.xadj[v0] > (uint64_t)kItvMax;
  // chunks of the vertex continued from the stretch before; unsplit vertices;
  // the last one alone; chunks of the last one (one call: the code is long)
  for (int step = 0; step < 4; ++step) {
    ItvRun r;
    r.nseg = 0;
    if (step == 0 || step == 3) {
      const int64_t u = step == 0 ? v0 - 1 : v1 - 1;
      if (step == 0 ? v0 == 0 : !split) continue;
      const uint64_t x = g.xadj[u], d = g.xadj[u + 1] - x;
      if (d <= LP_ITV_CHUNK_THRESHOLD) continue;
      const uint64_t nch = (d + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN;
      if (step == 3) {
        if (WRITE && threadIdx.x == 0) {
          offs[u] = pos;
          (void)varint_put(out + pos, x);
          split_list[atomicAdd(nsplit, 1u)] = (int32_t)u;
        }
        pos += varint_len(x) + 4 * (nch - 1);
      }
      // the chunks that start in [e0, e1)
      const uint64_t k0 = e0 > x ? (e0 - x + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN : 0;
      const uint64_t k1 = e1 > x ? min((e1 - x + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN, nch) : 0;
      if (k0 >= k1) continue;
      r.e0 = x + k0 * LP_CHUNK_LEN;
      r.m = (int32_t)(min(d, k1 * LP_CHUNK_LEN) - k0 * LP_CHUNK_LEN);
      r.nseg = (int32_t)(k1 - k0);
      r.u = u;
      r.ustep = 0;
      r.hdr = false;
      r.chunk0 = k0 == 0;
      for (int32_t i = threadIdx.x; i <= r.nseg; i += kItvThreads)
        sh.es[i] = (uint16_t)min(i * (int32_t)LP_CHUNK_LEN, r.m);
    } else {
      const int64_t a = step == 1 ? v0 : v1 - 1, b = step == 2 || !(split || alone) ? v1 : v1 - 1;
      if (a >= b || (step == 2 && !alone)) continue;
      r.e0 = g.xadj[a];
      r.m = (int32_t)(g.xadj[b] - r.e0);
      r.nseg = (int32_t)(b - a);
      r.u = a;
      r.ustep = 1;
      r.hdr = true;
      r.chunk0 = false;
      for (int32_t i = threadIdx.x; i <= r.nseg; i += kItvThreads) sh.es[i] = (uint16_t)(g.xadj[a + i] - r.e0);
    }
    __syncthreads();
    pos += itv_run<WGT, WRITE>(g, sh, r, pos, offs, cpos, out);
  }
  if (!WRITE && threadIdx.x == 0) tsize[c] = pos - start;
}

// Bounded VarInt read for decompression: false past `end` or beyond 64 bits.
__device__ __forceinline__ bool varint_read_to(const uint8_t* b, uint64_t end, uint64_t& pos, uint64_t& x) {
  x = 0;
  for (int shift = 0; shift < 64; shift += 7) {
    if (pos >= end) return false;
    const uint32_t c = b[pos++];
    x |= (uint64_t)(c & 0x7F) << shift;
    if (!(c & 0x80)) return true;
  }
  return false;
}

// One chunk of an interval-coded record written in (ID, weight) order: the
// interval neighbours and the other neighbours are each increasing in that
// order, so one lane merges the two on the fly. False on a malformed chunk.
__device__ bool itv_chunk_sorted(const GraphView& g, int32_t u, uint64_t pos, uint64_t end, uint32_t cnt,
                                 int32_t* ids, int32_t* wts) {
  const uint8_t* B = g.bytes;
  uint64_t kk, x;
  if (!varint_read_to(B, end, pos, kk) || kk > cnt) return false;
  const uint64_t pairs = pos;
  uint64_t L = 0;
  for (uint64_t j = 0; j < kk; ++j) {
    uint64_t len;
    if (!varint_read_to(B, end, pos, x) || !varint_read_to(B, end, pos, len)) return false;
    L += len + 3;
  }
  if (L > cnt) return false;
  // interval weights start at pos; the residuals after them
  const uint64_t wstart = pos;
  int64_t wlast = 0;
  if (g.weighted)
    for (uint64_t t = 0; t < L; ++t) {
      if (!varint_read_to(B, end, pos, x)) return false;
      wlast += unzigzag(x);
    }
  uint64_t pa = pairs, pw = wstart, pr = pos;
  // cursor A: interval neighbours; cursor B: the other neighbours
  uint64_t ja = 0, rema = 0, nb_left = cnt - L;
  int64_t va = 0, wa = 0, vb = 0, wb = wlast;
  bool has_a = false, has_b = false, first_b = true;
  auto next_a = [&]() -> bool {
    if (rema == 0) {
      if (ja == kk) {
        has_a = false;
        return true;
      }
      uint64_t zs, len;
      if (!varint_read_to(B, end, pa, zs) || !varint_read_to(B, end, pa, len)) return false;
      va = (int64_t)u + unzigzag(zs);
      rema = len + 3;
      ++ja;
    } else {
      ++va;
    }
    --rema;
    if (g.weighted) {
      uint64_t c;
      if (!varint_read_to(B, end, pw, c)) return false;
      wa += unzigzag(c);
    } else {
      wa = 1;
    }
    has_a = true;
    return va >= 0 && va < g.n;
  };
  auto next_b = [&]() -> bool {
    if (nb_left == 0) {
      has_b = false;
      return true;
    }
    uint64_t c;
    if (!varint_read_to(B, end, pr, c)) return false;
    vb = first_b ? (int64_t)u + unzigzag(c) : vb + (int64_t)c;
    first_b = false;
    if (g.weighted) {
      if (!varint_read_to(B, end, pr, c)) return false;
      wb += unzigzag(c);
    } else {
      wb = 1;
    }
    --nb_left;
    has_b = true;
    return vb >= 0 && vb < g.n;
  };
  if (!next_a() || !next_b()) return false;
  for (uint32_t i = 0; i < cnt; ++i) {
    const bool take_a = has_a && (!has_b || va < vb || (va == vb && wa <= wb));
    if (take_a) {
      ids[i] = (int32_t)va;
      if (wts) wts[i] = (int32_t)wa;
      if (!next_a()) return false;
    } else {
      if (!has_b) return false;
      ids[i] = (int32_t)vb;
      if (wts) wts[i] = (int32_t)wb;
      if (!next_b()) return false;
    }
  }
  return pr == end;
}

// Decompression of an interval-coded graph: one lane per chunk; the whole
// record must be consumed. Lanes [0, n) take every vertex's first chunk (its
// only one below the chunking threshold); lane n + q takes the later chunk that
// starts at one of the entries [1000 q, 1000 q + 1000), of which there is at
// most one, since it starts a multiple of 1000 entries after its vertex's first.
// Bound by the longest serial walk, an unsplit record or a chunk: a lane per
// vertex walked a hub's chunks one after another (R-MAT with 251,161 vertices:
// 16.1 ms, 4.3 now).
__global__ void k_decode_all_itv(GraphView g, const uint64_t* xadj, int32_t* adjncy, int32_t* adjwgt,
                                 uint32_t* err) {
  const int64_t m = g.n + (int64_t)((g.two_m + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    int64_t u = i;
    uint64_t e = 0;
    if (i >= g.n) {
      e = (uint64_t)(i - g.n) * LP_CHUNK_LEN;
      int64_t lo = 0, hi = g.n;  // xadj[lo] <= e < xadj[hi]
      while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (xadj[mid] <= e) lo = mid;
        else hi = mid;
      }
      u = lo;
    }
    const uint64_t fe = xadj[u];
    const uint32_t deg = (uint32_t)(xadj[u + 1] - fe);
    if (deg == 0) continue;
    uint32_t ch = 0;
    if (i >= g.n) {
      if (deg <= (uint32_t)LP_ITV_CHUNK_THRESHOLD || e < fe || e - fe >= deg) continue;
      ch = (uint32_t)((e - fe + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN);
      if (ch == 0 || (uint64_t)ch * LP_CHUNK_LEN >= deg) continue;
    }
    const Nbh h = nbh_locate(g, (int32_t)u, deg);
    const uint64_t p0 = nbh_chunk_pos(g, h, ch);
    const uint64_t p1 = ch + 1 < h.nchunks ? nbh_chunk_pos(g, h, ch + 1) : g.offs[u + 1];
    const uint32_t first = ch * LP_CHUNK_LEN;
    const uint32_t cnt = (h.nchunks > 1) ? min((uint32_t)LP_CHUNK_LEN, deg - first) : deg;
    if (p1 < p0 || p1 > g.offs[u + 1] ||
        !itv_chunk_sorted(g, (int32_t)u, p0, p1, cnt, adjncy + fe + first, adjwgt ? adjwgt + fe + first : nullptr)) {
      atomicOr(err, 1u);
      continue;
    }
    if (adjwgt && !g.weighted)
      for (uint32_t k = 0; k < cnt; ++k) adjwgt[fe + first + k] = 1;
  }
}

__global__ void k_degrees_comp(GraphView g, int32_t* deg) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < g.n; u += (int64_t)gridDim.x * blockDim.x) {
    uint64_t p;
    const uint64_t a = read_header(g, (int32_t)u, p);
    const uint64_t b = (u + 1 < g.n) ? read_header(g, (int32_t)(u + 1), p) : g.two_m;
    deg[u] = (int32_t)(b - a);
  }
}

__global__ void k_degrees_plain(GraphView g, int32_t* deg) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < g.n; u += (int64_t)gridDim.x * blockDim.x)
    deg[u] = (int32_t)(g.xadj[u + 1] - g.xadj[u]);
}

__global__ void k_xadj_from_headers(GraphView g, uint64_t* xadj) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u <= g.n; u += (int64_t)gridDim.x * blockDim.x) {
    uint64_t p;
    xadj[u] = (u < g.n) ? read_header(g, (int32_t)u, p) : g.two_m;
  }
}

// ------------------------------------------ decompression (gap format) ----
// One workgroup per stretch of kDecWork positions of the merged sequence
// (which is also the sequence of the numbers in the code bytes: a header per
// vertex, a code per entry, two with weights). It decodes the unsplit
// vertices that start in its stretch, whose records are one run of bytes, and
// the chunks of split ones that start there, another. A run goes through in
// windows of 4096 bytes, 16 per thread: every thread reads its bytes once,
// the numbers that end in them go to LDS in order (prefix count of
// terminators), then every thread takes an equal share of the numbers, a
// segmented prefix sum (segments = vertices or chunks) turns them into IDs
// and weights, and those leave through LDS as whole lines. kDecWork numbers
// of a power-law graph (2.2 bytes on average) fill one window. Bound by the
// instructions per byte. A wave per vertex, as before, took a round trip to
// memory and a scan for every 64 numbers of every vertex: 7.5 ms for a
// weighted R-MAT graph of 3e6 vertices and 8.6e7 entries, which now takes
// 0.63 ms (1.0 GB read and written: 1.6 TB/s).
constexpr int kDecThreads = 256;
constexpr int kDecBytes = 16 * kDecThreads;  // bytes per window
constexpr int kDecWork = 1664;
constexpr int kDecShare = kDecBytes / kDecThreads;  // most numbers per thread and window

struct DecShared {
  uint32_t qs[kDecWork + 2];               // first number of every segment, and the end
  __align__(16) int32_t val[kDecBytes + 4];  // the window's numbers, then its IDs (and weights)
  int32_t scan[kDecThreads / kWave], scan2[kDecThreads / kWave];
  uint32_t flags, flags2;
  int32_t carry_v, carry_w;
};

struct DecRun {
  uint64_t lo, hi;    // code bytes
  uint32_t nseg, Q;   // segments (starts in DecShared::qs), numbers
  int32_t u, ustep;   // vertex of segment i: u + i * ustep
  uint32_t hdr;       // numbers before the first code of a segment (1: a header)
  uint64_t out;       // first entry
};

// How many of the run's first q numbers are neighbour codes and weight codes.
template <bool WGT>
__device__ __forceinline__ void dec_counts(const DecShared& sh, const DecRun& r, uint32_t q, uint32_t& nv,
                                           uint32_t& nw) {
  nv = nw = 0;
  if (q == 0) return;
  const uint32_t i = (uint32_t)tile_find(sh.qs, (int32_t)r.nseg, q - 1);
  const uint32_t before = sh.qs[i] - i * r.hdr;         // codes of the segments before
  const uint32_t in = q - sh.qs[i] > r.hdr ? q - sh.qs[i] - r.hdr : 0u;
  if constexpr (WGT) {
    nv = before / 2 + (in + 1) / 2;
    nw = before / 2 + in / 2;
  } else {
    nv = before + in;
  }
}

template <bool WGT>
__device__ __forceinline__ bool decode_run(const uint8_t* __restrict__ bytes, DecShared& sh, const DecRun& r,
                                           int32_t* adjncy, int32_t* adjwgt) {
  const int tid = threadIdx.x;
  uint32_t qb = 0, nb = 0, wb = 0;  // numbers, neighbours, weights of earlier windows
  int32_t cv = 0, cw = 0;           // the segment's neighbour and weight so far
  for (uint64_t base = r.lo & ~15ull; base < r.hi; base += kDecBytes) {
    const uint64_t p = base + 16ull * (uint64_t)tid;
    uint4 cur = make_uint4(0, 0, 0, 0);
    uint32_t prev = 0;
    if (p < r.hi) {
      cur = *(const uint4*)(bytes + p);
      if (p > r.lo) prev = *(const uint32_t*)(bytes + p - 4);  // p >= 16 then
    }
    uint32_t w[4] = {cur.x, cur.y, cur.z, cur.w};
    // bytes before the run read as ends of numbers that are not counted,
    // bytes behind it as numbers that go on
    const int32_t b0 = p < r.lo ? (int32_t)min(r.lo - p, (uint64_t)16) : 0;
    const int32_t b1 = p < r.hi ? (int32_t)min(r.hi - p, (uint64_t)16) : 0;
    if (p > r.lo && p - r.lo < 4) prev &= ~0u << (8 * (4 - (uint32_t)(p - r.lo)));
    uint32_t term = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t t = ~w[k] & 0x80808080u;
      term |= (((t >> 7) | (t >> 14) | (t >> 21) | (t >> 28)) & 15u) << (4 * k);
    }
    term &= ((1u << b1) - 1u) & ~((1u << b0) - 1u);
    int32_t tot;
    const uint32_t idx0 = (uint32_t)(block_incl_scan_add<kDecThreads, int32_t>(__popc(term), sh.scan, &tot)) -
                          (uint32_t)__popc(term);
    // the first number may begin in the bytes before
    uint32_t acc = 0, shift = 0;
    {
      const uint32_t t = ~prev & 0x80808080u;
      const uint32_t s = t ? (32u - (uint32_t)__clz((int)t)) >> 3 : 0u;  // bytes up to the last end
      if (b0 == 0) {
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
          if (k >= s) {
            acc |= ((prev >> (8 * k)) & 0x7Fu) << shift;
            shift += 7;
          }
      }
    }
    uint32_t idx = idx0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (k >= b0) {
        acc |= ((w[k / 4] >> (8 * (k % 4))) & 0x7Fu) << (shift & 31u);
        shift += 7;
      }
      if ((term >> k) & 1u) {
        sh.val[idx++] = (int32_t)acc;
        acc = 0;
        shift = 0;
      }
    }
    if (tid == 0) sh.flags = sh.flags2 = 0;
    __syncthreads();
    // this thread's share of the window's numbers
    const uint32_t end = min((uint32_t)tot, r.Q - qb);
    const uint32_t share = (end + kDecThreads - 1) / kDecThreads;
    const uint32_t k0 = tid * share;
    int32_t x[kDecShare];
    uint32_t at[kDecShare];  // 2 * position in the window's output + (1 for a weight)
    uint32_t hv = 0, hw = 0;   // numbers that begin a chain
    int32_t a = tid == 0 ? cv : 0, aw = tid == 0 ? cw : 0;
    uint32_t i = k0 < end ? (uint32_t)tile_find(sh.qs, (int32_t)r.nseg, qb + k0) : 0u;
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kDecShare; ++k) {
      at[k] = ~0u;
      if (k >= share || k0 + k >= end) continue;
      const uint32_t q = qb + k0 + k;
      if (q >= sh.qs[i + 1]) ++i;  // every segment has a number
      const uint32_t in = q - sh.qs[i];
      if (in < r.hdr) continue;
      const uint32_t code = (uint32_t)sh.val[k0 + k];
      const uint32_t c = in - r.hdr, first = sh.qs[i] - i * r.hdr;
      if (!WGT || (c & 1u) == 0) {
        if (c == 0) {
          a = r.u + (int32_t)i * r.ustep + unzigzag32(code);
          hv |= 1u << k;
        } else {
          a += (int32_t)code;
        }
        x[k] = a;
        at[k] = 2 * ((WGT ? (first + c) / 2 : first + c) - nb);
      } else {
        if (c == 1) {
          aw = unzigzag32(code);
          hw |= 1u << k;
        } else {
          aw += unzigzag32(code);
        }
        x[k] = aw;
        at[k] = 2 * ((first + c) / 2 - wb) + 1;
      }
    }
    int32_t ex, exw = 0, unused;
    tile_seg_scan<kDecThreads>(hv != 0, a, 0, sh.scan, sh.scan2, &sh.flags, ex, unused);
    if constexpr (WGT) {
      __syncthreads();
      tile_seg_scan<kDecThreads>(hw != 0, aw, 0, sh.scan, sh.scan2, &sh.flags2, exw, unused);
    }
    if (tid == kDecThreads - 1) {
      sh.carry_v = hv ? a : ex + a;
      if constexpr (WGT) sh.carry_w = hw ? aw : exw + aw;
    }
    // the seg scan's barriers: every number has been read from val
    uint32_t nb2, wb2;
    dec_counts<WGT>(sh, r, qb + end, nb2, wb2);
    const uint32_t fv = hv ? (uint32_t)__ffs(hv) - 1u : 32u, fw = hw ? (uint32_t)__ffs(hw) - 1u : 32u;
    constexpr uint32_t kW = kDecBytes / 2 + 2;  // weights of a window start here
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kDecShare; ++k) {
      if (at[k] == ~0u) continue;
      if (WGT && (at[k] & 1u)) sh.val[kW + (at[k] >> 1)] = x[k] + (k < fw ? exw : 0);
      else sh.val[at[k] >> 1] = x[k] + (k < fv ? ex : 0);
    }
    __syncthreads();
    for (uint32_t j = tid; j < nb2 - nb; j += kDecThreads) adjncy[r.out + nb + j] = sh.val[j];
    if (adjwgt) {
      if constexpr (WGT) {
        for (uint32_t j = tid; j < wb2 - wb; j += kDecThreads) adjwgt[r.out + wb + j] = sh.val[kW + j];
      } else {
        for (uint32_t j = tid; j < nb2 - nb; j += kDecThreads) adjwgt[r.out + nb + j] = 1;
      }
    }
    cv = sh.carry_v;
    cw = WGT ? sh.carry_w : 0;
    nb = nb2;
    wb = wb2;
    qb += end;
    __syncthreads();
  }
  return qb == r.Q;
}

// err[0]: malformed records; err[1]: the offsets decrease (blk is incomplete).
template <bool WGT>
__global__ __launch_bounds__(kDecThreads) void k_decode(GraphView g, const uint64_t* xadj, const int64_t* blk,
                                                        int64_t nb, int64_t c0, int32_t* adjncy, int32_t* adjwgt,
                                                        uint32_t* err) {
  __shared__ DecShared sh;
  if (err[1]) return;
  constexpr uint32_t per = WGT ? 2u : 1u;
  const int64_t c = c0 + blockIdx.x;
  const int64_t v0 = blk[c], v1 = blk[c + 1];
  const uint64_t e0 = (uint64_t)c * kDecWork - (uint64_t)v0;
  const uint64_t e1 = c + 1 < nb ? (uint64_t)(c + 1) * kDecWork - (uint64_t)v1 : g.two_m;
  bool ok = true;
  // chunks that start in [e0, e1) of the split vertex u
  auto chunks = [&](int64_t u) {
    const uint64_t x = xadj[u], d = xadj[u + 1] - x;
    const uint64_t nch = (d + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN;
    const uint64_t j0 = e0 > x ? (e0 - x + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN : 0;
    const uint64_t j1 = e1 > x ? min((e1 - x + LP_CHUNK_LEN - 1) / LP_CHUNK_LEN, nch) : 0;
    if (j0 >= j1) return;
    const Nbh h = nbh_locate(g, (int32_t)u, (uint32_t)d);
    DecRun r;
    r.lo = nbh_chunk_pos(g, h, (uint32_t)j0);
    r.hi = j1 < nch ? nbh_chunk_pos(g, h, (uint32_t)j1) : g.offs[u + 1];
    r.nseg = (uint32_t)(j1 - j0);
    r.Q = per * (uint32_t)(min(d, j1 * LP_CHUNK_LEN) - j0 * LP_CHUNK_LEN);
    r.u = (int32_t)u;
    r.ustep = 0;
    r.hdr = 0;
    r.out = x + j0 * LP_CHUNK_LEN;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i <= r.nseg; i += kDecThreads) sh.qs[i] = min(per * i * LP_CHUNK_LEN, r.Q);
    __syncthreads();
    ok &= r.hi >= r.lo && r.hi <= g.offs[u + 1] && decode_run<WGT>(g.bytes, sh, r, adjncy, adjwgt);
  };
  if (v0 > 0 && xadj[v0] - xadj[v0 - 1] > LP_CHUNK_THRESHOLD) chunks(v0 - 1);
  if (v1 > v0) {
    const bool split = xadj[v1] - xadj[v1 - 1] > LP_CHUNK_THRESHOLD;
    const int64_t ve = v1 - (split ? 1 : 0);
    const uint64_t x = xadj[v0];
    if (ve > v0 && xadj[ve] > x) {
      DecRun r;
      r.lo = g.offs[v0];
      r.hi = g.offs[ve];
      r.nseg = (uint32_t)(ve - v0);
      r.Q = per * (uint32_t)(xadj[ve] - x) + r.nseg;
      r.u = (int32_t)v0;
      r.ustep = 1;
      r.hdr = 1;
      r.out = x;
      __syncthreads();
      for (uint32_t i = threadIdx.x; i <= r.nseg; i += kDecThreads)
        sh.qs[i] = per * (uint32_t)(xadj[v0 + i] - x) + i;
      __syncthreads();
      ok &= decode_run<WGT>(g.bytes, sh, r, adjncy, adjwgt);
    }
    if (split) chunks(v1 - 1);
  }
  if (!ok && threadIdx.x == 0) atomicOr(err, 1u);
}
static_assert(LP_CHUNK_THRESHOLD >= kDecWork, "only the last vertex a stretch starts can be split");

__global__ void k_set_u64(uint64_t* p, uint64_t v) { *p = v; }

__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) a[i] = v;
}

// Input checks of a CSR, cut into stretches of the merged sequence; with
// `size`, also the code bytes of every stretch (gap-only format) and their
// prefix sum. Synchronises the scratch stream.
struct CsrPlan {
  uint64_t two_m = 0;
  int64_t max_wdeg = 0, max_deg = 0, total_vwgt = 0;
  uint64_t nbytes = 0;   // all records (with `size`)
  int64_t* blk = nullptr;
  int64_t nb = 0;
  uint64_t* tbase = nullptr;  // first byte of every stretch (with `size`)
  CsrAcc* acc = nullptr;
};

lp_status check_csr(const CsrIn& in, bool size, Scratch& sc, CsrPlan* P) {
  hipStream_t s = sc.stream();
  uint64_t x0 = 0, xn = 0;
  LP_CHECK_HIP(hipMemcpyAsync(&x0, in.xadj, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
  LP_CHECK_HIP(hipMemcpyAsync(&xn, in.xadj + in.n, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
  LP_CHECK_HIP(hipStreamSynchronize(s));
  if (x0 != 0) return LP_EINVAL;
  P->two_m = xn;
  P->nb = merged_stretches(xn, in.n, kCtWork);
  const bool wgt = in.adjwgt != nullptr;
  P->blk = sc.alloc<int64_t>((size_t)P->nb + 1);
  CsrAcc* acc = sc.alloc<CsrAcc>(1);
  uint32_t* tdeg = sc.alloc<uint32_t>(P->nb);
  unsigned long long* tw = wgt ? sc.alloc<unsigned long long>(P->nb) : nullptr;
  unsigned long long* wspan = wgt ? sc.alloc<unsigned long long>(P->nb) : nullptr;
  P->tbase = size ? sc.alloc<uint64_t>(P->nb) : nullptr;
  P->acc = acc;
  if (sc.failed) return LP_ENOMEM;
  LP_CHECK_HIP(hipMemsetAsync(acc, 0, sizeof(CsrAcc), s));
  if (wgt) LP_CHECK_HIP(hipMemsetAsync(wspan, 0, (size_t)P->nb * sizeof(unsigned long long), s));
  LP_CHECK(merged_blocks(in.xadj, in.n, kCtWork, P->nb, P->blk, &acc->xerr, s));
  auto kern = wgt ? (size ? k_csr_scan<true, true> : k_csr_scan<true, false>)
                  : (size ? k_csr_scan<false, true> : k_csr_scan<false, false>);
  LP_CHECK(launch_sliced(P->nb, kCtThreads, [&](int64_t first, dim3 grid) {
    hipLaunchKernelGGL(kern, grid, dim3(kCtThreads), 0, s, in, P->blk, P->nb, first, acc, tdeg, tw, wspan, P->tbase);
  }));
  hipLaunchKernelGGL(k_csr_max, dim3(grid_for(P->nb, 1024, 64)), dim3(256), 0, s, tdeg, tw, wspan, P->nb, acc);
  LP_CHECK_LAUNCH();
  if (in.vwgt && in.n > 0) {
    // few workgroups: each ends with an atomic on one address
    hipLaunchKernelGGL(k_vwgt_check, dim3(grid_for(in.n, 2048, 512)), dim3(256), 0, s, in.vwgt, in.n, &acc->err,
                       &acc->vtot);
    LP_CHECK_LAUNCH();
  }
  if (size) LP_CHECK(scan_exclusive_u64(P->tbase, P->tbase, P->nb, &acc->nbytes, sc));
  CsrAcc h;
  LP_CHECK_HIP(hipMemcpyAsync(&h, acc, sizeof(CsrAcc), hipMemcpyDeviceToHost, s));
  LP_CHECK_HIP(hipStreamSynchronize(s));
  if (h.xerr || h.err) return LP_EINVAL;
  P->max_deg = (int64_t)h.deg;
  P->max_wdeg = wgt ? (int64_t)h.wdeg : P->max_deg;
  P->total_vwgt = in.vwgt ? (int64_t)h.vtot : (int64_t)in.n;
  P->nbytes = h.nbytes;
  return LP_OK;
}

template <typename T>
lp_status dev_copy(T** dst, const T* src, size_t count, hipStream_t s, size_t pad = 0) {
  *dst = nullptr;
  size_t bytes = count * sizeof(T) + pad;
  *dst = (T*)handle_alloc(bytes ? bytes : 1);
  if (!*dst) return LP_ENOMEM;
  if (count) LP_CHECK_HIP(hipMemcpyAsync(*dst, src, count * sizeof(T), hipMemcpyDeviceToDevice, s));
  if (pad) LP_CHECK_HIP(hipMemsetAsync((uint8_t*)*dst + count * sizeof(T), 0, pad, s));
  return LP_OK;
}

}  // namespace

lp_status merged_blocks(const uint64_t* xadj, int64_t n, uint64_t work, int64_t nb, int64_t* blk, uint32_t* err,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_codec_blocks, dim3(grid_for(n + 1, 256, 65536)), dim3(256), 0, s, xadj, n, work, nb, blk, err);
  return last_error();
}

lp_status compute_degrees(const lp_graph* g, int32_t* deg, hipStream_t s) {
  if (g->n == 0) return LP_OK;
  if (g->deg) {
    LP_CHECK_HIP(hipMemcpyAsync(deg, g->deg, (size_t)g->n * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    return LP_OK;
  }
  if (g->compressed)
    hipLaunchKernelGGL(k_degrees_comp, dim3(grid_for(g->n, 256, 65536)), dim3(256), 0, s, g->view(), deg);
  else
    hipLaunchKernelGGL(k_degrees_plain, dim3(grid_for(g->n, 256, 65536)), dim3(256), 0, s, g->view(), deg);
  return last_error();
}

}  // namespace lp

using namespace lp;

static lp_status make_handle(int32_t n, const uint64_t* xadj, const int32_t* adjncy, const int32_t* adjwgt,
                             const int32_t* vwgt, void* stream, bool compress, lp_graph** out,
                             bool intervals = false) {
  if (!out || n < 0 || (n > 0 && (!xadj || !adjncy)) || (n == 0 && !xadj)) return LP_EINVAL;
  *out = nullptr;
  hipStream_t s = (hipStream_t)stream;
  Scratch sc(s);
  CsrIn in{n, xadj, adjncy, adjwgt, vwgt};
  CsrPlan cp;
  LP_CHECK(check_csr(in, compress && !intervals, sc, &cp));
  const uint64_t two_m = cp.two_m;
  if (cp.max_deg > 0x7FFFFFFF) return LP_EUNSUPPORTED;
  lp_graph* g = new lp_graph();
  (void)hipGetDevice(&g->device);
  g->n = n;
  g->two_m = two_m;
  g->weighted = adjwgt != nullptr;
  g->total_vwgt = cp.total_vwgt;
  g->max_wdeg = cp.max_wdeg;
  g->max_deg = cp.max_deg;
  lp_status st = LP_OK;
  do {
    if (vwgt) {
      st = dev_copy(&g->vwgt, vwgt, (size_t)n, s);
      if (st) break;
    }
    if (!compress) {
      st = dev_copy(&g->xadj, xadj, (size_t)n + 1, s);
      if (st) break;
      st = dev_copy(&g->adjncy, adjncy, (size_t)two_m, s);
      if (st) break;
      if (adjwgt) {
        st = dev_copy(&g->adjwgt, adjwgt, (size_t)two_m, s);
        if (st) break;
      }
      break;
    }
    g->compressed = 1;
    g->intervals = intervals ? 1 : 0;
    if (graph_alloc(g, (void**)&g->offs, ((size_t)n + 1) * sizeof(uint64_t)) != hipSuccess) {
      st = LP_ENOMEM;
      break;
    }
    uint64_t nbytes = cp.nbytes;
    if (intervals && n > 0) {
      cp.nb = merged_stretches(two_m, n, kItvWork);
      cp.blk = sc.alloc<int64_t>((size_t)cp.nb + 1);
      cp.tbase = sc.alloc<uint64_t>(cp.nb);
      if (sc.failed) {
        st = LP_ENOMEM;
        break;
      }
      st = merged_blocks(xadj, n, kItvWork, cp.nb, cp.blk, &cp.acc->xerr, s);
      if (st) break;
      st = launch_sliced(cp.nb, kItvThreads, [&](int64_t first, dim3 grid) {
        hipLaunchKernelGGL((g->weighted ? k_itv<true, false> : k_itv<false, false>), grid, dim3(kItvThreads), 0, s, in,
                           cp.blk, cp.nb, first, cp.tbase, (uint64_t*)nullptr, (uint64_t*)nullptr, (int32_t*)nullptr,
                           (uint32_t*)nullptr, (uint8_t*)nullptr);
      });
      if (!st) st = scan_exclusive_u64(cp.tbase, cp.tbase, cp.nb, &cp.acc->nbytes, sc);
      if (st) break;
      if (hipMemcpyAsync(&nbytes, &cp.acc->nbytes, sizeof(uint64_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
          hipStreamSynchronize(s) != hipSuccess) {
        st = LP_EDEVICE;
        break;
      }
    }
    hipLaunchKernelGGL(k_set_u64, dim3(1), dim3(1), 0, s, g->offs + n, nbytes);
    st = last_error();
    if (st) break;
    g->nbytes = nbytes;
    if (graph_alloc(g, (void**)&g->bytes, nbytes + kBytePad) != hipSuccess) {
      st = LP_ENOMEM;
      break;
    }
    if (hipMemsetAsync(g->bytes + nbytes, 0, kBytePad, s) != hipSuccess) {
      st = LP_EDEVICE;
      break;
    }
    if (n > 0) {
      const uint64_t thr = chunk_threshold(intervals);
      const bool split = cp.max_deg > (int64_t)thr;
      uint64_t* cpos = split ? sc.alloc<uint64_t>(two_m / LP_CHUNK_LEN + 1) : nullptr;
      int32_t* list = split ? sc.alloc<int32_t>(two_m / thr + 1) : nullptr;
      if (sc.failed) {
        st = LP_ENOMEM;
        break;
      }
      if (intervals) {
        st = launch_sliced(cp.nb, kItvThreads, [&](int64_t first, dim3 grid) {
          hipLaunchKernelGGL((g->weighted ? k_itv<true, true> : k_itv<false, true>), grid, dim3(kItvThreads), 0, s, in,
                             cp.blk, cp.nb, first, cp.tbase, g->offs, cpos, list, &cp.acc->nsplit, g->bytes);
        });
      } else {
        auto kern = g->weighted ? k_csr_encode<true, true>
                                : two_m < (1ull << 35) ? k_csr_encode<false, false> : k_csr_encode<false, true>;
        st = launch_sliced(cp.nb, kCtThreads, [&](int64_t first, dim3 grid) {
          hipLaunchKernelGGL(kern, grid, dim3(kCtThreads), 0, s, in, cp.blk, cp.nb, first, cp.tbase, g->offs, cpos, list,
                             &cp.acc->nsplit, g->bytes);
        });
      }
      if (st || !split) break;
      hipLaunchKernelGGL(k_chunk_tables, dim3(grid_for((int64_t)(two_m / thr + 1), 4, 1024)), dim3(256),
                         0, s, in, list, &cp.acc->nsplit, g->offs, cpos, g->bytes);
      st = last_error();
    }
  } while (0);
  if (st == LP_OK && hipStreamSynchronize(s) != hipSuccess) st = LP_EDEVICE;
  if (st != LP_OK) {
    lp_graph_free(g);
    return st;
  }
  *out = g;
  return LP_OK;
}

extern "C" lp_status lp_compress(int32_t n, const uint64_t* xadj, const int32_t* adjncy, const int32_t* adjwgt,
                                 const int32_t* vwgt, void* stream, lp_graph** out) {
  clear_error();
  return make_handle(n, xadj, adjncy, adjwgt, vwgt, stream, true, out);
}

extern "C" lp_status lp_compress_ex(int32_t n, const uint64_t* xadj, const int32_t* adjncy, const int32_t* adjwgt,
                                    const int32_t* vwgt, int32_t flags, void* stream, lp_graph** out) {
  clear_error();
  if (flags & ~LP_COMPRESS_INTERVALS) return LP_EINVAL;
  return make_handle(n, xadj, adjncy, adjwgt, vwgt, stream, true, out, (flags & LP_COMPRESS_INTERVALS) != 0);
}

extern "C" lp_status lp_graph_from_csr(int32_t n, const uint64_t* xadj, const int32_t* adjncy,
                                       const int32_t* adjwgt, const int32_t* vwgt, void* stream, lp_graph** out) {
  clear_error();
  return make_handle(n, xadj, adjncy, adjwgt, vwgt, stream, false, out);
}

extern "C" lp_status lp_graph_export(const lp_graph* g, uint64_t* offs_dev, uint8_t* bytes_dev, void* stream) {
  clear_error();
  if (!g || !g->compressed || !offs_dev || (!bytes_dev && g->nbytes)) return LP_EINVAL;
  if (g->nbatch) return LP_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  LP_CHECK_HIP(hipMemcpyAsync(offs_dev, g->offs, ((size_t)g->n + 1) * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
  if (g->nbytes) LP_CHECK_HIP(hipMemcpyAsync(bytes_dev, g->bytes, g->nbytes, hipMemcpyDeviceToDevice, s));
  return LP_OK;
}

extern "C" lp_status lp_decompress(const lp_graph* g, uint64_t* xadj, int32_t* adjncy, int32_t* adjwgt,
                                   int32_t* vwgt, void* stream) {
  clear_error();
  if (!g || !xadj || (!adjncy && g->two_m)) return LP_EINVAL;
  if (g->nbatch) return LP_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  Scratch sc(s);
  if (vwgt) {
    if (g->vwgt) {
      if (g->n) LP_CHECK_HIP(hipMemcpyAsync(vwgt, g->vwgt, (size_t)g->n * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    } else if (g->n) {
      hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(g->n, 256, 65536)), dim3(256), 0, s, vwgt, (int64_t)g->n, 1);
      LP_CHECK_LAUNCH();
    }
  }
  if (!g->compressed) {
    LP_CHECK_HIP(hipMemcpyAsync(xadj, g->xadj, ((size_t)g->n + 1) * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
    if (g->two_m) {
      LP_CHECK_HIP(hipMemcpyAsync(adjncy, g->adjncy, g->two_m * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
      if (adjwgt) {
        if (g->adjwgt)
          LP_CHECK_HIP(hipMemcpyAsync(adjwgt, g->adjwgt, g->two_m * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
        else {
          hipLaunchKernelGGL(k_fill_i32, dim3(grid_for((int64_t)g->two_m, 256, 65536)), dim3(256), 0, s, adjwgt,
                             (int64_t)g->two_m, 1);
          LP_CHECK_LAUNCH();
        }
      }
    }
    return LP_OK;
  }
  uint32_t* err = sc.alloc<uint32_t>(2);
  if (!err) return LP_ENOMEM;
  LP_CHECK_HIP(hipMemsetAsync(err, 0, 2 * sizeof(uint32_t), s));
  GraphView v = g->view();
  hipLaunchKernelGGL(k_xadj_from_headers, dim3(grid_for((int64_t)g->n + 1, 256, 65536)), dim3(256), 0, s, v, xadj);
  LP_CHECK_LAUNCH();
  if (g->n && g->intervals) {
    hipLaunchKernelGGL(k_decode_all_itv, dim3(grid_for(g->n + (int64_t)(g->two_m / LP_CHUNK_LEN) + 1, 256, 65536)),
                       dim3(256), 0, s, v, xadj, adjncy, adjwgt,
                       err);
    LP_CHECK_LAUNCH();
  } else if (g->two_m) {
    const int64_t nb = merged_stretches(g->two_m, g->n, kDecWork);
    int64_t* blk = sc.alloc<int64_t>((size_t)nb + 1);
    if (!blk) return LP_ENOMEM;
    LP_CHECK(merged_blocks(xadj, g->n, kDecWork, nb, blk, err + 1, s));
    LP_CHECK(launch_sliced(nb, kDecThreads, [&](int64_t first, dim3 grid) {
      hipLaunchKernelGGL(g->weighted ? k_decode<true> : k_decode<false>, grid, dim3(kDecThreads), 0, s, v, xadj, blk, nb,
                         first, adjncy, adjwgt, err);
    }));
  }
  uint32_t h[2] = {0, 0};
  LP_CHECK_HIP(hipMemcpyAsync(h, err, sizeof(h), hipMemcpyDeviceToHost, s));
  LP_CHECK_HIP(hipStreamSynchronize(s));
  return h[0] || h[1] ? LP_EINVAL : LP_OK;
}

extern "C" lp_status lp_graph_info(const lp_graph* g, int32_t* n, uint64_t* two_m, uint64_t* nbytes,
                                   int32_t* is_compressed, int32_t* has_edge_weights, int64_t* total_vwgt) {
  clear_error();
  if (!g) return LP_EINVAL;
  if (n) *n = g->n;
  if (two_m) *two_m = g->two_m;
  if (nbytes) *nbytes = g->nbytes;
  if (is_compressed) *is_compressed = g->compressed ? (g->intervals ? 2 : 1) : 0;
  if (has_edge_weights) *has_edge_weights = g->weighted;
  if (total_vwgt) *total_vwgt = g->total_vwgt;
  return LP_OK;
}

extern "C" void lp_graph_free(lp_graph* g) {
  if (!g) return;
  void* bufs[] = {g->offs, g->bytes, g->xadj, g->adjncy, g->adjwgt, g->vwgt, g->gid, g->gbase, g->deg};
  int cur = g->device;
  (void)hipGetDevice(&cur);
  if (cur != g->device) (void)hipSetDevice(g->device);
  if (g->stream_mem) {
    // released in the order of the stream that made the handle, to the
    // memory cache of the handle's device
    if (g->plan && g->plan_free) g->plan_free(g->plan);
    if (g->reord && g->reord_free) g->reord_free(g->reord);
    for (void* p : bufs) cache_free(p, g->mem_stream);
  } else {
    (void)hipDeviceSynchronize();
    if (g->plan && g->plan_free) g->plan_free(g->plan);
    if (g->reord && g->reord_free) g->reord_free(g->reord);
    for (void* p : bufs) handle_free(p);
  }
  if (cur != g->device) (void)hipSetDevice(cur);
  clear_error();
  delete g;
}

extern "C" void lp_trim_memory(void) { cache_trim_all(); }

extern "C" lp_status lp_set_allocator(const lp_allocator* a) { return set_allocator(a); }

extern "C" lp_status lp_memory_info(uint64_t* live_bytes, uint64_t* cached_bytes, uint64_t* external_bytes) {
  memory_info(live_bytes, cached_bytes, external_bytes);
  return LP_OK;
}

extern "C" const char* lp_strerror(lp_status s) {
  switch (s) {
    case LP_OK: return "ok";
    case LP_EINVAL: return "invalid argument or malformed graph";
    case LP_ENOMEM: return "device out of memory";
    case LP_EOVERFLOW: return "coarse weight exceeds INT32_MAX";
    case LP_EDEVICE: return "HIP device error";
    case LP_EUNSUPPORTED: return "input outside the supported range";
    default: return "unknown status";
  }
}

extern "C" const char* lp_version(void) { return "lpgpu 0.1 gfx950"; }

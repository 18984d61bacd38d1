// Bucket accumulation (Sec. II-C): every bucket receives the sum of its
// entries' points (negated for negative signed digits), with the mixed
// addition (bucket XYTZ + prepared XYU, Sec. II-D).
//
// The digit-sorted entry list is cut into chunks of K entries and each lane
// sums one chunk, so every lane does the same number of additions whatever
// the bucket sizes.  Inside a chunk, runs of equal key are bucket pieces:
//   * a piece that is a whole bucket is written to buckets[key];
//   * the first piece, if its bucket began in an earlier chunk, goes to
//     head[chunk] (it may also continue into later chunks);
//   * otherwise the last piece, if its bucket continues into later chunks,
//     goes to tail[chunk] (the bucket starts in this chunk).
// A split bucket starting in chunk c0 and ending in chunk c1 is then
// tail[c0] + head[c0+1] + ... + head[c1]: one quad sums it when the span
// c1 - c0 is small; longer spans are cut into segments that many blocks fold.
//
// Buckets are stored as signed records (fe29.hpp) for the aggregation tree, or, UNS,
// with coordinates in [0, 2p), what the caller of msm_bucket_accumulate gets: at the
// store, because a pass over all buckets afterwards reads and writes the empty ones
// too (plain digits, c = 20, 13.6 M buckets: one point 1.72 ms with it, 0.77 without;
// 2^20 points 3.69, 2.78).  Pieces are of the same form as their buckets; merges read both.
//
// A chunk is summed by one lane, or, when there are too few entries to give
// every SIMD a wave of lanes a few entries each, by one quad (quad29.hpp).
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.hpp"
#include "curve29.hpp"
#include "quad29.hpp"

namespace msm {
namespace {

constexpr uint32_t SMALL_SPAN = 63;  // chunks beyond the first of a span that k_merge sums
constexpr uint32_t SEG_HEADS = 128;  // heads of a segment of a longer span

// An entry's index word is the point index in its job with the digit's sign in
// bit 31; segoff[s] is the word offset of segment s's point array from pts
// (NULL: one job, points at pts).  Addressing from the kernel argument keeps
// the point loads global (not flat) memory instructions.  Entries with key
// KEY_NONE (digit zero, kept in place by the one-kernel sort) add nothing.

__device__ __forceinline__ const uint32_t* entry_point(const uint32_t* __restrict__ pts,
                                                       const int64_t* __restrict__ segoff,
                                                       uint32_t bb, uint32_t k, uint32_t e) {
  const int64_t off = segoff ? segoff[k >> bb] : 0;
  return pts + off + (int64_t)(e & 0x7fffffffu) * XYU_WORDS;
}

// The chunks of E entries: the first X hold K + 4 entries, the rest K (both
// multiples of 4, so that keys and indices are read in aligned groups).  One
// chunk per unit of `units` x the waves per SIMD that E is worth, so that no
// second, mostly idle round follows; K + 4 first, so that the units' work
// differs by at most 4 entries.
struct Chunks {
  uint32_t K, X;
  __device__ __forceinline__ uint64_t start(uint32_t ch) const {
    return (uint64_t)ch * K + 4ull * (ch < X ? ch : X);
  }
  __device__ __forceinline__ uint32_t length(uint32_t ch) const { return K + (ch < X ? 4u : 0u); }
  // the chunk holding entry e
  __device__ __forceinline__ uint32_t of(uint32_t e) const {
    const uint32_t longer = X * (K + 4);  // <= the entries
    return e < longer ? e / (K + 4) : X + (e - longer) / K;
  }
};

__device__ __forceinline__ Chunks chunks_of(const AccumGeom& g, uint32_t E) {
  Chunks c = {g.fixed, 0u};
  if (g.fixed == 0) {
    const uint32_t units = accum_units(g, E);
    c.K = max(g.least, (E / units) & ~3u);
    const uint64_t even = (uint64_t)c.K * units;
    c.X = E > even ? (uint32_t)((E - even + 3) / 4) : 0u;
  }
  return c;
}

// One lane per chunk, on the signed 29-bit field form (curve29.hpp): points
// are converted from their 12-word records as they are loaded, the running
// sum stays in that form and is converted when it is stored (as signed
// words, fe29.hpp: 28 shifts and ors a coordinate).  Bound by VALU issue at
// a power-limited clock: 3090 VALU instructions an entry, 2350 of them
// multiply-adds, issued in 90% of SIMD cycles at 2.0 GHz; n = 2^20 with split
// digits, sustained: 2.14 ms with the 28-bit core, 1.90 with this one, 1.75-1.81
// (9.4 G entries/s) with a column's multiply-adds in one block.  Waves per SIMD:
// see accum_units; four measured no faster than three.  (Reading keys and
// indices in groups of four cut the kernel's HBM reads by 31%.)
template <bool UNS>
__device__ __forceinline__ void accum_chunk(const uint32_t* __restrict__ pts,
                                            const int64_t* __restrict__ segoff, uint32_t bb,
                                            const uint32_t* __restrict__ key,
                                            const uint32_t* __restrict__ idx,
                                            const uint32_t* __restrict__ total, const AccumGeom& g,
                                            uint32_t* __restrict__ buckets,
                                            uint32_t* __restrict__ head,
                                            uint32_t* __restrict__ tail) {
  auto store = [](uint32_t* dst, const xytz29& v) {
    st_xytz(dst, UNS ? pt29_to_unsigned(v) : pt29_to_words(v));
  };
  const uint32_t E1 = *total;
  const Chunks c = chunks_of(g, E1);
  const uint32_t ch = blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t s64 = c.start(ch);
  if (s64 >= E1) return;
  const uint32_t s = (uint32_t)s64;
  const uint64_t e64 = s64 + c.length(ch);
  const uint32_t e = (uint32_t)(e64 < E1 ? e64 : E1);

  uint32_t cur = key[s];
  const bool open_left = (s > 0) && (key[s - 1] == cur);
  bool first_seg = true;
  xytz29 acc = pt29_identity();
  // Keys and indices are read four at a time with 16-byte loads (the arrays
  // carry 32 bytes of padding for a last group that ends past E1).  A lane's
  // 128-byte line of keys would otherwise be fetched again for every entry:
  // the point gathers of all resident waves evict it between iterations.
  // The next group is loaded two entries ahead, while the current one's
  // last entry waits in (k3, i3).
  uint4 kq = *reinterpret_cast<const uint4*>(key + s);
  uint4 iq = *reinterpret_cast<const uint4*>(idx + s);
  uint32_t k3 = 0, i3 = 0;
  for (uint32_t i = 0; s + i < e; ++i) {
    const uint32_t r = i & 3u;
    uint32_t k, ie;
    if (r == 0) {
      k = kq.x;
      ie = iq.x;
    } else if (r == 1) {
      k = kq.y;
      ie = iq.y;
    } else if (r == 2) {
      k = kq.z;
      ie = iq.z;
      k3 = kq.w;
      i3 = iq.w;
      const uint32_t q = s + i + 2;  // the next group (in the padded arrays)
      kq = *reinterpret_cast<const uint4*>(key + q);
      iq = *reinterpret_cast<const uint4*>(idx + q);
    } else {
      k = k3;
      ie = i3;
    }
    if (k != cur) {
      uint32_t* dst = (first_seg && open_left) ? head + (size_t)ch * XYTZ_WORDS
                                               : buckets + (size_t)cur * XYTZ_WORDS;
      if (cur != KEY_NONE) store(dst, acc);
      acc = pt29_identity();
      cur = k;
      first_seg = false;
    }
    if (k != KEY_NONE) {
      const xyu29 P = pt29_from(ld_xyu(entry_point(pts, segoff, bb, k, ie)));
      acc = padd29_mixed_signed(acc, P, (ie >> 31) != 0u);
    }
  }
  if (cur == KEY_NONE) return;
  const bool open_right = (e < E1) && (key[e] == cur);
  uint32_t* dst;
  if (first_seg && open_left)
    dst = head + (size_t)ch * XYTZ_WORDS;
  else if (open_right)
    dst = tail + (size_t)ch * XYTZ_WORDS;
  else
    dst = buckets + (size_t)cur * XYTZ_WORDS;
  store(dst, acc);
}

#define ACCUM_KERNEL(name, UNS)                                                          \
  __global__ void __launch_bounds__(256) name(                                           \
      const uint32_t* __restrict__ pts, const int64_t* __restrict__ segoff, uint32_t bb, \
      const uint32_t* __restrict__ key, const uint32_t* __restrict__ idx,                \
      const uint32_t* __restrict__ total, AccumGeom g, uint32_t* __restrict__ buckets,   \
      uint32_t* __restrict__ head, uint32_t* __restrict__ tail) {                        \
    accum_chunk<UNS>(pts, segoff, bb, key, idx, total, g, buckets, head, tail);          \
  }
ACCUM_KERNEL(k_accum, false)
ACCUM_KERNEL(k_accum_unsigned, true)
#undef ACCUM_KERNEL

// The same with one quad per chunk, for up to ACCUM_QUAD_MAX digit slots: the
// time is then that of one wave's dependent additions (~2.1 us each here,
// ~6.7 us on one lane), whose chunks can be as short as four entries.  Each
// lane loads its own coordinate of a point, one entry ahead.  n = 33, signed
// digits: 108 us on lanes of 16 entries -> 13 us; n = 4099, split digits
// (123 K slots): 112 -> 27 us.  At 2^18 slots both take ~30 us (16 entries a
// quad, 4 a lane), but the quads' chunks split a quarter as many buckets; from 2^19
// on their 1.4 times as many instructions cost more than that (ACCUM_QUAD_MAX).
template <bool UNS>
__global__ void __launch_bounds__(256) k_accum_quad(const uint32_t* __restrict__ pts,
                                                      const int64_t* __restrict__ segoff,
                                                      uint32_t bb,
                                                      const uint32_t* __restrict__ key,
                                                      const uint32_t* __restrict__ idx,
                                                      const uint32_t* __restrict__ total,
                                                      AccumGeom g, uint32_t* __restrict__ buckets,
                                                      uint32_t* __restrict__ head,
                                                      uint32_t* __restrict__ tail) {
  const uint32_t E1 = *total;
  const Chunks c = chunks_of(g, E1);
  const uint32_t ch = (blockIdx.x * blockDim.x + threadIdx.x) >> 2;
  const uint64_t s64 = c.start(ch);
  if (s64 >= E1) return;  // whole quads
  const uint32_t s = (uint32_t)s64;
  const uint64_t e64 = s64 + c.length(ch);
  const uint32_t e = (uint32_t)(e64 < E1 ? e64 : E1);
  // the words of this lane's coordinate of entry (k, ie)
  auto load = [&](uint32_t k, uint32_t ie) {
    const uint32_t* rec = k == KEY_NONE ? pts : entry_point(pts, segoff, bb, k, ie);
    return ld_aos(quad_xyu(rec), 0);
  };
  uint4 kq = *reinterpret_cast<const uint4*>(key + s);
  uint4 iq = *reinterpret_cast<const uint4*>(idx + s);
  uint32_t k = kq.x, ie = iq.x;
  uint32_t cur = k;
  const bool open_left = (s > 0) && (key[s - 1] == cur);
  bool first_seg = true;
  fe29 acc = quad_identity();
  fe w = load(k, ie);
  for (uint32_t i = 0; s + i < e; ++i) {
    // entry i + 1 (past the chunk's end: loaded from the padded arrays, not
    // dereferenced)
    const uint32_t r = i & 3u;
    uint32_t kn = r == 0 ? kq.y : (r == 1 ? kq.z : kq.w);
    uint32_t in = r == 0 ? iq.y : (r == 1 ? iq.z : iq.w);
    if (r == 3) {
      kq = *reinterpret_cast<const uint4*>(key + s + i + 1);
      iq = *reinterpret_cast<const uint4*>(idx + s + i + 1);
      kn = kq.x;
      in = iq.x;
    }
    if (s + i + 1 >= e) kn = KEY_NONE;
    const fe wn = load(kn, in);
    if (k != cur) {
      uint32_t* dst = (first_seg && open_left) ? head + (size_t)ch * XYTZ_WORDS
                                               : buckets + (size_t)cur * XYTZ_WORDS;
      if (cur != KEY_NONE) quad_st_as<UNS>(dst, acc);
      acc = quad_identity();
      cur = k;
      first_seg = false;
    }
    if (k != KEY_NONE) acc = quad_add_mixed(acc, f29_from_words(w), (ie >> 31) != 0u);
    k = kn;
    ie = in;
    w = wn;
  }
  if (cur == KEY_NONE) return;
  const bool open_right = (e < E1) && (key[e] == cur);
  uint32_t* dst;
  if (first_seg && open_left)
    dst = head + (size_t)ch * XYTZ_WORDS;
  else if (open_right)
    dst = tail + (size_t)ch * XYTZ_WORDS;
  else
    dst = buckets + (size_t)cur * XYTZ_WORDS;
  quad_st_as<UNS>(dst, acc);
}

// chunk ch holds a tail partial: returns true, the bucket and its last chunk
__device__ __forceinline__ bool tail_of(const uint32_t* __restrict__ key,
                                        const uint32_t* __restrict__ offsets, uint32_t E1,
                                        uint32_t bb, const Chunks& c, uint32_t ch, uint32_t& b,
                                        uint32_t& c1) {
  const uint64_t s64 = c.start(ch);
  if (s64 >= E1) return false;
  const uint32_t s = (uint32_t)s64;
  const uint64_t e64 = s64 + c.length(ch);
  const uint32_t e = (uint32_t)(e64 < E1 ? e64 : E1);
  const uint32_t last = key[e - 1];
  if (last == KEY_NONE || !(e < E1 && key[e] == last)) return false;  // last piece ends here
  if (s > 0 && key[s - 1] == key[s] && key[s] == last)  // whole chunk is a middle piece
    return false;
  b = last;
  c1 = c.of(offsets[offset_index(b, bb) + 1] - 1);
  return true;
}

// The work list of the long spans, in words: [0] items, [1] segments, then
// each item's chunk, each item's count of finished segments, and (item,
// segment) pairs.  A long span has more than SMALL_SPAN heads of its own.
struct LongList {
  uint32_t* w;
  uint32_t items;  // capacity
  __device__ __forceinline__ uint32_t* item(uint32_t i) const { return w + 2 + i; }
  __device__ __forceinline__ uint32_t* done(uint32_t i) const { return w + 2 + items + i; }
  __device__ __forceinline__ uint32_t* segment(uint32_t i) const { return w + 2 + 2 * items + 2 * i; }
};

// Split buckets: tail + heads, up to SMALL_SPAN heads; longer spans (skewed
// inputs) are listed for k_merge_long.  A block looks at MERGE_CHUNKS chunks
// and cuts their spans into runs of at most MERGE_RUN records, one quad a
// run, ordered by length, longest first, so that the quads of a wave do sums
// of one length and none idles for a chunk without a tail; the runs of a span
// of several are folded pairwise through LDS.  Bound by VALU issue when
// every chunk boundary splits a bucket, by the latency of a span's additions,
// ~3 us each behind ~13 us of start and index loads, when there are few.
// With spans of up to 8 on one quad each, 256 chunks a block: n = 65536 (split
// digits, spans of 3-4, of 24 in the top window) 51 us and 39 in k_merge_long
// -> 49 and 5; n = 2^20 in two waves a SIMD (spans of 1-2) 46 -> 42.  Runs of 3 or
// 64 chunks a block: n = 65536 8-14 us slower, no gain elsewhere.
constexpr uint32_t MERGE_CHUNKS = 128;
constexpr uint32_t MERGE_RUN = 4;
constexpr uint32_t MERGE_RUNS = MERGE_CHUNKS + SMALL_SPAN;        // a span of n heads has <= n
constexpr uint32_t MERGE_PARTS = (MERGE_CHUNKS + SMALL_SPAN) / 2;  // of several runs, <= n / 2
constexpr uint32_t MERGE_PAIRS = 64;  // a span of R > 1 runs has R / 2 <= n / 4
static_assert(MERGE_CHUNKS + SMALL_SPAN <= 4 * MERGE_PAIRS && MERGE_RUNS < 256, "");

template <bool UNS>
__global__ void __launch_bounds__(256) k_merge(const uint32_t* __restrict__ key,
                                               const uint32_t* __restrict__ offsets,
                                               const uint32_t* __restrict__ total, uint32_t bb,
                                               AccumGeom g, const uint32_t* __restrict__ head,
                                               const uint32_t* __restrict__ tail,
                                               uint32_t* __restrict__ buckets, LongList list) {
  __shared__ uint32_t runs[MERGE_RUN + 1];  // runs of each length
  __shared__ uint32_t parts, pairs, most;   // places, quads and most runs of spans of several
  // a run: its first record's chunk in the block's order | length << 8 | its
  // place in part << 16 (0xff: the whole span), its bucket; bit 31 of the
  // first word: that record is a tail
  __shared__ uint2 run[MERGE_RUNS];
  // a quad of a span's fold: first place in part | runs << 8 | its number << 16,
  // the bucket
  __shared__ uint2 pair[MERGE_PAIRS];
  __shared__ int32_t part[MERGE_PARTS][4][NL29];
  const uint32_t tid = threadIdx.x, q = quad_lane();
  if (tid <= MERGE_RUN) runs[tid] = 0;
  if (tid == 0) parts = pairs = most = 0;
  __syncthreads();
  const uint32_t E1 = *total;
  const Chunks c = chunks_of(g, E1);
  const uint32_t ch0 = blockIdx.x * MERGE_CHUNKS;
  uint32_t b = 0, c1 = 0, span = 0;
  if (tid < MERGE_CHUNKS && tail_of(key, offsets, E1, bb, c, ch0 + tid, b, c1)) span = c1 - (ch0 + tid);
  if (span > SMALL_SPAN) {
    const uint32_t item = atomicAdd(&list.w[0], 1u), segs = (span + SEG_HEADS - 1) / SEG_HEADS;
    *list.item(item) = ch0 + tid;
    *list.done(item) = 0u;
    const uint32_t at = atomicAdd(&list.w[1], segs);
    for (uint32_t t = 0; t < segs; ++t) {
      list.segment(at + t)[0] = item;
      list.segment(at + t)[1] = t;
    }
    span = 0;
  }
  // the span's runs: `more` of len + 1 records, the others of len
  const uint32_t nr = span ? (span + MERGE_RUN) / MERGE_RUN : 0u;
  const uint32_t len = nr ? (span + 1) / nr : 0u, more = nr ? (span + 1) % nr : 0u;
  uint32_t at_more = 0, at_len = 0, place = 0xffu;
  if (nr) {
    if (more) at_more = atomicAdd(&runs[len + 1], more);
    at_len = atomicAdd(&runs[len], nr - more);
    if (nr > 1) {
      place = atomicAdd(&parts, nr);
      const uint32_t at = atomicAdd(&pairs, nr / 2);
      for (uint32_t i = 0; i < nr / 2; ++i) pair[at + i] = make_uint2(place | nr << 8 | i << 16, b);
      atomicMax(&most, nr);
    }
  }
  __syncthreads();
  uint32_t nruns = 0;
  for (uint32_t t = MERGE_RUN; t >= 1; --t) {
    if (t == len + 1) at_more += nruns;
    if (t == len) at_len += nruns;
    nruns += runs[t];
  }
  for (uint32_t i = 0, rec = 0; i < nr; ++i) {
    const uint32_t l = i < more ? len + 1 : len;
    run[i < more ? at_more + i : at_len + (i - more)] =
        make_uint2((tid + rec) | l << 8 | (nr > 1 ? place + i : 0xffu) << 16 |
                       (rec == 0 ? 1u << 31 : 0u),
                   b);
    rec += l;
  }
  __syncthreads();
  for (uint32_t i = tid >> 2; i < nruns; i += 64) {
    const uint2 t = run[i];
    const size_t ch = ch0 + (t.x & 0xffu);
    const uint32_t n = (t.x >> 8) & 0xffu, at = (t.x >> 16) & 0xffu;
    const uint32_t* h = head + ch * XYTZ_WORDS;
    fe29 acc = quad_ld((t.x >> 31 ? tail : head) + ch * XYTZ_WORDS);
    fe w = ld_aos(h + XYTZ_WORDS, (int)q);
    for (uint32_t j = 1; j < n; ++j) {
      const fe29 r = f29_from_words(w);
      w = ld_aos(h + (j + 1 < n ? j + 1 : j) * XYTZ_WORDS, (int)q);
      acc = quad_add(acc, r);
    }
    if (at == 0xffu) {
      quad_st_as<UNS>(buckets + (size_t)t.y * XYTZ_WORDS, acc);
    } else {
#pragma unroll
      for (int k = 0; k < NL29; ++k) part[at][q][k] = acc.v[k];
    }
  }
  // fold a span's m runs into (m + 1) / 2 until one is left
  const uint32_t quad = tid >> 2;
  const uint2 t = quad < pairs ? pair[quad] : make_uint2(0u, 0u);
  const uint32_t at = (t.x & 0xffu) + (t.x >> 16);
  uint32_t m = (t.x >> 8) & 0xffu;
  for (uint32_t left = most; left > 1; left = (left + 1) >> 1) {
    __syncthreads();
    const uint32_t half = (m + 1) >> 1;
    if ((t.x >> 16) + half < m) {
      fe29 l, r;
#pragma unroll
      for (int k = 0; k < NL29; ++k) {
        l.v[k] = part[at][q][k];
        r.v[k] = part[at + half][q][k];
      }
      l = quad_add(l, r);
      if (half == 1) {
        quad_st_as<UNS>(buckets + (size_t)t.y * XYTZ_WORDS, l);
      } else {
#pragma unroll
        for (int k = 0; k < NL29; ++k) part[at][q][k] = l.v[k];
      }
    }
    m = half;
  }
}

// Sum of count records at stride `stride` (in records) by the block's quads:
// each sums every 64th, then they fold pairwise through LDS.  The result is
// in quad 0.
constexpr uint32_t LONG_QUADS = 64;
__device__ __forceinline__ fe29 block_sum(const uint32_t* __restrict__ rec, uint32_t count,
                                          uint32_t stride, int32_t (*part)[4][NL29]) {
  const uint32_t quad = threadIdx.x >> 2, q = quad_lane();
  const uint32_t n = count < LONG_QUADS ? count : LONG_QUADS;
  fe29 acc = quad_identity();
  if (quad < n) {
    acc = quad_ld(rec + (size_t)quad * stride * XYTZ_WORDS);
    for (uint32_t j = quad + LONG_QUADS; j < count; j += LONG_QUADS)
      acc = quad_add(acc, quad_ld(rec + (size_t)j * stride * XYTZ_WORDS));
  }
  // fold [0, m) into [0, ceil(m / 2))
  for (uint32_t m = n; m > 1; m = (m + 1) >> 1) {
    const uint32_t half = (m + 1) >> 1;
    if (quad >= half && quad < m)
#pragma unroll
      for (int i = 0; i < NL29; ++i) part[quad][q][i] = acc.v[i];
    __syncthreads();
    if (quad + half < m) {
      fe29 o;
#pragma unroll
      for (int i = 0; i < NL29; ++i) o.v[i] = part[quad + half][q][i];
      acc = quad_add(acc, o);
    }
    __syncthreads();
  }
  return acc;
}

// Long split buckets: one block per segment of SEG_HEADS heads (two
// additions and a fold of six, whatever the span; one block of lanes a span
// took 267 us for n = 300 K with half the scalars 0 or 1, this 56).  The block that finishes
// an item's last segment sums the segments' results, left in the place of
// their first heads, and adds the tail.
template <bool UNS>
__global__ void __launch_bounds__(256) k_merge_long(const uint32_t* __restrict__ key,
                                                    const uint32_t* __restrict__ offsets,
                                                    const uint32_t* __restrict__ total,
                                                    uint32_t bb, AccumGeom g,
                                                    uint32_t* __restrict__ head,
                                                    const uint32_t* __restrict__ tail,
                                                    uint32_t* __restrict__ buckets,
                                                    LongList list) {
  __shared__ int32_t part[LONG_QUADS][4][NL29];
  __shared__ uint32_t last;
  const uint32_t count = list.w[1];
  if (blockIdx.x >= count) return;
  const Chunks c = chunks_of(g, *total);
  for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
    const uint32_t item = list.segment(i)[0], t = list.segment(i)[1];
    const uint32_t ch = *list.item(item);
    const uint32_t b = key[(uint32_t)c.start(ch + 1) - 1];  // the tail's bucket ends after chunk ch
    const uint32_t span = c.of(offsets[offset_index(b, bb) + 1] - 1) - ch;
    const uint32_t segs = (span + SEG_HEADS - 1) / SEG_HEADS;
    const uint32_t h0 = t * SEG_HEADS, h1 = min(h0 + SEG_HEADS, span);
    uint32_t* first = head + (size_t)(ch + 1) * XYTZ_WORDS;
    fe29 sum = block_sum(first + (size_t)h0 * XYTZ_WORDS, h1 - h0, 1, part);
    if (segs > 1) {
      if (threadIdx.x < 4) {
        quad_st(first + (size_t)h0 * XYTZ_WORDS, sum);
        __threadfence();
      }
      __syncthreads();
      if (threadIdx.x == 0) last = atomicAdd(list.done(item), 1u) + 1 == segs ? 1u : 0u;
      __syncthreads();
      const bool mine = last != 0u;
      __syncthreads();  // read before the next segment's write
      if (!mine) continue;
      __threadfence();
      sum = block_sum(first, segs, SEG_HEADS, part);
    }
    if (threadIdx.x < 4)
      quad_st_as<UNS>(buckets + (size_t)b * XYTZ_WORDS,
                      quad_add(quad_ld(tail + (size_t)ch * XYTZ_WORDS), sum));
    __syncthreads();
  }
}

template <bool UNS>
int accumulate(const Plan& pl, uint32_t* buckets, void* ws, hipStream_t st) {
  const uint32_t* offsets = ws_at<uint32_t>(ws, pl.o_offsets);
  const uint32_t* total = ws_at<uint32_t>(ws, pl.o_total);
  const uint32_t* key = ws_at<uint32_t>(ws, pl.o_key);
  const uint32_t* idx = ws_at<uint32_t>(ws, pl.o_idx);
  uint32_t* head = ws_at<uint32_t>(ws, pl.o_head);
  uint32_t* tail = ws_at<uint32_t>(ws, pl.o_tail);
  // its two counters were cleared by the digit sort
  const LongList list = {ws_at<uint32_t>(ws, pl.o_longlist), (uint32_t)pl.long_items};
  const int64_t* segoff = pl.J == 1 ? nullptr : ws_at<const int64_t>(ws, pl.o_segoff);
  const uint32_t bb = (uint32_t)pl.bb;
  const AccumGeom g = pl.accum;
  const unsigned grid = grid_for((g.quad ? 4 : 1) * pl.chunks, 256);
  const auto kernel = g.quad ? k_accum_quad<UNS> : (UNS ? k_accum_unsigned : k_accum);
  hipEvent_t ea = nullptr, eb = nullptr;
  if (prof_kernel_events(PT_ACCUM, st, &ea, &eb)) {
    // timed by events attached to the dispatch itself
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, ea, eb, 0, pl.one.xyu, segoff, bb,
                          key, idx, total, g, buckets, head, tail);
    prof_kernel_record(PT_ACCUM, ea, eb);
  } else {
    ProfScope prof(PT_ACCUM, st);
    kernel<<<grid, 256, 0, st>>>(pl.one.xyu, segoff, bb, key, idx, total, g, buckets, head, tail);
  }
  ProfScope prof(PT_MERGE, st);
  k_merge<UNS><<<grid_for(pl.chunks, MERGE_CHUNKS), 256, 0, st>>>(key, offsets, total, bb, g, head,
                                                                  tail, buckets, list);
  k_merge_long<UNS><<<(unsigned)std::min<size_t>(1024, pl.long_segs), 256, 0, st>>>(
      key, offsets, total, bb, g, head, tail, buckets, list);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

}  // namespace

int launch_accumulate(const Plan& pl, uint32_t* buckets, void* ws, hipStream_t st,
                      bool unsigned_buckets) {
  return unsigned_buckets ? accumulate<true>(pl, buckets, ws, st)
                          : accumulate<false>(pl, buckets, ws, st);
}

}  // namespace msm

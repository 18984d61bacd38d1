// Scalar slicing and digit sort (Sec. II-C: points are assigned to buckets by
// their sliced scalar values).
//
// The entries are the (segment, point) pairs with a non-zero digit, where a
// segment is one window of one job.  An entry's key is s * 2^bb + m (segment
// s, bucket m of bb bits) and its index word is the point's index in its job
// with the digit's sign in bit 31.  Over all M = segments * 2^bb buckets the
// sort produces
//   offsets[]      the start of each bucket's entries, and per segment their end
//                  (offset_index); the entry count goes to *total
//   key[], idx[]   the entries in bucket order,
// and writes the identity into every empty bucket.
//
// Small jobs take one kernel (k_small_sort).  Otherwise it is a two-pass
// most-significant-digit counting sort, with global atomics for large
// partitions alone, in seven launches: each costs ~4.6 us however little it
// does, and twelve of them (flags cleared, three scan passes, a plan and a scan
// for large partitions on their own) took 72 us at n = 65536 with split digits
// where these take 51, and 120 -> 88 us at n = 300007 signed:
//   slice   digits of every window, stored segment-major (coalesced);
//   pass 1  per tile of one segment, an LDS histogram of the bucket index's
//           high bits; the (partition, tile) count matrix is scanned, and each
//           tile scatters its entries to (partition, tile) ranges through LDS
//           cursors;
//   pass 2  one block per partition (segment, high bits) counts the low
//           <= 8 bits in LDS, writes the bucket offsets, and places the
//           entries in bucket order.  Partitions up to PART_CAP entries are
//           staged in LDS; larger ones (skewed inputs) are sorted by many
//           blocks (k_big_*).
// Segments of one job hold n entries each; jobs may differ in n, so a block
// finds its job by binary search over the job table.
#include <algorithm>

#include "common.hpp"
#include "convert.hpp"
#include "small_sort.hpp"

namespace msm {
namespace {

constexpr int SORT_THREADS = 256;
constexpr uint32_t TILE = SORT_TILE;  // entries per pass-1 tile
constexpr uint32_t PER_THREAD = TILE / SORT_THREADS;
constexpr uint32_t PART_CAP = SORT_PART_CAP;  // entries staged in LDS by pass 2
constexpr unsigned BIG_GRID = 512;    // blocks of the large-partition kernels
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER_THREAD = 16;
constexpr int SCAN_ITEMS = SCAN_THREADS * SCAN_PER_THREAD;

struct SortGeom {
  JobView jv;
  uint32_t W, S, bb, lo_bits, hi_bits;
  uint32_t tpb;  // pass-1 tiles per block: a block's group of tpb tiles shares one histogram
};

// The scanned count matrix: starts within each SCAN_ITEMS counts and the
// starts of those groups, added as they are read (a pass over the matrix for
// that was a launch of its own).
struct Scanned {
  const uint32_t* __restrict__ counts;
  const uint32_t* __restrict__ sums;
  const uint32_t* __restrict__ total;
  size_t n;
  __device__ __forceinline__ uint32_t operator[](size_t i) const {
    return counts[i] + sums[i / SCAN_ITEMS];
  }
  // the start of element i <= n, n being the end of all
  __device__ __forceinline__ uint32_t start(size_t i) const { return i < n ? (*this)[i] : *total; }
};

// Digit words: q | sign << 31, and in window 0's word RANGE_BIT when the
// point's scalar is out of range; its job's status flag is set from that in
// pass 1, after k_slice has cleared it.
constexpr uint32_t RANGE_BIT = 1u << 30;

// Staged entries between the passes (tmp): the index word (point index |
// sign << 31) and the bucket key, 8 bytes; or, for jobs of at most 2^23
// points (PK), one word: index bits 0..22, the key's low (<= 8) bucket bits
// at 23..30, the sign at 31.  Pass 2 and the many-block sort need only the
// index word and the low bits (a partition's keys are its first bucket plus
// the low bits), so the packed form loses nothing and halves the staging
// traffic.
template <bool PK>
struct TmpEnt;
template <>
struct TmpEnt<false> {
  using T = uint2;
  __device__ static T make(uint32_t idxw, uint32_t key, uint32_t) { return make_uint2(idxw, key); }
  __device__ static uint32_t lo(const T& e, uint32_t L) { return e.y & (L - 1); }
  __device__ static uint32_t idx(const T& e) { return e.x; }
};
template <>
struct TmpEnt<true> {
  using T = uint32_t;
  __device__ static T make(uint32_t idxw, uint32_t, uint32_t lo) {
    return (idxw & 0x807fffffu) | (lo << 23);
  }
  __device__ static uint32_t lo(const T& e, uint32_t) { return (e >> 23) & 0xffu; }
  __device__ static uint32_t idx(const T& e) { return e & 0x807fffffu; }
};

// largest j with key(j) <= x, for a key non-decreasing in j (J >= 1)
template <typename F>
__device__ __forceinline__ uint32_t find_job(uint32_t J, uint32_t x, F key) {
  uint32_t lo = 0, hi = J - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (key(mid) <= x)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// the segment, tile group and job of pass-1 block b (tile = the group's
// index in its segment; a group is tpb consecutive tiles of TILE digits)
struct TileRef {
  JobDesc d;
  uint32_t j, w, tile;
};

__device__ __forceinline__ TileRef tile_ref(const SortGeom& g, uint32_t b) {
  TileRef r;
  r.j = g.jv.tab ? find_job(g.jv.J, b, [&](uint32_t j) { return g.W * g.jv.tab[j].tile_off; }) : 0u;
  r.d = g.jv.get(r.j);
  const uint32_t local = b - g.W * r.d.tile_off;
  r.w = local / r.d.tps;
  r.tile = local % r.d.tps;
  return r;
}

// count-matrix index of (segment of job d window w, high bits hi, tile group)
__device__ __forceinline__ size_t count_index(const SortGeom& g, const JobDesc& d, uint32_t w,
                                              uint32_t hi, uint32_t tile) {
  const size_t seg_tile0 = (size_t)g.W * d.tile_off + (size_t)w * d.tps;
  return (seg_tile0 << g.hi_bits) + (size_t)hi * d.tps + tile;
}

// One signed digit: v (the window's c bits) plus the carry of the window
// below, as q | sign << 31; negative (v - 2^c) from 2^(c-1) on, except in
// the top window, which takes the carry.
__device__ __forceinline__ uint32_t signed_digit(uint32_t v0, uint32_t& carry, int c, bool top) {
  const uint32_t v = v0 + carry;
  if (v >= (1u << (c - 1)) && !top) {  // d = v - 2^c < 0
    carry = 1;
    return ((1u << c) - v) | (v == (1u << c) ? 0u : 0x80000000u);
  }
  carry = 0;
  return v;
}

// Digits of every window of every job.  Word (segment s = j W + w, point i)
// at W pt_off + w n + i holds q | sign << 31, where q = 0 drops the entry and
// otherwise bucket m = q - 1 (signed digits, q = |d|) or m = q (unsigned
// digits, q = d, so unsigned bucket 0 never receives points).  With the
// endomorphism split a job's n points are its n / 2 input points and their
// images, interleaved: point 2i takes the digits of s0 of scalar i, point
// 2i + 1 those of s1; one thread splits scalar i and writes both digit words
// of each window (n and pt_off are even there).  N counts threads: points,
// or point pairs with the split.  They also clear the J status flags, the
// counters of later passes and the scan's nb block sums.
__global__ void __launch_bounds__(256) k_slice(JobView jv, uint32_t N, int c, int W, int encoding,
                                               uint32_t* __restrict__ digits,
                                               uint32_t* __restrict__ flags,
                                               uint32_t* __restrict__ counters,
                                               uint32_t* __restrict__ blocksums, uint32_t nb,
                                               uint32_t* __restrict__ longlist) {
  const uint32_t gt = blockIdx.x * blockDim.x + threadIdx.x;
  if (gt >= N) return;
  if (gt < jv.J) flags[gt] = 0u;  // J <= N
  for (uint32_t i = gt; i < nb; i += N) blocksums[i] = 0u;
  if (gt == 0) {
    for (int i = 0; i < SORT_COUNTERS; ++i) counters[i] = 0u;
    longlist[0] = 0u;  // of the accumulation's merges
    longlist[1] = 0u;
  }
  const uint32_t gi = encoding == MSM_DIGITS_GLV ? 2u * gt : gt;  // first point
  const uint32_t j = jv.tab ? find_job(jv.J, gi, [&](uint32_t k) { return jv.tab[k].pt_off; }) : 0u;
  const JobDesc d = jv.get(j);
  const uint32_t i = gi - d.pt_off;
  uint32_t* out = digits + (size_t)W * d.pt_off + i;
  if (encoding == MSM_DIGITS_GLV) {
    scalar256 s0, s1;
    uint32_t over = 0;
    glv_split(ld_scalar_flag(d.scalars, i >> 1, over), s0, s1);
    uint2* out2 = reinterpret_cast<uint2*>(out);
    uint32_t carry0 = 0, carry1 = 0;
    for (int w = 0; w < W; ++w) {
      const bool top = w + 1 == W;
      uint2 q;
      q.x = signed_digit(digit_at(s0, w * c, c), carry0, c, top);
      q.y = signed_digit(digit_at(s1, w * c, c), carry1, c, top);
      if (w == 0 && over) q.x |= RANGE_BIT;
      out2[(size_t)w * (d.n >> 1)] = q;
    }
    return;
  }
  uint32_t over = 0, carry = 0;
  const scalar256 s = ld_scalar_flag(d.scalars, i, over);
  const bool is_signed = encoding != MSM_DIGITS_UNSIGNED;
  for (int w = 0; w < W; ++w) {
    const uint32_t v = digit_at(s, w * c, c);
    uint32_t q = is_signed ? signed_digit(v, carry, c, w + 1 == W) : v;
    if (w == 0 && over) q |= RANGE_BIT;
    out[(size_t)w * d.n] = q;
  }
}

// pass 1a: per-group histogram of the high bits (the group's tiles one
// after another into one LDS histogram)
__global__ void __launch_bounds__(SORT_THREADS) k_part_count(SortGeom g, uint32_t off,
                                                             const uint32_t* __restrict__ digits,
                                                             uint32_t* __restrict__ counts,
                                                             uint32_t* __restrict__ flags) {
  __shared__ uint32_t hist[1u << 12];
  const TileRef t = tile_ref(g, blockIdx.x);
  const uint32_t H = 1u << g.hi_bits;
  for (uint32_t b = threadIdx.x; b < H; b += SORT_THREADS) hist[b] = 0;
  __syncthreads();
  const uint32_t g0 = t.tile * TILE * g.tpb, g1 = min(g0 + TILE * g.tpb, t.d.n);
  const uint32_t* dg = digits + (size_t)g.W * t.d.pt_off + (size_t)t.w * t.d.n;
  uint32_t over = 0;
  for (uint32_t e0 = g0; e0 < g1; e0 += TILE) {
    const uint32_t e1 = min(e0 + TILE, g1);
    uint32_t dq[PER_THREAD];
#pragma unroll
    for (uint32_t r = 0; r < PER_THREAD; ++r) {  // loads first, clamped (e1 > e0)
      const uint32_t e = e0 + r * SORT_THREADS + threadIdx.x;
      dq[r] = dg[e < e1 ? e : e1 - 1];
    }
#pragma unroll
    for (uint32_t r = 0; r < PER_THREAD; ++r) {
      over |= dq[r];
      const uint32_t q = e0 + r * SORT_THREADS + threadIdx.x < e1 ? dq[r] & ~RANGE_BIT : 0u;
      if (q) atomicAdd(&hist[bucket_of(q, off) >> g.lo_bits], 1u);
    }
  }
  if (over & RANGE_BIT) atomicOr(flags + t.j, (uint32_t)MSM_FLAG_RANGE);
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < H; b += SORT_THREADS)
    counts[count_index(g, t.d, t.w, b, t.tile)] = hist[b];
}

// block-wide exclusive scan of the first L (<= 256) entries of v, in place;
// all SORT_THREADS threads must call it
__device__ void lds_exclusive_scan256(uint32_t* v, uint32_t L) {
  __shared__ uint32_t t[SORT_THREADS];
  const uint32_t i = threadIdx.x;
  uint32_t x = (i < L) ? v[i] : 0u;
  t[i] = x;
  __syncthreads();
  for (uint32_t d = 1; d < SORT_THREADS; d <<= 1) {
    uint32_t y = (i >= d) ? t[i - d] : 0u;
    __syncthreads();
    t[i] += y;
    __syncthreads();
  }
  if (i < L) v[i] = t[i] - x;
  __syncthreads();
}

// block-wide exclusive scan of v[0..n) (n <= 16 SORT_THREADS) in place;
// returns the total; all SORT_THREADS threads must call it
__device__ uint32_t lds_exclusive_scan(uint32_t* v, uint32_t n) {
  __shared__ uint32_t sums[SORT_THREADS];
  __shared__ uint32_t total;
  const uint32_t per = (n + SORT_THREADS - 1) / SORT_THREADS;
  const uint32_t b0 = min(threadIdx.x * per, n), b1 = min(b0 + per, n);
  uint32_t sum = 0;
  for (uint32_t i = b0; i < b1; ++i) sum += v[i];
  sums[threadIdx.x] = sum;
  __syncthreads();
  lds_exclusive_scan256(sums, SORT_THREADS);
  uint32_t run = sums[threadIdx.x];
  if (threadIdx.x == SORT_THREADS - 1) total = run + sum;
  for (uint32_t i = b0; i < b1; ++i) {
    const uint32_t x = v[i];
    v[i] = run;
    run += x;
  }
  __syncthreads();
  return total;
}

// pass 1b: scatter into (partition, tile group) ranges; tmp entry =
// {idx | sign, key}.  Each tile of the group is first ordered by partition in
// LDS, so that consecutive threads write consecutive entries of each
// partition's range; a partition's cursor (gstart) then moves past the
// tile's entries for the next tile of the group.
template <bool PK>
__global__ void __launch_bounds__(SORT_THREADS) k_part_scatter(SortGeom g, uint32_t off,
                                                               const uint32_t* __restrict__ digits,
                                                               Scanned scanned,
                                                               typename TmpEnt<PK>::T* __restrict__ tmp) {
  // dynamic LDS, sized by the launch for H = 2^hi_bits partitions: the tile
  // stage, then per partition its global start and its local count / start
  extern __shared__ uint2 scatter_lds[];
  const uint32_t H = 1u << g.hi_bits;
  uint2* stage = scatter_lds;
  uint32_t* gstart = reinterpret_cast<uint32_t*>(scatter_lds + TILE);
  uint32_t* lstart = gstart + H;
  const TileRef t = tile_ref(g, blockIdx.x);
  for (uint32_t b = threadIdx.x; b < H; b += SORT_THREADS) {
    gstart[b] = scanned[count_index(g, t.d, t.w, b, t.tile)];
    lstart[b] = 0;
  }
  __syncthreads();
  const uint32_t g0 = t.tile * TILE * g.tpb, g1 = min(g0 + TILE * g.tpb, t.d.n);
  const uint32_t* dg = digits + (size_t)g.W * t.d.pt_off + (size_t)t.w * t.d.n;
  const uint32_t keybase = (t.j * g.W + t.w) << g.bb;
  for (uint32_t e0 = g0; e0 < g1; e0 += TILE) {
    const uint32_t e1 = min(e0 + TILE, g1);
    uint32_t part[PER_THREAD], rank[PER_THREAD], dq[PER_THREAD];
    uint2 ent[PER_THREAD];
    // all loads first (clamped, unconditional), so that they overlap
#pragma unroll
    for (uint32_t r = 0; r < PER_THREAD; ++r) {
      const uint32_t e = e0 + r * SORT_THREADS + threadIdx.x;
      dq[r] = dg[e < e1 ? e : e1 - 1];
    }
#pragma unroll
    for (uint32_t r = 0; r < PER_THREAD; ++r) {
      const uint32_t e = e0 + r * SORT_THREADS + threadIdx.x;
      const uint32_t q = e < e1 ? dq[r] & ~RANGE_BIT : 0u;
      part[r] = H;  // no entry
      rank[r] = 0;
      ent[r] = make_uint2(0u, 0u);
      if (q) {
        const uint32_t m = bucket_of(q, off);
        part[r] = m >> g.lo_bits;
        rank[r] = atomicAdd(&lstart[part[r]], 1u);
        ent[r] = make_uint2(e | (q & 0x80000000u), keybase + m);
      }
    }
    __syncthreads();
    const uint32_t count = lds_exclusive_scan(lstart, H);
#pragma unroll
    for (uint32_t r = 0; r < PER_THREAD; ++r)
      if (part[r] < H) stage[lstart[part[r]] + rank[r]] = ent[r];
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < count; k += SORT_THREADS) {
      const uint2 en = stage[k];
      const uint32_t pr = (en.y - keybase) >> g.lo_bits;
      tmp[gstart[pr] + (k - lstart[pr])] =
          TmpEnt<PK>::make(en.x, en.y, (en.y - keybase) & ((1u << g.lo_bits) - 1));
    }
    if (g.tpb == 1) break;  // (a single tile needs no cursor update)
    __syncthreads();  // the stage and the local starts are read
    for (uint32_t b = threadIdx.x; b < H; b += SORT_THREADS)
      gstart[b] += (b + 1 < H ? lstart[b + 1] : count) - lstart[b];
    __syncthreads();  // every local start is read before the reset
    for (uint32_t b = threadIdx.x; b < H; b += SORT_THREADS) lstart[b] = 0;
    __syncthreads();
  }
}

// partition p's range [start, start + size) in tmp; partitions are contiguous
// in the count matrix, the next one starting tps entries later
__device__ __forceinline__ void part_range(const SortGeom& g, const Scanned& scanned, uint32_t p,
                                           uint32_t& start, uint32_t& size) {
  const uint32_t s = p >> g.hi_bits, hi = p & ((1u << g.hi_bits) - 1);
  const JobDesc d = g.jv.get(s / g.W);
  const size_t ci = count_index(g, d, s % g.W, hi, 0);
  start = scanned[ci];
  size = scanned.start(ci + d.tps) - start;
}

// first bucket of partition p
__device__ __forceinline__ uint32_t part_bucket0(const SortGeom& g, uint32_t p) {
  const uint32_t s = p >> g.hi_bits, hi = p & ((1u << g.hi_bits) - 1);
  return (s << g.bb) + (hi << g.lo_bits);
}

// pass 2: one block per partition (segment s, high bits hi).  Each thread
// keeps its share of the partition's entries in registers (ROWS rows of the
// block); after the bucket histogram and its scan, every entry takes its place
// in bucket order in LDS (index word and low bucket bits, 5 bytes an entry)
// and the block writes the partition out linearly.
template <uint32_t ROWS, bool PK>
__device__ __forceinline__ void part_sort_rows(const SortGeom& g, uint32_t p, uint32_t start,
                                               uint32_t size,
                                               const typename TmpEnt<PK>::T* __restrict__ tmp,
                                               uint32_t* __restrict__ key,
                                               uint32_t* __restrict__ idx,
                                               uint32_t* __restrict__ offsets,
                                               uint32_t* __restrict__ buckets, uint32_t* out_idx,
                                               uint8_t* out_lo, uint32_t* hist, uint32_t* cur) {
  const uint32_t L = 1u << g.lo_bits;
  if (threadIdx.x < 256) hist[threadIdx.x] = 0;
  __syncthreads();
  typename TmpEnt<PK>::T ev[ROWS];
  if (size > 0) {
    // all loads first (clamped, unconditional), so that they overlap
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r) {
      const uint32_t k = r * SORT_THREADS + threadIdx.x;
      ev[r] = tmp[start + (k < size ? k : size - 1)];
    }
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r)
      if (r * SORT_THREADS + threadIdx.x < size) atomicAdd(&hist[TmpEnt<PK>::lo(ev[r], L)], 1u);
  }
  __syncthreads();
  for (uint32_t lo = threadIdx.x; lo < L; lo += SORT_THREADS) cur[lo] = hist[lo];
  __syncthreads();
  lds_exclusive_scan256(cur, L);  // cur[lo] = local start of bucket lo
  const uint32_t bucket0 = part_bucket0(g, p);
  if (threadIdx.x < L) {
    const uint32_t lo = threadIdx.x;
    offsets[offset_index(bucket0, g.bb) + lo] = start + cur[lo];
    if (hist[lo] == 0 && buckets)
      st_xytz(buckets + (size_t)(bucket0 + lo) * XYTZ_WORDS, pt_identity());
  }
  __syncthreads();
  if (size > 0) {
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r) {
      if (r * SORT_THREADS + threadIdx.x < size) {
        const uint32_t lo = TmpEnt<PK>::lo(ev[r], L);
        const uint32_t q = atomicAdd(&cur[lo], 1u);
        out_idx[q] = TmpEnt<PK>::idx(ev[r]);
        out_lo[q] = (uint8_t)lo;
      }
    }
  }
  __syncthreads();
  for (uint32_t q = threadIdx.x; q < size; q += SORT_THREADS) {
    key[start + q] = bucket0 + out_lo[q];
    idx[start + q] = out_idx[q];
  }
}

// The large partitions' list.  count[0] partitions of count[1] items; an item
// is BIG_CH consecutive entries of one partition.  desc[4b ..] = id, start,
// size and first item of partition b; item_of[item] its partition; cnt[item *
// 256 + lo] the item's count of bucket lo; sum[b * 512 + lo] the partition's,
// and 256 words on, how many of them have their places.
constexpr uint32_t BIG_CH = SORT_BIG_ITEM;
struct BigList {
  uint32_t *count, *desc, *item_of, *cnt, *sum;
};

// Partitions of up to SHORT_ROWS rows (evenly spread digits) take the short
// form, larger ones up to PART_CAP entries the long one.  A partition of more
// than PART_CAP entries (skewed digits) is only listed here; the k_big_*
// kernels sort it with many blocks.
constexpr uint32_t SHORT_ROWS = 20;

template <bool PK>
__global__ void __launch_bounds__(SORT_THREADS) k_part_sort(
    SortGeom g, Scanned scanned, const typename TmpEnt<PK>::T* __restrict__ tmp,
    uint32_t* __restrict__ key, uint32_t* __restrict__ idx, uint32_t* __restrict__ offsets,
    uint32_t* __restrict__ buckets, BigList big) {
  __shared__ uint32_t out_idx[PART_CAP];  // index words in bucket order
  __shared__ uint8_t out_lo[PART_CAP];    // their low bucket bits
  __shared__ uint32_t hist[256], cur[256];
  constexpr uint32_t ROWS = (PART_CAP + SORT_THREADS - 1) / SORT_THREADS;
  const uint32_t p = blockIdx.x;
  uint32_t start, size;
  part_range(g, scanned, p, start, size);
  // a segment's last partition ends it
  if (((p + 1) & ((1u << g.hi_bits) - 1)) == 0 && threadIdx.x == 0)
    offsets[(size_t)((p >> g.hi_bits) + 1) * ((1u << g.bb) + 1) - 1] = start + size;
  if (size > PART_CAP) {
    const uint32_t items = (size + BIG_CH - 1) / BIG_CH;
    if (threadIdx.x == 0) {
      const uint32_t b = atomicAdd(&big.count[0], 1u), first = atomicAdd(&big.count[1], items);
      uint32_t* d = big.desc + 4 * b;
      d[0] = p;
      d[1] = start;
      d[2] = size;
      d[3] = first;
      cur[0] = b;
      cur[1] = first;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < items; k += SORT_THREADS) big.item_of[cur[1] + k] = cur[0];
    for (uint32_t k = threadIdx.x; k < 512; k += SORT_THREADS) big.sum[512 * cur[0] + k] = 0u;
    return;
  }
  if (size <= SHORT_ROWS * SORT_THREADS)
    part_sort_rows<SHORT_ROWS, PK>(g, p, start, size, tmp, key, idx, offsets, buckets, out_idx,
                                   out_lo, hist, cur);
  else
    part_sort_rows<ROWS, PK>(g, p, start, size, tmp, key, idx, offsets, buckets, out_idx, out_lo,
                             hist, cur);
}

// Large partitions, per item: histogram of the low bucket bits
template <bool PK>
__global__ void __launch_bounds__(SORT_THREADS) k_big_count(
    SortGeom g, BigList big, const typename TmpEnt<PK>::T* __restrict__ tmp) {
  __shared__ uint32_t hist[256];
  const uint32_t items = big.count[1], L = 1u << g.lo_bits, lo = threadIdx.x;
  for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
    const uint32_t b = big.item_of[item];
    const uint32_t start = big.desc[4 * b + 1], size = big.desc[4 * b + 2];
    const uint32_t e0 = (item - big.desc[4 * b + 3]) * BIG_CH, e1 = min(e0 + BIG_CH, size);
    hist[lo] = 0;
    __syncthreads();
    constexpr uint32_t PER = BIG_CH / SORT_THREADS;
    uint32_t kv[PER];
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r) {  // loads first, clamped (e1 > e0)
      const uint32_t k = e0 + r * SORT_THREADS + threadIdx.x;
      kv[r] = TmpEnt<PK>::lo(tmp[start + (k < e1 ? k : e1 - 1)], L);
    }
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r)
      if (e0 + r * SORT_THREADS + threadIdx.x < e1) atomicAdd(&hist[kv[r]], 1u);
    __syncthreads();
    const uint32_t n = hist[lo];
    big.cnt[(size_t)item * 256 + lo] = n;
    if (n) atomicAdd(&big.sum[512 * b + lo], n);
    __syncthreads();
  }
}

// Per item: reserves its entries' places in the partition's buckets and fills
// them (the order of a bucket's entries is free); the partition's first item
// also writes the bucket offsets and the empty buckets' identities.
template <bool PK>
__global__ void __launch_bounds__(SORT_THREADS) k_big_scatter(
    SortGeom g, BigList big, const typename TmpEnt<PK>::T* __restrict__ tmp,
    uint32_t* __restrict__ key, uint32_t* __restrict__ idx, uint32_t* __restrict__ offsets,
    uint32_t* __restrict__ buckets) {
  __shared__ uint32_t cur[256];
  const uint32_t items = big.count[1], L = 1u << g.lo_bits, lo = threadIdx.x;
  for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
    const uint32_t b = big.item_of[item];
    const uint32_t p = big.desc[4 * b], start = big.desc[4 * b + 1], size = big.desc[4 * b + 2];
    const uint32_t it0 = big.desc[4 * b + 3];
    const uint32_t e0 = (item - it0) * BIG_CH, e1 = min(e0 + BIG_CH, size);
    const uint32_t bucket0 = part_bucket0(g, p);
    constexpr uint32_t PER = BIG_CH / SORT_THREADS;
    typename TmpEnt<PK>::T ev[PER];
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r) {  // loads first, clamped (e1 > e0)
      const uint32_t k = e0 + r * SORT_THREADS + threadIdx.x;
      ev[r] = tmp[start + (k < e1 ? k : e1 - 1)];
    }
    const uint32_t n = big.cnt[(size_t)item * 256 + lo], all = big.sum[512 * b + lo];
    const uint32_t before = n ? atomicAdd(&big.sum[512 * b + 256 + lo], n) : 0u;
    cur[lo] = all;
    __syncthreads();
    lds_exclusive_scan256(cur, 256);  // (counts from L on are 0)
    const uint32_t first = start + cur[lo];
    if (item == it0 && lo < L) {
      offsets[offset_index(bucket0, g.bb) + lo] = first;
      if (all == 0 && buckets)
        st_xytz(buckets + (size_t)(bucket0 + lo) * XYTZ_WORDS, pt_identity());
    }
    cur[lo] = first + before;
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r) {
      if (e0 + r * SORT_THREADS + threadIdx.x < e1) {
        const uint32_t m = TmpEnt<PK>::lo(ev[r], L);
        const uint32_t pos = atomicAdd(&cur[m], 1u);
        key[pos] = bucket0 + m;
        idx[pos] = TmpEnt<PK>::idx(ev[r]);
      }
    }
    __syncthreads();
  }
}

// The whole sort in one kernel for small jobs: one block per segment forms the
// segment's digits straight from the scalars, counts its buckets in LDS and
// writes the entries in bucket order.  A segment keeps its n places in the
// entry list (those of zero digits, at its end, get key KEY_NONE), so no block
// waits for another's count.  Twelve launches with little to do at this size
// become one: MSM of n = 33 317 -> 277 us, n = 4099 (split digits) 315 -> 287.
// Every segment's block reads all scalars and splits them again, which at
// SMALL_SORT_MAX points still costs less than the launches (signed digits:
// 451 us at 16384 points, 470 at 16385).
constexpr uint32_t SMALL_ROWS = 16;  // entries per thread

__global__ void __launch_bounds__(1024) k_small_sort(SortGeom g, int c, int encoding, Bias bias,
                                                     uint32_t* __restrict__ key,
                                                     uint32_t* __restrict__ idx,
                                                     uint32_t* __restrict__ offsets,
                                                     uint32_t* __restrict__ buckets,
                                                     uint32_t* __restrict__ flags,
                                                     uint32_t* __restrict__ total,
                                                     uint32_t NW, uint32_t* __restrict__ longlist) {
  extern __shared__ uint32_t start[];  // 2^bb + 1: counts, then starts
  __shared__ uint32_t wsum[16];
  const uint32_t tid = threadIdx.x, T = blockDim.x, B = 1u << g.bb, seg = blockIdx.x;
  const uint32_t j = seg / g.W, w = seg % g.W;
  const JobDesc d = g.jv.get(j);
  const bool glv = encoding == MSM_DIGITS_GLV, top = w + 1 == g.W;
  if (seg == 0 && tid == 0) {
    *total = NW;
    longlist[0] = 0u;
    longlist[1] = 0u;
  }
  for (uint32_t b = tid; b < B; b += T) start[b] = 0;
  __syncthreads();
  uint32_t ent[SMALL_ROWS];
  const uint32_t range = small_entries<SMALL_ROWS>(ent, start, d, bias, w, c, encoding, top);
  const int any = __syncthreads_or((int)range);
  if (w == 0 && tid == 0) flags[j] = any ? MSM_FLAG_RANGE : 0u;
  small_starts(start, wsum, B);
  const uint32_t count = start[B], base = g.W * d.pt_off + w * d.n;
  uint32_t* offs = offsets + (size_t)seg * (B + 1);
  for (uint32_t b = tid; b <= B; b += T) {
    offs[b] = base + start[b];
    if (b < B && start[b] == start[b + 1])
      st_xytz(buckets + (size_t)((seg << g.bb) + b) * XYTZ_WORDS, pt_identity());
  }
#pragma unroll
  for (uint32_t r = 0; r < SMALL_ROWS; ++r) {
    if (ent[r] == 0xffffffffu) continue;
    const uint32_t m = ent[r] & 0x1fffu;
    const uint32_t pos = base + start[m] + ((ent[r] >> 13) & 0x3fffu);
    const uint32_t i = small_index(r, glv);
    key[pos] = (seg << g.bb) + m;
    idx[pos] = i | (ent[r] & 0x80000000u);
  }
  for (uint32_t k = count + tid; k < d.n; k += T) {
    key[base + k] = KEY_NONE;
    idx[base + k] = 0u;
  }
}

// Exclusive scan of the count matrix, SCAN_ITEMS elements per block.

__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t& excl) {
  __shared__ uint32_t wsum[SCAN_THREADS / 64];
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int j = 0; j < SCAN_THREADS / 64; ++j) {
    uint32_t t = wsum[j];
    base += (j < wid) ? t : 0u;
    total += t;
  }
  excl = base + x - v;
  __syncthreads();
  return total;
}

// Starts within each block's elements; the block that finishes last scans the
// blocks' sums.  A sum and the bit that says it is there are one word (cleared by
// k_slice), which that block reads until the bit is set: no order between the sums
// and the count of finished blocks is needed, where a fence would write back all
// that each block wrote (8-16 us a scan, this 5.7-8.6).  Every sum is on its way by
// then, from a block that waits for nothing.
constexpr uint32_t SUM_READY = 1u << 31;  // digit slots are fewer

__global__ void __launch_bounds__(SCAN_THREADS) k_scan(uint32_t* __restrict__ data, size_t n,
                                                       uint32_t* __restrict__ blocksums,
                                                       uint32_t* __restrict__ total_out,
                                                       uint32_t* __restrict__ done) {
  __shared__ uint32_t last;
  size_t base = (size_t)blockIdx.x * SCAN_ITEMS + (size_t)threadIdx.x * SCAN_PER_THREAD;
  uint32_t v[SCAN_PER_THREAD];
  // a thread's 16 words are 64-byte aligned: 16-byte loads when all in range
  const bool whole = base + SCAN_PER_THREAD <= n;
  if (whole) {
    const uint4* q = reinterpret_cast<const uint4*>(data + base);
#pragma unroll
    for (int j = 0; j < SCAN_PER_THREAD / 4; ++j) {
      const uint4 w = q[j];
      v[4 * j] = w.x;
      v[4 * j + 1] = w.y;
      v[4 * j + 2] = w.z;
      v[4 * j + 3] = w.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < SCAN_PER_THREAD; ++j) v[j] = (base + j < n) ? data[base + j] : 0u;
  }
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < SCAN_PER_THREAD; ++j) sum += v[j];
  uint32_t excl;
  uint32_t total = block_exclusive_scan(sum, excl);
#pragma unroll
  for (int j = 0; j < SCAN_PER_THREAD; ++j) {
    const uint32_t x = v[j];
    v[j] = excl;
    excl += x;
  }
  if (whole) {
    uint4* q = reinterpret_cast<uint4*>(data + base);
#pragma unroll
    for (int j = 0; j < SCAN_PER_THREAD / 4; ++j)
      q[j] = make_uint4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
  } else {
#pragma unroll
    for (int j = 0; j < SCAN_PER_THREAD; ++j)
      if (base + j < n) data[base + j] = v[j];
  }
  if (threadIdx.x == 0) {
    __hip_atomic_store(&blocksums[blockIdx.x], total | SUM_READY, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    last = atomicAdd(done, 1u) + 1 == gridDim.x ? 1u : 0u;
  }
  __syncthreads();
  if (last == 0) return;
  const uint32_t nb = gridDim.x;  // <= SCAN_ITEMS
  uint32_t ready;
  do {
    ready = SUM_READY;
#pragma unroll
    for (int j = 0; j < SCAN_PER_THREAD; ++j) {
      const uint32_t i = threadIdx.x * SCAN_PER_THREAD + j;
      v[j] = i < nb ? __hip_atomic_load(&blocksums[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                    : SUM_READY;
      ready &= v[j];
    }
  } while (ready == 0u);
  sum = 0;
#pragma unroll
  for (int j = 0; j < SCAN_PER_THREAD; ++j) {
    v[j] &= ~SUM_READY;
    sum += v[j];
  }
  total = block_exclusive_scan(sum, excl);
#pragma unroll
  for (int j = 0; j < SCAN_PER_THREAD; ++j) {
    const uint32_t i = threadIdx.x * SCAN_PER_THREAD + j;
    if (i < nb) blocksums[i] = excl;
    excl += v[j];
  }
  if (threadIdx.x == 0) *total_out = total;
}

}  // namespace

// Split of the bb bucket bits: enough high bits that a partition of uniformly
// distributed digits of the largest job holds about max_n / 2^hi <=
// sort_part_target entries, at most 8 low bits (pass-2 histogram) and at most 12
// high bits (pass-1 histogram).  Also the tile grouping and the count-matrix
// size.  A pass-1 block takes a group of tpb tiles with one histogram: tpb =
// 2^hi / (32 x staged entry bytes) keeps about 256 bytes of staged entries
// per (group, partition) for uniform digits (64 one-word or 32 two-word
// entries), so that the scatter writes long runs and the count matrix (groups
// x 2^hi, which with single tiles grows with the square of the input) stays
// small.  If the matrix still exceeds the two-level scan (SCAN_ITEMS^2
// counts), groups grow to 64 tiles, then the split takes fewer high bits
// (down to bb - 8), whose partitions, larger than the LDS stage, go to the
// many-block path.  Every single job the interface takes then fits (at
// n < 2^26 the matrix stays within 2^24 counts); plans that still do not
// (batches of thousands of jobs at widths of 18 and up, whose buckets alone
// would need hundreds of GB) are refused.
void sort_geometry(Plan& pl, const size_t* ns, uint32_t J, size_t mult) {
  const uint32_t bb = (uint32_t)pl.bb;
  uint32_t want = 0;
  while (want < 12 && (pl.max_n >> want) > sort_part_target(pl.max_n)) ++want;
  const uint32_t hi_min = bb > 8 ? bb - 8 : 0;
  uint32_t hi = std::max<uint32_t>(want, hi_min);
  hi = std::min<uint32_t>(hi, std::min<uint32_t>(bb, 12));
  auto groups = [&](uint32_t tpb) {
    size_t gs = 0;
    for (uint32_t j = 0; j < J; ++j) gs += (mult * ns[j] + (size_t)SORT_TILE * tpb - 1) / ((size_t)SORT_TILE * tpb);
    return gs * (size_t)pl.W;
  };
  const size_t two_level = (size_t)SCAN_ITEMS * SCAN_ITEMS;
  // staged entry bytes: one word for jobs of at most 2^23 point records
  const uint32_t sb = pl.max_n <= ((size_t)1 << 23) ? 4u : 8u;
  uint32_t tpb = std::max<uint32_t>(1u, (1u << hi) / (32u * sb));
  while (tpb < 64 && (groups(tpb) << hi) > two_level) tpb <<= 1;
  while (hi > hi_min && (groups(tpb) << hi) > two_level) --hi;
  pl.hi_bits = hi;
  pl.lo_bits = bb - hi;
  pl.tpb = tpb;
  pl.tile_digits = SORT_TILE * tpb;
  pl.tiles = groups(tpb);
  pl.ncounts = pl.tiles << hi;
  pl.nb = (pl.ncounts + SCAN_ITEMS - 1) / SCAN_ITEMS;
  // one-word staged entries: 23 index bits and 8 low bucket bits
  pl.tmp_packed = pl.max_n <= ((size_t)1 << 23) && pl.lo_bits <= 8;
}

namespace {
struct SortBufs {
  uint32_t *digits, *offsets, *key, *idx, *buckets;
};

// pass-1 scatter, pass 2 and the many-block sort, on staged entries of
// either form
template <bool PK>
void sort_passes(const Plan& pl, const SortGeom& g, uint32_t off, const Scanned& sc,
                 const SortBufs& b, const BigList& big, typename TmpEnt<PK>::T* tmp,
                 size_t scatter_lds, hipStream_t st) {
  k_part_scatter<PK><<<(unsigned)pl.tiles, SORT_THREADS, scatter_lds, st>>>(g, off, b.digits, sc,
                                                                          tmp);
  k_part_sort<PK><<<(unsigned)(pl.S << pl.hi_bits), SORT_THREADS, 0, st>>>(
      g, sc, tmp, b.key, b.idx, b.offsets, b.buckets, big);
  // large partitions (none for evenly spread digits: these return at once)
  k_big_count<PK><<<BIG_GRID, SORT_THREADS, 0, st>>>(g, big, tmp);
  k_big_scatter<PK><<<BIG_GRID, SORT_THREADS, 0, st>>>(g, big, tmp, b.key, b.idx, b.offsets,
                                                       b.buckets);
}
}  // namespace

int launch_sort(const Plan& pl, uint32_t* buckets, void* ws, hipStream_t st) {
  uint32_t* flags = ws_at<uint32_t>(ws, pl.o_flags);
  uint32_t* total = ws_at<uint32_t>(ws, pl.o_total);
  uint32_t* offsets = ws_at<uint32_t>(ws, pl.o_offsets);
  uint32_t* counts = ws_at<uint32_t>(ws, pl.o_counts);
  uint32_t* blocksums = ws_at<uint32_t>(ws, pl.o_blocksums);
  uint32_t* digits = ws_at<uint32_t>(ws, pl.o_digits);
  uint32_t* key = ws_at<uint32_t>(ws, pl.o_key);
  uint32_t* idx = ws_at<uint32_t>(ws, pl.o_idx);

  SortGeom g;
  g.jv = job_view(pl, ws);
  g.W = (uint32_t)pl.W;
  g.S = (uint32_t)pl.S;
  g.bb = (uint32_t)pl.bb;
  g.lo_bits = pl.lo_bits;
  g.hi_bits = pl.hi_bits;
  g.tpb = pl.tpb;
  const uint32_t off = pl.encoding == MSM_DIGITS_UNSIGNED ? 0u : 1u;

  if (pl.small_sort) {
    // a few entries a thread, at most SMALL_ROWS
    const unsigned threads = (unsigned)std::min<size_t>(1024, (pl.max_n / 4 + 256) / 256 * 256);
    k_small_sort<<<(unsigned)pl.S, threads, ((size_t)4 << pl.bb) + 4, st>>>(
        g, pl.c, pl.encoding, small_bias(pl), key, idx, offsets, buckets, flags, total, (uint32_t)pl.NW,
        ws_at<uint32_t>(ws, pl.o_longlist));
    HIPCHK(hipGetLastError());
    return MSM_OK;
  }
  if (pl.lo_bits > 8 || pl.hi_bits > 12 || pl.nb > (size_t)SCAN_ITEMS) return MSM_EINVAL;

  // counters: finished scan blocks, then the large-partition list's two
  uint32_t* counters = ws_at<uint32_t>(ws, pl.o_counters);
  const size_t slice_threads = pl.encoding == MSM_DIGITS_GLV ? pl.N / 2 : pl.N;
  k_slice<<<grid_for(slice_threads, 256), 256, 0, st>>>(g.jv, (uint32_t)slice_threads, pl.c, pl.W,
                                                        pl.encoding, digits, flags, counters,
                                                        blocksums, (uint32_t)pl.nb,
                                                        ws_at<uint32_t>(ws, pl.o_longlist));
  k_part_count<<<(unsigned)pl.tiles, SORT_THREADS, 0, st>>>(g, off, digits, counts, flags);
  k_scan<<<(unsigned)pl.nb, SCAN_THREADS, 0, st>>>(counts, pl.ncounts, blocksums, total, counters);
  const size_t scatter_lds = TILE * sizeof(uint2) + 2 * ((size_t)4 << pl.hi_bits);
  const Scanned sc{counts, blocksums, total, pl.ncounts};
  const SortBufs sb{digits, offsets, key, idx, buckets};
  const BigList big{counters + 1, ws_at<uint32_t>(ws, pl.o_bigdesc),
                    ws_at<uint32_t>(ws, pl.o_bigitem), ws_at<uint32_t>(ws, pl.o_bigcnt),
                    ws_at<uint32_t>(ws, pl.o_bigsum)};
  if (pl.tmp_packed)
    sort_passes<true>(pl, g, off, sc, sb, big, ws_at<uint32_t>(ws, pl.o_tmp), scatter_lds, st);
  else
    sort_passes<false>(pl, g, off, sc, sb, big, ws_at<uint2>(ws, pl.o_tmp), scatter_lds, st);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

}  // namespace msm

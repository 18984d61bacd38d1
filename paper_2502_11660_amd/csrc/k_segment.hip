// Windows of small jobs whole: digits, bucket order, accumulation, merges,
// aggregation and the Horner pass over the bits, one block per segment (a window
// of a job), from the scalars to the window's sum.
//
// For a few entries a window each of those is a few microseconds of dependent
// additions in a launch of its own, whose results go through memory.  Here the
// entries stay in LDS; the block's quads (quad29.hpp) take chunks of them as
// k_accum_quad does, a split bucket's pieces are folded pairwise in LDS by the
// quads that hold them, and window_tail does the levels.  Bound by the latency
// of those additions, one wave a SIMD of a compute unit: n = 33, signed digits,
// five launches of 51 us -> one of 37 (251.7 -> 238.4 us in all).
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.hpp"
#include "convert.hpp"
#include "curve29.hpp"
#include "quad29.hpp"
#include "small_sort.hpp"
#include "window_tail.hpp"

namespace msm {
namespace {

constexpr uint32_t SEG_CHUNK = 4;  // entries of a quad
constexpr uint32_t SEG_ROWS = 2;   // entries per thread: a scalar's two halves
static_assert(SEGMENT_MAX <= TAIL_THREADS && SEGMENT_MAX <= SEG_CHUNK * (TAIL_THREADS / 4), "");

// words of LDS: bucket starts (B + 1), entries, then per chunk the piece that
// ends there (0) and the one that goes on (1)
__host__ __device__ inline uint32_t seg_entries_at(uint32_t bb) { return ((1u << bb) + 4u) & ~3u; }
__host__ __device__ inline uint32_t seg_pieces_at(uint32_t bb, uint32_t n) {
  return seg_entries_at(bb) + ((n + 3u) & ~3u);
}
inline size_t seg_words(uint32_t bb, uint32_t n) {
  return seg_pieces_at(bb, n) + (size_t)((n + SEG_CHUNK - 1) / SEG_CHUNK) * 2 * 4 * NL29;
}

// An entry: point | bucket << 16 | sign << 31.  Of a bucket whose entries lie in
// chunks base .. base + L - 1 the first holds piece 1, the others piece 0.
__global__ void __launch_bounds__(TAIL_THREADS) k_segment(
    JobView jv, const uint32_t* __restrict__ pts, const int64_t* __restrict__ segoff, uint32_t W,
    uint32_t bb, int c, int encoding, Bias bias, uint32_t second_at, uint32_t* buckets,
    uint32_t* flags, uint32_t* wsum) {
  extern __shared__ __attribute__((aligned(16))) int32_t mem[];
  __shared__ __attribute__((aligned(16))) tail_lds sh;
  __shared__ uint32_t scan[TAIL_THREADS / 64];
  __shared__ uint32_t longest;
  const uint32_t tid = threadIdx.x, seg = blockIdx.x, j = seg / W, w = seg % W, B = 1u << bb;
  const JobDesc d = jv.get(j);
  const bool glv = encoding == MSM_DIGITS_GLV;
  uint32_t* start = reinterpret_cast<uint32_t*>(mem);
  uint32_t* ent = start + seg_entries_at(bb);
  int32_t(*piece)[2][4][NL29] =
      reinterpret_cast<int32_t(*)[2][4][NL29]>(mem + seg_pieces_at(bb, d.n));
  uint32_t* bk = buckets + ((size_t)seg << bb) * XYTZ_WORDS;
  const uint32_t* P = pts + (segoff ? segoff[seg] : 0);
  for (uint32_t b = tid; b < B; b += TAIL_THREADS) start[b] = 0;
  if (tid == 0) longest = 0;
  __syncthreads();
  uint32_t mine[SEG_ROWS];
  const uint32_t range =
      small_entries<SEG_ROWS>(mine, start, d, bias, w, c, encoding, w + 1 == W);
  const int any = __syncthreads_or((int)range);
  if (w == 0 && tid == 0) flags[j] = any ? MSM_FLAG_RANGE : 0u;
  small_starts(start, scan, B);
#pragma unroll
  for (uint32_t r = 0; r < SEG_ROWS; ++r) {
    if (mine[r] == 0xffffffffu) continue;
    const uint32_t m = mine[r] & 0x1fffu;
    ent[start[m] + ((mine[r] >> 13) & 0x3fffu)] =
        small_index(r, glv) | m << 16 | (mine[r] & 0x80000000u);
  }
  for (uint32_t b = tid; b < B; b += TAIL_THREADS)
    if (start[b] == start[b + 1]) st_xytz(bk + (size_t)b * XYTZ_WORDS, pt_identity());
  __syncthreads();
  const uint32_t count = start[B], quad = tid >> 2, q = quad_lane();
  const uint32_t s0 = quad * SEG_CHUNK, e0 = min(s0 + SEG_CHUNK, count);
  auto bucket = [](uint32_t x) { return (x >> 16) & 0x7fffu; };
  auto put = [&](uint32_t ch, int which, const fe29& v) {
#pragma unroll
    for (int i = 0; i < NL29; ++i) piece[ch][which][q][i] = v.v[i];
  };
  auto get = [&](uint32_t ch, int which) {
    fe29 v;
#pragma unroll
    for (int i = 0; i < NL29; ++i) v.v[i] = piece[ch][which][q][i];
    return v;
  };
  // the split bucket in whose fold this quad takes part: its first chunk, its
  // number of chunks (0: none)
  uint32_t base = 0, L = 0, cur = 0;
  if (s0 < count) {
    auto load = [&](uint32_t x) { return ld_aos(quad_xyu(P + (size_t)(x & 0xffffu) * XYU_WORDS), 0); };
    uint32_t x = ent[s0];
    cur = bucket(x);
    const bool open_left = s0 > 0 && bucket(ent[s0 - 1]) == cur;
    bool first = true;
    fe29 acc = quad_identity();
    fe v = load(x);
    for (uint32_t i = s0; i < e0; ++i) {
      const uint32_t xn = ent[min(i + 1, e0 - 1)];
      const fe vn = load(xn);
      if (bucket(x) != cur) {
        if (first && open_left)
          put(quad, 0, acc);
        else
          quad_st(bk + (size_t)cur * XYTZ_WORDS, acc);
        acc = quad_identity();
        cur = bucket(x);
        first = false;
      }
      acc = quad_add_mixed(acc, f29_from_words(v), (x >> 31) != 0u);
      x = xn;
      v = vn;
    }
    const bool open_right = e0 < count && bucket(ent[e0]) == cur;
    const bool goes_on = first && open_left;
    if (goes_on)
      put(quad, 0, acc);
    else if (open_right)
      put(quad, 1, acc);
    else
      quad_st(bk + (size_t)cur * XYTZ_WORDS, acc);
    if (open_right) {  // the last chunk of a span has no part in its fold
      base = goes_on ? start[cur] / SEG_CHUNK : quad;
      L = (start[cur + 1] - 1) / SEG_CHUNK - base + 1;
      if (q == 0 && !goes_on) atomicMax(&longest, L);
    }
  }
  __syncthreads();
  // fold a span's m pieces into (m + 1) / 2 until one is left
  const uint32_t r = quad - base;
  for (uint32_t left = longest, m = L; left > 1; left = (left + 1) >> 1) {
    const uint32_t half = (m + 1) >> 1;
    if (r + half < m) {
      const int which = r == 0 ? 1 : 0;
      const fe29 sum = quad_add(get(quad, which), get(quad + half, 0));
      if (half == 1)
        quad_st(bk + (size_t)cur * XYTZ_WORDS, sum);
      else
        put(quad, which, sum);
    }
    m = half;
    __syncthreads();
  }
  __syncthreads();
  window_tail(bk, 0, bb, second_at, encoding == MSM_DIGITS_UNSIGNED ? 0 : 1,
              wsum + (size_t)2 * seg * XYTZ_WORDS, mem, sh);
}

}  // namespace

int launch_segments(const Plan& pl, void* ws, hipStream_t st) {
  const uint32_t bb = (uint32_t)pl.bb;
  size_t second = 0;
  const size_t first = tail_words(0, bb, second);
  const size_t words = std::max(seg_words(bb, (uint32_t)pl.max_n), first + second);
  const JobView jv = job_view(pl, ws);
  const int64_t* segoff = pl.J == 1 ? nullptr : ws_at<const int64_t>(ws, pl.o_segoff);
  const Bias bias = small_bias(pl);
  uint32_t* buckets = ws_at<uint32_t>(ws, pl.o_buckets);
  uint32_t* flags = ws_at<uint32_t>(ws, pl.o_flags);
  uint32_t* wsum = ws_at<uint32_t>(ws, pl.o_wsum);
  const uint32_t W = (uint32_t)pl.W, S = (uint32_t)pl.S, lds = (uint32_t)(words * 4);
  hipEvent_t ea = nullptr, eb = nullptr;
  if (prof_kernel_events(PT_ACCUM, st, &ea, &eb)) {
    hipExtLaunchKernelGGL(k_segment, dim3(S), dim3(TAIL_THREADS), lds, st, ea, eb, 0, jv,
                          pl.one.xyu, segoff, W, bb, pl.c, pl.encoding, bias, (uint32_t)first,
                          buckets, flags, wsum);
    prof_kernel_record(PT_ACCUM, ea, eb);
  } else {
    ProfScope prof(PT_ACCUM, st);
    k_segment<<<S, TAIL_THREADS, lds, st>>>(jv, pl.one.xyu, segoff, W, bb, pl.c, pl.encoding, bias,
                                            (uint32_t)first, buckets, flags, wsum);
  }
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

}  // namespace msm

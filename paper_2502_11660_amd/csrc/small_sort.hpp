// Digits and bucket order of a segment with few entries, by one block (device
// code of k_small_sort and k_segment).
#pragma once
#include "common.hpp"
#include "convert.hpp"

namespace msm {

// bucket index and the entry's index word of a digit word q != 0
__device__ __forceinline__ uint32_t bucket_of(uint32_t q, uint32_t off) {
  return (q & 0x7fffffffu) - off;
}

// Signed digits by their place alone: with B = sum_{w < W-1} 2^(w c + c - 1)
// added to the scalar, window w < W - 1 holds d_w + 2^(c-1), and the top window
// its digit (the recoding's carries are the addition's).
struct Bias {
  uint32_t w[SCALAR_WORDS];
};

// digit word of window w (top: the last): q | sign << 31
__device__ __forceinline__ uint32_t small_digit(scalar256 s, const Bias& bias, int w, int c,
                                                bool top, bool is_signed) {
  if (is_signed) {
    uint64_t t = 0;
#pragma unroll
    for (int i = 0; i < SCALAR_WORDS; ++i) {
      t += (uint64_t)s.w[i] + bias.w[i];
      s.w[i] = (uint32_t)t;
      t >>= 32;
    }
  }
  const uint32_t v = digit_at(s, w * c, c);
  if (!is_signed || top) return v;
  const int32_t d = (int32_t)v - (1 << (c - 1));
  return d < 0 ? (uint32_t)-d | 0x80000000u : (uint32_t)d;
}

// the bias of a plan's signed digits
inline Bias small_bias(const Plan& pl) {
  Bias bias = {};
  if (pl.encoding != MSM_DIGITS_UNSIGNED)
    for (int w = 0; w + 1 < pl.W; ++w) {
      const int bit = w * pl.c + pl.c - 1;
      bias.w[bit >> 5] |= 1u << (bit & 31);
    }
  return bias;
}

// The entries of window w of job d, ROWS a thread, and the buckets' counts
// (zeroed before): bucket | rank << 13 | sign << 31, all ones for none.  Returns
// whether one of the thread's scalars is out of range.
template <uint32_t ROWS>
__device__ __forceinline__ uint32_t small_entries(uint32_t* ent, uint32_t* counts, const JobDesc& d,
                                                  const Bias& bias, uint32_t w, int c,
                                                  int encoding, bool top) {
  const uint32_t tid = threadIdx.x, T = blockDim.x;
  const bool glv = encoding == MSM_DIGITS_GLV, is_signed = encoding != MSM_DIGITS_UNSIGNED;
  const uint32_t off = is_signed ? 1u : 0u;
  const uint32_t ns = glv ? d.n >> 1 : d.n;  // scalars
  uint32_t range = 0;
  auto place = [&](uint32_t q) {
    if (q == 0) return 0xffffffffu;
    const uint32_t m = bucket_of(q, off);
    return m | (atomicAdd(&counts[m], 1u) << 13) | (q & 0x80000000u);
  };
#pragma unroll
  for (uint32_t r = 0; r < ROWS; r += 2) {
    ent[r] = ent[r + 1] = 0xffffffffu;
    if (glv) {
      const uint32_t i = (r >> 1) * T + tid;
      if (i < ns) {
        scalar256 s0, s1;
        uint32_t out = 0;
        glv_split(ld_scalar_flag(d.scalars, i, out), s0, s1);
        range |= out;
        ent[r] = place(small_digit(s0, bias, (int)w, c, top, true));
        ent[r + 1] = place(small_digit(s1, bias, (int)w, c, top, true));
      }
    } else {
#pragma unroll
      for (uint32_t t = r; t < r + 2; ++t) {
        const uint32_t i = t * T + tid;
        if (i < ns) {
          uint32_t out = 0;
          const scalar256 s = ld_scalar_flag(d.scalars, i, out);
          range |= out;
          ent[t] = place(small_digit(s, bias, (int)w, c, top, is_signed));
        }
      }
    }
  }
  return range;
}

// the point of a thread's entry r
__device__ __forceinline__ uint32_t small_index(uint32_t r, bool glv) {
  const uint32_t tid = threadIdx.x, T = blockDim.x;
  return glv ? 2u * ((r >> 1) * T + tid) + (r & 1u) : r * T + tid;
}

// Counts of B buckets -> their starts, and the end in start[B], by the whole
// block (wsum: a word for each of its waves); a few buckets a thread.
__device__ __forceinline__ void small_starts(uint32_t* start, uint32_t* wsum, uint32_t B) {
  const uint32_t tid = threadIdx.x, T = blockDim.x;
  const uint32_t per = (B + T - 1) / T, b0 = min(tid * per, B), b1 = min(b0 + per, B);
  uint32_t sum = 0;
  for (uint32_t b = b0; b < b1; ++b) sum += start[b];
  uint32_t x = sum;
  const uint32_t lane = tid & 63u, wave = tid >> 6;
#pragma unroll
  for (int dd = 1; dd < 64; dd <<= 1) {
    const uint32_t y = __shfl_up(x, dd, 64);
    if (lane >= (uint32_t)dd) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint32_t run = x - sum;
  for (uint32_t k = 0; k < wave; ++k) run += wsum[k];
  for (uint32_t b = b0; b < b1; ++b) {
    const uint32_t v = start[b];
    start[b] = run;
    run += v;
  }
  if (tid == T - 1) start[B] = run;
  __syncthreads();
}

}  // namespace msm

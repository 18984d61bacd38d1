// The end of a window's aggregation by one block (device code of k_window_tail
// and k_segment).
#pragma once
#include "common.hpp"
#include "curve29.hpp"
#include "quad29.hpp"
#include "wide26.hpp"

namespace msm {

// A window's last levels h0 .. bb - 1 and its Horner pass, one block per window
// (w).  The levels run on the block's quads, the records between them in
// LDS; the root goes to LDS in the form the latency unit reads, and waves 0..2
// form S_w = sum_t 2^t X_t (+ S for signed digits) by Horner's rule over the
// bits t (X_t: slot t < bb of the root, S: slot bb).  Writes S_w as XYTZ
// (record 2w) and XYUZ (record 2w + 1).  Wave 2 loads each slot a step ahead
// and lays it out as the next addition's operand.
// A level costs its ~3 us of one quad addition where a launch of its own took
// 6: n = 1024, unsigned digits of 8 bits, all eight levels and the Horner pass
// 61 -> 48 us; n = 2^20, four levels 49 -> 43.
constexpr uint32_t TAIL_THREADS = 512;
constexpr uint32_t TAIL_ADDS = 128;  // one addition per quad at level h0

// words of LDS for the records after level h0 (the largest) and after the next
inline size_t tail_words(uint32_t h0, uint32_t bb, size_t& second) {
  const size_t rec = 4 * NL29, n0 = (size_t)1 << (bb - 1 - h0);
  second = h0 + 2 < bb ? (n0 >> 1) * (h0 + 3) * rec : 0;
  return h0 + 1 < bb ? n0 * (h0 + 2) * rec : 0;
}

struct tail_lds {
  w26_lds s;
  uint32_t root[21 * XYTZ_WORDS];  // bb + 1 <= 21 slots
};

// base: the window's records after h0 levels; lv: tail_words words of LDS;
// wsum: the window's two results.  Waves 0..2 return, the others end before.
__device__ __forceinline__ void window_tail(const uint32_t* base, uint32_t h0, uint32_t bb,
                                            uint32_t second_at, int add_total, uint32_t* wsum,
                                            int32_t* lv, tail_lds& sh) {
  w26_lds& s = sh.s;
  uint32_t* root = sh.root;
  const uint32_t quad = threadIdx.x >> 2, c = quad_lane();
  const int32_t* from = lv;
  int32_t* to = lv;
  for (uint32_t h = h0; h < bb; ++h) {
    const uint32_t nodes = 1u << (bb - 1 - h), adds = nodes * (h + 1);
    auto load = [&](uint32_t r) {
      if (h == h0) return quad_ld(base + (size_t)r * XYTZ_WORDS);
      fe29 v;
#pragma unroll
      for (int i = 0; i < NL29; ++i) v.v[i] = from[(4 * r + c) * NL29 + i];
      return v;
    };
    // the additions, then the copies of R.S
    for (uint32_t a = quad; a < adds + nodes; a += TAIL_THREADS / 4) {
      const bool add = a < adds;
      const uint32_t n = add ? a / (h + 1) : a - adds, src = add ? a % (h + 1) : h;
      fe29 r = load((2 * n + 1) * (h + 1) + src);
      if (add) r = quad_add(load(2 * n * (h + 1) + src), r);
      const uint32_t slot = !add ? h : (src < h ? src : h + 1);
      if (h + 1 == bb) {
        quad_st_unsigned(root + slot * XYTZ_WORDS, quad_to_u(r));
      } else {
#pragma unroll
        for (int i = 0; i < NL29; ++i) to[(4 * (n * (h + 2) + slot) + c) * NL29 + i] = r.v[i];
      }
    }
    __syncthreads();
    from = to;
    to = lv + (to == lv ? second_at : 0);
  }
  if (threadIdx.x >= W26_THREADS) return;  // the barriers below are the first three waves'
  const w26_lane q = w26_lane_here(s);
  const int steps = (int)bb + (add_total ? 1 : 0);
  // step i adds slot bb - 1 - i (i < bb) or the total (slot bb); clamped
  auto slot = [&](int i) { return root + (i < (int)bb ? (int)bb - 1 - i : (int)bb) * XYTZ_WORDS; };
  w26_init(s);
  w26_sync();
  w26_fetch f;
  if (q.wave == 2) {
    w26_put_identity(s);
    w26_put_operand(s, q, w26_load(slot(0)), 0);
    f = w26_load(slot(1));
  }
  w26_sync();
  for (int i = 0; i < steps; ++i) {
    if (i >= 1 && i < (int)bb) w26_dbl(q);
    w26_add(q, i & 1, [&] {
      w26_put_operand(s, q, f, (i & 1) ^ 1);
      f = w26_load(slot(i + 2 < steps ? i + 2 : steps - 1));
    });
  }
  if (q.wave == 0) {
    w26_store(s, wsum, W26_T);
  } else if (q.wave == 1) {
    const uint32_t u = w26_mul(q, s.at(W26_T), s.at(W26_K) + (wlane() & 31u));
    if (wlane() < 16) s.at(W26_E)[q.j] = u;
    wave_lds_sync();
    w26_store(s, wsum + XYTZ_WORDS, W26_E);
  }
}

}  // namespace msm

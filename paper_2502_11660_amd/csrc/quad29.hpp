// Latency-oriented point arithmetic: four lanes per point (device code).
//
// A lone wave issues one instruction every ~4.6 cycles, so the latency of an
// addition done by one lane is the length of its instruction stream.  Here
// four consecutive lanes ("a quad") share one point: lane q of the quad holds
// coordinate q (0: X, 1: Y, 2: T or U = kT, 3: Z) in the signed 29-bit form
// (fe29.hpp).  Every formula has four independent products per phase, one per
// lane; sums and differences of two lanes' values are formed by DPP quad
// permutes, three instructions a limb:
//
//   mixed addition (Z2 = 1)        2 phases, ~1100 instructions (one lane: 3100)
//   addition, both XYTZ            3 phases (k T2 first), ~1550 (one lane: 4000)
//
// It takes 1.4 times the one-lane unit's instructions in all, and a third of
// its time when the chip is not full: used for bucket accumulation of small
// MSMs, the split-bucket merges and the middle levels of the aggregation tree.
//
// All lanes of a quad must be active.  Limb classes and value bounds are those
// of fe29.hpp and curve29.hpp.
#pragma once
#include "curve29.hpp"

namespace msm {

// 2^385 mod p in words: the factor whose product with Z1 is the D = 2 Z1
// 2^384 2^-406 of a prepared point; read like a record's coordinate, in 16-byte loads
__device__ const uint32_t __align__(16) kTwoR[NL] = {
    0xfffffed0u, 0x059bffffu, 0xffffff62u, 0xa2813f06u, 0x14fa7fe4u, 0x3efb6753u,
    0xdcf8c60bu, 0xf69d2f6eu, 0x007909d0u, 0x99e92b7fu, 0xc5fbe934u, 0x011accc3u};

__device__ __forceinline__ uint32_t quad_lane() { return threadIdx.x & 3u; }

// quad_perm:[a,b,c,d]
template <int A, int B, int C, int D>
__device__ __forceinline__ int32_t qperm(int32_t x) {
  return __builtin_amdgcn_mov_dpp(x, A | (B << 2) | (C << 4) | (D << 6), 0xF, 0xF, true);
}

// A sum of two lanes' values of class d: x + (y ^ mask) + add, where mask is
// all ones for x - y (the complement plus one) and add is 1 then, or takes
// 2^29 a limb from a sum of two n (f29_add).
struct qsum {
  int32_t mask, add0, add1, add12;
  __device__ __forceinline__ int32_t add(int i) const {
    return i == 0 ? add0 : (i + 1 < NL29 ? add1 : add12);
  }
};
__device__ __forceinline__ qsum qsum_of(bool minus) {
  qsum s;
  s.mask = minus ? -1 : 0;
  s.add0 = minus ? 1 : -(1 << 29);
  s.add1 = minus ? 1 : -M29;
  s.add12 = 1;
  return s;
}

// The first phase's operand: Y - X, Y + X, T or U, and Z or (TWICE) 2 Z.
template <bool TWICE>
__device__ __forceinline__ fe29 quad_first(const fe29& v) {
  const uint32_t q = quad_lane();
  const bool crossed = q < 2 || (TWICE && q == 3);
  const int32_t cross = crossed ? -1 : 0;
  const qsum s = qsum_of(q == 0);
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i)
    r.v[i] = (v.v[i] ^ s.mask) + (qperm<1, 0, 2, 3>(v.v[i]) & cross) + (crossed ? s.add(i) : 0);
  return r;
}

// The same of a prepared point (lane 3: kTwoR, taken as it is) or its
// negative: Y - X and Y + X exchanged, U negated.
__device__ __forceinline__ fe29 quad_first_signed(const fe29& v, bool neg) {
  const uint32_t q = quad_lane();
  const int32_t n = neg ? -1 : 0;
  const int32_t cross = q < 2 ? -1 : 0;
  const int32_t own = (q == 0 ? -1 : 0) ^ ((q & 1u) ? 0 : n);  // sign of this lane's value
  const int32_t other = q == 1 ? n : 0;                         // of the crossed one
  qsum s = qsum_of((q == 0) != neg);
  const int32_t alone = q == 2 && neg ? 1 : 0;
  s.add0 = q < 2 ? s.add0 : alone;
  s.add1 = q < 2 ? s.add1 : alone;
  s.add12 = q < 2 ? s.add12 : alone;
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i)
    r.v[i] = (v.v[i] ^ own) + ((qperm<1, 0, 2, 3>(v.v[i]) & cross) ^ other) + s.add(i);
  return r;
}

// The second phase: from A, B, C, D in lanes 0..3, E F, G H, E H, F G.
__device__ __forceinline__ fe29 quad_finish(const fe29& p) {
  const uint32_t q = quad_lane();
  const qsum sl = qsum_of(q != 1), sr = qsum_of(q == 0);
  fe29 l, r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) {
    // E, G, E, F = B - A, D + C, B - A, D - C
    l.v[i] = qperm<1, 3, 1, 3>(p.v[i]) + (qperm<0, 2, 0, 2>(p.v[i]) ^ sl.mask) + sl.add(i);
    // F, H, H, G = D - C, B + A, B + A, D + C
    r.v[i] = qperm<3, 1, 1, 3>(p.v[i]) + (qperm<2, 0, 0, 2>(p.v[i]) ^ sr.mask) + sr.add(i);
  }
  return f29_mul(l, r);
}

// a + b or a - b (neg), b prepared (quad_ld_xyu); a's coordinates are products
__device__ __forceinline__ fe29 quad_add_mixed(const fe29& a, const fe29& b, bool neg) {
  return quad_finish(f29_mul(quad_first<false>(a), quad_first_signed(b, neg)));
}

// T -> U = k T in lane 2
__device__ __forceinline__ fe29 quad_to_u(const fe29& v) {
  return f29_select(quad_lane() == 2, f29_mul_const(v, kK29), v);
}

// a + b, both XYTZ
__device__ __forceinline__ fe29 quad_add(const fe29& a, const fe29& b) {
  return quad_finish(f29_mul(quad_first<false>(a), quad_first<true>(quad_to_u(b))));
}

// identity (0, 1, 0, 1): coordinate q
__device__ __forceinline__ fe29 quad_identity() { return f29_small((int32_t)(quad_lane() & 1u)); }

// coordinate q of an XYTZ record (signed words)
__device__ __forceinline__ fe29 quad_ld(const uint32_t* __restrict__ rec) {
  return f29_from_words(ld_aos(rec, (int)quad_lane()));
}

// word address of a prepared record's coordinate q (lane 3: kTwoR)
__device__ __forceinline__ const uint32_t* quad_xyu(const uint32_t* __restrict__ rec) {
  const uint32_t q = quad_lane();
  return q < 3 ? rec + q * NL : kTwoR;
}

// store as signed words, or with coordinates in [0, 2p)
__device__ __forceinline__ void quad_st(uint32_t* __restrict__ rec, const fe29& v) {
  st_aos(rec, (int)quad_lane(), f29_to_words(v));
}
__device__ __forceinline__ void quad_st_unsigned(uint32_t* __restrict__ rec, const fe29& v) {
  st_aos(rec, (int)quad_lane(), fe_unsigned(f29_to_words(v)));
}
template <bool UNS>
__device__ __forceinline__ void quad_st_as(uint32_t* __restrict__ rec, const fe29& v) {
  if (UNS)
    quad_st_unsigned(rec, v);
  else
    quad_st(rec, v);
}

}  // namespace msm

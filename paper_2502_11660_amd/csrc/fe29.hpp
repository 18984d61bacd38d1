// Signed 29-bit base-field arithmetic of the one-lane throughput PADD unit
// (device code).
//
// An element is thirteen 29-bit limbs (13 x 29 = 377 = the bit length of p),
// each in its own 32-bit register, of which the top limb carries the sign.  A
// product is 25 columns of v_mad_i64_i32 into one 64-bit accumulator per
// column: with limbs of magnitude below 2^29 a column stays below 2^63, so
// there are no carry words (the carry-save idea of Sec. III-D, the saved
// bits being the upper half of each column sum), and sums and differences
// need no multiple of p added to stay non-negative.
//
// Reduction.  p = 1 (mod 2^46): with m = t mod 2^29 the column sum t has its
// low 29 bits cleared by subtracting m p, whose lowest limb is m itself, so
// the digit is one mask and the carry one arithmetic shift.  p's other limbs
// are taken balanced (in [-2^28, 2^28)) and negated, so that the reduction is
// added like the product.  Fourteen digits: R' = 2^406 and
//     out = (a b - m p) / R',   -p - |a b| / R' < out <= |a b| / R',
// where |a b| / R' < 2^-20 p for every product formed here (|a|, |b| < 8p).
// A product is 169 + 168 = 337 multiply-adds and 52 masks and shifts (389
// instructions); the 14-limb unsigned core it replaced took 378 and 86
// (464).  Bucket accumulation issues 3620 -> 3090 VALU instructions per mixed
// addition; the chip is power-limited under them (its clock falls from 2.2 to
// 1.9 GHz within a few launches), so the gain is that of the multiply-adds
// saved: split digits at n = 2^20 2.60 -> 2.36 ms, at 2^22 9.38 -> 8.52 ms.
//
// Stored records hold the 12-word form: the same integers in 384-bit two's
// complement (above -(1 + 2^-4) p and below 2p), in Montgomery form with
// R = 2^384.  Projective points do not change under a common factor of their
// coordinates, so extended points carry over as they are.  A prepared point
// has Z = 1, that is the integer 2^384: the mixed addition's products with it
// are reduced by thirteen digits, 2^377, so that D = 2 Z1 2^384 2^-377 =
// 2^8 Z1 (f29_shl8; with fourteen, D is the as costly 2^-21 Z1, and the three
// products take 42 instructions more).
//
// Limb classes:
//   n  limbs 0..11 in [0, 2^29), any sign in the top limb: every product
//   d  limbs 0..11 in [-2^29, 2^29]: a difference of two n, or a sum of two n
//      less 2^29 per limb (f29_add: the 2^29 moves as a carry of one into the
//      next limb, so the value is unchanged)
// Operands are n or d with top limbs of magnitude below 2^31, that is values
// below 4.76p.  The largest column of d times d, top limbs 2^31 included, is
// 0.72 x 2^63 with the reduction's share (digits of 2^29 against the balanced
// limbs of p, whose magnitudes add up to 7.9 x 2^28); one operand with limbs
// of 3 x 2^28 (f29_add_p, values below 2p) against d below 2p gives 0.77.
#pragma once
#include "field.hpp"
#include "mad64.hpp"

namespace msm {

constexpr int NL29 = 13;
constexpr int32_t M29 = 0x1fffffff;

struct fe29 {
  int32_t v[NL29];
};

// -p in balanced 29-bit limbs (limb 0 is -1)
constexpr int32_t kNP29[NL29] = {-1,         -138805248, -33,       155547552, 192937615,
                                 250094331,  -238844878, 27255134,  82173222,  -56953418,
                                 242302608,  -260710870, -451126369};
// the curve constant k = 2d in R'-form (k 2^406 mod p)
constexpr int32_t kK29[NL29] = {0x114806b1, 0x4ef4e0d,  0x7df1bf4,  0x1a7dedd, 0x7626a98,
                                0x61c00c8,  0x1b3f730c, 0x37d439d,  0x1c957daa, 0x96f1594,
                                0x98747ae,  0x19dba77f, 0x3dbbc1f};

__device__ __forceinline__ fe29 f29_const(const int32_t (&c)[NL29]) {
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) r.v[i] = c[i];
  return r;
}

__device__ __forceinline__ fe29 f29_small(int32_t x) {
  fe29 r;
  r.v[0] = x;
#pragma unroll
  for (int i = 1; i < NL29; ++i) r.v[i] = 0;
  return r;
}

// 12 words (two's complement, magnitude below 2^379) -> 13 limbs, class n
__device__ __forceinline__ fe29 f29_from_words(const fe& x) {
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) {
    const int b = 29 * i, w = b >> 5, s = b & 31;
    uint32_t t = x.v[w];
    if (s) t = s + 29 <= 32 ? t >> s : __builtin_amdgcn_alignbit(x.v[w + 1], t, s);
    r.v[i] = (int32_t)(i + 1 < NL29 ? t & (uint32_t)M29 : t);
  }
  return r;
}

// 13 limbs of class n -> 12 words, two's complement
__device__ __forceinline__ fe f29_to_words(const fe29& x) {
  fe r;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int b = 32 * j, i = b / 29, s = b % 29;
    if (i + 1 < NL29) {
      uint32_t w = (uint32_t)x.v[i] >> s;
      w |= (uint32_t)x.v[i + 1] << (29 - s);
      if (58 - s < 32) w |= (uint32_t)x.v[i + 2] << (58 - s);
      r.v[j] = w;
    } else {
      r.v[j] = (uint32_t)(x.v[i] >> s);  // the sign fills the top word
    }
  }
  return r;
}

// column K of a b - m p without the digits m_j p_0: the products a_i b_{K-i}
// and m_j (-p)_{K-j} with indices in [0, 13) and j < DIGITS; b in SGPRs when SB
template <int K, int DIGITS, bool SB = false>
__device__ __forceinline__ void f29_column(const fe29& a, const fe29& b, const int32_t* m,
                                           int64_t& acc) {
  constexpr int I0 = K < NL29 ? 0 : K - (NL29 - 1);
  constexpr int I1 = K < NL29 ? K : NL29 - 1;
  constexpr int J1 = K - 1 < DIGITS - 1 ? K - 1 : DIGITS - 1;
  constexpr int NA = I1 >= I0 ? I1 - I0 + 1 : 0, NM = J1 >= I0 ? J1 - I0 + 1 : 0;
  int32_t x[NL29], y[NL29], u[NL29], q[NL29];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    x[i] = a.v[I0 + i];
    y[i] = b.v[K - I0 - i];
  }
#pragma unroll
  for (int j = 0; j < NM; ++j) {
    u[j] = m[I0 + j];
    q[j] = kNP29[K - I0 - j];
  }
  if constexpr (SB) {
    if constexpr (NA > 0) mad64_block<true, 0, NA>(acc, x, y, x, y);
    if constexpr (NM > 0) mad64_block<true, 0, NM>(acc, u, q, u, q);
  } else {
    mad64_block<true, NA, NM>(acc, x, y, u, q);
  }
}

// columns [K, DIGITS): reduction digits
template <int K, int DIGITS, bool SB = false>
__device__ __forceinline__ void f29_low(const fe29& a, const fe29& b, int32_t* m, int64_t& acc) {
  if constexpr (K < DIGITS) {
    f29_column<K, DIGITS, SB>(a, b, m, acc);
    m[K] = (int32_t)acc & M29;
    acc >>= 29;
    f29_low<K + 1, DIGITS, SB>(a, b, m, acc);
  }
}

// columns [K, DIGITS + 12): result limbs
template <int K, int DIGITS, bool SB = false>
__device__ __forceinline__ void f29_high(const fe29& a, const fe29& b, const int32_t* m,
                                         int64_t& acc, fe29& r) {
  if constexpr (K < DIGITS + NL29 - 1) {
    f29_column<K, DIGITS, SB>(a, b, m, acc);
    r.v[K - DIGITS] = (int32_t)acc & M29;
    acc >>= 29;
    f29_high<K + 1, DIGITS, SB>(a, b, m, acc, r);
  }
}

// a b 2^-(29 DIGITS) mod p, product scanning with the reduction interleaved
// per column.  Operands n or d; result n, in (-(1 + 2^-20) p, 2^-20 p) with
// fourteen digits, in (-|a b| / 2^377 - p, |a b| / 2^377] with thirteen.
template <int DIGITS = 14, bool SB = false>
__device__ __forceinline__ fe29 f29_mul(const fe29& a, const fe29& b) {
  int32_t m[DIGITS];
  fe29 r;
  int64_t acc = 0;
  f29_low<0, DIGITS, SB>(a, b, m, acc);
  f29_high<DIGITS, DIGITS, SB>(a, b, m, acc, r);
  r.v[NL29 - 1] = (int32_t)acc;
  return r;
}

// a times a constant (in SGPRs)
__device__ __forceinline__ fe29 f29_mul_const(const fe29& a, const int32_t (&c)[NL29]) {
  return f29_mul<14, true>(a, f29_const(c));
}

// columns [K, 26) of the 385-bit reduction: limbs straddle two columns
template <int K>
__device__ __forceinline__ void f29_high385(const fe29& a, const fe29& b, const int32_t* m,
                                            int64_t& acc, uint32_t& below, fe29& r) {
  if constexpr (K < 26) {
    f29_column<K, 14>(a, b, m, acc);
    const uint32_t lo = (uint32_t)acc;
    r.v[K - 14] = (int32_t)(__builtin_amdgcn_alignbit(lo, below << 3, 11) & (uint32_t)M29);
    below = lo;
    acc >>= 29;
    f29_high385<K + 1>(a, b, m, acc, below, r);
  }
}

// a b 2^-385 mod p: thirteen digits of 29 bits and one of 8.  Operands n or
// d; result n, in (-(1 + 2^-4) p, 2^-4 p) for |a b| < 8 p^2.  With it the
// additions keep the projective scale of R-form data (2 x 2^384 = 2^385:
// D = 2 Z1 Z2 2^-385 = Z1 for Z2 = 1), 26 more instructions than f29_mul.
__device__ __forceinline__ fe29 f29_mul385(const fe29& a, const fe29& b) {
  int32_t m[14];
  fe29 r;
  int64_t acc = 0;
  f29_low<0, 13>(a, b, m, acc);
  f29_column<13, 13>(a, b, m, acc);
  uint32_t below = (uint32_t)acc;
  m[13] = (int32_t)(below & 0xffu);
  acc >>= 29;
  f29_high385<14>(a, b, m, acc, below, r);
  // limb 12: the rest of column 25 and the carry above it, with its sign
  r.v[NL29 - 1] = (int32_t)(((uint32_t)acc << 21) | ((below & (uint32_t)M29) >> 8));
  return r;
}

// a + b, class d: 2^29 less per limb, one more in the next
__device__ __forceinline__ fe29 f29_add(const fe29& a, const fe29& b) {
  fe29 r;
  r.v[0] = a.v[0] + b.v[0] - (1 << 29);
#pragma unroll
  for (int i = 1; i < NL29 - 1; ++i) r.v[i] = a.v[i] + b.v[i] - M29;
  r.v[NL29 - 1] = a.v[NL29 - 1] + b.v[NL29 - 1] + 1;
  return r;
}

// a - b, class d
__device__ __forceinline__ fe29 f29_sub(const fe29& a, const fe29& b) {
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) r.v[i] = a.v[i] - b.v[i];
  return r;
}

// neg ? -a : a, limb-wise (one v_xad_u32 a limb)
__device__ __forceinline__ fe29 f29_negate_if(bool neg, const fe29& a) {
  const uint32_t mask = neg ? 0xffffffffu : 0u, one = neg ? 1u : 0u;
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) r.v[i] = (int32_t)(((uint32_t)a.v[i] ^ mask) + one);
  return r;
}

// r = (lane condition) ? x : y
__device__ __forceinline__ fe29 f29_select(bool c, const fe29& x, const fe29& y) {
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) r.v[i] = c ? x.v[i] : y.v[i];
  return r;
}

// a + b + p less 2^29 per limb: limbs within 3 x 2^28 of zero
__device__ __forceinline__ fe29 f29_add_p(const fe29& a, const fe29& b) {
  fe29 r;
  r.v[0] = a.v[0] + b.v[0] + (-kNP29[0] - (1 << 29));
#pragma unroll
  for (int i = 1; i < NL29 - 1; ++i) r.v[i] = a.v[i] + b.v[i] + (-kNP29[i] - M29);
  r.v[NL29 - 1] = a.v[NL29 - 1] + b.v[NL29 - 1] + (1 - kNP29[NL29 - 1]);
  return r;
}

// 2^8 z mod p: z class n with |z| < 2p; result n, magnitude below 0.51 p
// (the quotient by p comes from the top limb, off by less than 2^-12).
template <int K>
__device__ __forceinline__ void f29_shl8_limbs(const fe29& z, int32_t q, int64_t& acc, fe29& r) {
  if constexpr (K < NL29) {
    const int32_t x[2] = {z.v[K], q}, y[2] = {256, kNP29[K]};
    mad64_block<true, 0, 2>(acc, x, y, x, y);
    if constexpr (K + 1 < NL29) {
      r.v[K] = (int32_t)acc & M29;
      acc >>= 29;
    }
    f29_shl8_limbs<K + 1>(z, q, acc, r);
  }
}
__device__ __forceinline__ fe29 f29_shl8(const fe29& z) {
  const int32_t q = (int32_t)rintf((float)z.v[NL29 - 1] * (256.0f / 451126368.5f));
  fe29 r;
  int64_t acc = 0;
  f29_shl8_limbs<0>(z, q, acc, r);
  r.v[NL29 - 1] = (int32_t)acc;
  return r;
}

// z 2^-S mod p (S <= 29): 2^(29-S) z with one reduction digit.  z class n with
// |z| < 2p; result n, in (-(1 + 2^-20) p, 2^-20 p) for S > 20.
template <int S, int K>
__device__ __forceinline__ void f29_shift_limbs(const fe29& z, int32_t m, int64_t& acc, fe29& r) {
  if constexpr (K < NL29) {
    const int32_t x[2] = {z.v[K], m}, y[2] = {1 << (29 - S), kNP29[K]};
    mad64_block<true, 0, 2>(acc, x, y, x, y);
    r.v[K - 1] = (int32_t)acc & M29;
    acc >>= 29;
    f29_shift_limbs<S, K + 1>(z, m, acc, r);
  }
}
template <int S>
__device__ __forceinline__ fe29 f29_shift_right(const fe29& z) {
  const int32_t m = (int32_t)((uint32_t)z.v[0] << (29 - S)) & M29;
  fe29 r;
  int64_t acc = z.v[0] >> S;  // (2^(29-S) z_0 - m) / 2^29
  f29_shift_limbs<S, 1>(z, m, acc, r);
  r.v[NL29 - 1] = (int32_t)acc;
  return r;
}

// A stored coordinate (two's complement, in (-(1 + 2^-4) p, 2p)) as an
// unsigned value of the same residue in [0, 2p): a negative one gets p added,
// twice when it is below -p.  A value below p comes out canonical.
__device__ __forceinline__ fe fe_unsigned(const fe& x) {
  fe r = x;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint32_t mask = (uint32_t)((int32_t)r.v[NL - 1] >> 31);
    uint64_t c = 0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      c += (uint64_t)r.v[i] + (kP[i] & mask);
      r.v[i] = (uint32_t)c;
      c >>= 32;
    }
  }
  return r;
}

}  // namespace msm

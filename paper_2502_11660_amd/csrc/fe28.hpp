// Carry-free 28-bit field multiplication, one of the cores that
// msm_fe_mul_chain compares (device code).
//
// An element is fourteen 28-bit limbs, each in its own 32-bit word, so a
// 32x32->64 multiply-add of two limbs leaves room above the product: a 64-bit
// column accumulator absorbs every product of a column with no carry word.
// Montgomery form with R' = 2^392 = 2^(14*28).
//
// Bounds.  p < 2^377, R'/p > 38996.  For operands with limbs below 2^30 the
// largest column sum is 14 (2^30)^2 + 13 (2^28)^2 + 2^36 < 2^64, and
// REDC(a b) < 2p whenever a b < R' p.  Products return limbs 0..12 below
// 2^28 and the value below 2p.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "field.hpp"
#include "mad64.hpp"

namespace msm {

constexpr int NL28 = 14;
constexpr uint32_t M28 = 0x0fffffffu;

struct fe28 {
  uint32_t v[NL28];
};

// p in 28-bit limbs
constexpr uint32_t kP28[NL28] = {0x0000001u, 0x08c0000u, 0x0000085u, 0x5d44300u, 0x800170bu,
                                 0x2fba094u, 0xf1ef362u, 0x00f5138u, 0xa22d9f3u, 0xa1493b1u,
                                 0xb05c06cu, 0x10eac63u, 0xa4617c5u, 0x0001ae3u};
// 12 words (value < 2^392) -> 14 limbs: limb i holds bits 28i .. 28i + 27.
__device__ __forceinline__ fe28 f28_from_words(const fe& x) {
  fe28 r;
#pragma unroll
  for (int i = 0; i < NL28; ++i) {
    const int b = 28 * i, w = b >> 5, s = b & 31;
    if (s + 28 <= 32)
      r.v[i] = s + 28 == 32 ? x.v[w] >> s : (x.v[w] >> s) & M28;
    else if (w + 1 < NL)
      r.v[i] = __builtin_amdgcn_alignbit(x.v[w + 1], x.v[w], s) & M28;
    else
      r.v[i] = x.v[w] >> s;
  }
  return r;
}

// 14 limbs with limbs 0..12 normalised (value < 2^384) -> 12 words.
__device__ __forceinline__ fe f28_to_words(const fe28& x) {
  fe r;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int b = 32 * j, i = b / 28, s = b % 28;
    uint32_t w = x.v[i] >> s;
    w |= x.v[i + 1] << (28 - s);
    if (56 - s < 32) w |= x.v[i + 2] << (56 - s);
    r.v[j] = w;
  }
  return r;
}

// column K of a b + m p: the products a_i b_{K-i} and m_j p_{K-j} whose
// indices lie in [0, 14) (j < K below column 14, where m_K is not known yet)
template <int K>
__device__ __forceinline__ void f28_column(const fe28& a, const fe28& b, const uint32_t* m,
                                           uint64_t& acc) {
  constexpr int I0 = K < NL28 ? 0 : K - (NL28 - 1);
  constexpr int I1 = K < NL28 ? K : NL28 - 1;
  constexpr int J1 = K < NL28 ? K - 1 : NL28 - 1;
  uint32_t x[NL28], y[NL28];
#pragma unroll
  for (int i = I0; i <= I1; ++i) {
    x[i - I0] = a.v[i];
    y[i - I0] = b.v[K - i];
  }
  mad64_block<false, I1 - I0 + 1, 0>(acc, x, y, x, y);
  if constexpr (J1 >= I0) {
    uint32_t u[NL28], q[NL28];
#pragma unroll
    for (int j = I0; j <= J1; ++j) {
      u[j - I0] = m[j];
      q[j - I0] = kP28[K - j];
    }
    mad64_block<false, 0, J1 - I0 + 1>(acc, u, q, u, q);
  }
}

// low column K < 14 with column sum t: the reduction digit m_K = -t mod 2^28
// (-p^-1 = -1 mod 2^28 since p = 1 mod 2^46) clears the column's low 28 bits
// when m_K p_0 = m_K is added, so the carry is (t + m_K) >> 28, which equals
// (t + 2^28 - 1) >> 28; with u = t + 2^28 - 1, m_K is also ~u mod 2^28 (one
// and-not of u's low word)
template <int K>
__device__ __forceinline__ void f28_low(const fe28& a, const fe28& b, uint32_t* m, uint64_t& acc) {
  f28_column<K>(a, b, m, acc);
  acc += M28;
  m[K] = ~(uint32_t)acc & M28;
  acc >>= 28;
}

// high column K >= 14: result limb K - 14
template <int K>
__device__ __forceinline__ void f28_high(const fe28& a, const fe28& b, const uint32_t* m,
                                         uint64_t& acc, fe28& r) {
  f28_column<K>(a, b, m, acc);
  r.v[K - NL28] = (uint32_t)acc & M28;
  acc >>= 28;
}

// Montgomery product a b 2^-392 mod p, product scanning with the reduction
// interleaved per column: column k's products are added onto the carry of
// column k - 1 in one 64-bit accumulator.  Operands: limbs < 2^30 and
// a b < R' p.  Result: limbs 0..12 normalised, value < 2p.
__device__ __forceinline__ fe28 f28_mul(const fe28& a, const fe28& b) {
  uint32_t m[NL28];
  fe28 r;
  uint64_t acc = 0;
  f28_low<0>(a, b, m, acc);
  f28_low<1>(a, b, m, acc);
  f28_low<2>(a, b, m, acc);
  f28_low<3>(a, b, m, acc);
  f28_low<4>(a, b, m, acc);
  f28_low<5>(a, b, m, acc);
  f28_low<6>(a, b, m, acc);
  f28_low<7>(a, b, m, acc);
  f28_low<8>(a, b, m, acc);
  f28_low<9>(a, b, m, acc);
  f28_low<10>(a, b, m, acc);
  f28_low<11>(a, b, m, acc);
  f28_low<12>(a, b, m, acc);
  f28_low<13>(a, b, m, acc);
  f28_high<14>(a, b, m, acc, r);
  f28_high<15>(a, b, m, acc, r);
  f28_high<16>(a, b, m, acc, r);
  f28_high<17>(a, b, m, acc, r);
  f28_high<18>(a, b, m, acc, r);
  f28_high<19>(a, b, m, acc, r);
  f28_high<20>(a, b, m, acc, r);
  f28_high<21>(a, b, m, acc, r);
  f28_high<22>(a, b, m, acc, r);
  f28_high<23>(a, b, m, acc, r);
  f28_high<24>(a, b, m, acc, r);
  f28_high<25>(a, b, m, acc, r);
  f28_high<26>(a, b, m, acc, r);
  r.v[NL28 - 1] = (uint32_t)acc;
  return r;
}

}  // namespace msm

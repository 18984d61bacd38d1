// Twisted-Edwards point additions on the signed 29-bit field form (fe29.hpp):
// the one-lane throughput unit of bucket accumulation, the standalone PADD
// kernel, the split-bucket merges and the large aggregation levels.
//
// Same unified law as curve.hpp (Hisil, Wong, Carter and Dawson 2008, a = -1,
// Sec. II-D):
//   A = (Y1 - X1)(Y2 - X2)   B = (Y1 + X1)(Y2 + X2)   C = T1 k T2   D = 2 Z1 Z2
//   E = B - A   F = D - C   G = D + C   H = B + A
//   X3 = E F    Y3 = G H    T3 = E H    Z3 = F G
//
// Bounds (fe29.hpp's limb classes; values in units of p, "~" up to a relative
// 2^-20, or 2^-4 after f29_mul385):
//   inputs: n, products in (-~1, ~0] or stored values in (-~1, 2)
//   Y1 - X1, Y2 - X2: d, magnitude < 3~    Y1 + X1, Y2 + X2: d, magnitude < 4
//   2 Z2 (complete): d, magnitude < 4
//   A, B, C, D: n, in (-~1, ~0]
//   E = B - A, F = D - C: d, magnitude < ~1    H = B + A, G = D + C: d, < ~2
// so every operand is n or d and below 4.76p, every product below 16 p^2, and
// the outputs are n, in (-~1, ~0].
// The mixed addition reduces A, B, C by 2^377 (p / 2^377 = 0.841) and takes
// Y1 + X1 + p, in (-~1, ~1], for Y1 + X1, with a's coordinates products
// (in (-~1, ~0]) and b canonical:
//   Y1 - X1, Y2 - X2: magnitude < ~1   Y2 + X2: [0, 2)
//   A, B: the product with Y2 + X2 in (-2.69, 1.69), the other in (-1.85, 0.85)
//   C in (-1.85, 0.85)   D = 2^8 Z1: magnitude < 0.51
//   E: < 3.54   H: < 4.54   F, G: < 2.4
#pragma once
#include "curve.hpp"
#include "fe29.hpp"

namespace msm {

struct xytz29 {
  fe29 X, Y, T, Z;
};

struct xyu29 {
  fe29 X, Y, U;
};

// identity (0 : 1 : 0 : 1); any common non-zero Y = Z is the same point
__device__ __forceinline__ xytz29 pt29_identity() {
  xytz29 r;
  r.X = f29_small(0);
  r.Y = f29_small(1);
  r.T = f29_small(0);
  r.Z = f29_small(1);
  return r;
}

__device__ __forceinline__ xytz29 pt29_from(const xytz& p) {
  xytz29 r;
  r.X = f29_from_words(p.X);
  r.Y = f29_from_words(p.Y);
  r.T = f29_from_words(p.T);
  r.Z = f29_from_words(p.Z);
  return r;
}

__device__ __forceinline__ xyu29 pt29_from(const xyu& p) {
  xyu29 r;
  r.X = f29_from_words(p.X);
  r.Y = f29_from_words(p.Y);
  r.U = f29_from_words(p.U);
  return r;
}

// products only (class n)
__device__ __forceinline__ xytz pt29_to_words(const xytz29& p) {
  xytz r;
  r.X = f29_to_words(p.X);
  r.Y = f29_to_words(p.Y);
  r.T = f29_to_words(p.T);
  r.Z = f29_to_words(p.Z);
  return r;
}

// the same with coordinates in [0, 2p), the form of the library's outputs
__device__ __forceinline__ xytz pt29_to_unsigned(const xytz29& p) {
  const xytz w = pt29_to_words(p);
  xytz r;
  r.X = fe_unsigned(w.X);
  r.Y = fe_unsigned(w.Y);
  r.T = fe_unsigned(w.T);
  r.Z = fe_unsigned(w.Z);
  return r;
}

__device__ __forceinline__ xytz29 padd29_tail(const fe29& A, const fe29& B, const fe29& C,
                                              const fe29& D) {
  const fe29 E = f29_sub(B, A), H = f29_add(B, A), F = f29_sub(D, C), G = f29_add(D, C);
  xytz29 r;
  r.X = f29_mul(E, F);
  r.Y = f29_mul(G, H);
  r.T = f29_mul(E, H);
  r.Z = f29_mul(F, G);
  return r;
}

// a + b (neg = false) or a - b (neg = true), b prepared.  -b = (-X2, Y2, -U2)
// exchanges Y2 - X2 with Y2 + X2 and negates U2.  7 products.
__device__ __forceinline__ xytz29 padd29_mixed_signed(const xytz29& a, const xyu29& b, bool neg) {
  const fe29 bm = f29_sub(b.Y, b.X), bp = f29_add(b.Y, b.X);
  const fe29 A = f29_mul<13>(f29_sub(a.Y, a.X), f29_select(neg, bp, bm));
  const fe29 B = f29_mul<13>(f29_add_p(a.Y, a.X), f29_select(neg, bm, bp));
  const fe29 C = f29_mul<13>(a.T, f29_negate_if(neg, b.U));
  return padd29_tail(A, B, C, f29_shl8(a.Z));
}

__device__ __forceinline__ xytz29 padd29_mixed(const xytz29& a, const xyu29& b) {
  return padd29_mixed_signed(a, b, false);
}

// a + b, both extended: 9 products (k T2 formed on the fly).
__device__ __forceinline__ xytz29 padd29_full(const xytz29& a, const xytz29& b) {
  const fe29 A = f29_mul(f29_sub(a.Y, a.X), f29_sub(b.Y, b.X));
  const fe29 B = f29_mul(f29_add(a.Y, a.X), f29_add(b.Y, b.X));
  const fe29 C = f29_mul(a.T, f29_mul_const(b.T, kK29));
  const fe29 D = f29_mul(a.Z, f29_add(b.Z, b.Z));
  return padd29_tail(A, B, C, D);
}

// The two additions with the first four products reduced by 2^385, which
// leaves the result's projective scale what the R = 2^384 form's formulas
// give it (3 reductions by 2^392 in all): msm_padd_batch returns these
// coordinates themselves.
__device__ __forceinline__ xytz29 padd29_mixed_scaled(const xytz29& a, const xyu29& b) {
  const fe29 A = f29_mul385(f29_sub(a.Y, a.X), f29_sub(b.Y, b.X));
  const fe29 B = f29_mul385(f29_add(a.Y, a.X), f29_add(b.Y, b.X));
  const fe29 C = f29_mul385(a.T, b.U);
  return padd29_tail(A, B, C, a.Z);  // D = 2 Z1 2^384 2^-385
}

__device__ __forceinline__ xytz29 padd29_full_scaled(const xytz29& a, const xytz29& b) {
  const fe29 A = f29_mul385(f29_sub(a.Y, a.X), f29_sub(b.Y, b.X));
  const fe29 B = f29_mul385(f29_add(a.Y, a.X), f29_add(b.Y, b.X));
  const fe29 C = f29_mul385(a.T, f29_mul_const(b.T, kK29));
  const fe29 D = f29_mul385(a.Z, f29_add(b.Z, b.Z));
  return padd29_tail(A, B, C, D);
}

}  // namespace msm

// Elementwise kernels: batched field multiply, batched PADD (the paper's
// "task", Sec. II-D / V-A), point preparation and the synthetic point
// generator.
#include <algorithm>

#include "common.hpp"
#include "convert.hpp"
#include "curve29.hpp"

namespace msm {
namespace {

__global__ void __launch_bounds__(256) k_fe_mul(const uint32_t* __restrict__ a,
                                                const uint32_t* __restrict__ b,
                                                uint32_t* __restrict__ out, uint32_t count,
                                                int canonical) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  fe r = fe_mul(ld_soa(a, count, 0, i), ld_soa(b, count, 0, i));
  if (canonical) r = fe_canon(r);
  st_soa(out, count, 0, i, r);
}

// SoA rows through buffer instructions: row r of an array (word r count + i
// of element i) is a wave-uniform base, so its buffer descriptor lives in
// scalar registers and every load or store takes the one per-lane byte
// offset 4 i, with no per-access address arithmetic on the vector unit.
// Requires count < 2^29 (4 count fits a descriptor's 32-bit byte range).
constexpr uint32_t kBufferFlags = 0x00020000u;  // raw 32-bit buffer access

__device__ __forceinline__ fe ld_rows(const uint32_t* __restrict__ base, uint32_t count, int coord,
                                      uint32_t voff) {
  fe r;
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const uint32_t* row = base + (size_t)(coord * NL + l) * count;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)row, 0, (int)(count * 4u), kBufferFlags);
    r.v[l] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, 0, 0);
  }
  return r;
}

__device__ __forceinline__ void st_rows(uint32_t* __restrict__ base, uint32_t count, int coord,
                                        uint32_t voff, const fe& x) {
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    uint32_t* row = base + (size_t)(coord * NL + l) * count;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)row, 0, (int)(count * 4u), kBufferFlags);
    __builtin_amdgcn_raw_buffer_store_b32(x.v[l], rs, voff, 0, 0);
  }
}

// out_i = a_i + b_i, SoA limb-major operands; FORM selects the mixed
// (b prepared: X, Y, U, Z = 1) or the complete (b extended) addition.  On the
// signed 29-bit field form (curve29.hpp); outputs canonical.
template <int FORM>
__global__ void __launch_bounds__(256) k_padd(const uint32_t* __restrict__ a,
                                              const uint32_t* __restrict__ b,
                                              uint32_t* __restrict__ out, uint32_t count) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t vo = 4u * i;
  xytz29 pa;
  pa.X = f29_from_words(ld_rows(a, count, 0, vo));
  pa.Y = f29_from_words(ld_rows(a, count, 1, vo));
  pa.T = f29_from_words(ld_rows(a, count, 2, vo));
  pa.Z = f29_from_words(ld_rows(a, count, 3, vo));
  xytz29 r;
  if (FORM == MSM_FORM_XYU) {
    xyu29 pb;
    pb.X = f29_from_words(ld_rows(b, count, 0, vo));
    pb.Y = f29_from_words(ld_rows(b, count, 1, vo));
    pb.U = f29_from_words(ld_rows(b, count, 2, vo));
    r = padd29_mixed_scaled(pa, pb);
  } else {
    xytz29 pb;
    pb.X = f29_from_words(ld_rows(b, count, 0, vo));
    pb.Y = f29_from_words(ld_rows(b, count, 1, vo));
    pb.T = f29_from_words(ld_rows(b, count, 2, vo));
    pb.Z = f29_from_words(ld_rows(b, count, 3, vo));
    r = padd29_full_scaled(pa, pb);
  }
  st_rows(out, count, 0, vo, fe_unsigned(f29_to_words(r.X)));
  st_rows(out, count, 1, vo, fe_unsigned(f29_to_words(r.Y)));
  st_rows(out, count, 2, vo, fe_unsigned(f29_to_words(r.T)));
  st_rows(out, count, 3, vo, fe_unsigned(f29_to_words(r.Z)));
}

// Weierstrass affine (ordinary form) -> prepared (X, Y, U = k x y), Z = 1
// (Sec. II-D: inputs enter as (X, Y, U, Z = 1)):
//   w = x + 1,  x_e = (beta/alpha) w / y,  y_e = (w - alpha) / (w + alpha)
// so each point needs the inverses of y and w + alpha, and its image phi(P) =
// (omega x, y) that of omega x + 1 + alpha.  They come from one inversion per
// wave (Montgomery's trick, on three levels).  Each lane walks its points
// forward multiplying their denominators d = y (w + alpha) (omega x + 1 + alpha)
// into a running product (each point's record slot keeps the product before
// it); the wave then forms prefix and suffix products of the 64 lane products
// (six shuffle-and-multiply steps each), inverts the wave's total once with
// all lanes cooperating (fe_inv_lanes), and gives each lane the inverse of its
// own product as total^-1 x prefix x suffix.  Walking back, the inverse of
// point j's d is (inverse of the product up to j) times (product before j),
// multiplying by d steps the inverse back, and d's factors split the inverse.
// A zero denominator (an exceptional point, flagged; it cannot lie in the
// prime-order subgroup) enters the product as 1 so that it does not spoil the
// batch; its own record is then unspecified.
//
// On the signed 29-bit form (fe29.hpp), whose products reduce by 2^406: an
// input x as it is stands for x 2^-406 there, every denominator with it, and
// the constants below bring the outputs into R = 2^384 form, so that nothing is
// converted on the way in.  Bound by VALU issue: 26 products a point with its
// image, 16 without (34 and 21 on the out-of-line 12-word multiply before):
// n = 2^20 with images 764 -> 457 us, without 489 -> 302; few points take the
// wave inversion's latency, 92 -> 68 and 73 -> 60 us.
// 1 in the 2^406 form, and 2^812, which takes a value into it
constexpr int32_t kPrepOne[NL29] = {0x19eaf730, 0x171ffffe, 0xd714cf8, 0x44e31d8, 0x1eb6e262,
    0xbfad163, 0xd46e9c, 0x10b6ddbf, 0x13b9cbdd,
    0x75782af, 0x3bd1d8a, 0x1557cab6, 0x15742a14};
constexpr int32_t kPrepIn[NL29] = {0x1c14cc5c, 0x7b8df46, 0x4c74875, 0xd6832fa,
    0x5f4afc1, 0x11ea1ee5, 0x9265a5f, 0x9fa84f9, 0x12f6f558,
    0x18644b2b, 0x1caa9452, 0x11db07d, 0xef492d1};
// omega 2^406: x -> omega x
constexpr int32_t kPrepOmega[NL29] = {0x1c8a7893, 0xb7d08f2, 0x6b88506, 0x162aa2ed, 0x1c5fdf80,
    0x11b95a22, 0x3b86dd7, 0x1191f770, 0x10701220,
    0x1501c11f, 0x1cee88bb, 0x118d05ec, 0x6f2fa26};
// 1 + alpha and 1 - alpha
constexpr int32_t kPrepPlus[NL29] = {0x109adc02, 0x2c1256, 0x71e9f27, 0x17651e1c, 0x64272e6,
    0x5b2fe0b, 0x1690bf8b, 0x663068c, 0xe86ef0d,
    0x10ae65fc, 0x16505bb3, 0xc5a693c, 0x32d7560};
constexpr int32_t kPrepMinus[NL29] = {0xf652401, 0x819eda9, 0x18e160fa, 0x1f556a43,
    0xe3d8e89, 0xb64def9, 0x17abbc42, 0x17fd1815, 0xc9333cc,
    0x12b6a44d, 0x1b3e65bc, 0x32fb898, 0x17b62f01};
// 2^1218: a plain inverse of a value of the 2^406 form -> its inverse there
constexpr int32_t kPrepInv[NL29] = {0x116ee469, 0x193358dc, 0x5d36c9a, 0x8690878, 0x7b9a713,
    0x31c169b, 0x1de45103, 0x94b9b1e, 0x140c4b90,
    0xe3a757c, 0x1315b3f7, 0x393cb0b, 0xfeb6639};
// (beta / alpha) 2^384 and k 2^428: the outputs' R = 2^384 form
constexpr int32_t kPrepX[NL29] = {0xad605e4, 0x1be055c7, 0x1d4b1ebe, 0x1727a3c4, 0x1e536363,
    0x141a8a25, 0x1df4891, 0x1ba853e4, 0x3eb8bf6,
    0x1011a6a1, 0xea7bf68, 0x1418e548, 0x13c7943b};
constexpr int32_t kPrepU[NL29] = {0xc36d10f, 0x57c900d, 0x1bd871b8, 0x1d41bd7,
    0xc494f80, 0xbb719fe, 0x3a2ee3b, 0x15c2767f, 0x1aff76a6,
    0xea89726, 0x107baa55, 0x1c32e522, 0x8af1458};

// lane-to-lane moves of a field element (lanes without a source keep x)
__device__ __forceinline__ fe29 f29_shfl_up(const fe29& x, int d) {
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) r.v[i] = __shfl_up(x.v[i], d, 64);
  return r;
}

__device__ __forceinline__ fe29 f29_shfl_down(const fe29& x, int d) {
  fe29 r;
#pragma unroll
  for (int i = 0; i < NL29; ++i) r.v[i] = __shfl_down(x.v[i], d, 64);
  return r;
}

// canonical words of a product
__device__ __forceinline__ fe f29_canon(const fe29& x) { return fe_unsigned(f29_to_words(x)); }

// Every lane's v^-1 (2^406 form) for a non-zero product v, with one inversion
// for the wave.  All 64 lanes of the wave must take part.
__device__ __forceinline__ fe29 wave_batch_inverse(const fe29& v) {
  const int lane = (int)__lane_id();
  fe29 A = v, B = v;  // inclusive prefix and suffix products over the lanes
#pragma unroll 1
  for (int d = 1; d < 64; d <<= 1) {
    const fe29 au = f29_mul(A, f29_shfl_up(A, d));
    const fe29 bd = f29_mul(B, f29_shfl_down(B, d));
    A = f29_select(lane >= d, au, A);
    B = f29_select(lane + d < 64, bd, B);
  }
  fe29 total;
#pragma unroll
  for (int i = 0; i < NL29; ++i) total.v[i] = __builtin_amdgcn_readlane(A.v[i], 63);
  const fe29 E = f29_select(lane == 0, f29_const(kPrepOne), f29_shfl_up(A, 1));     // lanes below
  const fe29 S = f29_select(lane == 63, f29_const(kPrepOne), f29_shfl_down(B, 1));  // lanes above
  const fe29 es = f29_mul(E, S);
  const fe inv = fe_inv_lanes(f29_canon(total));
  return f29_mul(f29_mul_const(f29_from_words(inv), kPrepInv), es);
}

__device__ __forceinline__ void prepare_identity(uint32_t* rec) {
  st_aos(rec, 0, fe_zero());
  st_aos(rec, 1, fe_const(kOne));
  st_aos(rec, 2, fe_zero());
}

// Point i.  Points come from outside: coordinates that are not canonical (any 384 bits)
// are brought below p + 2^352, for one comparison where both are.
__device__ __forceinline__ void prep_load(const uint32_t* __restrict__ xy, uint32_t n, size_t i,
                                          fe29& x, fe29& y) {
  fe v[2] = {ld_soa(xy, n, 0, i), ld_soa(xy, n, 1, i)};
  if (max(v[0].v[NL - 1], v[1].v[NL - 1]) > kP[NL - 1]) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll 1
      while (v[c].v[NL - 1] > kP[NL - 1]) {
        uint64_t borrow;
        v[c] = fe_sub_mask(v[c], fe_const(kP), borrow);
      }
  }
  x = f29_from_words(v[0]);
  y = f29_from_words(v[1]);
}

// the image's x, the product of the w + alpha (of the point and its image),
// and the factor d of the batch (1 for a zero denominator)
struct prep_den {
  fe29 xb, P, d;
};
template <bool ENDO>
__device__ __forceinline__ prep_den prep_denominators(const fe29& x, const fe29& y,
                                                      uint32_t& flags) {
  prep_den r;
  const fe29 wa = f29_add(x, f29_const(kPrepPlus));
  if (ENDO) {
    r.xb = f29_mul_const(x, kPrepOmega);
    r.P = f29_mul(wa, f29_add(r.xb, f29_const(kPrepPlus)));
  } else {
    r.xb = x;
    r.P = wa;
  }
  r.d = f29_mul(r.P, y);
  if (fe_is_zero_canon(f29_canon(r.d))) {
    flags |= MSM_FLAG_EXCEPT;
    r.d = f29_const(kPrepOne);
  }
  return r;
}

// Thread t prepares points i = t + j T, j = 0 .. m-1 (i < n), T = threads;
// threads t >= T take part in the wave-wide inversion only.
// ENDO: records 2i and 2i + 1 hold point i and its image (omega x, y).
template <bool ENDO>
__global__ void __launch_bounds__(256, ENDO ? 2 : 4) k_prepare(const uint32_t* __restrict__ xy,
                                                 const uint32_t* __restrict__ inf,
                                                 uint32_t* __restrict__ out, uint32_t n,
                                                 uint32_t T, uint32_t m,
                                                 uint32_t* __restrict__ status) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t mine = t < T ? m : 0u;
  uint32_t flags = 0;
  fe29 c = f29_const(kPrepOne);  // product of the factors so far
  uint32_t last = 0;             // points of this thread
#pragma unroll 1
  for (uint32_t j = 0; j < mine; ++j) {
    const uint64_t i = (uint64_t)t + (uint64_t)j * T;
    if (i >= n) break;
    last = j + 1;
    if (inf && inf[i]) continue;
    fe29 x, y;
    prep_load(xy, n, (size_t)i, x, y);
    // y^2 - 1 = x^3
    fe29 ym = y, yp = y;
    ym.v[0] -= 1;
    yp.v[0] += 1;
    const fe lhs = f29_canon(f29_mul(ym, yp));
    const fe rhs = f29_canon(f29_mul(f29_mul(x, x), f29_mul_const(x, kPrepIn)));
    if (!fe_eq_canon(lhs, rhs)) flags |= MSM_FLAG_OFFCURVE;
    const prep_den e = prep_denominators<ENDO>(x, y, flags);
    st_aos(out + (size_t)(ENDO ? 2 * i : i) * XYU_WORDS, 0, f29_to_words(c));  // product before i
    c = f29_mul(c, e.d);
  }
  fe29 tinv = wave_batch_inverse(c);  // inverse of this thread's product
#pragma unroll 1
  for (uint32_t jj = last; jj-- > 0;) {
    const uint64_t i = (uint64_t)t + (uint64_t)jj * T;
    uint32_t* rec = out + (size_t)(ENDO ? 2 * i : i) * XYU_WORDS;
    if (inf && inf[i]) {
      prepare_identity(rec);
      if (ENDO) prepare_identity(rec + XYU_WORDS);
      continue;
    }
    fe29 x, y;
    prep_load(xy, n, (size_t)i, x, y);
    uint32_t dummy = 0;
    const prep_den e = prep_denominators<ENDO>(x, y, dummy);
    const fe29 inv_d = f29_mul(tinv, f29_from_words(ld_aos(rec, 0)));  // 1 / d
    tinv = f29_mul(tinv, e.d);  // 1 / (product before this point)
    const fe29 xs = f29_mul_const(f29_mul(inv_d, e.P), kPrepX);  // (beta / alpha) / y
    // 1 / P in the outputs' form (2^406 to 2^384)
    const fe29 inv_p = f29_shift_right<22>(f29_mul(inv_d, y));
#pragma unroll 1
    for (uint32_t im = 0; im < (ENDO ? 2u : 1u); ++im) {
      const fe29 px = ENDO ? f29_select(im != 0, e.xb, x) : x;
      const fe29 other = f29_add(f29_select(im != 0, x, e.xb), f29_const(kPrepPlus));
      fe29 w = px;
      w.v[0] += 1;
      const fe29 xe = f29_mul(w, xs);
      const fe29 inv_w = ENDO ? f29_mul(inv_p, other) : inv_p;
      const fe29 ye = f29_mul(f29_add(px, f29_const(kPrepMinus)), inv_w);
      const fe29 u = f29_mul(f29_mul_const(xe, kPrepU), ye);
      st_aos(rec, 0, f29_canon(xe));
      st_aos(rec, 1, f29_canon(ye));
      st_aos(rec, 2, f29_canon(u));
      rec += XYU_WORDS;
    }
  }
  if (flags) atomicOr(status, flags);
}

// P_i = k_i G: most-significant-bit-first double-and-add in twisted-Edwards
// coordinates, then mapped to Weierstrass affine.
__global__ void __launch_bounds__(256) k_gen_points(const uint32_t* __restrict__ kk,
                                                    uint32_t* __restrict__ xy,
                                                    uint32_t* __restrict__ inf, uint32_t n) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const fe p2 = fe_const(kP2);
  xyu g;
  g.X = fe_const(kGteX);
  g.Y = fe_const(kGteY);
  g.U = fe_const(kGteU);
  uint32_t kw[SCALAR_WORDS];
#pragma unroll
  for (int j = 0; j < SCALAR_WORDS; ++j) kw[j] = kk[(size_t)i * SCALAR_WORDS + j];
  xytz acc = pt_identity();
  for (int j = SCALAR_WORDS - 1; j >= 0; --j) {
    uint32_t word = kw[j];
    for (int bit = 31; bit >= 0; --bit) {
      acc = pdbl(acc, p2);
      if ((word >> bit) & 1u) acc = padd_mixed(acc, g, p2);
    }
  }
  fe xw, yw;
  bool fin = te_to_weierstrass(acc, xw, yw);
  st_soa(xy, n, 0, i, xw);
  st_soa(xy, n, 1, i, yw);
  inf[i] = fin ? 0u : 1u;
}

}  // namespace

int launch_fe_mul(const uint32_t* a, const uint32_t* b, uint32_t* out, uint32_t count,
                  int canonical, hipStream_t st) {
  k_fe_mul<<<grid_for(count, 256), 256, 0, st>>>(a, b, out, count, canonical);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

int launch_padd(const uint32_t* a, const uint32_t* b, uint32_t* out, uint32_t count, int form,
                hipStream_t st) {
  if (form == MSM_FORM_XYU)
    k_padd<MSM_FORM_XYU><<<grid_for(count, 256), 256, 0, st>>>(a, b, out, count);
  else
    k_padd<MSM_FORM_XYTZ><<<grid_for(count, 256), 256, 0, st>>>(a, b, out, count);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

int launch_prepare(const uint32_t* xy, const uint32_t* inf, uint32_t* xyu, uint32_t n,
                   uint32_t* status, bool endo, hipStream_t st) {
  // points per thread: at most two waves per SIMD, the most the registers of the
  // form with images allow (256 CUs x 4 SIMDs x 64 lanes x 2), the rest of the
  // points batched; n = 2^20 with images at three waves and spills 504 us, at one
  // 514, against 457.  Rounded up, so that no second round follows for a few
  // threads: n = 1500000 with images 501 -> 397 us, without 322 -> 272, n = 700000
  // 248 -> 199 and 168 -> 135 (n = 262145 without 78 -> 81).
  const uint32_t m = std::max<uint32_t>(1u, std::min<uint32_t>(64u, (n + 131071u) / 131072u));
  const uint32_t T = (uint32_t)(((uint64_t)n + m - 1) / m);
  if (endo)
    k_prepare<true><<<grid_for(T, 256), 256, 0, st>>>(xy, inf, xyu, n, T, m, status);
  else
    k_prepare<false><<<grid_for(T, 256), 256, 0, st>>>(xy, inf, xyu, n, T, m, status);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

int launch_gen_points(const uint32_t* k, uint32_t* xy, uint32_t* inf, uint32_t n, hipStream_t st) {
  k_gen_points<<<grid_for(n, 256), 256, 0, st>>>(k, xy, inf, n);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

}  // namespace msm

// Grouped 32x32->64 multiply-adds without carry words (device code): the
// building block of the one-lane field cores (fe29.hpp, fe28.hpp).
//
// N products are added into one 64-bit column accumulator by one asm block
// (written as asm so that the column's products are added in order onto the
// incoming carry: as plain C the compiler sums each column from zero and adds
// the carry afterwards, one extra 64-bit add per column; grouped because the
// compiler puts a wait state after every asm block).  OP is v_mad_u64_u32 or
// v_mad_i64_i32, CB the second factor's constraint ("v" for a VGPR, "s" for an
// SGPR such as a limb of p).  The carry-out goes to a scratch SGPR pair (cc)
// that nothing reads; it is early-clobber ("=&s") because the block's first
// multiply-add writes it before the later ones read their factors, so it must
// not share a register with an SGPR factor.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace msm {
#define MSM_MAD64_1(OP, CB, acc, cc, a0, b0) \
  asm(OP" %0, %1, %2, %3, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0))

#define MSM_MAD64_2(OP, CB, acc, cc, a0, b0, a1, b1) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1))

#define MSM_MAD64_3(OP, CB, acc, cc, a0, b0, a1, b1, a2, b2) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0\n\t" \
      OP" %0, %1, %6, %7, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1), "v"(a2), CB(b2))

#define MSM_MAD64_4(OP, CB, acc, cc, a0, b0, a1, b1, a2, b2, a3, b3) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0\n\t" \
      OP" %0, %1, %6, %7, %0\n\t" \
      OP" %0, %1, %8, %9, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1), "v"(a2), CB(b2), "v"(a3), CB(b3))

#define MSM_MAD64_5(OP, CB, acc, cc, a0, b0, a1, b1, a2, b2, a3, b3, a4, b4) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0\n\t" \
      OP" %0, %1, %6, %7, %0\n\t" \
      OP" %0, %1, %8, %9, %0\n\t" \
      OP" %0, %1, %10, %11, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1), "v"(a2), CB(b2), "v"(a3), CB(b3), "v"(a4), CB(b4))

#define MSM_MAD64_6(OP, CB, acc, cc, a0, b0, a1, b1, a2, b2, a3, b3, a4, b4, a5, b5) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0\n\t" \
      OP" %0, %1, %6, %7, %0\n\t" \
      OP" %0, %1, %8, %9, %0\n\t" \
      OP" %0, %1, %10, %11, %0\n\t" \
      OP" %0, %1, %12, %13, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1), "v"(a2), CB(b2), "v"(a3), CB(b3), "v"(a4), CB(b4), "v"(a5), CB(b5))

#define MSM_MAD64_7(OP, CB, acc, cc, a0, b0, a1, b1, a2, b2, a3, b3, a4, b4, a5, b5, a6, b6) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0\n\t" \
      OP" %0, %1, %6, %7, %0\n\t" \
      OP" %0, %1, %8, %9, %0\n\t" \
      OP" %0, %1, %10, %11, %0\n\t" \
      OP" %0, %1, %12, %13, %0\n\t" \
      OP" %0, %1, %14, %15, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1), "v"(a2), CB(b2), "v"(a3), CB(b3), "v"(a4), CB(b4), "v"(a5), CB(b5), "v"(a6), CB(b6))

#define MSM_MAD64_8(OP, CB, acc, cc, a0, b0, a1, b1, a2, b2, a3, b3, a4, b4, a5, b5, a6, b6, a7, b7) \
  asm(OP" %0, %1, %2, %3, %0\n\t" \
      OP" %0, %1, %4, %5, %0\n\t" \
      OP" %0, %1, %6, %7, %0\n\t" \
      OP" %0, %1, %8, %9, %0\n\t" \
      OP" %0, %1, %10, %11, %0\n\t" \
      OP" %0, %1, %12, %13, %0\n\t" \
      OP" %0, %1, %14, %15, %0\n\t" \
      OP" %0, %1, %16, %17, %0" \
      : "+v"(acc), "=&s"(cc) \
      : "v"(a0), CB(b0), "v"(a1), CB(b1), "v"(a2), CB(b2), "v"(a3), CB(b3), "v"(a4), CB(b4), "v"(a5), CB(b5), "v"(a6), CB(b6), "v"(a7), CB(b7))


template <int N, bool SIGNED, bool SGPR_Y, typename A, typename W>
__device__ __forceinline__ void mad64_group(A& acc, const W* x, const W* y) {
  uint64_t cc;
#define MSM_G1 x[0], y[0]
#define MSM_G2 MSM_G1, x[1], y[1]
#define MSM_G3 MSM_G2, x[2], y[2]
#define MSM_G4 MSM_G3, x[3], y[3]
#define MSM_G5 MSM_G4, x[4], y[4]
#define MSM_G6 MSM_G5, x[5], y[5]
#define MSM_G7 MSM_G6, x[6], y[6]
#define MSM_G8 MSM_G7, x[7], y[7]
#define MSM_CALL(f, ...) f(__VA_ARGS__)
#define MSM_GROUP(n)                                                        \
  if constexpr (N == n) {                                                   \
    if constexpr (SIGNED && SGPR_Y)                                         \
      MSM_CALL(MSM_MAD64_##n, "v_mad_i64_i32", "s", acc, cc, MSM_G##n);     \
    else if constexpr (SIGNED)                                              \
      MSM_CALL(MSM_MAD64_##n, "v_mad_i64_i32", "v", acc, cc, MSM_G##n);     \
    else if constexpr (SGPR_Y)                                              \
      MSM_CALL(MSM_MAD64_##n, "v_mad_u64_u32", "s", acc, cc, MSM_G##n);     \
    else                                                                    \
      MSM_CALL(MSM_MAD64_##n, "v_mad_u64_u32", "v", acc, cc, MSM_G##n);     \
  }
  MSM_GROUP(1)
  MSM_GROUP(2)
  MSM_GROUP(3)
  MSM_GROUP(4)
  MSM_GROUP(5)
  MSM_GROUP(6)
  MSM_GROUP(7)
  MSM_GROUP(8)
#undef MSM_GROUP
#undef MSM_CALL
#undef MSM_G8
#undef MSM_G7
#undef MSM_G6
#undef MSM_G5
#undef MSM_G4
#undef MSM_G3
#undef MSM_G2
#undef MSM_G1
  (void)cc;
}

// acc += sum of the L products x[t] y[t] (y in SGPRs when SGPR_Y)
template <int L, bool SIGNED, bool SGPR_Y, typename A, typename W>
__device__ __forceinline__ void mad64_run(A& acc, const W* x, const W* y) {
  if constexpr (L > 0) {
    constexpr int G = L < 8 ? L : 8;
    mad64_group<G, SIGNED, SGPR_Y>(acc, x, y);
    if constexpr (L > G) mad64_run<L - G, SIGNED, SGPR_Y>(acc, x + G, y + G);
  }
}

}  // namespace msm

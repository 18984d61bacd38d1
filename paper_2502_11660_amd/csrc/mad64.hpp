// Column sums of 32x32->64 multiply-adds without carry words (device code): the
// building block of the one-lane field cores (fe29.hpp, fe28.hpp).
//
// All of a column's products are added into one 64-bit accumulator by one asm
// block (written as asm so that they are added in order onto the incoming
// carry: as plain C the compiler sums each column from zero and adds the carry
// afterwards, one extra 64-bit add per column; one block, because the compiler
// puts a wait state after every one, an instruction slot to a lone wave).  The
// products of a block are of two VGPRs first, then of a VGPR and an SGPR
// (such as a limb of p).  The carry-out goes to a scratch SGPR pair that
// nothing reads; it is early-clobber ("=&s") because the block's first
// multiply-add writes it before the later ones read their factors, so it must
// not share a register with an SGPR factor.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace msm {

// the first n lines of a block: line i multiplies operands 2 + 2 i and 3 + 2 i
#define MSM_MADL_1(OP) OP " %0, %1, %2, %3, %0"
#define MSM_MADL_2(OP) MSM_MADL_1(OP) "\n\t" OP " %0, %1, %4, %5, %0"
#define MSM_MADL_3(OP) MSM_MADL_2(OP) "\n\t" OP " %0, %1, %6, %7, %0"
#define MSM_MADL_4(OP) MSM_MADL_3(OP) "\n\t" OP " %0, %1, %8, %9, %0"
#define MSM_MADL_5(OP) MSM_MADL_4(OP) "\n\t" OP " %0, %1, %10, %11, %0"
#define MSM_MADL_6(OP) MSM_MADL_5(OP) "\n\t" OP " %0, %1, %12, %13, %0"
#define MSM_MADL_7(OP) MSM_MADL_6(OP) "\n\t" OP " %0, %1, %14, %15, %0"
#define MSM_MADL_8(OP) MSM_MADL_7(OP) "\n\t" OP " %0, %1, %16, %17, %0"
#define MSM_MADL_9(OP) MSM_MADL_8(OP) "\n\t" OP " %0, %1, %18, %19, %0"
#define MSM_MADL_10(OP) MSM_MADL_9(OP) "\n\t" OP " %0, %1, %20, %21, %0"
#define MSM_MADL_11(OP) MSM_MADL_10(OP) "\n\t" OP " %0, %1, %22, %23, %0"
#define MSM_MADL_12(OP) MSM_MADL_11(OP) "\n\t" OP " %0, %1, %24, %25, %0"
#define MSM_MADL_13(OP) MSM_MADL_12(OP) "\n\t" OP " %0, %1, %26, %27, %0"
#define MSM_MADL_14(OP) MSM_MADL_13(OP) "\n\t" OP " %0, %1, %28, %29, %0"
#define MSM_MADL_15(OP) MSM_MADL_14(OP) "\n\t" OP " %0, %1, %30, %31, %0"
#define MSM_MADL_16(OP) MSM_MADL_15(OP) "\n\t" OP " %0, %1, %32, %33, %0"
#define MSM_MADL_17(OP) MSM_MADL_16(OP) "\n\t" OP " %0, %1, %34, %35, %0"
#define MSM_MADL_18(OP) MSM_MADL_17(OP) "\n\t" OP " %0, %1, %36, %37, %0"
#define MSM_MADL_19(OP) MSM_MADL_18(OP) "\n\t" OP " %0, %1, %38, %39, %0"
#define MSM_MADL_20(OP) MSM_MADL_19(OP) "\n\t" OP " %0, %1, %40, %41, %0"
#define MSM_MADL_21(OP) MSM_MADL_20(OP) "\n\t" OP " %0, %1, %42, %43, %0"
#define MSM_MADL_22(OP) MSM_MADL_21(OP) "\n\t" OP " %0, %1, %44, %45, %0"
#define MSM_MADL_23(OP) MSM_MADL_22(OP) "\n\t" OP " %0, %1, %46, %47, %0"
#define MSM_MADL_24(OP) MSM_MADL_23(OP) "\n\t" OP " %0, %1, %48, %49, %0"
#define MSM_MADL_25(OP) MSM_MADL_24(OP) "\n\t" OP " %0, %1, %50, %51, %0"

// the first n operand pairs: two VGPRs (x, y), a VGPR and an SGPR (u, q)
#define MSM_MADV_1 "v"(x[0]), "v"(y[0])
#define MSM_MADV_2 MSM_MADV_1, "v"(x[1]), "v"(y[1])
#define MSM_MADV_3 MSM_MADV_2, "v"(x[2]), "v"(y[2])
#define MSM_MADV_4 MSM_MADV_3, "v"(x[3]), "v"(y[3])
#define MSM_MADV_5 MSM_MADV_4, "v"(x[4]), "v"(y[4])
#define MSM_MADV_6 MSM_MADV_5, "v"(x[5]), "v"(y[5])
#define MSM_MADV_7 MSM_MADV_6, "v"(x[6]), "v"(y[6])
#define MSM_MADV_8 MSM_MADV_7, "v"(x[7]), "v"(y[7])
#define MSM_MADV_9 MSM_MADV_8, "v"(x[8]), "v"(y[8])
#define MSM_MADV_10 MSM_MADV_9, "v"(x[9]), "v"(y[9])
#define MSM_MADV_11 MSM_MADV_10, "v"(x[10]), "v"(y[10])
#define MSM_MADV_12 MSM_MADV_11, "v"(x[11]), "v"(y[11])
#define MSM_MADV_13 MSM_MADV_12, "v"(x[12]), "v"(y[12])
#define MSM_MADV_14 MSM_MADV_13, "v"(x[13]), "v"(y[13])
#define MSM_MADS_1 "v"(u[0]), "s"(q[0])
#define MSM_MADS_2 MSM_MADS_1, "v"(u[1]), "s"(q[1])
#define MSM_MADS_3 MSM_MADS_2, "v"(u[2]), "s"(q[2])
#define MSM_MADS_4 MSM_MADS_3, "v"(u[3]), "s"(q[3])
#define MSM_MADS_5 MSM_MADS_4, "v"(u[4]), "s"(q[4])
#define MSM_MADS_6 MSM_MADS_5, "v"(u[5]), "s"(q[5])
#define MSM_MADS_7 MSM_MADS_6, "v"(u[6]), "s"(q[6])
#define MSM_MADS_8 MSM_MADS_7, "v"(u[7]), "s"(q[7])
#define MSM_MADS_9 MSM_MADS_8, "v"(u[8]), "s"(q[8])
#define MSM_MADS_10 MSM_MADS_9, "v"(u[9]), "s"(q[9])
#define MSM_MADS_11 MSM_MADS_10, "v"(u[10]), "s"(q[10])
#define MSM_MADS_12 MSM_MADS_11, "v"(u[11]), "s"(q[11])
#define MSM_MADS_13 MSM_MADS_12, "v"(u[12]), "s"(q[12])
#define MSM_MADS_14 MSM_MADS_13, "v"(u[13]), "s"(q[13])

#define MSM_MAD_ASM(OP, n, ...) \
  asm(MSM_MADL_##n(OP) : "+v"(acc), "=&s"(cc) : __VA_ARGS__)
#define MSM_MAD_V(na)                                              \
  if constexpr (NA == na && NM == 0) {                             \
    if constexpr (SIGNED) MSM_MAD_ASM("v_mad_i64_i32", na, MSM_MADV_##na); \
    else MSM_MAD_ASM("v_mad_u64_u32", na, MSM_MADV_##na);          \
  }
#define MSM_MAD_S(nm)                                              \
  if constexpr (NA == 0 && NM == nm) {                             \
    if constexpr (SIGNED) MSM_MAD_ASM("v_mad_i64_i32", nm, MSM_MADS_##nm); \
    else MSM_MAD_ASM("v_mad_u64_u32", nm, MSM_MADS_##nm);          \
  }
#define MSM_MAD_VS(na, nm, n)                                      \
  if constexpr (NA == na && NM == nm)                              \
    MSM_MAD_ASM("v_mad_i64_i32", n, MSM_MADV_##na, MSM_MADS_##nm);

// the numbers of products that there are blocks for (V: x y, S: u q, VS: both)
#define MSM_MAD_LIST(V, S, VS)                                                              \
  V(1) V(2) V(3) V(4) V(5) V(6) V(7) V(8) V(9) V(10) V(11) V(12) V(13) V(14)                \
  S(1) S(2) S(3) S(4) S(5) S(6) S(7) S(8) S(9) S(10) S(11) S(12) S(13) S(14)                \
  VS(1, 1, 2) VS(1, 2, 3) VS(2, 1, 3) VS(2, 2, 4) VS(2, 3, 5) VS(3, 2, 5) VS(3, 3, 6)       \
  VS(3, 4, 7) VS(4, 3, 7) VS(4, 4, 8) VS(4, 5, 9) VS(5, 4, 9) VS(5, 5, 10) VS(5, 6, 11)     \
  VS(6, 5, 11) VS(6, 6, 12) VS(6, 7, 13) VS(7, 6, 13) VS(7, 7, 14) VS(7, 8, 15)             \
  VS(8, 7, 15) VS(8, 8, 16) VS(8, 9, 17) VS(9, 8, 17) VS(9, 9, 18) VS(9, 10, 19)            \
  VS(10, 9, 19) VS(10, 10, 20) VS(10, 11, 21) VS(11, 10, 21) VS(11, 11, 22) VS(11, 12, 23)  \
  VS(12, 11, 23) VS(12, 12, 24) VS(13, 12, 25)
#define MSM_MAD_IS_V(na) +(NA == na && NM == 0)
#define MSM_MAD_IS_S(nm) +(NA == 0 && NM == nm)
#define MSM_MAD_IS_VS(na, nm, n) +(NA == na && NM == nm)

// acc += sum of NA products x[t] y[t] and NM products u[t] q[t] (q in SGPRs)
template <bool SIGNED, int NA, int NM, typename A, typename W>
__device__ __forceinline__ void mad64_block(A& acc, const W* x, const W* y, const W* u,
                                            const W* q) {
  static_assert(0 MSM_MAD_LIST(MSM_MAD_IS_V, MSM_MAD_IS_S, MSM_MAD_IS_VS) == 1,
                "no block for these numbers of products");
  static_assert(SIGNED || NA == 0 || NM == 0, "blocks of both kinds are signed");
  uint64_t cc;
  MSM_MAD_LIST(MSM_MAD_V, MSM_MAD_S, MSM_MAD_VS)
  (void)cc;
}

#undef MSM_MAD_IS_VS
#undef MSM_MAD_IS_S
#undef MSM_MAD_IS_V
#undef MSM_MAD_LIST
#undef MSM_MAD_VS
#undef MSM_MAD_S
#undef MSM_MAD_V
#undef MSM_MAD_ASM

}  // namespace msm

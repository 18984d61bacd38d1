// The latency unit of the dependent chains (window and group Horner): point
// arithmetic on three waves, field elements as 16 limbs of 26 bits, one limb
// per lane (device code).
//
// A lone wave issues one VALU instruction every ~4.6 cycles, dependent or
// not (multiply-adds, DPP moves and s_nop alike), and waits ~50-100 cycles for
// an LDS read, so a dependent product costs its instruction count plus its
// LDS round trips.  Here a product has one of each that it cannot do without:
//
//   columns   lane jj of a 32-lane half sums sum_i a_i b_{jj-i}: a broadcast
//             from LDS in four 16-byte reads, b read at a lane-shifted address
//             (16 zero words on either side of every array)
//   carries   the middle 26 bits of a column go one lane up, the rest two:
//             limbs below 2^27.1
//   fold      limbs 15..31 times 2^(26 k) mod p, a constant matrix, added to
//             limbs 0..14.  Lane j of a 16-lane row needs all 16 high limbs:
//             rotations of the row (DPP) against the matrix's diagonals, half
//             of them in each row of the half, then one cross-row sum; no
//             LDS, and no Montgomery digits (two more products of 16
//             multiply-adds and two more LDS round trips in wide.hpp)
//   carries   as above
//
// The result is a plain product mod p below 2^407, not a Montgomery one:
// coordinates are projective, every formula here is homogeneous, and a common
// power of R = 2^384 in all of a point's coordinates changes nothing.
//
// Every wave computes two products (one per half), chosen so that the sums
// the next phase needs are formed in registers from the wave's two results
// (v_permlane32_swap) before they are written to LDS: each phase is one LDS
// round trip and one barrier.  Addition: wave 0 A, B -> E, H; wave 1 C, D ->
// F, G.  Doubling: wave 0 X^2, Y^2 -> H; wave 1 (Y - X)(Y + X), Z^2 -> G, F;
// wave 2 T Z -> E = 2 T Z.  Second phase: wave 0 X, Y (and Y - X, Y + X), wave 1
// T, Z.
// Measured, group Horner of 112 doublings and 7 additions (n = 2^20, split
// digits): 125 -> 75 us against the Montgomery unit of wide_unit.hpp on two
// waves; 252 and 62 (n = 33, signed digits): 302 -> 178 us, 0.57 us an
// operation.
//
// Bounds: limbs of products below 2^27.01 (limb 15 below 2^18.2);
// differences add kOff26, a multiple of p whose limbs (2^28.9 .. 2^29, limb 15
// 2^21) exceed twice a product's; the largest operand, D - C + kOff26, has
// limbs below 2^29.6, so column sums stay below 2^62.3 and the product below
// 2^832 (nothing is carried out of column 31).
#pragma once
#include "curve.hpp"
#include "wide.hpp"

namespace msm {

constexpr uint32_t M26 = 0x3ffffffu;

// limbs of 2^(26 (15 + k)) mod p
__device__ const uint32_t kFold26[17][16] = {
    {0x3ffd9ebu, 0x20fffffu, 0x2c35c9cu, 0x1203fffu, 0x26c393au, 0x3234524u, 0x35dc785u, 0x09aa955u,
     0x0ec8afeu, 0x16bb283u, 0x25e6384u, 0x137dc5cu, 0x2c350fau, 0x02e3314u, 0x00000edu, 0x0000000u},
    {0x3dcbccfu, 0x0cfd9eau, 0x0de2ff1u, 0x04e9c53u, 0x2fd57bdu, 0x203bc13u, 0x237c3a6u, 0x1a2b356u,
     0x255a9bdu, 0x2318f21u, 0x129d194u, 0x1ed2244u, 0x26ef92fu, 0x2de34eau, 0x0000028u, 0x0000000u},
    {0x3f9f169u, 0x18cbcceu, 0x27342c0u, 0x17cefe4u, 0x3e83575u, 0x3a2d6d7u, 0x1459364u, 0x1dc802eu,
     0x381465bu, 0x37a1ec5u, 0x0692e7fu, 0x29bf8b2u, 0x3766dfau, 0x19e2cc4u, 0x0000b5eu, 0x0000000u},
    {0x24f0d7fu, 0x1c9f168u, 0x1c027e0u, 0x3827f3cu, 0x3befa6fu, 0x2af2534u, 0x3aa5da7u, 0x3c139f4u,
     0x1f056adu, 0x0475c11u, 0x2f660c1u, 0x0d4bb34u, 0x0a2ad4eu, 0x060b9dcu, 0x0000a29u, 0x0000000u},
    {0x27d10b1u, 0x17f0d7eu, 0x09115d9u, 0x254e4bcu, 0x2291a6bu, 0x2f0f744u, 0x2e94ebau, 0x2623660u,
     0x257a344u, 0x1e1ae09u, 0x003491eu, 0x01184cfu, 0x2883842u, 0x3e538a7u, 0x0000c27u, 0x0000000u},
    {0x231114cu, 0x0bd10b0u, 0x061aab4u, 0x24a1217u, 0x33f2323u, 0x241076bu, 0x23ea30eu, 0x03ec1d0u,
     0x2586596u, 0x250b80bu, 0x21f545du, 0x38f5bacu, 0x029a22cu, 0x0469b43u, 0x00005d7u, 0x0000000u},
    {0x321988au, 0x011114bu, 0x3876b3cu, 0x16928e5u, 0x3372d0au, 0x02a55d8u, 0x104690du, 0x07cb5b6u,
     0x052bfdeu, 0x393c692u, 0x2cfc4dbu, 0x0923b4bu, 0x3663391u, 0x0f8a79du, 0x00012a8u, 0x0000000u},
    {0x1397e55u, 0x1119889u, 0x076a4f2u, 0x0972577u, 0x09f751du, 0x2c869beu, 0x180cffeu, 0x0eb9687u,
     0x3fb5437u, 0x0b37bf1u, 0x09af39du, 0x2cf6e80u, 0x22fd330u, 0x08fed3eu, 0x000155bu, 0x0000000u},
    {0x0d2b773u, 0x0c97e54u, 0x2e9c0ccu, 0x03cde57u, 0x1821b7bu, 0x1b5fdb5u, 0x3036862u, 0x03af2b9u,
     0x3800486u, 0x2a4861bu, 0x0917c98u, 0x3b5dca2u, 0x2eced73u, 0x32783b7u, 0x0000e09u, 0x0000000u},
    {0x1e964c0u, 0x0d2b772u, 0x3ba9d6du, 0x279bc74u, 0x20c529du, 0x13b938fu, 0x01deed0u, 0x29698bfu,
     0x2af8612u, 0x06f205eu, 0x1956c57u, 0x213535au, 0x3d60757u, 0x12e0a64u, 0x00012eeu, 0x0000000u},
    {0x12f1298u, 0x26964bfu, 0x293051du, 0x32c9792u, 0x147ff70u, 0x320c948u, 0x126c804u, 0x224aea4u,
     0x2b44f8cu, 0x0382dc5u, 0x1e670cbu, 0x3996ae9u, 0x0546e00u, 0x1275c16u, 0x0000c8eu, 0x0000000u},
    {0x221d8f0u, 0x22f1297u, 0x2bf3262u, 0x047013bu, 0x2db5abbu, 0x29a1cc1u, 0x2946ed0u, 0x1e25ea3u,
     0x034c41cu, 0x2bb0831u, 0x2aeb7a9u, 0x27869e2u, 0x0a456cau, 0x356e7f0u, 0x00011cau, 0x0000000u},
    {0x15a6e07u, 0x171d8efu, 0x06f20f3u, 0x0b46ce2u, 0x2c7ccf5u, 0x398592eu, 0x1b1e757u, 0x2d2f05au,
     0x0dee6b2u, 0x3128592u, 0x3f09b09u, 0x08746cau, 0x1cfb16fu, 0x131f842u, 0x0001a9cu, 0x0000000u},
    {0x00a9ce9u, 0x30a6e06u, 0x37ff78eu, 0x1add8b8u, 0x12e8432u, 0x145a0bcu, 0x08179dbu, 0x36249a1u,
     0x2d8ae6fu, 0x00e675cu, 0x087a7ddu, 0x01d78feu, 0x2cff866u, 0x03d5f1eu, 0x0000f7cu, 0x0000000u},
    {0x1b25004u, 0x0ca9ce8u, 0x0011308u, 0x3c2f2c5u, 0x0a404dcu, 0x0ca86f3u, 0x120b89au, 0x34d6addu,
     0x2a7cfb8u, 0x0185538u, 0x1417d69u, 0x17f1cd2u, 0x0e30f47u, 0x0e63638u, 0x000155fu, 0x0000000u},
    {0x0d21be9u, 0x3625003u, 0x19584fbu, 0x07fcc6cu, 0x0605039u, 0x3d455f5u, 0x2a84fb8u, 0x30f4b26u,
     0x34ef1e7u, 0x184d1b5u, 0x091d1b4u, 0x329f86du, 0x058072du, 0x34f7770u, 0x00003c5u, 0x0000000u},
    {0x3705332u, 0x2321be8u, 0x0c74d22u, 0x11b03d1u, 0x138e6bfu, 0x267187fu, 0x0346ca2u, 0x1e8a69fu,
     0x3f9efdau, 0x1c2a3dbu, 0x294cdecu, 0x12f7205u, 0x114e50bu, 0x37b0868u, 0x0000f5bu, 0x0000000u},
};
// a multiple of p with large limbs, added before a limb-wise subtraction
__device__ const uint32_t kOff26[16] = {
    0x1ea24ac1u, 0x1e300129u, 0x1f7e252au, 0x1d2aa518u, 0x1e1a0d5fu, 0x1f607d63u,
    0x1f2b4317u, 0x1eb40f8du, 0x1c9fe237u, 0x1c3766c5u, 0x1ce83a5bu, 0x1f1447c9u,
    0x1fe103a3u, 0x1dba2683u, 0x1fffea46u, 0x00200000u};
// the curve constant k (plain residue)
__device__ const uint32_t kK26[16] = {
    0x0d6e016u, 0x30495a1u, 0x13e4e02u, 0x1e1c38fu, 0x1735d94u, 0x02cc84eu, 0x165b2feu, 0x0b485fcu,
    0x198c1a3u, 0x10dde1au, 0x2e65fc7u, 0x02dd9c2u, 0x1a4f2cau, 0x2ac0c5au, 0x000196bu, 0x0000000u};

// arrays of a unit: 16 zero words, 16 limbs, 16 zero words each
enum {
  W26_X, W26_Y, W26_T, W26_Z, W26_YM, W26_YP,  // accumulator, Y - X, Y + X
  W26_E, W26_F, W26_G, W26_H,                  // between the phases
  W26_O0,                                      // operand slots 0, 1: Y - X, Y + X, U, Z
  W26_K = W26_O0 + 8,                          // the constant k
  W26_ARRAYS
};
constexpr int W26_THREADS = 192;

struct w26_lds {
  uint32_t a[W26_ARRAYS][48];
  uint32_t sink[64];  // lanes with nothing to write
  __device__ __forceinline__ uint32_t* at(int k) { return a[k] + 16; }
};

// this lane's place, constants and LDS addresses
struct w26_lane {
  uint32_t wave;  // uniform
  uint32_t half, row, j;
  uint32_t m[9];  // fold: diagonals i = 0..7 of this row's rotations, limb 15
  uint32_t off;
  uint32_t low;   // 1 in row 0, limbs 0..14: adds the product's low limb
  // operands (the second one's address for column jj) and result of this
  // half in an addition, a doubling and the second phase
  const uint32_t *add_l, *add_r, *dbl_l, *dbl_r, *out_l, *out_r;
  uint32_t *add_d, *dbl_d, *out_d;
};

// LDS writes done, then all waves of the block meet (loads from memory are not
// waited for).  The wait is the builtin, which the compiler counts: the reads
// after it are then waited for one by one, under the multiply-adds.
__device__ __forceinline__ void w26_sync() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ w26_lane w26_lane_here(w26_lds& s) {
  w26_lane q;
  const uint32_t lane = wlane(), jj = lane & 31u;
  q.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  q.half = lane >> 5;
  q.row = (lane >> 4) & 1u;
  q.j = lane & 15u;
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) q.m[i] = kFold26[1 + ((q.j - i - 8 * q.row) & 15u)][q.j];
  q.m[8] = q.row ? 0u : kFold26[0][q.j];
  q.off = kOff26[q.j];
  q.low = q.row == 0 && q.j < 15 ? 1u : 0u;
  const bool h = q.half != 0, top = q.row != 0;
  uint32_t* sink = s.sink + lane;
  if (q.wave == 0) {
    q.add_l = s.at(h ? W26_YP : W26_YM);
    q.dbl_l = s.at(h ? W26_Y : W26_X);
    q.dbl_r = q.dbl_l + jj;
    q.out_l = s.at(h ? W26_G : W26_E);
    q.out_r = s.at(h ? W26_H : W26_F) + jj;
    q.add_d = top ? sink : s.at(h ? W26_H : W26_E) + q.j;
    q.dbl_d = top || h ? sink : s.at(W26_H) + q.j;
    q.out_d = s.at(top ? (h ? W26_YP : W26_YM) : (h ? W26_Y : W26_X)) + q.j;
  } else {
    q.add_l = s.at(h ? W26_Z : W26_T);
    q.dbl_l = s.at(q.wave == 2 ? W26_T : (h ? W26_Z : W26_YM));
    q.dbl_r = s.at(q.wave == 2 || h ? W26_Z : W26_YP) + jj;
    q.out_l = s.at(h ? W26_F : W26_E);
    q.out_r = s.at(h ? W26_G : W26_H) + jj;
    q.add_d = top ? sink : s.at(h ? W26_G : W26_F) + q.j;
    q.dbl_d = q.wave == 2 ? (top || h ? sink : s.at(W26_E) + q.j)
                          : (top ? sink : s.at(h ? W26_F : W26_G) + q.j);
    q.out_d = top ? sink : s.at(h ? W26_Z : W26_T) + q.j;
  }
  q.add_r = s.at(W26_O0 + (q.wave < 2 ? 2 * (int)q.wave + (int)q.half : 0)) + jj;
  return q;
}

// zero the arrays, write k; needs a w26_sync before use
__device__ __forceinline__ void w26_init(w26_lds& s) {
  for (uint32_t i = threadIdx.x; i < W26_ARRAYS * 48; i += W26_THREADS) {
    const uint32_t l = i - W26_K * 48 - 16;
    (&s.a[0][0])[i] = l < 16 ? kK26[l] : 0u;
  }
}

#define W26_DPP " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
#define W26_ROT(n) "v_mov_b32_dpp %" #n ", %10 row_ror:" #n W26_DPP

// From a half's column sums (col: lo, hi) to the fold's sums of this row:
// the middle 26 bits of a column move up one lane, those above two (columns
// run across the half's rows; nothing leaves column 31); then tl, th = limbs j
// and 16 + j in both rows, row 1's th turned by 8 lanes so that the same
// rotations 0 .. 7 give it 8 .. 15; then the nine multiply-adds.  One block,
// because the compiler places a wait state before every DPP move that reuses
// a register and after every block.
__device__ __forceinline__ uint64_t w26_fold(const w26_lane& q, uint64_t col) {
  uint64_t acc, cc;
  uint32_t r1, r2, r3, r4, r5, r6, r7, r8, th, tl = (uint32_t)col;
  const uint32_t hi = (uint32_t)(col >> 32);
  asm("v_lshrrev_b32 %1, 20, %13\n\t"
      "v_alignbit_b32 %2, %13, %9, 26\n\t"
      "v_and_b32 %2, 0x3ffffff, %2\n\t"
      "v_and_b32 %9, 0x3ffffff, %9\n\t"
      "v_add_u32_dpp %2, %1, %2 wave_shr:1" W26_DPP
      "s_nop 1\n\t"
      "v_add_u32_dpp %9, %2, %9 wave_shr:1" W26_DPP
      "v_mov_b32 %10, %9\n\t"
      "s_nop 1\n\t"
      "v_permlane16_swap_b32 %9, %10\n\t"
      "s_nop 1\n\t"
      "v_mov_b32_dpp %10, %10 row_ror:8 row_mask:0xa bank_mask:0xf\n\t"
      "v_mov_b32_dpp %8, %9 row_newbcast:15" W26_DPP
      "v_mad_u64_u32 %0, %11, %9, %12, 0\n\t"
      W26_ROT(1) W26_ROT(2) W26_ROT(3) W26_ROT(4) W26_ROT(5) W26_ROT(6) W26_ROT(7)
      "v_mad_u64_u32 %0, %11, %14, %10, %0\n\t"
      "v_mad_u64_u32 %0, %11, %15, %1, %0\n\t"
      "v_mad_u64_u32 %0, %11, %16, %2, %0\n\t"
      "v_mad_u64_u32 %0, %11, %17, %3, %0\n\t"
      "v_mad_u64_u32 %0, %11, %18, %4, %0\n\t"
      "v_mad_u64_u32 %0, %11, %19, %5, %0\n\t"
      "v_mad_u64_u32 %0, %11, %20, %6, %0\n\t"
      "v_mad_u64_u32 %0, %11, %21, %7, %0\n\t"
      "v_mad_u64_u32 %0, %11, %22, %8, %0"
      : "=&v"(acc), "=&v"(r1), "=&v"(r2), "=&v"(r3), "=&v"(r4), "=&v"(r5), "=&v"(r6), "=&v"(r7),
        "=&v"(r8), "+v"(tl), "=&v"(th), "=&s"(cc)
      : "v"(q.low), "v"(hi), "v"(q.m[0]), "v"(q.m[1]), "v"(q.m[2]), "v"(q.m[3]), "v"(q.m[4]),
        "v"(q.m[5]), "v"(q.m[6]), "v"(q.m[7]), "v"(q.m[8]));
  return acc;
}

// The two rows' sums added, and the carries as above within the row: the
// product's limb j in both rows.
__device__ __forceinline__ uint32_t w26_limbs(uint64_t acc) {
  uint32_t lo = (uint32_t)acc, hi = (uint32_t)(acc >> 32), c0, c1;
  asm("v_mov_b32 %2, %0\n\t"
      "v_mov_b32 %3, %1\n\t"
      "s_nop 1\n\t"
      "v_permlane16_swap_b32 %0, %2\n\t"
      "v_permlane16_swap_b32 %1, %3\n\t"
      "v_add_co_u32 %0, vcc, %0, %2\n\t"
      "v_addc_co_u32 %1, vcc, %1, %3, vcc\n\t"
      "v_alignbit_b32 %2, %1, %0, 26\n\t"
      "v_and_b32 %2, 0x3ffffff, %2\n\t"
      "v_lshrrev_b32 %3, 20, %1\n\t"
      "v_and_b32 %0, 0x3ffffff, %0\n\t"
      "v_add_u32_dpp %0, %2, %0 row_shr:1" W26_DPP
      "v_add_u32_dpp %0, %3, %0 row_shr:2" W26_DPP
      : "+v"(lo), "+v"(hi), "=&v"(c0), "=&v"(c1)
      :
      : "vcc");
  return lo;
}
#undef W26_ROT
#undef W26_DPP

// Limb j of a product mod p in both rows of the half (l: the first operand's
// limbs, r: the address of the second's limb jj).
__device__ __forceinline__ uint32_t w26_mul(const w26_lane& q, const uint32_t* l,
                                            const uint32_t* r) {
  const uint4* l4 = reinterpret_cast<const uint4*>(l);
  uint32_t a[16], b[16];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint4 v = l4[i];
    a[4 * i] = v.x;
    a[4 * i + 1] = v.y;
    a[4 * i + 2] = v.z;
    a[4 * i + 3] = v.w;
#pragma unroll
    for (int t = 4 * i; t < 4 * i + 4; ++t) b[t] = r[-t];
  }
  uint64_t col = (uint64_t)a[0] * b[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) col += (uint64_t)a[i] * b[i];
  return w26_limbs(w26_fold(q, col));
}

// this wave's two products in every lane: half 0's and half 1's limb j
struct w26_pair {
  uint32_t a, b;
};
__device__ __forceinline__ w26_pair w26_both(uint32_t v) {
  const auto sw = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return {sw[0], sw[1]};
}

// second phase of both operations, on waves 0 and 1
__device__ __forceinline__ void w26_out(const w26_lane& q) {
  if (q.wave < 2) {
    const uint32_t v = w26_mul(q, q.out_l, q.out_r);  // X, Y | T, Z
    const w26_pair p = w26_both(v);
    const uint32_t u = q.half ? p.a + p.b : (p.b + q.off) - p.a;  // Y + X, Y - X
    *q.out_d = q.row ? u : v;
  }
  w26_sync();
}

// acc + the operand of slot o (0, 1): Y2 - X2, Y2 + X2, U2 = k T2, Z2.  idle()
// runs on wave 2 meanwhile.
template <typename F>
__device__ __forceinline__ void w26_add(const w26_lane& q, int o, F idle) {
  if (q.wave < 2) {
    const uint32_t v = w26_mul(q, q.add_l, q.add_r + (o ? 4 * 48 : 0));
    const w26_pair p = w26_both(v);    // A, B | C, Z1 Z2
    const uint32_t d = p.b << q.wave;  // B | D = 2 Z1 Z2
    *q.add_d = q.half ? d + p.a : (d + q.off) - p.a;
  } else {
    idle();
  }
  w26_sync();
  w26_out(q);
}

// 2 acc (a = -1): A = X^2, B = Y^2, E = 2XY = 2TZ, G = B - A = (Y - X)(Y + X),
// F = G - 2 Z^2, H = -(A + B)
__device__ __forceinline__ void w26_dbl(const w26_lane& q) {
  uint32_t v = w26_mul(q, q.dbl_l, q.dbl_r);
  if (q.wave == 2) {
    v <<= 1;
  } else {
    const w26_pair p = w26_both(v);  // X^2, Y^2 | G, Z^2
    if (q.wave == 0)
      v = q.off - (p.a + p.b);
    else
      v = q.half ? (p.a + q.off) - (p.b << 1) : v;
  }
  *q.dbl_d = v;
  w26_sync();
  w26_out(q);
}

// The words of the limbs this lane of wave 2 loads of a record of four
// coordinates (12 words each): rows 0, 1 Y and X, row 2 T or U, row 3 Z.
struct w26_fetch {
  limb_src own, x;
};
__device__ __forceinline__ limb_src w26_words(const uint32_t* __restrict__ w, uint32_t j) {
  const uint32_t wi = (26u * j) >> 5;  // 12 for limb 15, which is zero
  limb_src r;
  r.lo = w[wi < (uint32_t)NL ? wi : (uint32_t)NL - 1];
  r.hi = w[wi + 1 < (uint32_t)NL ? wi + 1 : (uint32_t)NL - 1];
  return r;
}
__device__ __forceinline__ uint32_t w26_limb(const limb_src& s, uint32_t j) {
  const uint64_t v = ((uint64_t)(j < 14 ? s.hi : 0u) << 32) | s.lo;
  return j < 15 ? (uint32_t)(v >> ((26u * j) & 31u)) & M26 : 0u;
}
__device__ __forceinline__ w26_fetch w26_load(const uint32_t* __restrict__ rec) {
  const uint32_t lane = wlane(), row = lane >> 4, j = lane & 15u;
  w26_fetch f;
  f.own = w26_words(rec + (row < 1 ? 1 : row) * NL, j);
  f.x = w26_words(rec, j);
  return f;
}
// wave 2: the loaded record as the addition's operand of slot o
__device__ __forceinline__ void w26_put_operand(w26_lds& s, const w26_lane& q, const w26_fetch& f,
                                                int o) {
  const uint32_t row = wlane() >> 4;
  const uint32_t v = w26_limb(f.own, q.j), x = w26_limb(f.x, q.j);
  s.at(W26_O0 + 4 * o + (int)row)[q.j] = row == 0 ? (v + q.off) - x : (row == 1 ? v + x : v);
}
// wave 2: the loaded record (XYTZ) as the accumulator
__device__ __forceinline__ void w26_put_acc(w26_lds& s, const w26_lane& q, const w26_fetch& f) {
  const uint32_t row = wlane() >> 4;
  const uint32_t v = w26_limb(f.own, q.j), x = w26_limb(f.x, q.j);
  s.at(row == 0 ? W26_X : (int)row)[q.j] = row == 0 ? x : v;
  if (row < 2) s.at(row == 0 ? W26_YM : W26_YP)[q.j] = row == 0 ? (v + q.off) - x : v + x;
}
// wave 2: the identity (0, 1, 0, 1) as the accumulator
__device__ __forceinline__ void w26_put_identity(w26_lds& s) {
  const uint32_t row = wlane() >> 4;
  if ((wlane() & 15u) == 0) {
    if (row & 1u) s.at((int)row)[0] = 1u;          // Y, Z
    else s.at(row ? W26_YP : W26_YM)[0] = 1u;
  }
}

// The value of 16 limbs (below 2^408) as 12 words in [0, 2p): an exact carry
// chain, then the quotient by p from the top 56 bits (short of the true one
// by at most 1) times p subtracted.  One lane.
__device__ __forceinline__ fe w26_to_words(const uint32_t* limbs) {
  uint32_t n[17];
  uint64_t c = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    c += limbs[i];
    n[i] = i < 15 ? (uint32_t)c & M26 : (uint32_t)c;
    c >>= 26;
  }
  n[16] = 0;
  uint32_t w[13];
#pragma unroll
  for (int i = 0; i < 13; ++i) {
    const int b = 32 * i, l = b / 26, sh = b % 26;
    uint64_t v = (uint64_t)n[l] >> sh;
    if (l + 1 < 16) v |= (uint64_t)n[l + 1] << (26 - sh);
    if (l + 2 < 16 && 52 - sh < 32) v |= (uint64_t)n[l + 2] << (52 - sh);
    w[i] = (uint32_t)v;
  }
  // p / 2^352 = 28195398.093...; 2^-18 covers the rounding and the bits below 2^352
  const double top = (double)w[12] * 4294967296.0 + (double)w[11];
  const double est = top * (1.0 / 28195398.09285074) - 0x1p-18;
  const uint32_t qt = est > 0.0 ? (uint32_t)est : 0u;
  fe r;
  int64_t acc = 0;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    acc += (int64_t)w[i] - (int64_t)((uint64_t)qt * kP[i]);
    r.v[i] = (uint32_t)acc;
    acc >>= 32;
  }
  return r;
}

// lanes 0 .. 3 of the calling wave: the accumulator as an XYTZ record, U =
// k T in the place of T when `u` names its array
__device__ __forceinline__ void w26_store(w26_lds& s, uint32_t* __restrict__ rec, int t_array) {
  const uint32_t lane = wlane();
  if (lane < 4) st_aos(rec, (int)lane, w26_to_words(s.at(lane == 2 ? t_array : (int)lane)));
}

}  // namespace msm

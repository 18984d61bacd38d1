// Bucket aggregation and group aggregation (Sec. II-C).
//
// Bucket aggregation computes the window sum S_w = sum_b b B[w][b] (unsigned
// digits) or sum_m (m + 1) B[w][m] (signed digits: bucket m holds digit
// magnitude m + 1).  Writing the bucket index b in binary,
// sum_b b B[w][b] = sum_t 2^t X_t with X_t = sum of the buckets whose index
// has bit t set; signed digits add the sum of all buckets.
// The X_t are built by a binary tree over the bucket index: a node covering
// 2^h consecutive buckets keeps V[t] (t < h, the sum over its buckets with bit
// t set) and S (the sum of all its buckets).  Merging left child L and right
// child R gives V[t] = L.V[t] + R.V[t] (t < h), V[h] = R.S, S = L.S + R.S.
// Every output of a level is one independent addition, the whole tree costs
// about 2 * 2^c additions per window (as many as the running-sum method) and
// its dependent depth is only c additions.  Large levels run on lanes, two to
// a kernel; smaller ones use four-lane quads (quad29.hpp) to cut latency; the
// last ones of a window, and its Horner pass, share one block.
//
// Each window then forms S_w by Horner's rule on one latency unit, and group
// aggregation Q = sum_w 2^(w c) S_w is Horner's rule over the windows of a job
// (c doublings per window), the dependent chain the paper assigns to its
// low-latency unit: one three-wave unit per job (wide26.hpp).  The
// result is mapped back to Weierstrass affine form.  A "window" below is a
// segment: one window of one job of the batch.
#include "common.hpp"
#include "convert.hpp"
#include "curve29.hpp"
#include "quad29.hpp"
#include "wide26.hpp"
#include "wide_unit.hpp"
#include "window_tail.hpp"

namespace msm {
namespace {

// record of node n, slot s at a tree level with `slots` slots per node
__device__ __forceinline__ size_t rec_index(uint32_t w, uint32_t nodes, uint32_t n, uint32_t slots,
                                            uint32_t s) {
  return ((size_t)w * nodes + n) * slots + s;
}

// All records of the tree are signed (fe29.hpp) but the root's, which the
// latency unit reads: U = k T in the place of T and coordinates in [0, 2p).

// Levels 0 and 1 on two lanes per node of four buckets B0 .. B3: the even lane
// adds B0 + B1, the odd one B2 + B3 = V[1]; then the even lane adds both sums, S,
// and the odd one B1 + B3 = V[0].  One pass over the buckets where two levels
// write and read every record again: n = 2^20 (262 K buckets) 74 -> 50 us,
// n = 300007, signed digits (278 K) 84 -> 65.  Bound by VALU issue at two waves
// per SIMD; 1.8 M buckets (n = 2^22) take 291 us, 221 of it issue.
__global__ void __launch_bounds__(256) k_tree_first(const uint32_t* __restrict__ in,
                                                    uint64_t lanes,
                                                    uint32_t* __restrict__ out) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= lanes) return;  // whole pairs
  const bool odd = (g & 1u) != 0;
  const uint32_t* B = in + (g >> 1) * 4 * XYTZ_WORDS;
  uint32_t* O = out + (g >> 1) * 3 * XYTZ_WORDS;  // V[0], V[1], S
  const uint32_t* mine = B + (odd ? 2 : 0) * XYTZ_WORDS;
  const xytz29 s = padd29_full(pt29_from(ld_xytz(mine)), pt29_from(ld_xytz(mine + XYTZ_WORDS)));
  if (odd) st_xytz(O + XYTZ_WORDS, pt29_to_words(s));
  // the even lane's second operand is the odd lane's sum; the odd lane adds
  // B1 and B3, read again (its registers hold the sum)
  xytz29 l, r;
  const xytz b1 = ld_xytz(B + XYTZ_WORDS), b3 = ld_xytz(B + 3 * XYTZ_WORDS);
  auto other = [](const fe29& v) {
    fe29 o;
#pragma unroll
    for (int i = 0; i < NL29; ++i) o.v[i] = qperm<1, 0, 3, 2>(v.v[i]);
    return o;
  };
  auto pick = [&](const fe29& sum, const fe& x, const fe& y, fe29& lo, fe29& ro) {
    const fe29 so = other(sum);
    lo = f29_select(odd, f29_from_words(x), sum);
    ro = f29_select(odd, f29_from_words(y), so);
  };
  pick(s.X, b1.X, b3.X, l.X, r.X);
  pick(s.Y, b1.Y, b3.Y, l.Y, r.Y);
  pick(s.T, b1.T, b3.T, l.T, r.T);
  pick(s.Z, b1.Z, b3.Z, l.Z, r.Z);
  st_xytz(O + (odd ? 0 : 2) * XYTZ_WORDS, pt29_to_words(padd29_full(l, r)));
}

// One level h -> h+1, one addition per lane: addition a < h forms slot a,
// addition h the total (slot h + 1); the lane of addition 0 also copies
// slot h (= R.S), so that no lane of a wave idles through another's addition.
__global__ void __launch_bounds__(256) k_tree_level(const uint32_t* __restrict__ in, uint32_t h,
                                                    uint32_t nodes_in, uint32_t S,
                                                    uint32_t* __restrict__ out) {
  const uint32_t nodes_out = nodes_in >> 1, slots_in = h + 1, slots_out = h + 2;
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (uint64_t)S * nodes_out * slots_in) return;
  const uint32_t a = (uint32_t)(g % slots_in);
  const uint32_t t = (uint32_t)(g / slots_in);
  const uint32_t n = t % nodes_out, w = t / nodes_out;
  const uint32_t* L = in + rec_index(w, nodes_in, 2 * n, slots_in, 0) * XYTZ_WORDS;
  const uint32_t* R = L + (size_t)slots_in * XYTZ_WORDS;
  uint32_t* O = out + rec_index(w, nodes_out, n, slots_out, 0) * XYTZ_WORDS;
  if (a == 0)
    st_xytz(O + (size_t)h * XYTZ_WORDS, ld_xytz(R + (size_t)h * XYTZ_WORDS));
  const uint32_t s = a < h ? a : h + 1;  // output slot
  const xytz29 r = padd29_full(pt29_from(ld_xytz(L + (size_t)a * XYTZ_WORDS)),
                               pt29_from(ld_xytz(R + (size_t)a * XYTZ_WORDS)));
  st_xytz(O + (size_t)s * XYTZ_WORDS, pt29_to_words(r));
}

// Levels h and h + 1 on lanes, one per output record as k_tree_quad2's quads
// below (nodes: of level h + 1, over all windows): first the sums of four
// records, then those of two, so that a wave's lanes do one kind.  The next
// record loads during an addition, where a level of its own waits for its two
// and writes and reads every record between: two levels at n = 300007, signed
// digits (15 bits) 49 -> 36 us, at n = 2^20 48 -> 42, four at n = 2^22 (c = 19)
// 295 -> 279.
__global__ void __launch_bounds__(256) k_tree_level2(const uint32_t* __restrict__ in, uint32_t h,
                                                     uint64_t nodes, uint32_t* __restrict__ out) {
  const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t fours = nodes * (h + 1);
  if (g >= fours + 2 * nodes) return;
  const bool four = g < fours;
  const uint64_t node = four ? g / (h + 1) : (g - fours) >> 1;
  const uint32_t a = four ? (uint32_t)(g % (h + 1)) : h;  // slot of the grandchildren
  const uint32_t odd = (uint32_t)(g - fours) & 1u;
  const uint32_t s = !four ? h + odd : (a < h ? a : h + 2);
  const uint32_t* R = in + (node * 4 * (h + 1) + a) * XYTZ_WORDS;
  const size_t stride = (size_t)(h + 1) * XYTZ_WORDS;
  uint32_t left = four ? 0xfu : (odd ? 0xcu : 0xau);
  auto next = [&] {
    const uint32_t i = (uint32_t)__builtin_ctz(left);
    left &= left - 1;
    return ld_xytz(R + i * stride);
  };
  xytz29 acc = pt29_from(next());
  xytz w = next();
#pragma unroll 1
  for (;;) {
    const xytz29 v = pt29_from(w);
    const bool more = left != 0;
    if (more) w = next();
    acc = padd29_full(acc, v);
    if (!more) break;
  }
  st_xytz(out + (node * (h + 3) + s) * XYTZ_WORDS, pt29_to_words(acc));
}

// Levels h and h + 1 on quads, one per output record: slot t < h of a node is
// the sum of its four grandchildren's slot t, slots h and h + 1 of S1 + S3 and
// S2 + S3, the total of all four S (one addition more than the two levels
// take).  Three additions in a row in one launch where two launches of one
// addition each cost 6-8 us apiece once a level no longer fills the chip
// (n = 65536, seven levels 58 -> 53 us; n = 300007 six levels 56 -> 46).
__global__ void __launch_bounds__(256) k_tree_quad2(const uint32_t* __restrict__ in, uint32_t h,
                                                    uint64_t outs, uint32_t* __restrict__ out) {
  const uint64_t g = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
  if (g >= outs) return;  // whole quads
  const uint32_t s = (uint32_t)(g % (h + 3));
  const uint64_t node = g / (h + 3);  // over all windows
  const uint32_t* R = in + (node * 4 * (h + 1) + (s < h ? s : h)) * XYTZ_WORDS;
  const size_t stride = (size_t)(h + 1) * XYTZ_WORDS;
  // which of the four are summed
  uint32_t left = s == h ? 0xau : (s == h + 1 ? 0xcu : 0xfu);
  auto next = [&] {
    const uint32_t i = (uint32_t)__builtin_ctz(left);
    left &= left - 1;
    return ld_aos(R + i * stride, (int)quad_lane());
  };
  fe29 acc = f29_from_words(next());
  fe w = next();
  for (;;) {
    const fe29 v = f29_from_words(w);
    const bool more = left != 0;
    if (more) w = next();
    acc = quad_add(acc, v);
    if (!more) break;
  }
  quad_st(out + g * XYTZ_WORDS, acc);
}

// One level on quads, one per output record.
__global__ void __launch_bounds__(256) k_tree_level_quad(const uint32_t* __restrict__ in, uint32_t h,
                                                         uint32_t nodes_in, uint32_t S,
                                                         uint32_t* __restrict__ out) {
  const uint32_t nodes_out = nodes_in >> 1, slots_in = h + 1, slots_out = h + 2;
  const uint64_t g = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
  // whole quads only: the task count test is uniform across a quad
  if (g >= (uint64_t)S * nodes_out * slots_out) return;
  const uint32_t s = (uint32_t)(g % slots_out);
  const uint32_t t = (uint32_t)(g / slots_out);
  const uint32_t n = t % nodes_out, w = t / nodes_out;
  const uint32_t* L = in + rec_index(w, nodes_in, 2 * n, slots_in, 0) * XYTZ_WORDS;
  const uint32_t* R = L + (size_t)slots_in * XYTZ_WORDS;
  const uint32_t src = (s < h) ? s : h;
  fe29 r = quad_ld(R + (size_t)src * XYTZ_WORDS);
  if (s != h) r = quad_add(quad_ld(L + (size_t)src * XYTZ_WORDS), r);
  quad_st(out + rec_index(w, nodes_out, n, slots_out, s) * XYTZ_WORDS, r);
}

// The last levels and the Horner pass of window w = the block (window_tail).
__global__ void __launch_bounds__(TAIL_THREADS) k_window_tail(const uint32_t* __restrict__ in,
                                                              uint32_t h0, uint32_t bb,
                                                              uint32_t second_at, int add_total,
                                                              uint32_t* __restrict__ wsum) {
  extern __shared__ int32_t lv[];  // records [4][NL29], two buffers
  __shared__ __attribute__((aligned(16))) tail_lds sh;
  const uint32_t w = blockIdx.x;
  window_tail(in + ((size_t)w << (bb - h0)) * (h0 + 1) * XYTZ_WORDS, h0, bb, second_at, add_total,
              wsum + (size_t)2 * w * XYTZ_WORDS, lv, sh);
}

// Twisted-Edwards extended (Montgomery form) -> Weierstrass affine, ordinary
// form, canonical, on one wave: the field inversion is lane-parallel
// (fe_inv_lanes) and the ten products around it run as wide products, two at
// a time (one per half-wave), in five dependent steps:
//   d = (Z - Y) X, un = (Z + Y) X;   [d^-1]   im = d^-1 R^3 (Montgomery
//   inverse), vn = (Z + Y) Z;   u = un im, v = vn im;   u alpha, v beta;
//   x = (u alpha - 1) / R, y = v beta / R (out of Montgomery form).
// The steps are one loop over operands in LDS, and the reductions one
// function: code that a lone wave runs once costs its instruction fetches
// too (written out step by step the conversion was three times as long, and
// the kernel 10 us slower).
enum { AF_D, AF_UN, AF_VN, AF_X, AF_Z, AF_ZMY, AF_ZPY, AF_R3, AF_ALPHA, AF_BETA, AF_UNIT, AF_SLOTS };

struct affine_lds {
  uint32_t mul[WMUL2_WORDS];
  uint32_t slot[AF_SLOTS][16];
  uint32_t q[XYTZ_WORDS];  // the point
};
// kR3, kAlpha, kBeta, to be read limb by limb
struct affine_consts {
  uint32_t w[3][NL];
};
constexpr affine_consts affine_consts_table() {
  affine_consts t = {};
  for (int l = 0; l < NL; ++l) {
    t.w[0][l] = kR3[l];
    t.w[1][l] = kAlpha[l];
    t.w[2][l] = kBeta[l];
  }
  return t;
}
__device__ const affine_consts kAffineConsts = affine_consts_table();

// canonical words of 16 lazily reduced limbs
__device__ __noinline__ fe canon_of_limbs(const uint32_t* limbs) {
  return fe_canon(words_of_limbs(limbs));
}

// Lane 32 h gets x (h = 0) or y (h = 1) of the point s.q; false for the
// identity (zero for both).
__device__ __forceinline__ bool wide_to_weierstrass(affine_lds& s, fe& out) {
  const uint32_t lane = wlane(), h = lane >> 5, j = lane & 15u;
  const bool act = (lane & 31u) < 16u;
  const uint32_t c2p = 2u * kP24[j] + (j < 15 ? (1u << 26) : 0u) - (j >= 1 ? 4u : 0u);
  wmul2_init(s.mul);
  if (lane < 16) {
    const uint32_t X = limb_extract(limb_fetch(s.q, j), j),
                   Y = limb_extract(limb_fetch(s.q + NL, j), j),
                   Z = limb_extract(limb_fetch(s.q + 3 * NL, j), j);
    s.slot[AF_X][j] = X;
    s.slot[AF_Z][j] = Z;
    s.slot[AF_ZMY][j] = (Z + c2p) - Y;
    s.slot[AF_ZPY][j] = Z + Y;
    s.slot[AF_UNIT][j] = j == 0 ? 1u : 0u;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      s.slot[AF_R3 + k][j] = limb_extract(limb_fetch(kAffineConsts.w[k], j), j);
  }
  wave_lds_sync();
  // operands and results of the steps by half, a byte each: l, r, result
  constexpr uint32_t kStep[5][2] = {
      {AF_ZMY | AF_X << 8 | AF_D << 16, AF_ZPY | AF_X << 8 | AF_UN << 16},
      {AF_D | AF_R3 << 8 | AF_D << 16, AF_ZPY | AF_Z << 8 | AF_VN << 16},
      {AF_UN | AF_D << 8 | AF_D << 16, AF_VN | AF_D << 8 | AF_VN << 16},
      {AF_D | AF_ALPHA << 8 | AF_D << 16, AF_VN | AF_BETA << 8 | AF_VN << 16},
      {AF_D | AF_UNIT << 8 | AF_D << 16, AF_VN | AF_UNIT << 8 | AF_VN << 16}};
  bool finite = true;
#pragma unroll 1
  for (int i = 0; i < 5; ++i) {
    uint32_t op = h ? kStep[0][1] : kStep[0][0];
#pragma unroll
    for (int k = 1; k < 5; ++k) op = i == k ? (h ? kStep[k][1] : kStep[k][0]) : op;
    const uint32_t l = s.slot[op & 0xffu][j], r = s.slot[(op >> 8) & 0xffu][j];
    uint32_t v = wmul2_hi(act ? l : 0u, act ? r : 0u, s.mul);
    // u alpha - 1 (Montgomery)
    if (i == 3 && h == 0) v += c2p - limb_of_const(kOne, j);
    if (!act) s.slot[op >> 16][j] = v;
    wave_lds_sync();
    if (i == 0) {
      const fe d = canon_of_limbs(s.slot[AF_D]);  // 0 for the identity alone (y = 1 or x = 0)
      finite = !fe_is_zero_canon(d);
      const fe inv = fe_inv_lanes(d);
      wave_lds_sync();
      if (lane < NL) {
        uint32_t w = inv.v[0];
#pragma unroll
        for (uint32_t k = 1; k < (uint32_t)NL; ++k) w = lane == k ? inv.v[k] : w;
        s.q[lane] = w;
      }
      wave_lds_sync();
      if (lane < 16) s.slot[AF_D][j] = limb_extract(limb_fetch(s.q, j), j);
      wave_lds_sync();
    }
  }
  out = canon_of_limbs(s.slot[h ? AF_VN : AF_D]);
  if (!finite) out = fe_zero();
  return finite;
}

// Group aggregation and the affine result of job j (block j): Q = sum_w 2^(w c)
// S_w by Horner's rule over the job's W windows on one latency unit, wave 2
// loading the next window's sum during the doublings; then wave 0 maps Q
// back and writes the result.  One kernel: the conversion alone took 33 us, a
// launch and a round trip of Q through memory among them (n = 33: group
// aggregation and conversion 212 -> 202 us).
__global__ void __launch_bounds__(W26_THREADS) k_group(const uint32_t* __restrict__ wsum,
                                                       uint32_t W, uint32_t c, JobView jv,
                                                       const uint32_t* __restrict__ flags) {
  __shared__ __attribute__((aligned(16))) w26_lds s;
  __shared__ __attribute__((aligned(16))) affine_lds a;
  const uint32_t job = blockIdx.x;
  const w26_lane q = w26_lane_here(s);
  const uint32_t* ws = wsum + (size_t)2 * job * W * XYTZ_WORDS;
  // S_w, XYUZ (w clamped: W = 1 has none to add)
  auto sum = [&](int w) { return ws + (size_t)(2 * (w < 0 ? 0 : w) + 1) * XYTZ_WORDS; };
  w26_fetch top, f;
  if (q.wave == 2) {
    top = w26_load(ws + (size_t)(2 * (W - 1)) * XYTZ_WORDS);  // S_{W-1}, XYTZ
    f = w26_load(sum((int)W - 2));
  }
  w26_init(s);
  w26_sync();
  if (q.wave == 2) {
    w26_put_acc(s, q, top);
    w26_put_operand(s, q, f, 0);
    f = w26_load(sum((int)W - 3));
  }
  w26_sync();
  int o = 0;
  for (int w = (int)W - 2; w >= 0; --w) {
    for (uint32_t t = 0; t < c; ++t) w26_dbl(q);
    w26_add(q, o, [&] {
      w26_put_operand(s, q, f, o ^ 1);
      f = w26_load(sum(w - 2));
    });
    o ^= 1;
  }
  if (q.wave != 0) return;
  w26_store(s, a.q, W26_T);
  wave_lds_sync();
  fe out;
  const bool finite = wide_to_weierstrass(a, out);
  uint32_t* result = jv.get(job).result;
  const uint32_t lane = wlane();
  if ((lane & 31u) == 0)
#pragma unroll
    for (int l = 0; l < NL; ++l) result[(lane >> 5) * NL + l] = out.v[l];
  if (lane < MSM_RESULT_WORDS - 2 * NL)
    result[2 * NL + lane] = lane == 0 ? (finite ? 0u : 1u) : (lane == 1 ? flags[job] : 0u);
}

}  // namespace

int launch_aggregate(const Plan& pl, const uint32_t* buckets, void* ws, hipStream_t st) {
  const uint32_t bb = (uint32_t)pl.bb, S = (uint32_t)pl.S;
  uint32_t* lv[2] = {ws_at<uint32_t>(ws, pl.o_lvl0), ws_at<uint32_t>(ws, pl.o_lvl1)};
  uint32_t* wsum = ws_at<uint32_t>(ws, pl.o_wsum);
  ProfScope prof(PT_AGG, st);
  const uint32_t* in = buckets;
  uint32_t nodes = 1u << bb, h = 0, level = 0;
  // outputs and additions of level h over all windows
  auto outs = [&](uint32_t l) { return ((uint64_t)S << (bb - 1 - l)) * (l + 2); };
  auto adds = [&](uint32_t l) { return ((uint64_t)S << (bb - 1 - l)) * (l + 1); };
  // the fused tail: from the first level with one addition per quad of a
  // window's block on (or a schedule's number of outputs over all windows)
  auto tail = [&](uint32_t l) {
    return l + 1 == bb || (adds(l) <= (uint64_t)S * TAIL_ADDS &&
                           (pl.tree_wide == 0 || outs(l) <= pl.tree_wide));
  };
  while (!tail(h)) {
    uint32_t* out = lv[level++ & 1];
    // one lane per addition down to tree_quad outputs, then quads
    if (h == 0 && !tail(1) && outs(1) >= pl.tree_quad) {
      const uint64_t lanes = (uint64_t)S << (bb - 1);
      k_tree_first<<<(unsigned)((lanes + 255) / 256), 256, 0, st>>>(in, lanes, out);
      ++h;
      nodes >>= 1;
    } else if (outs(h + 1) >= pl.tree_quad && !tail(h + 1)) {
      const uint64_t n1 = (uint64_t)S << (bb - 2 - h);
      k_tree_level2<<<(unsigned)((n1 * (h + 3) + 255) / 256), 256, 0, st>>>(in, h, n1, out);
      ++h;
      nodes >>= 1;
    } else if (outs(h) >= pl.tree_quad) {
      k_tree_level<<<(unsigned)((adds(h) + 255) / 256), 256, 0, st>>>(in, h, nodes, S, out);
    } else if (!tail(h + 1)) {
      const uint64_t o2 = outs(h + 1);
      k_tree_quad2<<<(unsigned)((4 * o2 + 255) / 256), 256, 0, st>>>(in, h, o2, out);
      ++h;
      nodes >>= 1;
    } else {
      k_tree_level_quad<<<(unsigned)((4 * outs(h) + 255) / 256), 256, 0, st>>>(in, h, nodes, S, out);
    }
    in = out;
    ++h;
    nodes >>= 1;
  }
  size_t second = 0;
  const size_t first = tail_words(h, bb, second);
  k_window_tail<<<S, TAIL_THREADS, (first + second) * 4, st>>>(
      in, h, bb, (uint32_t)first, pl.encoding == MSM_DIGITS_UNSIGNED ? 0 : 1, wsum);
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

int launch_horner(const Plan& pl, void* ws, hipStream_t st) {
  ProfScope prof(PT_HORNER, st);
  const JobView jv = job_view(pl, ws);
  k_group<<<(unsigned)pl.J, W26_THREADS, 0, st>>>(ws_at<uint32_t>(ws, pl.o_wsum), (uint32_t)pl.W,
                                                  (uint32_t)pl.c, jv,
                                                  ws_at<uint32_t>(ws, pl.o_flags));
  HIPCHK(hipGetLastError());
  return MSM_OK;
}

}  // namespace msm

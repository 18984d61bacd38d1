// Declarations shared by the translation units of libmsm_gfx950.so.
#pragma once
#include <hip/hip_runtime.h>

#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "../../include/msm.h"
#include "curve.hpp"
#include "field.hpp"

namespace msm {

// Constants of the Weierstrass <-> twisted-Edwards map, Montgomery form:
//   x_w = alpha u - 1,  y_w = beta v,  u = (1 + y_e)/(1 - y_e),  v = u / x_e
constexpr uint32_t kAlpha[NL] = {0x8894e1e4u, 0x3fabdfd0u, 0xcc1f55aau, 0xcbf921ddu,
                                 0x460edc0cu, 0xd17deff1u, 0x7897028du, 0xd394e81eu,
                                 0x0912681au, 0xc29c995du, 0xaff9d568u, 0x01515e6cu};
constexpr uint32_t kBeta[NL] = {0xa38cfd11u, 0xface0c97u, 0x0adb8383u, 0x8cc7c229u,
                                0xd44ae9cbu, 0x4765cd5fu, 0x22354029u, 0x9ae986d8u,
                                0x252ab9bdu, 0xc3dc7860u, 0xc8942395u, 0x00486011u};
// R^3 mod p: turns a plain inverse of a Montgomery value into Montgomery form
constexpr uint32_t kR3[NL] = {0x8815de20u, 0x581f532fu, 0xbe329585u, 0xe50f4148u,
                              0x0449f513u, 0x2be8b118u, 0xc804a20eu, 0x6a2a9516u,
                              0x13590cb9u, 0x3f725407u, 0xc0e7dda5u, 0x01065ab4u};
// conventional generator G of BLS12-377 G1, Weierstrass affine (Montgomery form)
constexpr uint32_t kGx[NL] = {0x772451f4u, 0x260f33b9u, 0x169d5658u, 0xc54dd773u,
                              0x69a510ddu, 0x5c1551c4u, 0x425e1698u, 0x761662e4u,
                              0x6f065272u, 0xc97d78ccu, 0xb361fd4du, 0x00a41206u};
constexpr uint32_t kGy[NL] = {0xb8cb81f3u, 0x8193961fu, 0x5f44adb8u, 0x00638d4cu,
                              0xd4daf54au, 0xfafaf3dau, 0xd655cd18u, 0xc27849e2u,
                              0x01d52814u, 0x2ec3ddb4u, 0x26303c71u, 0x007da933u};
// G in prepared twisted-Edwards form (x_e, y_e, k x_e y_e), Montgomery form
constexpr uint32_t kGteX[NL] = {0x654b417fu, 0x5bab21b3u, 0x1d3e1fe0u, 0x042fff8au,
                                0xdf39dc37u, 0xb702072eu, 0x39426b02u, 0xa5625e78u,
                                0xb51c7d03u, 0xbf2dc368u, 0x28ac3263u, 0x00b3ad90u};
constexpr uint32_t kGteY[NL] = {0xef15101du, 0x3904973cu, 0xb1f14456u, 0xb45ed211u,
                                0x5dfac94eu, 0x90a86b86u, 0xfe3945cdu, 0xcdb19c57u,
                                0xef4f7097u, 0x972a8d46u, 0xa3d9cf77u, 0x00281a91u};
constexpr uint32_t kGteU[NL] = {0x4f3f8d58u, 0x719243efu, 0x4a7b9d48u, 0xf744d1fcu,
                                0xa77008dcu, 0x0ab712e3u, 0x1e09b26fu, 0x53f80798u,
                                0xef3f9f1bu, 0x24125ab8u, 0xfb63f6d1u, 0x01959f77u};

constexpr int SCALAR_BITS = 253;  // scalars are below 2^253
constexpr int GLV_BITS = 127;     // halves of the endomorphism split are below 2^127
constexpr int SCALAR_WORDS = 8;

inline unsigned grid_for(size_t n, unsigned block) { return (unsigned)((n + block - 1) / block); }

// ---------------------------------------------------------------------------
// error reporting and optional per-phase timing (msm_api.hip)
// ---------------------------------------------------------------------------
void set_last_hip_error(int e);

#define HIPCHK(x)                         \
  do {                                    \
    hipError_t e_ = (x);                  \
    if (e_ != hipSuccess) {               \
      ::msm::set_last_hip_error((int)e_); \
      return MSM_EHIP;                    \
    }                                     \
  } while (0)

enum ProfTag { PT_SORT = 0, PT_ACCUM, PT_MERGE, PT_AGG, PT_HORNER, PT_COUNT };

// Records HIP events around its lifetime on `st` while profiling is enabled.
struct ProfScope {
  bool active = false;
  int tag = 0;
  hipStream_t st = nullptr;
  hipEvent_t a = nullptr;
  ProfScope(int t, hipStream_t s);
  ~ProfScope();
};

// Start and stop events for one kernel dispatch of phase `tag`, when the
// profiling mode times that kernel alone (false otherwise); the caller
// launches with them (hipExtLaunchKernelGGL) and then records the pair.
bool prof_kernel_events(int tag, hipStream_t st, hipEvent_t* a, hipEvent_t* b);
void prof_kernel_record(int tag, hipEvent_t a, hipEvent_t b);

// Digit sort geometry: partitions of uniformly spread digits hold at most
// sort_part_target entries; pass 2 stages up to SORT_PART_CAP in LDS and
// sorts larger partitions on many blocks, in items of SORT_BIG_ITEM entries.
// 8192 from jobs of more than 2^21 point records on: half the partitions, so a
// tile's runs to each are twice as long (split digits, n = 2^22: sort 787 ->
// 648 us; signed, 2^22: 627 -> 552).  4096 below, where the scatter is not what
// counts and a window of fewer digit values (twice the entries a bucket) then
// exceeds the stage (split digits, n = 2^20: 193 us, with 8192 197; n = 65536:
// 73, 79).
inline uint32_t sort_part_target(size_t max_n) {
  return max_n > (size_t)1 << 21 ? 8192u : 4096u;
}
constexpr uint32_t SORT_PART_CAP = 10240;
constexpr uint32_t SORT_BIG_ITEM = 4096;
constexpr int SORT_COUNTERS = 3;  // cleared by each sort's first kernel

// ---------------------------------------------------------------------------
// jobs and workspace plans (msm_api.hip)
// ---------------------------------------------------------------------------
// One pipeline runs a batch of J independent MSMs that share the window width
// c and the digit encoding; a single MSM is a batch of one.  Window w of job j
// is segment s = j W + w.  Segment s holds the job's n digits at
// [W pt_off + w n, W pt_off + (w+1) n) of the digit array and owns the
// pass-1 sort tiles [W tile_off + w tps, W tile_off + (w+1) tps).
struct JobDesc {
  const uint32_t* xyu;      // prepared points (AoS XYU records)
  const uint32_t* scalars;  // 8 words per scalar
  uint32_t* result;         // MSM_RESULT_WORDS words
  uint32_t n;               // points of the job
  uint32_t pt_off;          // points of the jobs before it
  uint32_t tile_off;        // tile groups per window of the jobs before it
  uint32_t tps;             // sort tile groups per window, ceil(n / tile_digits)
};

// Kernel-argument view of a batch's jobs: a device table, or (J = 1) the one
// job by value so that a single MSM needs no table upload.
struct JobView {
  const JobDesc* tab;
  JobDesc one;
  uint32_t J;
  __device__ __forceinline__ JobDesc get(uint32_t j) const { return tab ? tab[j] : one; }
};

constexpr uint32_t SORT_TILE = 8192;  // digits per pass-1 sort tile

// Accumulation chunks (k_accum.hip).  Their length follows from the number of
// entries, which only the device knows (zero digits have none): one chunk per
// unit, where `units` units give every SIMD one wave.
struct AccumGeom {
  uint32_t units;  // lanes or quads of one wave per SIMD
  uint32_t least;  // entries of a chunk, at least (a multiple of 4)
  uint32_t fixed;  // a schedule's chunk length (0: from the entries)
  uint32_t quad;   // a unit is a quad
};
// Quads up to 2^19 digit slots: a quarter of the lanes' chunks, and so of the
// split buckets, for 1.4 times the instructions (split digits, c = 8: n = 10000 325
// us on lanes, 265 on quads, n = 16384 328, 295).  Above, lanes of more than
// eight entries are as fast (n = 24000, c = 13: 349, 353; n = 50000 402, 424).
constexpr size_t ACCUM_QUAD_MAX = (size_t)1 << 19;
// Units for E entries.  Lanes: a lone wave a SIMD leaves 13% of its issue slots
// empty, and each further wave doubles or halves again the split buckets to
// merge.  One wave up to 16 entries a lane (n = 40000, split digits, 13: 442 us,
// with two waves 457; n = 90000, 27: 502, 485), two up to 160 (n = 262144, 80: two
// 821, three 834; n = 700000 signed, 171: 1768, 1756; n = 2^21, 512: 4297, 4128),
// three above, the most that its registers allow.
__host__ __device__ inline uint32_t accum_units(const AccumGeom& g, uint32_t E) {
  const uint64_t u = g.units;
  return g.quad || E < 16 * u ? g.units : (E < 160 * u ? 2 * g.units : 3 * g.units);
}

// The one-kernel sort takes jobs of at most SMALL_SORT_MAX point records (16 for
// each of a block's 1024 threads) and buckets that fit its LDS counts.
constexpr size_t SMALL_SORT_MAX = 16384;
constexpr int SMALL_SORT_BITS = 13;

// Windows of jobs of at most SEGMENT_MAX point records and SEGMENT_BITS bucket
// bits (one addition per quad of a block at the first level) run whole in one
// block each (k_segment), when there are compute units for all of them: n = 128
// split digits 178 -> 174 us, n = 256 signed 266 -> 246.  With more records a block's
// own quads take longer than the chip's (512 signed 263 -> 279; 180 split, 360
// records, 179 -> 192), and with more windows than compute units the blocks' idle
// lanes cost (64 jobs of 32 to 128 points, 428 -> 493 us).
constexpr size_t SEGMENT_MAX = 256;
constexpr int SEGMENT_BITS = 8;

// key of the entries that the one-kernel sort keeps for zero digits
constexpr uint32_t KEY_NONE = 0xffffffffu;
// bucket b's place in the offsets array: each segment has its 2^bb buckets'
// starts and its own end
__host__ __device__ inline size_t offset_index(uint32_t b, uint32_t bb) {
  return (size_t)b + (b >> bb);
}

struct Plan {
  int c = 0, W = 0;
  int encoding = MSM_DIGITS_SIGNED;
  int bb = 0;  // bucket-index bits: c (unsigned digits) or c - 1 (signed)
  uint32_t J = 1;
  size_t N = 0;       // points over all jobs
  size_t max_n = 0;   // largest job
  size_t S = 0;       // segments J W
  size_t M = 0;       // buckets S 2^bb
  size_t NW = 0;      // digits N W
  size_t tiles = 0;   // pass-1 sort tiles over all segments
  AccumGeom accum{};      // how entries are cut into accumulation chunks
  size_t chunks = 0;      // accumulation chunks, at most
  size_t long_items = 0;  // capacity of the long-span list: items and segments
  size_t long_segs = 0;
  uint64_t tree_quad = 65536;  // tree levels with fewer outputs run on quads
  uint64_t tree_wide = 0;      // outputs from which a window's levels run in one block (0: k_agg.hip's rule)
  bool small_sort = false;            // the one-kernel sort
  bool segment = false;  // windows run whole, one block each (k_segment)
  uint32_t lo_bits = 0, hi_bits = 0;  // split of the bb bucket bits in the sort
  uint32_t tpb = 1;                   // pass-1 tiles per block (one histogram per group)
  uint32_t tile_digits = SORT_TILE;   // digits per group, SORT_TILE tpb
  bool tmp_packed = false;            // staged sort entries in one word (jobs <= 2^23 points)
  size_t ncounts = 0, nb = 0;         // sort count matrix size, its scan blocks
  JobDesc one{};  // the job when J = 1; otherwise one.xyu is the base of segment offsets
  // byte offsets into the workspace
  size_t o_flags = 0, o_total = 0, o_offsets = 0, o_counts = 0, o_blocksums = 0, o_digits = 0,
         o_tmp = 0, o_key = 0, o_idx = 0, o_head = 0, o_tail = 0, o_buckets = 0, o_lvl0 = 0,
         o_lvl1 = 0, o_wsum = 0, o_longlist = 0, o_counters = 0, o_bigdesc = 0, o_bigsum = 0, o_bigcnt = 0, o_bigitem = 0, o_jobs = 0, o_segoff = 0, bytes = 0;
};

// schedule of a plan (0 = default for each; msm_job's chunk, tree_quad,
// tree_wide)
struct Schedule {
  int chunk = 0, tree_quad = 0, tree_wide = 0;
  bool operator<(const Schedule& o) const {
    if (chunk != o.chunk) return chunk < o.chunk;
    if (tree_quad != o.tree_quad) return tree_quad < o.tree_quad;
    return tree_wide < o.tree_wide;
  }
};

int num_windows(int c, int encoding);
int window_bits(int c, int encoding);
int default_window(size_t n);                     // signed-digit model (msm_default_window)
// the width c = 0 picks for an MSM of an encoding that is one of `jobs` run
// together, among those whose workspace (on a schedule, and compact: see
// make_plan) is within `limit` bytes (0: any); 0 when none is
int default_window_for(size_t n, int encoding, size_t jobs = 1, size_t limit = 0,
                       const Schedule& sched = Schedule(), bool compact = false);
// work of `jobs` MSMs of n points in all at width c, in digit entries
double window_work(double n, double jobs, int c, int encoding);

// Picks for many sizes: what a width costs whatever the size is worked out once (a
// batch of 20000 jobs with c = 0 planned in 14 ms before, 2.8 with this).
class WidthPicker {
 public:
  WidthPicker(int encoding, size_t jobs);
  int pick(size_t n) const;
  // among the widths c that may(c) allows; 0 when none is
  template <typename F>
  int pick(size_t n, F may) const {
    int best = 0;
    double best_cost = 1e300;
    for (int i = 0; i < count_; ++i) {
      const double x = cost(widths_[i], mult_ * (double)n);
      if (x < best_cost && may(widths_[i].c)) {
        best_cost = x;
        best = widths_[i].c;
      }
    }
    return best;
  }

 private:
  struct Width {
    int c;
    double W, work, latency;
    double digits, crowd;  // the top window's: how many, and the share of entries that has one
  };
  double cost(const Width& w, double points) const;
  double mult_, jobs_;
  uint32_t simds_;
  int count_ = 0;
  Width widths_[17];  // 4 .. 20
};

// Entries of an accumulation chunk, at least.  Four, the group in which keys are
// read, give most units a chunk (13 us of accumulation at n = 33 against 108 with
// sixteen).  A chunk's head and tail take 384 bytes, though, and with four entries
// they are most of a small job's workspace: a compact plan has sixteen.
constexpr uint32_t CHUNK_LEAST = 4, CHUNK_LEAST_COMPACT = 16;

// plan of a batch with job sizes ns[0..J); false for invalid sizes, c or
// schedule values.  compact: less workspace, for callers who have no more
bool make_plan(const size_t* ns, uint32_t J, int c, int encoding, Plan& pl,
               const Schedule& sched = Schedule(), bool compact = false);

// plan of one MSM in `limit` bytes of workspace, at width c, or for c = 0 at the
// width picked for one of `jobs`, or if that takes more at the best that fits;
// compact when nothing else fits: MSM_OK, MSM_EINVAL (as make_plan) or MSM_ENOSPC
int plan_within(size_t n, int c, int encoding, size_t jobs, size_t limit, Plan& pl,
                const Schedule& sched = Schedule());

template <typename T>
inline T* ws_at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// every phase of a planned batch on one stream (msm_api.hip); with an event
// `accum_after`, the accumulation first waits for that event's last recording
// (the digit sort does not)
int enqueue_msm(const Plan& pl, void* ws, hipStream_t st, hipEvent_t accum_after = nullptr);

inline JobView job_view(const Plan& pl, void* ws) {
  JobView v;
  v.tab = pl.J == 1 ? nullptr : ws_at<const JobDesc>(ws, pl.o_jobs);
  v.one = pl.one;
  v.J = pl.J;
  return v;
}

// ---------------------------------------------------------------------------
// kernel launchers (each returns MSM_OK or MSM_EHIP)
// ---------------------------------------------------------------------------
// k_sort.hip: digits -> CSR offsets, sorted (key, idx | sign << 31); empty
// buckets set to the identity
// fills lo_bits, hi_bits, tpb, tile_digits, tiles (groups over all segments),
// ncounts, nb for jobs of mult * ns[j] points
void sort_geometry(Plan& pl, const size_t* ns, uint32_t J, size_t mult);
int launch_sort(const Plan& pl, uint32_t* buckets, void* ws, hipStream_t st);
// k_accum.hip: bucket accumulation and split-bucket merge, buckets as signed
// records (fe29.hpp) or with coordinates in [0, 2p)
int launch_accumulate(const Plan& pl, uint32_t* buckets, void* ws, hipStream_t st,
                      bool unsigned_buckets = false);
// k_agg.hip: bucket aggregation (window sums), group aggregation and the
// affine results of every job
int launch_aggregate(const Plan& pl, const uint32_t* buckets, void* ws, hipStream_t st);
int launch_horner(const Plan& pl, void* ws, hipStream_t st);
// k_segment.hip: all of that up to the window sums for small jobs (Plan::segment)
int launch_segments(const Plan& pl, void* ws, hipStream_t st);
// k_elementwise.hip
int launch_fe_mul(const uint32_t* a, const uint32_t* b, uint32_t* out, uint32_t count,
                  int canonical, hipStream_t st);
int launch_padd(const uint32_t* a, const uint32_t* b, uint32_t* out, uint32_t count, int form,
                hipStream_t st);
int launch_prepare(const uint32_t* xy, const uint32_t* inf, uint32_t* xyu, uint32_t n,
                   uint32_t* status, bool endo, hipStream_t st);
int launch_gen_points(const uint32_t* k, uint32_t* xy, uint32_t* inf, uint32_t n, hipStream_t st);

}  // namespace msm

// C ABI of libmsm_gfx950.so (include/msm.h): argument checks, workspace plans,
// per-phase timing and the entry points, which enqueue the kernels of the
// other translation units on the caller's stream.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <mutex>
#include <vector>

#include "common.hpp"

namespace msm {

namespace {
thread_local int g_last_hip = 0;

const char* const kProfNames[PT_COUNT] = {"sort", "accum", "merge", "agg", "horner"};

struct ProfState {
  std::mutex mu;
  int mode = MSM_PROFILE_OFF;
  struct Rec {
    int tag;
    hipEvent_t a, b;
  };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;
};
ProfState g_prof;

hipEvent_t prof_event() {
  if (!g_prof.pool.empty()) {
    hipEvent_t e = g_prof.pool.back();
    g_prof.pool.pop_back();
    return e;
  }
  // timing only: no system-scope fence (cache writeback and invalidation)
  // when the event is recorded
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
  return e;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace

void set_last_hip_error(int e) { g_last_hip = e; }

// set while msm_run_noalloc enqueues: no timing events are taken then (an
// event pool refill would create events)
static thread_local bool t_no_events = false;

ProfScope::ProfScope(int t, hipStream_t s) : tag(t), st(s) {
  if (t_no_events) return;
  std::lock_guard<std::mutex> g(g_prof.mu);
  if (g_prof.mode != MSM_PROFILE_PHASES) return;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return;
  a = prof_event();
  if (a && hipEventRecord(a, st) == hipSuccess) active = true;
}

ProfScope::~ProfScope() {
  if (!active) return;
  std::lock_guard<std::mutex> g(g_prof.mu);
  hipEvent_t b = prof_event();
  if (b && hipEventRecord(b, st) == hipSuccess) g_prof.recs.push_back({tag, a, b});
}

bool prof_kernel_events(int tag, hipStream_t st, hipEvent_t* a, hipEvent_t* b) {
  if (t_no_events) return false;
  std::lock_guard<std::mutex> g(g_prof.mu);
  if (g_prof.mode != MSM_PROFILE_ACCUM_KERNEL || tag != PT_ACCUM) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return false;
  *a = prof_event();
  *b = prof_event();
  if (*a && *b) return true;
  if (*a) g_prof.pool.push_back(*a);
  if (*b) g_prof.pool.push_back(*b);
  return false;
}

void prof_kernel_record(int tag, hipEvent_t a, hipEvent_t b) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.recs.push_back({tag, a, b});
}

int num_windows(int c, int encoding) {
  if (encoding == MSM_DIGITS_SIGNED) return (c >= 2 && c <= 20) ? (SCALAR_BITS + c) / c : 0;
  if (encoding == MSM_DIGITS_GLV) return (c >= 2 && c <= 20) ? (GLV_BITS + c) / c : 0;
  if (encoding == MSM_DIGITS_UNSIGNED) return (c >= 1 && c <= 20) ? (SCALAR_BITS + c - 1) / c : 0;
  return 0;
}

// Window width actually used for a requested width c: the smallest width
// that covers the digit bits with the same number of windows, so that no
// window (in particular the top one) is left with a few bits whose digits
// would crowd a handful of buckets.
int window_bits(int c, int encoding) {
  const int W = num_windows(c, encoding);
  if (W == 0) return 0;
  const int bits = encoding == MSM_DIGITS_UNSIGNED ? SCALAR_BITS
                   : encoding == MSM_DIGITS_GLV    ? GLV_BITS + 1
                                                   : SCALAR_BITS + 1;
  return (bits + W - 1) / W;
}

// compute units of the current device (256 on MI355X; also the answer when
// no device is visible, e.g. for workspace queries on a host without GPU)
static unsigned device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0) {
    (void)hipGetLastError();
    return 256;
  }
  return (unsigned)cus;
}

// Cost of an MSM of n points at width c, in digit entries (8.8 G a second), one
// of `jobs` that run together.  Work: the entries, 2.6 for each bucket (tree,
// merges, the sort's identities) and 100 for each window.  Latency, which jobs
// running together hide from each other: 5.5 us for each bucket bit (a level
// of the tree and a step of the window's combination), 0.8 us for each window
// (its step in the group aggregation), 11 us for the larger sort and the lanes'
// merges beyond the quads' range, and a crowded top window: when its few
// digits spread their entries over more than 64 chunks, k_merge_long has work
// (11 us, and 23 more beyond 128 chunks, two stages).  Hence the widths whose top
// window is nearly full, c' = 8, 11 (plain), 13 and 16, hold over long ranges of n.
// Fitted to the widths around the pick by entries and buckets alone, 39 sizes of
// single MSMs of each encoding and 21 batches: on average 0.6% above the best
// width, that pick 4.5%.  Split digits, n = 4099: c' = 10 246 us, 8 229; n =
// 24000: 12 398, 13 352; 64 jobs of 8192: 10 1.97 ms, 8 2.13.  Signed, n = 8192:
// 10 366 us, 8 312.  Plain, n = 65536: 13 586 us, 11 513.
double window_work(double n, double jobs, int c, int encoding) {
  const double W = num_windows(c, encoding);
  const int bits = window_bits(c, encoding);
  const int bb = encoding == MSM_DIGITS_UNSIGNED ? bits : bits - 1;
  return (encoding == MSM_DIGITS_GLV ? 2.0 : 1.0) * n * W +
         jobs * (2.6 * std::ldexp(1.0, bb) + 100.0) * W;
}

WidthPicker::WidthPicker(int encoding, size_t jobs)
    : mult_(encoding == MSM_DIGITS_GLV ? 2.0 : 1.0), jobs_((double)jobs), simds_(4u * device_cus()) {
  // the digits of the top window run to the largest scalar's (split half's)
  const double largest = encoding == MSM_DIGITS_GLV ? std::ldexp((double)0x452217cc, 96)
                                                    : std::ldexp((double)0x12ab655e, 224);
  for (int c = 4; c <= 20; ++c) {
    const int W = num_windows(c, encoding), bits = window_bits(c, encoding);
    if (W == 0) continue;
    const int bb = encoding == MSM_DIGITS_UNSIGNED ? bits : bits - 1;
    Width w = {};
    w.c = c;
    w.W = W;
    w.work = window_work(0.0, 1.0, c, encoding);
    w.latency = 48e3 * bb + 7e3 * W;
    w.digits = std::floor(std::ldexp(largest, -bits * (W - 1)));
    w.crowd = 1.0;
    if (w.digits < 1.0) {  // the carry alone
      const double below = std::floor(std::ldexp(largest, -bits * (W - 2)));
      w.crowd = std::max(0.0, 1.0 - std::ldexp(0.5, bits) / below);
    }
    widths_[count_++] = w;
  }
}

double WidthPicker::cost(const Width& w, double points) const {
  const double entries = points * w.W;
  const double all = std::min(entries * jobs_, 2147483648.0);
  AccumGeom g = {};
  g.quad = all <= (double)ACCUM_QUAD_MAX ? 1u : 0u;
  g.units = simds_ * (g.quad ? 16u : 64u);
  const double chunk = std::max((double)CHUNK_LEAST, all / accum_units(g, (uint32_t)all));
  // chunks of the entries of one of the top window's digits
  const double span = points / std::max(1.0, w.digits) / chunk * w.crowd;
  const double latency = w.latency + (g.quad ? 0.0 : 1e5) + (span > 64 ? 1e5 : 0.0) +
                         (span > 128 ? 2e5 : 0.0);
  return entries + w.work + latency / jobs_;
}

int WidthPicker::pick(size_t n) const {
  return pick(n, [](int) { return true; });
}

int default_window_for(size_t n, int encoding, size_t jobs, size_t limit, const Schedule& sched,
                       bool compact) {
  const WidthPicker picker(encoding, jobs);
  if (limit == 0) return picker.pick(n);
  return picker.pick(n, [&](int c) {
    Plan pl;
    return make_plan(&n, 1, c, encoding, pl, sched, compact) && pl.bytes <= limit;
  });
}

int default_window(size_t n) { return default_window_for(n, MSM_DIGITS_SIGNED); }

bool make_plan(const size_t* ns, uint32_t J, int c_req, int encoding, Plan& pl,
               const Schedule& sched, bool compact) {
  pl = Plan();
  const int W = num_windows(c_req, encoding);
  if (W == 0 || J == 0 || !ns) return false;
  if (sched.chunk < 0 || sched.tree_quad < 0 || sched.tree_wide < 0) return false;
  if (sched.tree_quad) pl.tree_quad = (uint64_t)sched.tree_quad;
  if (sched.tree_wide) pl.tree_wide = (uint64_t)sched.tree_wide;
  const int c = window_bits(c_req, encoding);
  pl.c = c;
  pl.W = W;
  pl.encoding = encoding;
  pl.bb = encoding == MSM_DIGITS_UNSIGNED ? c : c - 1;
  pl.J = J;
  // with the endomorphism split every input point contributes two points
  const size_t mult = encoding == MSM_DIGITS_GLV ? 2 : 1;
  for (uint32_t j = 0; j < J; ++j) {
    if (ns[j] == 0 || ns[j] >= ((size_t)1 << 26)) return false;
    const size_t nv = mult * ns[j];
    pl.N += nv;
    pl.max_n = std::max(pl.max_n, nv);
  }
  pl.S = (size_t)J * W;
  pl.M = pl.S << pl.bb;
  pl.NW = pl.N * (size_t)W;
  // entry positions, keys (s 2^bb + m) and point indices are 32-bit words
  if (pl.N >= ((size_t)1 << 31) || pl.NW >= ((size_t)1 << 31) || pl.M >= ((size_t)1 << 31))
    return false;
  sort_geometry(pl, ns, J, mult);
  pl.small_sort = pl.max_n <= SMALL_SORT_MAX && pl.bb <= SMALL_SORT_BITS;
  // (a schedule is for the kernels that it schedules)
  pl.segment = pl.max_n <= SEGMENT_MAX && pl.bb <= SEGMENT_BITS &&
               pl.S <= (size_t)device_cus() && sched.chunk == 0 && sched.tree_quad == 0 &&
               sched.tree_wide == 0;
  if (pl.lo_bits > 8 || pl.nb > 4096 || pl.tiles >= ((size_t)1 << 31)) return false;
  if (J == 1) {
    pl.one.n = (uint32_t)(mult * ns[0]);
    pl.one.tps = (uint32_t)((mult * ns[0] + pl.tile_digits - 1) / pl.tile_digits);
  }
  // accumulation chunks (AccumGeom): at most one per unit, each of at least
  // `least` entries, or all of a schedule's length
  const size_t simds = (size_t)device_cus() * 4;
  if (sched.chunk) pl.accum.fixed = ((uint32_t)std::max(4, sched.chunk) + 3u) & ~3u;
  pl.accum.least = compact ? CHUNK_LEAST_COMPACT : CHUNK_LEAST;
  pl.accum.quad = pl.NW <= ACCUM_QUAD_MAX ? 1u : 0u;
  pl.accum.units = (uint32_t)(simds * (pl.accum.quad ? 16 : 64));
  pl.chunks = pl.accum.fixed
                  ? (pl.NW + pl.accum.fixed - 1) / pl.accum.fixed
                  : std::min<size_t>(accum_units(pl.accum, (uint32_t)pl.NW),
                                     (pl.NW + pl.accum.least - 1) / pl.accum.least);
  pl.long_items = pl.chunks / 8 + 1;
  pl.long_segs = pl.long_items + pl.chunks / 128;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = align_up(o + bytes, 256);
    return at;
  };
  const size_t rec = XYTZ_WORDS * 4;
  pl.o_flags = take((size_t)J * 4);
  pl.o_total = take(4);
  pl.o_offsets = take((pl.M + pl.S) * 4);
  pl.o_counts = take(pl.ncounts * 4);
  pl.o_blocksums = take(4096 * 4);
  // large sort partitions: each holds more than SORT_PART_CAP entries, so
  // there are at most NW / SORT_PART_CAP of them, and NW / SORT_BIG_ITEM +
  // that many items; their 512 counts each take the place of the digits (more),
  // which pass 1 has read
  const size_t nbig_max = pl.NW / SORT_PART_CAP;
  static_assert(SORT_PART_CAP >= 512, "");
  pl.o_digits = take(pl.NW * 4);
  pl.o_bigsum = pl.o_digits;
  pl.o_tmp = take(pl.NW * 8);
  pl.o_key = take(pl.NW * 4 + 32);  // + 16-byte groups read past the end
  pl.o_idx = take(pl.NW * 4 + 32);
  pl.o_longlist = take((2 + 2 * pl.long_items + 2 * pl.long_segs) * 4);
  pl.o_counters = take(SORT_COUNTERS * 4);
  pl.o_bigdesc = take(nbig_max * 16);
  pl.o_bigcnt = take((pl.NW / SORT_BIG_ITEM + nbig_max + 1) * 256 * 4);
  pl.o_bigitem = take((pl.NW / SORT_BIG_ITEM + nbig_max + 1) * 4);
  // buckets, then the tree levels ping-pong between lvl0 (level 0's M
  // records) and the bucket array, which level 0 has consumed; before level 0,
  // lvl0 holds the accumulation's heads and tails
  pl.o_buckets = take(pl.M * rec);
  pl.o_lvl0 = take(std::max(pl.M, 2 * pl.chunks) * rec);
  pl.o_head = pl.o_lvl0;
  pl.o_tail = pl.o_head + pl.chunks * rec;
  pl.o_lvl1 = pl.o_buckets;
  pl.o_wsum = take(2 * pl.S * rec);
  pl.o_jobs = take((size_t)J * sizeof(JobDesc));
  pl.o_segoff = take(pl.S * 8);
  pl.bytes = o;
  return true;
}

// The picked width's workspace does not grow with n throughout (split digits: 512
// points 3.9 MB, 513 2.4 MB), so one sized for more points may be too small for it
// and yet hold a plan at the larger size's width.
int plan_within(size_t n, int c, int encoding, size_t jobs, size_t limit, Plan& pl,
                const Schedule& sched) {
  const int pick = c == 0 ? default_window_for(n, encoding, jobs) : c;
  if (!make_plan(&n, 1, pick, encoding, pl, sched)) return MSM_EINVAL;
  if (pl.bytes <= limit) return MSM_OK;
  for (const bool compact : {false, true}) {
    const int w = c == 0 ? default_window_for(n, encoding, jobs, limit, sched, compact) : c;
    if (w && make_plan(&n, 1, w, encoding, pl, sched, compact) && pl.bytes <= limit) return MSM_OK;
  }
  return MSM_ENOSPC;
}

int enqueue_msm(const Plan& pl, void* ws, hipStream_t st, hipEvent_t accum_after) {
  uint32_t* buckets = ws_at<uint32_t>(ws, pl.o_buckets);
  int rc;
  if (pl.segment) {
    if (accum_after) HIPCHK(hipStreamWaitEvent(st, accum_after, 0));
    if ((rc = launch_segments(pl, ws, st)) != MSM_OK) return rc;
    return launch_horner(pl, ws, st);
  }
  {
    ProfScope prof(PT_SORT, st);
    rc = launch_sort(pl, buckets, ws, st);
  }
  if (rc != MSM_OK) return rc;
  if (accum_after) HIPCHK(hipStreamWaitEvent(st, accum_after, 0));
  if ((rc = launch_accumulate(pl, buckets, ws, st)) != MSM_OK) return rc;
  if ((rc = launch_aggregate(pl, buckets, ws, st)) != MSM_OK) return rc;
  return launch_horner(pl, ws, st);
}

// Scratch of msm_run_noalloc: a file-scope device array, one copy per GPU,
// held until the process ends.  Host code must not use the array's name as a
// device address; the address comes from hipGetSymbolAddress, taken once per
// device (with that device current) on the entry point's first call there.
constexpr size_t kScratchBytes = (size_t)MSM_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

static int scratch_of_current_device(void** out) {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return MSM_EINVAL;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return MSM_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return MSM_OK;
}

}  // namespace msm

using namespace msm;

extern "C" {

int msm_last_hip_error(void) { return g_last_hip; }

const char* msm_status_string(int status) {
  switch (status) {
    case MSM_OK: return "MSM_OK";
    case MSM_EINVAL: return "MSM_EINVAL: invalid argument";
    case MSM_ENOSPC: return "MSM_ENOSPC: workspace too small";
    case MSM_EHIP: return "MSM_EHIP: HIP runtime error";
    default: return "unknown status";
  }
}

int msm_num_windows(int c, int encoding) { return num_windows(c, encoding); }

int msm_default_window(size_t n) { return default_window(n); }

int msm_window_bits(int c, int encoding) { return window_bits(c, encoding); }

size_t msm_workspace_bytes(size_t n, int c, int encoding) {
  if (c == 0) c = default_window_for(n, encoding);
  Plan pl;
  if (!make_plan(&n, 1, c, encoding, pl)) return 0;
  return pl.bytes;
}

int msm_fe_mul_batch(const uint32_t* a, const uint32_t* b, uint32_t* out, size_t count,
                     int canonical, void* stream) {
  if (!a || !b || !out || count == 0 || count >= (1u << 31)) return MSM_EINVAL;
  return launch_fe_mul(a, b, out, (uint32_t)count, canonical, (hipStream_t)stream);
}

int msm_padd_batch(const uint32_t* a_xytz, const uint32_t* b, uint32_t* out_xytz, size_t count,
                   int b_form, void* stream) {
  if (!a_xytz || !b || !out_xytz || count == 0 || count >= (1u << 29)) return MSM_EINVAL;
  if (b_form != MSM_FORM_XYTZ && b_form != MSM_FORM_XYU) return MSM_EINVAL;
  return launch_padd(a_xytz, b, out_xytz, (uint32_t)count, b_form, (hipStream_t)stream);
}

int msm_points_prepare(const uint32_t* xy_std, const uint32_t* inf, uint32_t* xyu, size_t n,
                       uint32_t* status, void* stream) {
  if (!xy_std || !xyu || !status || n == 0 || n >= (1u << 31)) return MSM_EINVAL;
  return launch_prepare(xy_std, inf, xyu, (uint32_t)n, status, false, (hipStream_t)stream);
}

int msm_points_prepare_endo(const uint32_t* xy_std, const uint32_t* inf, uint32_t* xyu, size_t n,
                            uint32_t* status, void* stream) {
  if (!xy_std || !xyu || !status || n == 0 || n >= (1u << 30)) return MSM_EINVAL;
  return launch_prepare(xy_std, inf, xyu, (uint32_t)n, status, true, (hipStream_t)stream);
}

int msm_gen_points(const uint32_t* k, size_t n, uint32_t* xy_std, uint32_t* inf, void* stream) {
  if (!k || !xy_std || !inf || n == 0 || n >= (1u << 31)) return MSM_EINVAL;
  return launch_gen_points(k, xy_std, inf, (uint32_t)n, (hipStream_t)stream);
}

int msm_bucket_accumulate(const uint32_t* xyu, const uint32_t* scalars, size_t n, int c,
                          int encoding, uint32_t* buckets, void* ws, size_t ws_bytes,
                          void* stream) {
  if (!xyu || !scalars || !buckets || !ws || c == 0) return MSM_EINVAL;
  Plan pl;
  int rc = plan_within(n, c, encoding, 1, ws_bytes, pl);
  if (rc != MSM_OK) return rc;
  pl.one.xyu = xyu;
  pl.one.scalars = scalars;
  hipStream_t st = (hipStream_t)stream;
  {
    ProfScope prof(PT_SORT, st);
    rc = launch_sort(pl, buckets, ws, st);
  }
  if (rc != MSM_OK) return rc;
  return launch_accumulate(pl, buckets, ws, st, true);
}

int msm_run(const uint32_t* xyu, const uint32_t* scalars, size_t n, int c, int encoding,
            uint32_t* result, void* ws, size_t ws_bytes, void* stream) {
  if (!xyu || !scalars || !result || !ws) return MSM_EINVAL;
  Plan pl;
  const int rc = plan_within(n, c, encoding, 1, ws_bytes, pl);
  if (rc != MSM_OK) return rc;
  pl.one.xyu = xyu;
  pl.one.scalars = scalars;
  pl.one.result = result;
  return enqueue_msm(pl, ws, (hipStream_t)stream);
}

int msm_run_noalloc(const uint32_t* xyu, const uint32_t* scalars, size_t n, int c, int encoding,
                    uint32_t* result, void* stream) {
  if (!xyu || !scalars || !result) return MSM_EINVAL;
  Plan pl;
  int rc = plan_within(n, c, encoding, 1, kScratchBytes, pl);
  if (rc != MSM_OK) return rc;
  void* ws = nullptr;
  if ((rc = scratch_of_current_device(&ws)) != MSM_OK) return rc;
  pl.one.xyu = xyu;
  pl.one.scalars = scalars;
  pl.one.result = result;
  t_no_events = true;
  const int rc2 = enqueue_msm(pl, ws, (hipStream_t)stream);
  t_no_events = false;
  return rc2;
}

int msm_profile_enable(int mode) {
  if (mode < MSM_PROFILE_OFF || mode > MSM_PROFILE_ACCUM_KERNEL) return MSM_EINVAL;
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.mode = mode;
  return MSM_OK;
}

int msm_profile_read(const char* phase, double* total_ms, int* launches) {
  if (!phase || !total_ms || !launches) return MSM_EINVAL;
  int tag = -1;
  for (int t = 0; t < PT_COUNT; ++t)
    if (std::strcmp(phase, kProfNames[t]) == 0) tag = t;
  if (tag < 0) return MSM_EINVAL;
  std::lock_guard<std::mutex> g(g_prof.mu);
  double tot = 0.0;
  int cnt = 0;
  std::vector<ProfState::Rec> keep;
  int rc = MSM_OK;
  for (auto& r : g_prof.recs) {
    if (r.tag != tag) {
      keep.push_back(r);
      continue;
    }
    float ms = 0.f;
    hipError_t e = hipEventSynchronize(r.b);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
    if (e != hipSuccess) {
      set_last_hip_error((int)e);
      rc = MSM_EHIP;
    }
    tot += ms;
    ++cnt;
    g_prof.pool.push_back(r.a);
    g_prof.pool.push_back(r.b);
  }
  g_prof.recs.swap(keep);
  *total_ms = tot;
  *launches = cnt;
  return rc;
}

int msm_constants(uint32_t* out, size_t words) {
  if (!out || words < 96) return MSM_EINVAL;
  const uint32_t* tabs[8] = {kP, kOne, kR2, kK, kAlpha, kBeta, kGx, kGy};
  for (int t = 0; t < 8; ++t)
    for (int l = 0; l < NL; ++l) out[t * NL + l] = tabs[t][l];
  return MSM_OK;
}

}  // extern "C"

// C ABI of the FMMformer attention forward operator: argument validation,
// segment planning, the per-(device, stream) workspace cache and the optional
// kernel timer.  Every kernel is launched asynchronously on the caller's stream.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <random>
#include <utility>
#include <vector>

#include "../../include/fmm_attn.h"
#include "fmm_launch.h"
#include "fmm_fw.h"

namespace {

constexpr int kVersion = 1 * 10000 + 2 * 100 + 0;

// ------------------------------------------------------------------ planning
// Segments split the key axis of every (batch, head) slice for the far-field
// state: enough segments to give the GPU about 512 workgroups, but long enough
// that the per-segment state (rank * d * (d+1) floats) stays at most a quarter
// of the key/value bytes it summarises.
struct Plan {
  int nseg;
  int L;
  int nseg_apply;
  int L_apply;
  size_t ws_bytes;
  int fused_g = 0;  // workgroups per slice of the one-launch path (0: not available)
};

// Plans are made for MI355X's 256 compute units.
constexpr long long kCUs = 256;

// The one-launch path for short non-causal slices is planned at two workgroups
// per compute unit; a device with fewer CUs (checked per
// call) takes the three-launch path with the same workspace.
constexpr int kFusedPlanWorkgroups = 2 * kCUs;

// Rows per segment so that B*H*segments is about `target_wg` workgroups.
long long seg_rows(long long bh, int N, long long target_wg, int tm) {
  const long long per_slice = bh >= target_wg ? 1 : (target_wg + bh - 1) / bh;
  long long L = (N + per_slice - 1) / per_slice;
  L = (L + tm - 1) / tm * tm;
  return L < tm ? tm : L;
}

// The smallest multiple of a tile's rows whose K + V bytes are `share` times
// those of its state record.
long long record_rows(int d, int rank, int esize, int share) {
  const int tm = fmm::tile_rows();
  const long long l = 2LL * share * rank * (d + 1) / esize;
  return std::max<long long>(tm, (l + tm - 1) / tm * tm);
}

// Rows of a state segment: ~512 workgroups, each segment's state record
// (rank*d*(d+1) floats) at most a quarter of the K+V bytes it summarises.
long long segment_rows(long long bh, int N, int d, int rank, int esize) {
  return std::max(seg_rows(bh, N, 2 * kCUs, fmm::tile_rows()), record_rows(d, rank, esize, 4));
}

// Shorter ones, records of up to the K+V bytes themselves, where they leave at
// most `wg` workgroups in all and `per_slice` in a slice (else segment_rows).
// Up to one workgroup per CU a shorter walk is a shorter call; one more starts
// a second round (fp32 causal, 8 slices of 9000 rows, d = 64, rank 2, whole
// forward: 232 workgroups of 320 rows 106 us, 288 of 256 162, 376 of 192 126).
long long fill_rows(long long bh, int N, int d, int rank, int esize, long long wg,
                    long long per_slice) {
  const long long base = segment_rows(bh, N, d, rank, esize);
  const long long n = std::min(wg / bh, per_slice);
  if (n < 1) return base;
  const int tm = fmm::tile_rows();
  const long long l = ((N + n - 1) / n + tm - 1) / tm * tm;
  return std::min(base, std::max({l, seg_rows(bh, N, 2 * kCUs, tm), record_rows(d, rank, esize, 1)}));
}

// Segments of a slice beyond which the combine, which walks a slice's records
// in four ranges and keeps the first 32 of each in registers, costs more than
// the shorter walks save (one slice of 30000 rows, causal, us: bf16, d = 32,
// rank 2, 118 segments 18.0, 157 19.2, 235 24.7, 469 44).  The fp32 walk, that
// of rank 3 and the backward's cost more per row: up to 160 (10000 rows: fp32,
// d = 32, rank 2, 79 segments 27.2, 157 22.7; bf16, d = 16, rank 3, 22.2, 19.2),
// the causal fp32 one of wide heads up to one per CU (30000 rows, d = 64, rank
// 2, 157 segments 69.2, 235 60.2).
long long slice_segments(bool causal, int d, int rank, int esize, bool backward) {
  if (esize == 2) return rank == 3 ? 192 : backward ? 160 : 128;
  return causal && d >= 64 ? kCUs : 160;
}

// The rows of fill_rows for one workgroup per CU, or for two where that walk is
// shorter by more than the second round costs: `round2` tenths of a first one.
long long one_or_two_rows(long long bh, int N, int d, int rank, int esize, long long per_slice,
                          int round2) {
  const long long one = fill_rows(bh, N, d, rank, esize, kCUs, per_slice);
  const long long two = fill_rows(bh, N, d, rank, esize, 2 * kCUs, per_slice);
  auto cost = [&](long long L) { return L * (bh * ((N + L - 1) / L) <= kCUs ? 10 : round2); };
  return cost(two) < cost(one) ? two : one;
}

// L: rows of a state segment.
Plan make_plan(int B, int H, int N, int d, int rank, long long L, int apply_tm) {
  const long long bh = (long long)B * H;
  // non-causal apply walk: ~512 workgroups (two per CU), no state per segment
  const long long La = seg_rows(bh, N, 2 * kCUs, apply_tm);
  Plan p;
  p.L = (int)L;
  p.nseg = (int)((N + L - 1) / L);
  p.L_apply = (int)La;
  p.nseg_apply = (int)((N + La - 1) / La);
  typedef unsigned __int128 u128;
  const u128 rec = (u128)rank * d * (d + 1);
  const u128 ws = ((u128)bh * p.nseg + (u128)bh) * rec * sizeof(float);
  // a workspace beyond half the address space cannot exist: report it as 0
  p.ws_bytes = ws > (u128)(SIZE_MAX / 2) ? 0 : (size_t)((ws + 255) / 256 * 256);
  return p;
}

bool supported(int d, int rank) {
  return (d == 16 || d == 32 || d == 64 || d == 128) && rank >= 1 && rank <= 3;
}

bool overlaps(const void* a, const void* b, size_t n) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + n && y < x + n;
}
// [a, a + na) and [b, b + nb) share a byte
bool overlaps2(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

int validate(const void* q, const void* k, const void* v, void* out, int B, int H, int N,
             int d, int band_k, int rank, int causal, const float* w_near, const float* w_far,
             int dtype, int far_norm) {
  if (!q || !k || !v || !out || !w_near || !w_far) return FMM_ERR_INVALID_ARG;
  if (B < 1 || H < 1 || N < 1 || d < 1 || band_k < 0) return FMM_ERR_INVALID_ARG;
  if (causal != 0 && causal != 1) return FMM_ERR_INVALID_ARG;
  if (far_norm != FMM_FAR_NORM_PER_MAP && far_norm != FMM_FAR_NORM_JOINT)
    return FMM_ERR_INVALID_ARG;
  if (dtype != FMM_DTYPE_F32 && dtype != FMM_DTYPE_BF16) return FMM_ERR_UNSUPPORTED;
  if (!supported(d, rank)) return FMM_ERR_UNSUPPORTED;
  const size_t es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  // sizes in 128-bit arithmetic: four positive ints cannot overflow it
  typedef unsigned __int128 u128;
  const u128 bytes128 = (u128)(unsigned)B * (unsigned)H * (unsigned)N * (unsigned)d * es;
  if (bytes128 > (u128)INT64_MAX) return FMM_ERR_INVALID_ARG;
  // slices are counted in int by the launchers; grids are checked before launch
  if ((long long)B * H > INT32_MAX) return FMM_ERR_UNSUPPORTED;
  for (const void* p : {q, k, v, (const void*)out})
    if ((uintptr_t)p % 16) return FMM_ERR_INVALID_ARG;
  if ((uintptr_t)w_near % 4 || (uintptr_t)w_far % 4) return FMM_ERR_INVALID_ARG;
  const size_t bytes = (size_t)bytes128;
  if (overlaps(out, q, bytes) || overlaps(out, k, bytes) || overlaps(out, v, bytes))
    return FMM_ERR_INVALID_ARG;
  return FMM_OK;
}

// ------------------------------------------------------------------ timing
struct EventTimer : fmm::LaunchTimer {
  std::mutex mu;
  bool enabled = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending[FMM_KERNEL_COUNT];
  std::vector<hipEvent_t> pool;

  hipEvent_t take_one() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  bool take(int, hipEvent_t* start, hipEvent_t* stop) override {
    if (!enabled) return false;
    *start = take_one();
    *stop = take_one();
    if (*start && *stop) return true;
    if (*start) pool.push_back(*start);
    if (*stop) pool.push_back(*stop);
    return false;
  }
  void commit(int kernel, hipEvent_t start, hipEvent_t stop) override {
    pending[kernel].push_back({start, stop});
  }
};

EventTimer& timer() {
  static EventTimer* t = new EventTimer();
  return *t;
}

// ------------------------------------------------------------------ workspace
struct WsEntry {
  void* ptr = nullptr;
  size_t bytes = 0;
};

std::mutex& ws_mutex() {
  static std::mutex* m = new std::mutex();
  return *m;
}
std::map<std::pair<int, void*>, WsEntry>& ws_map() {
  static auto* m = new std::map<std::pair<int, void*>, WsEntry>();
  return *m;
}

size_t ws_limit() {
  const char* s = getenv("FMM_ATTN_WS_LIMIT");
  if (!s || !*s) return (size_t)-1;
  return (size_t)strtoull(s, nullptr, 10);
}

// Returns a workspace of at least `bytes` for (current device, stream).  The
// caller holds ws_mutex() until its kernels are enqueued, so no other thread
// can free the buffer between this lookup and the launches that use it.
// keep: the caller can do with less, so a failure leaves the present buffer.
int acquire_ws_locked(void* stream, size_t bytes, void** out, bool keep = false) {
  if (bytes > ws_limit()) return FMM_ERR_OOM;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return FMM_ERR_HIP;
  WsEntry& e = ws_map()[{dev, stream}];
  if (e.bytes < bytes) {
    // a stream under graph capture can neither allocate nor synchronise: its
    // workspace has to come from an earlier call outside the capture
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &cs) != hipSuccess) {
      (void)hipGetLastError();
      return FMM_ERR_HIP;
    }
    if (cs != hipStreamCaptureStatusNone) return FMM_ERR_UNSUPPORTED;
    void* p = nullptr;
    if (keep && hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      return FMM_ERR_OOM;
    }
    if (e.ptr) {
      // kernels enqueued earlier on this stream may still read the old buffer
      if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) {
        if (p) (void)hipFree(p);
        return FMM_ERR_HIP;
      }
      (void)hipFree(e.ptr);
      e.ptr = nullptr;
      e.bytes = 0;
    }
    if (!p && hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      return FMM_ERR_OOM;
    }
    e.ptr = p;
    e.bytes = bytes;
  }
  *out = e.ptr;
  return FMM_OK;
}

// Runs f(lean) with the preferred plan, then, where its workspace was not to be
// had (the limit, the device's memory, the caller's buffer, or a capture that
// finds a smaller one), with the leanest: what the shorter segments took is no
// reason to refuse a call.  f returns FMM_ERR_OOM, or FMM_ERR_UNSUPPORTED, only
// before it has enqueued anything.
template <typename F> int preferred_or_lean(F f) {
  const int st = f(false);
  return st == FMM_ERR_OOM || st == FMM_ERR_UNSUPPORTED ? f(true) : st;
}

// The dry pass over the launch sequence: grid limits and LDS limits, nothing
// enqueued.  Runs before any workspace is acquired.
int check_launch(const fmm::LaunchArgs& a) {
  EventTimer& t = timer();
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher dry;
  dry.timer = &t;
  dry.dry = true;
  if (fmm::launch_forward(a, dry) != hipSuccess)
    return dry.err == hipErrorInvalidConfiguration ? FMM_ERR_UNSUPPORTED : FMM_ERR_HIP;
  return FMM_OK;
}

// Enqueues the launch sequence (after check_launch passed).
int launch_now(const fmm::LaunchArgs& a) {
  EventTimer& t = timer();
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher L;
  L.timer = &t;
  return fmm::launch_forward(a, L) == hipSuccess ? FMM_OK : FMM_ERR_HIP;
}

// ------------------------------------------------------------------ one-launch path
// Mode: 0 never, 1 wherever it applies (default), 2 wherever it applies but
// with every workgroup forming its slice's state itself (no exchange).
std::atomic<int>& one_launch_mode() {
  static std::atomic<int> m{1};
  return m;
}

// Epochs of the one-launch path's stamps (56 bits, formed on the device): this
// call's number in bits 32-55, from a random start, and in bits 0-31 a random
// per-process offset to which each launch adds its dispatch id.  Eager calls
// differ in the call number, replays of a captured graph (frozen arguments)
// in the dispatch id; the random parts make a match with stale stamps left in
// memory by another process unlikely.
unsigned long long next_epoch() {
  static const unsigned long long offset = [] {
    std::random_device rd;
    return (unsigned long long)rd();
  }();
  static std::atomic<unsigned long long> n{[] {
    std::random_device rd;
    return (unsigned long long)rd();
  }()};
  const unsigned long long c = n.fetch_add(1, std::memory_order_relaxed) & 0xffffffull;
  return (c << 32) | (offset & 0xffffffffull);
}

// Workgroups of k_band_fused that fit on the current device at once (two per CU).
int resident_fused_workgroups() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  if (dev >= 0 && dev < 64) {
    const int c = cache[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  if (dev >= 0 && dev < 64) cache[dev].store(2 * cus, std::memory_order_relaxed);
  return 2 * cus;
}

fmm::LaunchArgs make_args(const void* q, const void* k, const void* v, void* out, int B, int H,
                          int N, int d, int band_k, int rank, int causal, const float* w_near,
                          const float* w_far, int dtype, int far_norm, void* ws, const Plan& p,
                          void* stream) {
  fmm::LaunchArgs a;
  a.far_norm = far_norm;
  a.q = q;
  a.k = k;
  a.v = v;
  a.out = out;
  a.w_near = w_near;
  a.w_far = w_far;
  a.B = B;
  a.H = H;
  a.N = N;
  a.d = d;
  // a half-width of N already covers every key; clamping keeps row +/- k in int range
  a.band_k = band_k < N ? band_k : N;
  a.rank = rank;
  a.causal = causal;
  a.dtype = dtype;
  a.stream = stream;
  a.ws = (float*)ws;
  a.nseg = p.nseg;
  a.L = p.L;
  a.nseg_apply = p.nseg_apply;
  a.L_apply = p.L_apply;
  const int mode = one_launch_mode().load(std::memory_order_relaxed);
  if (p.fused_g > 0 && mode != 0 && far_norm == FMM_FAR_NORM_PER_MAP &&
      (long long)B * H * p.fused_g <= resident_fused_workgroups()) {
    a.fused_g = p.fused_g;
    a.exchange = mode == 2 ? 0 : 1;
    a.epoch = next_epoch();
  }
  return a;
}

// Adds the one-launch path's workspace to a plan (the larger of the two).
void add_fused(Plan& p, long long bh, int G, int d, int rank) {
  p.fused_g = G;
  if (G <= 0 || p.ws_bytes == 0) return;
  const size_t f = fmm::fused_layout(bh, G, (long long)rank * d * (d + 1)).total;
  if (f > p.ws_bytes) p.ws_bytes = f;
}

// lean: the plan of the smallest workspace (segment_rows), for where the
// preferred one's is not to be had.
Plan plan_for(int B, int H, int N, int d, int band_k, int rank, int causal, int dtype,
              bool lean = false) {
  const int kc = band_k < N ? band_k : N;
  const int apply_tm = fmm::band_pair_applies(dtype, d, kc, causal, N) ? fmm::pair_tile_rows()
                                                                    : fmm::tile_rows();
  const int es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  const long long bh = (long long)B * H;
  // one workgroup per CU where the records fit the fixed array of the
  // no-allocation call (so that it takes every shape that it took).  Whole
  // causal calls, us with quarter records -> so: bf16, 2 slices of 3000 rows at
  // d = 64 36.9 -> 20.6; 2 of 16000 at d = 128 242 -> 88; fp32, 2 of 5000 at
  // d = 64, rank 2 97.8 -> 45.6
  const long long rec = (long long)rank * d * (d + 1) * (long long)sizeof(float);
  const long long fit = (long long)fmm_attn_noalloc_max_bytes() / rec / bh - 1;
  const long long base = segment_rows(bh, N, d, rank, es);
  long long most = std::min(slice_segments(causal, d, rank, es, false), fit);
  // narrow heads, one or two maps: less than twice the workspace (so that half
  // of what fmm_attn_workspace_bytes states is never enough); it holds back
  // fp32, d = 32, rank 2 on a few slices only (2 of 5000 27 us, 19.5 with four
  // times the records, 35 with the longest segments)
  if (d <= 32 && rank <= 2) most = std::min(most, 2 * ((N + base - 1) / base));
  // the causal walk of three maps fits twice on a CU (as in the backward; bf16,
  // 32 slices of 4000 rows at d = 64: 256 workgroups 131 us, 512 100; 8 of 5000
  // at d = 32: 216 35, 320 31); those of one or two gain nothing from a second
  // round
  // (non-causal only the state kernel walks segments: with narrow heads and one
  // or two maps most calls take as long either way, the best gain 5 %)
  const bool same = !causal && d <= 32 && rank <= 2;
  const long long rows = lean || same ? base
                         : causal && rank == 3
                             ? one_or_two_rows(bh, N, d, rank, es, most, es == 2 ? 14 : 17)
                             : fill_rows(bh, N, d, rank, es, kCUs, most);
  Plan p = make_plan(B, H, N, d, rank, rows, apply_tm);
  add_fused(p, bh, fmm::fused_groups(dtype, d, kc, rank, causal, bh, N, kFusedPlanWorkgroups), d,
            rank);
  return p;
}


int run_plan(const void* q, const void* k, const void* v, void* out, int B, int H, int N, int d,
             int band_k, int rank, int causal, const float* w_near, const float* w_far,
             int dtype, int far_norm, void* ws, size_t ws_bytes, bool own_ws, void* stream,
             bool lean) {
  int st = validate(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype,
                    far_norm);
  if (st != FMM_OK) return st;
  const Plan p = plan_for(B, H, N, d, band_k, rank, causal, dtype, lean);
  if (p.ws_bytes == 0) return FMM_ERR_UNSUPPORTED;
  fmm::LaunchArgs a = make_args(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far,
                                dtype, far_norm, nullptr, p, stream);
  st = check_launch(a);
  if (st != FMM_OK) return st;
  std::unique_lock<std::mutex> ws_lock(ws_mutex(), std::defer_lock);
  if (own_ws) {
    ws_lock.lock();
    st = acquire_ws_locked(stream, p.ws_bytes, &ws, !lean);
    if (st != FMM_OK) return st;
  } else {
    if (!ws || (uintptr_t)ws % 256) return FMM_ERR_INVALID_ARG;
    if (ws_bytes < p.ws_bytes) return FMM_ERR_OOM;
  }
  a.ws = (float*)ws;
  return launch_now(a);
}

int run(const void* q, const void* k, const void* v, void* out, int B, int H, int N, int d,
        int band_k, int rank, int causal, const float* w_near, const float* w_far, int dtype,
        int far_norm, void* ws, size_t ws_bytes, bool own_ws, void* stream) {
  return preferred_or_lean([&](bool lean) {
    return run_plan(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype,
                    far_norm, ws, ws_bytes, own_ws, stream, lean);
  });
}

// ------------------------------------------------------------------ backward
struct BwdPlan {
  Plan p;
  int nwalk, Lwalk;  // row segments of the row and key passes
  size_t off_dpart, off_rowstat, off_rowfar, off_dwpart, total;
};

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Workspace of the backward pass: the forward state records (as the forward
// plan), the dS records of the same shape, per-row softmax statistics and far
// quotients, and per-segment blend sums.  0 when it cannot exist.  lean: as
// plan_for.
BwdPlan bwd_plan(int B, int H, int N, int d, int rank, int causal, int dtype,
                 bool lean = false) {
  BwdPlan b;
  // One workgroup per CU as in the forward, or two where the shorter walk makes
  // up for it: two rounds cost 1.6 (causal bf16, two workgroups on a CU), 1.7
  // (causal fp32) or 2.1 times one (non-causal: only the state kernels walk
  // segments).  bf16 causal, d = 64, backward alone: 32 slices of 4000
  // rows, rank 2, 224 workgroups of 576 rows 156 us, 256 of 512 144, 512 of 256
  // 133; 8 of 9000, rank 1, 232 of 320 81, 376 of 192 75.  fp32, rank 2, 8 of
  // 9000: 232 of 320 266 us, 376 of 192 319
  const int es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  // (causal, three maps at d = 64: one workgroup per CU, 32 slices of 4000 rows
  // 370 us with 512 workgroups, 336 with 256)
  const int round2 = !causal ? 21 : rank == 3 && d == 64 ? 20 : es == 2 ? 16 : 17;
  const long long bh = (long long)B * H;
  b.p = make_plan(B, H, N, d, rank,
                  lean ? segment_rows(bh, N, d, rank, es)
                       : one_or_two_rows(bh, N, d, rank, es,
                                         slice_segments(causal, d, rank, es, true), round2),
                  fmm::tile_rows());
  // the causal walks start from their segment's prefix (suffix) record; the
  // non-causal ones need only the slice's totals and take the apply split of
  // about two workgroups per CU (row / key pass, us: rank 3, 16 slices of 4001
  // rows, 144 -> 512 workgroups and two per CU 41.7 / 28.6 -> 20.0 / 14.4;
  // fp32, 64 slices of 1024 rows, 384 -> 512 workgroups 54.9 / 40.1 ->
  // 41.4 / 32.5)
  b.nwalk = causal || lean ? b.p.nseg : b.p.nseg_apply;
  b.Lwalk = causal || lean ? b.p.L : b.p.L_apply;
  b.total = 0;
  if (b.p.ws_bytes == 0) return b;
  typedef unsigned __int128 u128;
  const u128 bhn = (u128)B * H * N;
  const u128 rowstat = (u128)align256((size_t)std::min<u128>(bhn * 12, SIZE_MAX / 8));
  const u128 rowfar = (u128)align256((size_t)std::min<u128>(bhn * rank * 8, SIZE_MAX / 8));
  const u128 dwp = align256((size_t)bh * b.nwalk * 8);
  const u128 tot = 2 * (u128)b.p.ws_bytes + rowstat + rowfar + dwp;
  if (tot > (u128)(SIZE_MAX / 4)) return b;
  b.off_dpart = b.p.ws_bytes;
  b.off_rowstat = 2 * b.p.ws_bytes;
  b.off_rowfar = b.off_rowstat + (size_t)rowstat;
  b.off_dwpart = b.off_rowfar + (size_t)rowfar;
  b.total = (size_t)tot;
  return b;
}

void fill_bwd_args(fmm::BwdArgs& a, const BwdPlan& bp, void* ws, int B, int H) {
  const uintptr_t w = reinterpret_cast<uintptr_t>(ws);
  const size_t rec = (size_t)a.rank * a.d * (a.d + 1);
  const size_t fin_off = (size_t)B * H * bp.p.nseg * rec * sizeof(float);
  a.part = reinterpret_cast<float*>(w);
  a.fin = reinterpret_cast<float*>(w + fin_off);
  a.dpart = reinterpret_cast<float*>(w + bp.off_dpart);
  a.dfin = reinterpret_cast<float*>(w + bp.off_dpart + fin_off);
  a.rowstat = reinterpret_cast<float*>(w + bp.off_rowstat);
  a.rowfar = reinterpret_cast<float*>(w + bp.off_rowfar);
  a.dwpart = reinterpret_cast<float*>(w + bp.off_dwpart);
  a.nwalk = bp.nwalk;
  a.Lwalk = bp.Lwalk;
}

int run_backward(const void* q, const void* k, const void* v, const void* dout, void* dq,
                 void* dk, void* dv, float* dw_near, float* dw_far, int B, int H, int N, int d,
                 int band_k, int rank, int causal, const float* w_near, const float* w_far,
                 int dtype, int far_norm, void* stream, bool lean) {
  // the inputs as in the forward (dout takes the place of out for the checks)
  int st = validate(q, k, v, dq, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype,
                    far_norm);
  if (st != FMM_OK) return st;
  if (!dout || !dk || !dv || !dw_near || !dw_far) return FMM_ERR_INVALID_ARG;
  const size_t es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  const size_t bytes = (size_t)B * H * N * d * es;  // fits: validate checked it
  for (const void* p : {dout, (const void*)dk, (const void*)dv})
    if ((uintptr_t)p % 16) return FMM_ERR_INVALID_ARG;
  if ((uintptr_t)dw_near % 4 || (uintptr_t)dw_far % 4) return FMM_ERR_INVALID_ARG;
  // gradients overlap neither the inputs nor one another
  const void* ins[4] = {q, k, v, dout};
  void* outs[3] = {dq, dk, dv};
  for (void* o : outs)
    for (const void* i : ins)
      if (overlaps(o, i, bytes)) return FMM_ERR_INVALID_ARG;
  if (overlaps(dq, dk, bytes) || overlaps(dq, dv, bytes) || overlaps(dk, dv, bytes))
    return FMM_ERR_INVALID_ARG;
  if (overlaps(dw_near, dw_far, (size_t)H * 4)) return FMM_ERR_INVALID_ARG;
  const BwdPlan bp = bwd_plan(B, H, N, d, rank, causal, dtype, lean);
  if (bp.total == 0) return FMM_ERR_UNSUPPORTED;
  fmm::LaunchArgs fa = make_args(q, k, v, dq, B, H, N, d, band_k, rank, causal, w_near, w_far,
                                 dtype, FMM_FAR_NORM_PER_MAP, nullptr, bp.p, stream);
  fmm::BwdArgs ba;
  ba.q = q;
  ba.k = k;
  ba.v = v;
  ba.dout = dout;
  ba.dq = dq;
  ba.dk = dk;
  ba.dv = dv;
  ba.dw_near = dw_near;
  ba.dw_far = dw_far;
  ba.w_near = w_near;
  ba.w_far = w_far;
  ba.B = B;
  ba.H = H;
  ba.N = N;
  ba.d = d;
  ba.band_k = fa.band_k;
  ba.rank = rank;
  ba.causal = causal;
  ba.dtype = dtype;
  ba.far_norm = far_norm;
  ba.stream = stream;
  ba.nseg = bp.p.nseg;
  ba.L = bp.p.L;
  fill_bwd_args(ba, bp, nullptr, B, H);
  EventTimer& t = timer();
  {
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher dry;
    dry.timer = &t;
    dry.dry = true;
    if (fmm::launch_state_only(fa, dry) != hipSuccess ||
        fmm::launch_backward_tail(ba, dry) != hipSuccess)
      return dry.err == hipErrorInvalidConfiguration ? FMM_ERR_UNSUPPORTED : FMM_ERR_HIP;
  }
  std::lock_guard<std::mutex> wl(ws_mutex());
  void* ws = nullptr;
  st = acquire_ws_locked(stream, bp.total, &ws, !lean);
  if (st != FMM_OK) return st;
  fa.ws = (float*)ws;
  fill_bwd_args(ba, bp, ws, B, H);
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher L;
  L.timer = &t;
  if (fmm::launch_state_only(fa, L) != hipSuccess) return FMM_ERR_HIP;
  return fmm::launch_backward_tail(ba, L) == hipSuccess ? FMM_OK : FMM_ERR_HIP;
}

// ------------------------------------------------------------------ layer
std::mutex& blas_mutex() {
  static std::mutex* m = new std::mutex();
  return *m;
}

// rocBLAS handle of the current device (created once per device).
void* blas_handle() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  static std::map<int, void*>* handles = new std::map<int, void*>();
  void*& h = (*handles)[dev];
  if (!h) h = fmm::layer_blas_handle_create();
  return h;
}

int run_layer(const void* x, const void* w_qkv, const void* w_out, void* y, int B, int N, int E,
              int H, int band_k, int rank, int causal, const float* w_near, const float* w_far,
              int dtype, void* stream, bool lean) {
  if (!x || !w_qkv || !w_out || !y || !w_near || !w_far) return FMM_ERR_INVALID_ARG;
  if (B < 1 || N < 1 || E < 1 || H < 1 || band_k < 0 || E % H) return FMM_ERR_INVALID_ARG;
  if (causal != 0 && causal != 1) return FMM_ERR_INVALID_ARG;
  if (dtype != FMM_DTYPE_F32 && dtype != FMM_DTYPE_BF16) return FMM_ERR_UNSUPPORTED;
  const int d = E / H;
  if (!supported(d, rank)) return FMM_ERR_UNSUPPORTED;
  const size_t es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  typedef unsigned __int128 u128;
  const u128 tokens = (u128)B * N;
  if (tokens > (u128)INT32_MAX || (u128)3 * E > (u128)INT32_MAX) return FMM_ERR_UNSUPPORTED;
  const u128 xbytes = tokens * E * es;
  if (xbytes * 8 > (u128)INT64_MAX) return FMM_ERR_INVALID_ARG;
  for (const void* p : {x, w_qkv, w_out, (const void*)y})
    if ((uintptr_t)p % 16) return FMM_ERR_INVALID_ARG;
  if ((uintptr_t)w_near % 4 || (uintptr_t)w_far % 4) return FMM_ERR_INVALID_ARG;
  const size_t xb = (size_t)xbytes, wq = (size_t)E * 3 * E * es, wo = (size_t)E * E * es;
  if (overlaps2(y, xb, x, xb) || overlaps2(y, xb, w_qkv, wq) || overlaps2(y, xb, w_out, wo))
    return FMM_ERR_INVALID_ARG;
  // workspace: the heads q, k, v and their outputs o, around rocBLAS products
  // also qkv and the merged heads m, then the operator's records
  const Plan p = plan_for(B, H, N, d, band_k, rank, causal, dtype, lean);
  if (p.ws_bytes == 0) return FMM_ERR_UNSUPPORTED;
  const bool own_proj = fmm::layer_proj_applies(E);
  const size_t seg = align256(xb);
  const size_t off_q = 0, off_k = seg, off_v = 2 * seg, off_o = 3 * seg, off_qkv = 4 * seg,
               off_m = 7 * seg, off_ws = own_proj ? 4 * seg : 8 * seg;
  const size_t total = off_ws + p.ws_bytes;
  auto at = [](void* base, size_t off) {
    return reinterpret_cast<void*>(reinterpret_cast<uintptr_t>(base) + off);
  };
  fmm::LaunchArgs a = make_args(at(nullptr, off_q), at(nullptr, off_k), at(nullptr, off_v),
                                at(nullptr, off_o), B, H, N, d, band_k, rank, causal, w_near,
                                w_far, dtype, FMM_FAR_NORM_PER_MAP, nullptr, p, stream);
  int st = check_launch(a);
  if (st != FMM_OK) return st;
  {
    EventTimer& t = timer();
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher dry;
    dry.timer = &t;
    dry.dry = true;
    // (the dry passes record their result in dry.err)
    if (own_proj) {
      for (fmm::LayerProj m : {fmm::LayerProj::kQkv, fmm::LayerProj::kOut})
        (void)fmm::launch_layer_proj(dry, m, dtype, nullptr, nullptr, nullptr, nullptr, nullptr,
                                     nullptr, nullptr, B, N, H, d, (hipStream_t)stream);
    } else {
      (void)fmm::launch_layer_copy(dry, true, dtype, nullptr, nullptr, nullptr, nullptr, B, N, H,
                                   d, (hipStream_t)stream);
      (void)fmm::launch_layer_copy(dry, false, dtype, nullptr, nullptr, nullptr, nullptr, B, N,
                                   H, d, (hipStream_t)stream);
    }
    if (dry.err != hipSuccess)
      return dry.err == hipErrorInvalidConfiguration ? FMM_ERR_UNSUPPORTED : FMM_ERR_HIP;
  }
  std::unique_lock<std::mutex> bl(blas_mutex(), std::defer_lock);
  void* hdl = nullptr;  // (the library's own products need none)
  if (!own_proj) {
    bl.lock();
    hdl = blas_handle();
    if (!hdl) return FMM_ERR_HIP;
  }
  std::lock_guard<std::mutex> wl(ws_mutex());
  void* ws = nullptr;
  st = acquire_ws_locked(stream, total, &ws, !lean);
  if (st != FMM_OK) return st;
  a.q = at(ws, off_q);
  a.k = at(ws, off_k);
  a.v = at(ws, off_v);
  a.out = at(ws, off_o);
  a.ws = (float*)at(ws, off_ws);
  const int M = B * N;
  if (own_proj) {
    EventTimer& t = timer();
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher L;
    L.timer = &t;
    if (fmm::launch_layer_proj(L, fmm::LayerProj::kQkv, dtype, x, nullptr, nullptr, w_qkv,
                               at(ws, off_q), at(ws, off_k), at(ws, off_v), B, N, H, d,
                               (hipStream_t)stream) != hipSuccess ||
        fmm::launch_forward(a, L) != hipSuccess ||
        fmm::launch_layer_proj(L, fmm::LayerProj::kOut, dtype, at(ws, off_o), nullptr, nullptr,
                               w_out, y, nullptr, nullptr, B, N, H, d,
                               (hipStream_t)stream) != hipSuccess)
      return FMM_ERR_HIP;
    return FMM_OK;
  }
  if (fmm::layer_gemm(hdl, stream, dtype, x, w_qkv, at(ws, off_qkv), M, E, 3 * E) != hipSuccess)
    return FMM_ERR_HIP;
  EventTimer& t = timer();
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher L;
  L.timer = &t;
  if (fmm::launch_layer_copy(L, true, dtype, at(ws, off_qkv), at(ws, off_q), at(ws, off_k),
                             at(ws, off_v), B, N, H, d, (hipStream_t)stream) != hipSuccess ||
      fmm::launch_forward(a, L) != hipSuccess ||
      fmm::launch_layer_copy(L, false, dtype, at(ws, off_o), at(ws, off_m), nullptr, nullptr, B,
                             N, H, d, (hipStream_t)stream) != hipSuccess)
    return FMM_ERR_HIP;
  if (fmm::layer_gemm(hdl, stream, dtype, at(ws, off_m), w_out, y, M, E, E) != hipSuccess)
    return FMM_ERR_HIP;
  return FMM_OK;
}

// Backward of the layer: the forward recomputed through the projections (this
// library's kernels or rocBLAS, as in the forward) and the operator: the heads
// q, k, v and their outputs o; then dm = dy W_out^T, dW_out = m^T dy, the
// operator's backward for the heads' share of dm, dx = dqkv W_qkv^T and dW_qkv
// = x^T dqkv with dqkv = [dq | dk | dv] per token.
int run_layer_backward(const void* x, const void* w_qkv, const void* w_out, const void* dy,
                       void* dx, void* dw_qkv, void* dw_out, float* dw_near, float* dw_far,
                       int B, int N, int E, int H, int band_k, int rank, int causal,
                       const float* w_near, const float* w_far, int dtype, void* stream, bool lean) {
  if (!x || !w_qkv || !w_out || !dy || !dx || !dw_qkv || !dw_out || !dw_near || !dw_far ||
      !w_near || !w_far)
    return FMM_ERR_INVALID_ARG;
  if (B < 1 || N < 1 || E < 1 || H < 1 || band_k < 0 || E % H) return FMM_ERR_INVALID_ARG;
  if (causal != 0 && causal != 1) return FMM_ERR_INVALID_ARG;
  if (dtype != FMM_DTYPE_F32 && dtype != FMM_DTYPE_BF16) return FMM_ERR_UNSUPPORTED;
  const int d = E / H;
  if (!supported(d, rank)) return FMM_ERR_UNSUPPORTED;
  const size_t es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  typedef unsigned __int128 u128;
  const u128 tokens = (u128)B * N;
  if (tokens > (u128)INT32_MAX || (u128)3 * E > (u128)INT32_MAX) return FMM_ERR_UNSUPPORTED;
  const u128 xbytes = tokens * E * es;
  if (xbytes * 16 > (u128)INT64_MAX) return FMM_ERR_INVALID_ARG;
  for (const void* p : {x, w_qkv, w_out, dy, (const void*)dx, (const void*)dw_qkv,
                        (const void*)dw_out})
    if ((uintptr_t)p % 16) return FMM_ERR_INVALID_ARG;
  if ((uintptr_t)w_near % 4 || (uintptr_t)w_far % 4 || (uintptr_t)dw_near % 4 ||
      (uintptr_t)dw_far % 4)
    return FMM_ERR_INVALID_ARG;
  const size_t xb = (size_t)xbytes, wq = (size_t)E * 3 * E * es, wo = (size_t)E * E * es;
  // outputs overlap neither the inputs nor one another
  const void* ins[4] = {x, w_qkv, w_out, dy};
  const size_t in_b[4] = {xb, wq, wo, xb};
  void* outs[3] = {dx, dw_qkv, dw_out};
  const size_t out_b[3] = {xb, wq, wo};
  for (int o = 0; o < 3; ++o) {
    for (int i = 0; i < 4; ++i)
      if (overlaps2(outs[o], out_b[o], ins[i], in_b[i])) return FMM_ERR_INVALID_ARG;
    for (int o2 = o + 1; o2 < 3; ++o2)
      if (overlaps2(outs[o], out_b[o], outs[o2], out_b[o2])) return FMM_ERR_INVALID_ARG;
  }
  if (overlaps(dw_near, dw_far, (size_t)H * 4)) return FMM_ERR_INVALID_ARG;
  const bool own_proj = fmm::layer_proj_applies(E);
  // workspace: the heads q, k, v, their outputs o and the gradients do, dq, dk,
  // dv, around rocBLAS products also qkv (later dqkv), m and dm, then the
  // forward operator's and the backward's records and the weight gradients'
  // chunks
  const Plan p = plan_for(B, H, N, d, band_k, rank, causal, dtype, lean);
  const BwdPlan bp = bwd_plan(B, H, N, d, rank, causal, dtype, lean);
  if (p.ws_bytes == 0 || bp.total == 0) return FMM_ERR_UNSUPPORTED;
  const size_t seg = align256(xb);
  const size_t off_q = 0, off_k = seg, off_v = 2 * seg, off_o = 3 * seg, off_do = 4 * seg,
               off_dq = 5 * seg, off_dk = 6 * seg, off_dv = 7 * seg, off_qkv = 8 * seg,
               off_m = 11 * seg, off_dm = 12 * seg, off_fws = own_proj ? 8 * seg : 13 * seg,
               off_bws = off_fws + align256(p.ws_bytes),
               off_wg = off_bws + align256(bp.total);
  const int Mtok = B * N;  // fits: checked above
  const size_t total =
      off_wg + align256(fmm::layer_wgrad_scratch_bytes(Mtok, E, 3 * E, lean));
  auto at = [](void* base, size_t off) {
    return reinterpret_cast<void*>(reinterpret_cast<uintptr_t>(base) + off);
  };
  fmm::LaunchArgs a = make_args(at(nullptr, off_q), at(nullptr, off_k), at(nullptr, off_v),
                                at(nullptr, off_o), B, H, N, d, band_k, rank, causal, w_near,
                                w_far, dtype, FMM_FAR_NORM_PER_MAP, nullptr, p, stream);
  int st = check_launch(a);
  if (st != FMM_OK) return st;
  fmm::LaunchArgs fa = make_args(at(nullptr, off_q), at(nullptr, off_k), at(nullptr, off_v),
                                 at(nullptr, off_dq), B, H, N, d, band_k, rank, causal, w_near,
                                 w_far, dtype, FMM_FAR_NORM_PER_MAP, nullptr, bp.p, stream);
  fmm::BwdArgs ba;
  ba.q = at(nullptr, off_q);
  ba.k = at(nullptr, off_k);
  ba.v = at(nullptr, off_v);
  ba.dout = at(nullptr, off_do);
  ba.dq = at(nullptr, off_dq);
  ba.dk = at(nullptr, off_dk);
  ba.dv = at(nullptr, off_dv);
  ba.dw_near = dw_near;
  ba.dw_far = dw_far;
  ba.w_near = w_near;
  ba.w_far = w_far;
  ba.B = B;
  ba.H = H;
  ba.N = N;
  ba.d = d;
  ba.band_k = fa.band_k;
  ba.rank = rank;
  ba.causal = causal;
  ba.dtype = dtype;
  ba.stream = stream;
  ba.nseg = bp.p.nseg;
  ba.L = bp.p.L;
  fill_bwd_args(ba, bp, nullptr, B, H);
  hipStream_t s = (hipStream_t)stream;
  {
    EventTimer& t = timer();
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher dry;
    dry.timer = &t;
    dry.dry = true;
    if (own_proj) {
      for (fmm::LayerProj m : {fmm::LayerProj::kQkv, fmm::LayerProj::kDm, fmm::LayerProj::kDx})
        (void)fmm::launch_layer_proj(dry, m, dtype, nullptr, nullptr, nullptr, nullptr, nullptr,
                                     nullptr, nullptr, B, N, H, d, s);
      for (bool qkv : {false, true})
        (void)fmm::launch_layer_wgrad(dry, dtype, qkv, nullptr, nullptr, nullptr, nullptr,
                                      nullptr, nullptr, B, N, H, d, s, lean);
    } else {
      (void)fmm::launch_layer_copy(dry, true, dtype, nullptr, nullptr, nullptr, nullptr, B, N, H,
                                   d, s);
      (void)fmm::launch_layer_copy(dry, false, dtype, nullptr, nullptr, nullptr, nullptr, B, N,
                                   H, d, s);
      (void)fmm::launch_layer_split1(dry, dtype, nullptr, nullptr, B, N, H, d, s);
      (void)fmm::launch_layer_merge_part(dry, dtype, nullptr, nullptr, 0, B, N, H, d, s);
    }
    if (dry.err == hipSuccess) (void)fmm::launch_state_only(fa, dry);
    if (dry.err == hipSuccess) (void)fmm::launch_backward_tail(ba, dry);
    if (dry.err == hipSuccess && !own_proj)
      (void)fmm::layer_wgrad(nullptr, dry, stream, dtype, nullptr, nullptr, nullptr, Mtok, E,
                             3 * E, nullptr);
    if (dry.err != hipSuccess)
      return dry.err == hipErrorInvalidConfiguration ? FMM_ERR_UNSUPPORTED : FMM_ERR_HIP;
  }
  std::unique_lock<std::mutex> bl(blas_mutex(), std::defer_lock);
  void* hdl = nullptr;  // (the library's own products need none)
  if (!own_proj) {
    bl.lock();
    hdl = blas_handle();
    if (!hdl) return FMM_ERR_HIP;
  }
  std::lock_guard<std::mutex> wl(ws_mutex());
  void* ws = nullptr;
  st = acquire_ws_locked(stream, total, &ws, !lean);
  if (st != FMM_OK) return st;
  a.q = ba.q = at(ws, off_q);
  a.k = ba.k = at(ws, off_k);
  a.v = ba.v = at(ws, off_v);
  a.out = at(ws, off_o);
  a.ws = (float*)at(ws, off_fws);
  fa.q = a.q;
  fa.k = a.k;
  fa.v = a.v;
  fa.ws = (float*)at(ws, off_bws);
  ba.dout = at(ws, off_do);
  ba.dq = at(ws, off_dq);
  ba.dk = at(ws, off_dk);
  ba.dv = at(ws, off_dv);
  fill_bwd_args(ba, bp, at(ws, off_bws), B, H);
  const int M = B * N;
  EventTimer& t = timer();
  if (own_proj) {
    // the forward up to the heads' outputs o, their gradient and dW_out, the
    // operator's backward, then dx and dW_qkv
    float* wgs = reinterpret_cast<float*>(at(ws, off_wg));
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher L;
    L.timer = &t;
    if (fmm::launch_layer_proj(L, fmm::LayerProj::kQkv, dtype, x, nullptr, nullptr, w_qkv,
                               at(ws, off_q), at(ws, off_k), at(ws, off_v), B, N, H, d, s) !=
            hipSuccess ||
        fmm::launch_forward(a, L) != hipSuccess ||
        fmm::launch_layer_proj(L, fmm::LayerProj::kDm, dtype, dy, nullptr, nullptr, w_out,
                               at(ws, off_do), nullptr, nullptr, B, N, H, d, s) != hipSuccess ||
        fmm::launch_layer_wgrad(L, dtype, false, a.out, dy, nullptr, nullptr, dw_out, wgs, B, N,
                                H, d, s, lean) != hipSuccess ||
        fmm::launch_state_only(fa, L) != hipSuccess ||
        fmm::launch_backward_tail(ba, L) != hipSuccess ||
        fmm::launch_layer_proj(L, fmm::LayerProj::kDx, dtype, ba.dq, ba.dk, ba.dv, w_qkv, dx,
                               nullptr, nullptr, B, N, H, d, s) != hipSuccess)
      return FMM_ERR_HIP;
    return fmm::launch_layer_wgrad(L, dtype, true, x, ba.dq, ba.dk, ba.dv, dw_qkv, wgs, B, N, H,
                                   d, s, lean) == hipSuccess
               ? FMM_OK
               : FMM_ERR_HIP;
  }
  // the forward: qkv, the heads, the operator, the merged rows
  if (fmm::layer_gemm(hdl, stream, dtype, x, w_qkv, at(ws, off_qkv), M, E, 3 * E) != hipSuccess)
    return FMM_ERR_HIP;
  {
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher L;
    L.timer = &t;
    if (fmm::launch_layer_copy(L, true, dtype, at(ws, off_qkv), at(ws, off_q), at(ws, off_k),
                               at(ws, off_v), B, N, H, d, s) !=
            hipSuccess ||
        fmm::launch_forward(a, L) != hipSuccess ||
        fmm::launch_layer_copy(L, false, dtype, a.out, at(ws, off_m), nullptr, nullptr, B, N, H,
                               d, s) != hipSuccess)
      return FMM_ERR_HIP;
  }
  // dm = dy W_out^T, dW_out = m^T dy
  float* wg = reinterpret_cast<float*>(at(ws, off_wg));
  if (fmm::layer_gemm(hdl, stream, dtype, dy, w_out, at(ws, off_dm), M, E, E, false, true) !=
      hipSuccess)
    return FMM_ERR_HIP;
  {
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher L;
    L.timer = &t;
    if (fmm::layer_wgrad(hdl, L, stream, dtype, at(ws, off_m), dy, dw_out, M, E, E, wg) !=
        hipSuccess)
      return FMM_ERR_HIP;
  }
  // the operator's backward on the heads' share of dm, then dqkv per token
  {
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher L;
    L.timer = &t;
    if (fmm::launch_layer_split1(L, dtype, at(ws, off_dm), at(ws, off_do), B, N, H, d, s) !=
            hipSuccess ||
        fmm::launch_state_only(fa, L) != hipSuccess ||
        fmm::launch_backward_tail(ba, L) != hipSuccess ||
        fmm::launch_layer_merge_part(L, dtype, ba.dq, at(ws, off_qkv), 0, B, N, H, d, s) !=
            hipSuccess ||
        fmm::launch_layer_merge_part(L, dtype, ba.dk, at(ws, off_qkv), 1, B, N, H, d, s) !=
            hipSuccess ||
        fmm::launch_layer_merge_part(L, dtype, ba.dv, at(ws, off_qkv), 2, B, N, H, d, s) !=
            hipSuccess)
      return FMM_ERR_HIP;
  }
  // dx = dqkv W_qkv^T, dW_qkv = x^T dqkv
  if (fmm::layer_gemm(hdl, stream, dtype, at(ws, off_qkv), w_qkv, dx, M, 3 * E, E, false,
                      true) != hipSuccess)
    return FMM_ERR_HIP;
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher L;
  L.timer = &t;
  return fmm::layer_wgrad(hdl, L, stream, dtype, x, at(ws, off_qkv), dw_qkv, M, E, 3 * E, wg) ==
                 hipSuccess
             ? FMM_OK
             : FMM_ERR_HIP;
}

// ------------------------------------------------------------------ fast weight
// level: 0 the preferred plan, 1 the leanest of the operator, then passes of
// half the chunks each time.  *last: a further level would take no less.
int run_fastweight(const void* q, const void* k, const void* v, const float* beta, void* out,
                   int B, int H, int N, int d, int band_k, int n_linear, const float* w_near,
                   const float* w_far, int dtype, void* stream, int level, bool* last) {
  *last = true;
  int st = validate(q, k, v, out, B, H, N, d, band_k, 1, 1, w_near, w_far, dtype,
                    FMM_FAR_NORM_PER_MAP);
  if (st != FMM_OK) return st;
  if (!beta || (uintptr_t)beta % 4 || (n_linear != 0 && n_linear != 1))
    return FMM_ERR_INVALID_ARG;
  const Plan p = plan_for(B, H, N, d, band_k, 1, 1, dtype, level > 0);
  if (p.ws_bytes == 0) return FMM_ERR_UNSUPPORTED;
  // the operator's records, then H floats of -inf that remove its linear far
  // part when n_linear = 0; once its kernels have run, the fast-weight kernels'
  // chunks in the same place
  const long long bh = (long long)B * H;
  const size_t pass = level < 2 ? fmm::kFwPassBytes
                                : fmm::fw_forward_bytes(bh, N, d, fmm::kFwPassBytes) >>
                                      std::min(level - 1, 60);
  const fmm::FwPlan fp = fmm::fw_plan(bh, N, d, pass);
  *last = level > 0 && fp.slices == 1 && fp.chunks == 1;
  const size_t total = std::max(p.ws_bytes + align256((size_t)H * 4),
                                align256(fmm::fw_forward_bytes(bh, N, d, pass)));
  fmm::LaunchArgs a = make_args(q, k, v, out, B, H, N, d, band_k, 1, 1, w_near, w_far, dtype,
                                FMM_FAR_NORM_PER_MAP, nullptr, p, stream);
  fmm::FwArgs f;
  f.q = q;
  f.k = k;
  f.v = v;
  f.beta = beta;
  f.out = out;
  f.w_far = w_far;
  f.B = B;
  f.H = H;
  f.N = N;
  f.d = d;
  f.dtype = dtype;
  f.stream = stream;
  f.pass_bytes = pass;
  f.ws = nullptr;
  EventTimer& t = timer();
  {
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher dry;
    dry.timer = &t;
    dry.dry = true;
    if (fmm::launch_forward(a, dry) != hipSuccess ||
        fmm::launch_fast_weight(dry, f) != hipSuccess)
      return dry.err == hipErrorInvalidConfiguration ? FMM_ERR_UNSUPPORTED : FMM_ERR_HIP;
  }
  std::lock_guard<std::mutex> wl(ws_mutex());
  void* ws = nullptr;
  st = acquire_ws_locked(stream, total, &ws, !*last);
  if (st != FMM_OK) return st;
  a.ws = (float*)ws;
  float* minus_inf =
      reinterpret_cast<float*>(reinterpret_cast<uintptr_t>(ws) + p.ws_bytes);
  f.ws = (float*)ws;
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher L;
  L.timer = &t;
  if (!n_linear) {
    if (fmm::launch_fill(L, minus_inf, H, -INFINITY, stream) != hipSuccess) return FMM_ERR_HIP;
    a.w_far = minus_inf;
  }
  if (fmm::launch_forward(a, L) != hipSuccess) return FMM_ERR_HIP;
  return fmm::launch_fast_weight(L, f) == hipSuccess ? FMM_OK : FMM_ERR_HIP;
}

// Backward of the fast-weight operator: the operator's backward at rank 1,
// causal (the near field, and the linear far part when n_linear = 1; with
// n_linear = 0 its far part is removed by -inf logits), then the fast-weight
// kernel, which adds its gradients to dq, dk, dv, writes dbeta and adds its
// share to dw_far.
int run_backward_fastweight(const void* q, const void* k, const void* v, const float* beta,
                            const void* dout, void* dq, void* dk, void* dv, float* dbeta,
                            float* dw_near, float* dw_far, int B, int H, int N, int d,
                            int band_k, int n_linear, const float* w_near, const float* w_far,
                            int dtype, void* stream, bool lean) {
  int st = validate(q, k, v, dq, B, H, N, d, band_k, 1, 1, w_near, w_far, dtype,
                    FMM_FAR_NORM_PER_MAP);
  if (st != FMM_OK) return st;
  if (!dout || !dk || !dv || !dw_near || !dw_far || !beta || !dbeta) return FMM_ERR_INVALID_ARG;
  if (n_linear != 0 && n_linear != 1) return FMM_ERR_INVALID_ARG;
  const size_t es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
  const size_t bytes = (size_t)B * H * N * d * es;  // fits: validate checked it
  for (const void* p : {dout, (const void*)dk, (const void*)dv})
    if ((uintptr_t)p % 16) return FMM_ERR_INVALID_ARG;
  if ((uintptr_t)dw_near % 4 || (uintptr_t)dw_far % 4 || (uintptr_t)beta % 4 ||
      (uintptr_t)dbeta % 4)
    return FMM_ERR_INVALID_ARG;
  const void* ins[4] = {q, k, v, dout};
  void* outs[3] = {dq, dk, dv};
  for (void* o : outs)
    for (const void* i : ins)
      if (overlaps(o, i, bytes)) return FMM_ERR_INVALID_ARG;
  if (overlaps(dq, dk, bytes) || overlaps(dq, dv, bytes) || overlaps(dk, dv, bytes))
    return FMM_ERR_INVALID_ARG;
  const size_t nb = (size_t)B * H * N * 4;
  for (const void* o : {(const void*)dq, (const void*)dk, (const void*)dv})
    if (overlaps2(dbeta, nb, o, bytes)) return FMM_ERR_INVALID_ARG;
  if (overlaps2(dbeta, nb, beta, nb) || overlaps(dw_near, dw_far, (size_t)H * 4))
    return FMM_ERR_INVALID_ARG;
  const BwdPlan bp = bwd_plan(B, H, N, d, 1, 1, dtype, lean);
  if (bp.total == 0) return FMM_ERR_UNSUPPORTED;
  // the backward's workspace and H floats of -inf, then, once its kernels have
  // run, the fast-weight kernels' chunks in the same place
  typedef unsigned __int128 u128;
  const u128 tot = std::max((u128)bp.total + align256((size_t)H * 4),
                            fmm::fw_backward_bytes((long long)B * H, N, d));
  if (tot > (u128)(SIZE_MAX / 4)) return FMM_ERR_UNSUPPORTED;
  const size_t off_m = bp.total;
  fmm::LaunchArgs fa = make_args(q, k, v, dq, B, H, N, d, band_k, 1, 1, w_near, w_far, dtype,
                                 FMM_FAR_NORM_PER_MAP, nullptr, bp.p, stream);
  fmm::BwdArgs ba;
  ba.q = q;
  ba.k = k;
  ba.v = v;
  ba.dout = dout;
  ba.dq = dq;
  ba.dk = dk;
  ba.dv = dv;
  ba.dw_near = dw_near;
  ba.dw_far = dw_far;
  ba.w_near = w_near;
  ba.w_far = w_far;
  ba.B = B;
  ba.H = H;
  ba.N = N;
  ba.d = d;
  ba.band_k = fa.band_k;
  ba.rank = 1;
  ba.causal = 1;
  ba.dtype = dtype;
  ba.stream = stream;
  ba.nseg = bp.p.nseg;
  ba.L = bp.p.L;
  fill_bwd_args(ba, bp, nullptr, B, H);
  fmm::FwBwdArgs fb;
  fb.q = q;
  fb.k = k;
  fb.v = v;
  fb.beta = beta;
  fb.dout = dout;
  fb.dq = dq;
  fb.dk = dk;
  fb.dv = dv;
  fb.dbeta = dbeta;
  fb.dw_far = dw_far;
  fb.w_far = w_far;
  fb.ws = nullptr;
  fb.B = B;
  fb.H = H;
  fb.N = N;
  fb.d = d;
  fb.dtype = dtype;
  fb.stream = stream;
  EventTimer& t = timer();
  {
    std::lock_guard<std::mutex> g(t.mu);
    fmm::Launcher dry;
    dry.timer = &t;
    dry.dry = true;
    if (fmm::launch_state_only(fa, dry) != hipSuccess ||
        fmm::launch_backward_tail(ba, dry) != hipSuccess ||
        fmm::launch_fast_weight_backward(dry, fb) != hipSuccess)
      return dry.err == hipErrorInvalidConfiguration ? FMM_ERR_UNSUPPORTED : FMM_ERR_HIP;
  }
  std::lock_guard<std::mutex> wl(ws_mutex());
  void* ws = nullptr;
  st = acquire_ws_locked(stream, (size_t)tot, &ws, !lean);
  if (st != FMM_OK) return st;
  const uintptr_t w = reinterpret_cast<uintptr_t>(ws);
  fa.ws = (float*)ws;
  fill_bwd_args(ba, bp, ws, B, H);
  fb.ws = (float*)ws;
  float* minus_inf = reinterpret_cast<float*>(w + off_m);
  std::lock_guard<std::mutex> g(t.mu);
  fmm::Launcher L;
  L.timer = &t;
  if (!n_linear) {
    if (fmm::launch_fill(L, minus_inf, H, -INFINITY, stream) != hipSuccess) return FMM_ERR_HIP;
    fa.w_far = minus_inf;
    ba.w_far = minus_inf;
  }
  if (fmm::launch_state_only(fa, L) != hipSuccess) return FMM_ERR_HIP;
  if (fmm::launch_backward_tail(ba, L) != hipSuccess) return FMM_ERR_HIP;
  return fmm::launch_fast_weight_backward(L, fb) == hipSuccess ? FMM_OK : FMM_ERR_HIP;
}

}  // namespace

namespace fmm {

int validate_forward(const void* q, const void* k, const void* v, void* out, int B, int H,
                     int N, int d, int band_k, int rank, int causal, const float* w_near,
                     const float* w_far, int dtype) {
  return validate(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype,
                  FMM_FAR_NORM_PER_MAP);
}

size_t forward_workspace_bytes(int B, int H, int N, int d, int band_k, int rank, int causal,
                               int dtype) {
  return plan_for(B, H, N, d, band_k, rank, causal, dtype).ws_bytes;
}

int forward_with_workspace(const void* q, const void* k, const void* v, void* out, int B, int H,
                           int N, int d, int band_k, int rank, int causal, const float* w_near,
                           const float* w_far, int dtype, void* ws, size_t ws_bytes,
                           void* stream) {
  return run(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype,
             FMM_FAR_NORM_PER_MAP, ws, ws_bytes, false, stream);
}

}  // namespace fmm

extern "C" {

int fmm_attn_forward(const void* q, const void* k, const void* v, void* out, int B, int H,
                     int N, int d, int band_k, int rank, int causal, const float* w_near,
                     const float* w_far, void* stream) {
  return run(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, FMM_DTYPE_F32,
             FMM_FAR_NORM_PER_MAP, nullptr, 0, true, stream);
}

int fmm_attn_forward_bf16(const void* q, const void* k, const void* v, void* out, int B, int H,
                          int N, int d, int band_k, int rank, int causal, const float* w_near,
                          const float* w_far, void* stream) {
  return run(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, FMM_DTYPE_BF16,
             FMM_FAR_NORM_PER_MAP, nullptr, 0, true, stream);
}

int fmm_attn_forward_ex(const void* q, const void* k, const void* v, void* out, int B, int H,
                        int N, int d, int band_k, int rank, int causal, const float* w_near,
                        const float* w_far, int dtype, int far_norm, void* stream) {
  return run(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype, far_norm,
             nullptr, 0, true, stream);
}

int fmm_attn_backward(const void* q, const void* k, const void* v, const void* dout, void* dq,
                      void* dk, void* dv, float* dw_near, float* dw_far, int B, int H, int N,
                      int d, int band_k, int rank, int causal, const float* w_near,
                      const float* w_far, int dtype, void* stream) {
  return fmm_attn_backward_ex(q, k, v, dout, dq, dk, dv, dw_near, dw_far, B, H, N, d, band_k,
                              rank, causal, w_near, w_far, dtype, FMM_FAR_NORM_PER_MAP, stream);
}

int fmm_attn_backward_ex(const void* q, const void* k, const void* v, const void* dout,
                         void* dq, void* dk, void* dv, float* dw_near, float* dw_far, int B,
                         int H, int N, int d, int band_k, int rank, int causal,
                         const float* w_near, const float* w_far, int dtype, int far_norm,
                         void* stream) {
  return preferred_or_lean([&](bool lean) {
    return run_backward(q, k, v, dout, dq, dk, dv, dw_near, dw_far, B, H, N, d, band_k, rank,
                        causal, w_near, w_far, dtype, far_norm, stream, lean);
  });
}

int fmm_attn_layer_backward(const void* x, const void* w_qkv, const void* w_out, const void* dy,
                            void* dx, void* dw_qkv, void* dw_out, float* dw_near, float* dw_far,
                            int B, int N, int E, int H, int band_k, int rank, int causal,
                            const float* w_near, const float* w_far, int dtype, void* stream) {
  return preferred_or_lean([&](bool lean) {
    return run_layer_backward(x, w_qkv, w_out, dy, dx, dw_qkv, dw_out, dw_near, dw_far, B, N, E,
                              H, band_k, rank, causal, w_near, w_far, dtype, stream, lean);
  });
}

int fmm_attn_backward_fastweight(const void* q, const void* k, const void* v, const float* beta,
                                 const void* dout, void* dq, void* dk, void* dv, float* dbeta,
                                 float* dw_near, float* dw_far, int B, int H, int N, int d,
                                 int band_k, int n_linear, const float* w_near,
                                 const float* w_far, int dtype, void* stream) {
  return preferred_or_lean([&](bool lean) {
    return run_backward_fastweight(q, k, v, beta, dout, dq, dk, dv, dbeta, dw_near, dw_far, B, H,
                                   N, d, band_k, n_linear, w_near, w_far, dtype, stream, lean);
  });
}

int fmm_attn_layer_forward(const void* x, const void* w_qkv, const void* w_out, void* y, int B,
                           int N, int E, int H, int band_k, int rank, int causal,
                           const float* w_near, const float* w_far, int dtype, void* stream) {
  return preferred_or_lean([&](bool lean) {
    return run_layer(x, w_qkv, w_out, y, B, N, E, H, band_k, rank, causal, w_near, w_far, dtype,
                     stream, lean);
  });
}

int fmm_attn_forward_fastweight(const void* q, const void* k, const void* v, const float* beta,
                                void* out, int B, int H, int N, int d, int band_k, int n_linear,
                                const float* w_near, const float* w_far, int dtype,
                                void* stream) {
  bool last = false;
  for (int level = 0;; ++level) {
    const int st = run_fastweight(q, k, v, beta, out, B, H, N, d, band_k, n_linear, w_near, w_far,
                                  dtype, stream, level, &last);
    if (last || (st != FMM_ERR_OOM && st != FMM_ERR_UNSUPPORTED)) return st;
  }
}

size_t fmm_attn_workspace_bytes(int B, int H, int N, int d, int rank, int causal) {
  if (B < 1 || H < 1 || N < 1 || (causal != 0 && causal != 1) || !supported(d, rank)) return 0;
  // the plan depends on the element size only through the segment length
  // floor; report the larger of the two dtypes' needs
  // (and, at any band the one-launch path takes, through its layout)
  const Plan a = plan_for(B, H, N, d, 0, rank, causal, FMM_DTYPE_BF16),
             b = plan_for(B, H, N, d, 0, rank, causal, FMM_DTYPE_F32);
  return a.ws_bytes > b.ws_bytes ? a.ws_bytes : b.ws_bytes;
}

int fmm_attn_set_one_launch(int mode) {
  if (mode < 0 || mode > 2) return -1;
  return one_launch_mode().exchange(mode);
}

int fmm_attn_forward_ws(const void* q, const void* k, const void* v, void* out, int B, int H,
                        int N, int d, int band_k, int rank, int causal, const float* w_near,
                        const float* w_far, int dtype, void* workspace, size_t ws_bytes,
                        void* stream) {
  return run(q, k, v, out, B, H, N, d, band_k, rank, causal, w_near, w_far, dtype,
             FMM_FAR_NORM_PER_MAP, workspace, ws_bytes, false, stream);
}

const char* fmm_attn_status_string(int status) {
  switch (status) {
    case FMM_OK: return "FMM_OK: success";
    case FMM_ERR_INVALID_ARG:
      return "FMM_ERR_INVALID_ARG: null, negative, misaligned or overlapping argument";
    case FMM_ERR_UNSUPPORTED:
      return "FMM_ERR_UNSUPPORTED: d must be 16, 32, 64 or 128 and rank 1, 2 or 3, within the "
             "dispatch limits";
    case FMM_ERR_HIP: return "FMM_ERR_HIP: a HIP runtime call or kernel launch failed";
    case FMM_ERR_OOM: return "FMM_ERR_OOM: workspace allocation failed or workspace too small";
    case FMM_ERR_SCRATCH:
      return "FMM_ERR_SCRATCH: the shape needs more scratch than the fixed no-allocation array";
    default: return "unknown fmm_attn status";
  }
}

void fmm_attn_release_workspace(void) {
  std::lock_guard<std::mutex> g(ws_mutex());
  int cur = 0;
  const bool have_cur = hipGetDevice(&cur) == hipSuccess;
  for (auto& kv : ws_map()) {
    if (!kv.second.ptr) continue;
    (void)hipSetDevice(kv.first.first);
    (void)hipDeviceSynchronize();
    (void)hipFree(kv.second.ptr);
  }
  ws_map().clear();
  if (have_cur) (void)hipSetDevice(cur);
}

int fmm_attn_version(void) { return kVersion; }

int fmm_attn_kernel_timing(int enable) {
  EventTimer& t = timer();
  std::lock_guard<std::mutex> g(t.mu);
  t.enabled = enable != 0;
  return FMM_OK;
}

int fmm_attn_kernel_timing_read(int kernel, double* total_ms, long long* launches) {
  if (kernel < 0 || kernel >= FMM_KERNEL_COUNT || !total_ms || !launches)
    return FMM_ERR_INVALID_ARG;
  EventTimer& t = timer();
  std::lock_guard<std::mutex> g(t.mu);
  double sum = 0.0;
  long long n = 0;
  int st = FMM_OK;
  for (auto& pr : t.pending[kernel]) {
    float ms = 0.f;
    if (hipEventSynchronize(pr.second) != hipSuccess ||
        hipEventElapsedTime(&ms, pr.first, pr.second) != hipSuccess)
      st = FMM_ERR_HIP;
    sum += ms;
    ++n;
    t.pool.push_back(pr.first);
    t.pool.push_back(pr.second);
  }
  t.pending[kernel].clear();
  *total_ms = sum;
  *launches = n;
  return st;
}

}  // extern "C"

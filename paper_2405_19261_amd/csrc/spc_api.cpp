// spc_api.cpp -- the C interface of libspeccascade (declared in
// include/speccascade.h): argument checks, workspace, kernel dispatch.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "spc_internal.h"

namespace {

thread_local std::string g_err;

spc_status fail(spc_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// The internal workspace of each device.  A buffer that had to grow is kept
// (not freed) until spc_release: kernels already enqueued, or captured in a
// graph, may still refer to it.
struct DevWorkspace {
  void* ptr = nullptr;
  size_t bytes = 0;
  std::vector<void*> retired;
};
std::mutex g_ws_mu;
std::map<int, DevWorkspace> g_ws;

std::mutex g_cu_mu;
std::map<int, int> g_cus;

// Compute units of device dev, read once per device; 0 on failure.
int cu_count(int dev) {
  std::lock_guard<std::mutex> lk(g_cu_mu);
  auto it = g_cus.find(dev);
  if (it != g_cus.end()) return it->second;
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) n = 0;
  if (n > 0) g_cus[dev] = n;
  return n;
}

int64_t stat_tiles(int dtype, int64_t V) {
  const int64_t n = spc::stat_tile_elems(dtype);
  return (V + n - 1) / n;
}

// Sequences per launch: whole sequences, at most kMaxRows rows (the
// statistics grid is tiles x rows; a row of V < 2^31 entries has fewer than
// 2^31 tiles).
int64_t seqs_per_launch(int64_t B, int64_t gamma) {
  return std::max<int64_t>(1, std::min(B, spc::kMaxRows / (gamma + 1)));
}

}  // namespace

namespace spc {

WsLayout ws_layout(int64_t B, int64_t gamma, int64_t V, int dtype) {
  // The zero region (job counter lines, per-row lines) has the same size
  // and offset for every shape, so one zeroed workspace serves calls of any
  // shape it is large enough for; launches leave it as found.
  const int64_t R = B * (gamma + 1);
  const int64_t nt = stat_tiles(dtype, V);
  WsLayout L;
  size_t o = 0;
  L.hdr = o;
  o = align_up(o + 4 * (size_t)(kHdrLines * kLineWords), 256);
  L.rowline = o;
  o = align_up(o + 4 * (size_t)(kMaxRows * kLineWords), 256);
  L.zero_end = o;
  // the job pass's list: a slice of every tile for TV or eta (a row has one
  // kind)
  L.jobs = o; o = align_up(o + 8 * (size_t)(R * nt * kSlices), 256);
  L.tiles = o; o = align_up(o + sizeof(TilePart) * R * nt, 256);
  L.tvpart = o; o = align_up(o + sizeof(double) * R * nt * kSlices, 256);
  // residual sub-chunk masses per sequence, or (small path) two sets per row
  L.submass = o;
  o = align_up(o + sizeof(double) * std::max<int64_t>(B * nt * tile_subchunks(dtype),
                                                       R * 2 * kSmallSub), 256);
  L.moms = o; o = align_up(o + sizeof(TileMom) * R * nt, 256);
  L.rowstat = o; o = align_up(o + sizeof(RowStat) * R, 256);
  L.rowdec = o; o = align_up(o + sizeof(int32_t) * R, 256);
  L.etalist = o; o = align_up(o + sizeof(int32_t) * R * nt, 256);
  L.etacnt = o; o = align_up(o + sizeof(int32_t) * R, 256);
  L.total = o;
  return L;
}

}  // namespace spc

namespace {

// Bound of a statistics workgroup's wait for a TV row's merge, in ticks of
// the 100 MHz real-time clock: 4000 (40 us).  SPC_TV_WAIT_TICKS overrides it
// (read at every call); a test sets 0 so that every wait gives up at once
// and the rows' merges take the tiles.
uint32_t tv_wait_ticks() {
  const char* e = getenv("SPC_TV_WAIT_TICKS");
  if (!e || !*e) return 4000u;
  char* end = nullptr;
  const unsigned long v = strtoul(e, &end, 10);
  return (end && *end == '\0' && v <= 1000000ul) ? (uint32_t)v : 4000u;
}

spc_status check_shape(int32_t B, int32_t gamma, int32_t V) {
  if (B < 1 || gamma < 1 || gamma > SPC_MAX_GAMMA || V < 2)
    return fail(SPC_E_SHAPE, "bad shape B=%d gamma=%d V=%d (need B>=1, 1<=gamma<=%d, V>=2)", B,
                gamma, V, SPC_MAX_GAMMA);
  return SPC_OK;
}

// The layout of one launch of a verify call of this shape.
spc::WsLayout launch_layout(int32_t B, int32_t gamma, int32_t V, int dtype) {
  return spc::ws_layout(seqs_per_launch(B, gamma), gamma, V, dtype);
}

bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return st != hipStreamCaptureStatusNone;
}

// The internal workspace of the current device, at least `bytes` long.  A
// new buffer has its zero region cleared on `stream` before any kernel that
// uses it; that cannot be recorded into a graph, so a call being captured
// that would need a larger buffer fails instead (make one eager call of the
// largest shape first, or pass a caller workspace).
spc_status internal_workspace(size_t bytes, size_t zero_bytes, hipStream_t stream, char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(SPC_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  std::lock_guard<std::mutex> lk(g_ws_mu);
  DevWorkspace& w = g_ws[dev];
  if (w.bytes < bytes) {
    if (capturing(stream))
      return fail(SPC_E_WORKSPACE,
                  "the internal workspace must grow to %zu bytes, which a stream capture cannot "
                  "record: make an eager call of this shape first, or pass a workspace",
                  bytes);
    const size_t want = bytes + bytes / 4;  // headroom for nearby shapes
    void* ptr = nullptr;
    e = hipMalloc(&ptr, want);
    if (e != hipSuccess) return fail(SPC_E_HIP, "hipMalloc(%zu): %s", want, hipGetErrorString(e));
    // zero the counters, ordered before this call's kernels on the same stream
    e = hipMemsetAsync(ptr, 0, zero_bytes, stream);
    if (e != hipSuccess) {
      (void)hipFree(ptr);
      return fail(SPC_E_HIP, "hipMemsetAsync: %s", hipGetErrorString(e));
    }
    if (w.ptr) w.retired.push_back(w.ptr);
    w.ptr = ptr;
    w.bytes = want;
  }
  *out = static_cast<char*>(w.ptr);
  return SPC_OK;
}

// Static scratch of spc_verify_noalloc: each device that runs it holds its
// own copy until the process ends.  Host code never uses the array's name as
// an address: noalloc_scratch looks up the device address once per device.
constexpr size_t kNoAllocBytes = size_t(32) << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];

struct NoAllocDev {
  void* ptr = nullptr;  // the device address of `scratch` on this device
  bool cleared = false; // its counter region zeroed by a fill kernel
};
std::mutex g_na_mu;
std::map<int, NoAllocDev> g_na;

// Sequences per launch that the static scratch holds for this row shape
// (0: not even one).
int64_t noalloc_seqs(int64_t gamma, int64_t V, int dtype) {
  const size_t one = spc::ws_layout(1, gamma, V, dtype).total;
  if (one > kNoAllocBytes) return 0;
  int64_t lo = 1, hi = spc::kMaxRows;  // largest b with layout(b) <= the scratch
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) / 2;
    if (spc::ws_layout(mid, gamma, V, dtype).total <= kNoAllocBytes) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The static scratch of device `dev` (the current device).  The first call
// on a device looks up its address and clears its counter region with a
// fill kernel on `stream`; the kernels leave that region zero after every
// call, so later calls find it cleared.  Nothing here allocates.
spc_status noalloc_scratch(int dev, size_t zero_bytes, hipStream_t stream, char** out) {
  std::lock_guard<std::mutex> lk(g_na_mu);
  NoAllocDev& d = g_na[dev];
  if (!d.ptr) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(SPC_E_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    d.ptr = ptr;
  }
  if (!d.cleared) {
    const hipError_t e = spc::launch_fill_zero(d.ptr, zero_bytes, stream);
    if (e != hipSuccess) return fail(SPC_E_HIP, "clearing the scratch: %s", hipGetErrorString(e));
    d.cleared = true;
  }
  *out = static_cast<char*>(d.ptr);
  return SPC_OK;
}

template <class T>
T* offset(T* p, int64_t n) {
  return p ? p + n : p;
}

// Rules by what they need of a row besides its maxima and normalisers.
constexpr uint32_t kAllRules = (1u << (SPC_RULE_OPTLOG + 1)) - 1u;
constexpr uint32_t kTvRules = (1u << SPC_RULE_OPT) | (1u << SPC_RULE_OPTLOG);
constexpr uint32_t kLogRules = (1u << SPC_RULE_BILD) | (1u << SPC_RULE_CHOWLOG) |
                               (1u << SPC_RULE_DIFFLOG) | (1u << SPC_RULE_OPTLOG);
constexpr uint32_t kTokRules = (1u << SPC_RULE_TOKEN_V1) | (1u << SPC_RULE_TOKEN_V2) |
                               (1u << SPC_RULE_TOKEN_V3);

struct Route {
  bool seq = false, small = false;  // the one-launch paths; neither: statistics tiles
  bool tv_self = false, tv_pass = false, tv_jobs = false, job_pass = false, pair = false;
  int mom_set = 0;  // first moments the statistics sum (kMom* bits)
};

// What a batch may ask of its rows.
struct Work {
  bool tv, tok, mom;  // D_TV, eta, first moments
  bool greedy;        // temperature 0 throughout
  bool mixed;         // rules per sequence: only some rows ask for it
};

// Whether a launch of B sequences takes the one-launch path with a workgroup
// per sequence (k_seq).  Its time grows with a sequence's gamma + 1 rows of ns
// sub-chunks (one compute unit reads them) and with the rounds of workgroups;
// the other paths' with the rows of the batch.  us per step, that path / the
// next best one (rows held by a workgroup, or statistics tiles), on 256
// compute units:
//   rows within the compute units, gamma = 4:
//     Diff bf16 V=2000 10.9 / 10.9, V=2560 12.9 / 10.8; f32 V=1000 9.6 / 10.5,
//     V=1501 11.5 / 10.2; greedy bf16 V=1001 7.7 / 8.3, V=1501 8.8 / 8.3; OPT
//     bf16 V=500 11.7 / 11.7, V=1501 14.9 / 11.7; TokenV2 bf16 V=1000 14.9 /
//     15.0, V=1501 17.1 / 15.6; CHOW, Diff and OPT mixed bf16 V=813 gamma=3
//     11.1 / 13.0; DiffLog bf16 gamma=1 V=1192 11.4 / 12.9, gamma=5 V=1800
//     13.9 / 12.2; OPTLog bf16 gamma=1 V=1600 13.6 / 13.2
//   one round, more rows: Diff bf16 B=256 gamma=7 V=4000 22 / 33; OPT bf16 B=40
//     gamma=7 V=2000 14.2 / 17.3, V=2560 19.9 / 17.6; greedy f32 B=64 gamma=4
//     V=1001 8.6 / 10.8, V=2560 10.8 / 9.9, gamma=3 V=3001 9.4 / 10.2, B=125
//     V=4024 12.1 / 10.4 (bf16 10.1 / 10.7)
//   two rounds (B = 400): Diff f32 gamma=4 V=2000 22.9 / 24.8, V=4000 33 / 28;
//     DiffLog f32 gamma=1 V=2000 21.5 / 22.6, V=4000 28.5 / 23.4
//   four (B = 1024): Diff bf16 gamma=7 V=1001 39 / 65, V=2560 66 / 65; gamma=1
//     V=1501 29 / 27; TokenV2 bf16 gamma=7 V=4000 195 / 385
bool short_sequences(int64_t B, int64_t g1, int64_t V, int dtype, const Work& w, int64_t cus) {
  const bool bf16 = dtype == SPC_BF16;
  const int64_t sub = spc::seq_sub_elems(dtype), ns = (V + sub - 1) / sub;
  if (ns > spc::kSeqSubs) return false;
  const int64_t n = g1 * V, rows = B * g1, rounds = (B + cus - 1) / cus;
  const bool four = ns <= 4;
  if (rows <= cus) {
    if (w.mom) return n <= (w.tv ? 3072 : w.greedy ? 4096 : bf16 ? 6144 : 4608);
    if (w.greedy) return n <= 4096 || (V <= 1024 && n <= 8192);
    if (w.tok || (w.tv && w.mixed)) return n <= 4096;
    if (w.tv) return g1 * ns <= 4;
    return g1 * ns <= 16 || (four && g1 * ns <= 32);
  }
  if (rounds == 1) {
    if (w.mom) return n <= (bf16 ? 32768 : rows > 2 * cus ? 20480 : 16384);
    if (w.greedy)
      return n <= 20480 && (four || g1 <= 2 || (g1 <= 4 && n <= (bf16 ? 16384 : 12288)) ||
                            rows > 4 * cus || (rows > 2 * cus && n <= 10240));
    if (w.tok) return n <= 40960;
    if (w.tv) return n <= 20480 && (g1 <= 5 || rows > 2 * cus || n <= (bf16 ? 16384 : 10240));
    return n <= 40960;
  }
  if (rounds == 2) {
    if (w.mom) return ns <= 8 && n <= 32768;
    if (w.greedy) return four && n <= 20480 && (g1 >= 4 || ns <= 2);
    if (w.tok) return n <= 40960;
    if (w.tv) return ns <= 12 && n <= 20480;
    return ns <= 8 && n <= 40960;
  }
  if (w.mom) return n <= 32768 && four && (g1 >= 4 || (bf16 && ns <= 3));
  if (w.greedy) return n <= 20480 && four && g1 >= 4;
  if (w.tok) return n <= 40960 && V <= 6400;
  return n <= 40960 && four && (g1 >= 4 || (bf16 && ns <= 2));
}

// Whether a launch of other sizes takes the one-launch path with a workgroup
// per row (k_small), whose rows fit a workgroup's registers, rather than
// statistics tiles and the passes after them: up to two rows per compute unit.
// us per step, as rows / as tiles:
//   rows within the compute units: Diff bf16 V=18565 17.6 / 18.4, V=22992 18.9 /
//     17.3 (8 to 27 rows), V=22695 19.7 / 21.7 (234 rows); OPT bf16 V=22176
//     21.4 / 22.9, V=28624 24.0 / 22.7, V=30824 25.7 / 31.0 (135 rows); TokenV2
//     V=30957 29.4 / 32.2; greedy V=8472 9.4 / 9.1, V=17848 11.6 / 9.6; DiffLog
//     bf16 V=8191 12.6 / 20.6, V=20003 19.3 / 20.7; OPTLog V=24001 22.0 / 26.5
//   more rows: Diff bf16 V=3929 19.3 / 19.9, V=5995 21.3 / 20.0, V=21355 32.7 /
//     23.2; f32 V=2584 17.9 / 17.0; OPT bf16 V=9721 28.0 / 35.3, V=16832 33.2 /
//     31.3; TokenV2 V=11264 35.5 / 42.8, V=29312 50.7 / 42.1; greedy V=1479
//     14.4 / 11.4; DiffLog V=2000 23.5 / 21.2
bool held_rows(int64_t rows, int64_t V, int64_t nt, int dtype, const Work& w, int64_t cus) {
  if (V > spc::small_row_elems(dtype) || rows > 2 * cus) return false;
  if (rows > cus) {
    if (w.greedy || w.mom) return false;
    return V <= (w.tok ? 16384 : w.tv ? 12288 : dtype == SPC_BF16 ? 4096 : 2048);
  }
  if (w.greedy) return V <= 8192;
  if (w.tok && !w.mom) return true;
  return V <= (w.tv ? 24576 : w.mom ? 16384 : 20480) || (!w.mom && rows * nt > 2 * cus);
}

// Which kernels one launch of a verify call runs, from its sizes and from the
// rules its sequences may hold (`rules`, a bitmask; `per_rule`: per-sequence
// rules).  B: sequences of the call, b_launch: the most of them in a launch,
// R: rows of this launch.  sampled: some sequence may be at temperature > 0,
// greedy: the batch is at temperature 0.
Route choose_route(int64_t B, int64_t b_launch, int64_t R, int64_t g1, int64_t V, int dtype,
                   uint32_t rules, bool per_rule, bool sampled, bool greedy, int64_t cus) {
  Route t;
  // first moments of the log-loss rules (BiLD* at temperature 0 reads one
  // logit instead): x for BiLD*, H(q) for ChowLog, H(q) and H(p) otherwise
  const bool need_mom = (rules & kLogRules) && !(rules == (1u << SPC_RULE_BILD) && greedy);
  t.mom_set = !need_mom ? 0
                        : ((rules & (1u << SPC_RULE_BILD)) ? spc::kMomX : 0) |
                              ((rules & (1u << SPC_RULE_CHOWLOG)) ? spc::kMomHQ : 0) |
                              ((rules & ((1u << SPC_RULE_DIFFLOG) | (1u << SPC_RULE_OPTLOG)))
                                   ? spc::kMomHQ | spc::kMomHP
                                   : 0);
  // Rows of OPT / OPTLOG at T > 0 are decided after their TV pass, rows of
  // a token rule after their eta pass (the job pass, for the tiles their
  // statistics leave open), every other row by its last statistics tile.
  const bool tv_rows = sampled && (rules & kTvRules);
  const bool tok_rows = sampled && (rules & kTokRules);
  const Work work{tv_rows, tok_rows, need_mom, !sampled, per_rule};
  t.seq = short_sequences(b_launch, g1, V, dtype, work, cus);
  if (t.seq) return t;
  const int64_t nt = stat_tiles(dtype, V);
  t.small = held_rows(b_launch * g1, V, nt, dtype, work, cus);
  if (t.small) return t;
  // Where TV rows get their TV pass.  In a grid that is resident at once
  // (at most two workgroups per compute unit) each TV row takes it from
  // its own tiles' registers once the row is merged (tv_self), up to the 62
  // tiles a row's gate holds.  (With more the second read is no slower: at 63,
  // float32 V = 256 000, rows that wait for 62 others, against k_tvpass:
  // gamma = 1 OPT 21.8 / 22.0 us, OPTLog 21.1 / 20.0; gamma = 7 OPT 26.9 /
  // 26.7, OPTLog 26.3 / 23.7.)  Otherwise
  // a kernel of its own reads the TV rows again after the statistics
  // kernel (k_tvpass) when the rule is batch-wide, so that most rows may
  // need it; with per-sequence rules (a few TV rows among others) their
  // slices are job-pass items (tv_jobs).
  t.tv_self = tv_rows && R * nt <= 2 * cus && nt <= spc::kTvTiles;
  // batches of at least 64 statistics tiles per compute unit stream two
  // tiles per workgroup (without first moments): B = 32 at the Gemma
  // vocabulary (32 per CU) is faster with one, B = 128 and 256 with two
  t.pair = !t.tv_self && !need_mom && R * nt >= 64 * cus;
  t.tv_jobs = tv_rows && !t.tv_self && per_rule;
  t.tv_pass = tv_rows && !t.tv_self && !t.tv_jobs;
  // the job pass: eta slices, and TV slices (tv_jobs)
  t.job_pass = tok_rows || t.tv_jobs;
  return t;
}

spc_status verify_impl(const void* q, const void* p, int32_t dtype, const int32_t* draft,
                       const float* uniforms, int32_t B, int32_t gamma, int32_t V, int32_t rule,
                       float alpha, float temperature, bool force_greedy, int32_t* out_accept,
                       int32_t* out_token, uint8_t* out_defer, const spc_verify_ex_args* ex,
                       hipStream_t stream, bool no_alloc = false) {
  g_err.clear();
  if (!q || !p || !draft || !out_accept || !out_token || !out_defer)
    return fail(SPC_E_NULL, "a required pointer is NULL");
  if (!force_greedy && !uniforms) return fail(SPC_E_NULL, "uniforms is NULL");
  spc_status st = check_shape(B, gamma, V);
  if (st != SPC_OK) return st;
  if (dtype != SPC_F32 && dtype != SPC_BF16) return fail(SPC_E_PARAM, "unknown dtype %d", dtype);
  const bool per_rule = ex && ex->rule_per_seq;
  const bool per_alpha = ex && ex->alpha_per_seq;
  const bool per_temp = ex && ex->temp_per_seq;
  if (!per_rule && (rule < SPC_RULE_CHOW || rule > SPC_RULE_OPTLOG))
    return fail(SPC_E_RULE, "unknown rule %d", rule);
  if (!per_alpha && !isfinite(alpha)) return fail(SPC_E_PARAM, "alpha is not finite");
  if (!per_rule && !per_alpha && rule == SPC_RULE_LOSSY && !(alpha < 1.0f))
    return fail(SPC_E_PARAM, "the lossy rule needs alpha < 1 (got %g)", (double)alpha);
  if (!force_greedy && !per_temp && !(isfinite(temperature) && temperature > 0.0f))
    return fail(SPC_E_PARAM, "temperature must be finite and > 0 (got %g)", (double)temperature);
  if (((uintptr_t)q | (uintptr_t)p) % 16 != 0)
    return fail(SPC_E_ALIGN, "logit base pointers must be 16-byte aligned");

  const int64_t g1 = (int64_t)gamma + 1;
  int64_t b_launch = seqs_per_launch(B, gamma);
  if (no_alloc) {
    if (ex && ex->workspace)
      return fail(SPC_E_WORKSPACE, "spc_verify_noalloc takes no caller workspace");
    // as many sequences per launch as the static scratch holds (the layout
    // grows with the sequences of a launch)
    b_launch = std::min<int64_t>(b_launch, noalloc_seqs(gamma, V, dtype));
    if (b_launch < 1)
      return fail(SPC_E_WORKSPACE,
                  "one sequence of gamma=%d V=%d needs %zu bytes of workspace, more than the "
                  "%zu-byte static scratch of spc_verify_noalloc",
                  gamma, V, spc::ws_layout(1, gamma, V, dtype).total, kNoAllocBytes);
  }
  const spc::WsLayout L = spc::ws_layout(b_launch, gamma, V, dtype);
  // argument checks end here: no HIP call precedes them
  if (ex && ex->workspace &&
      (ex->workspace_bytes < L.total || ((uintptr_t)ex->workspace % 256) != 0))
    return fail(SPC_E_WORKSPACE, "workspace of %zu bytes (need %zu, 256-byte aligned)",
                ex->workspace_bytes, L.total);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(SPC_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  const int cus = cu_count(dev);
  if (cus <= 0) return fail(SPC_E_HIP, "cannot read the compute-unit count of device %d", dev);
  char* ws = nullptr;
  if (no_alloc) {
    const spc_status wst = noalloc_scratch(dev, L.zero_end, stream, &ws);
    if (wst != SPC_OK) return wst;
  } else if (ex && ex->workspace) {
    ws = static_cast<char*>(ex->workspace);
  } else {
    const spc_status wst = internal_workspace(L.total, L.zero_end, stream, &ws);
    if (wst != SPC_OK) return wst;
  }

  // The rules the batch may hold decide what each launch computes.
  const uint32_t mask = ex ? ex->rules_present & kAllRules : 0u;
  const uint32_t rules = per_rule ? (mask ? mask : kAllRules) : (1u << rule);
  const bool may_sample = !force_greedy && (per_temp || temperature > 0.0f);
  const int64_t nt = stat_tiles(dtype, V);
  const int64_t eb = dtype == SPC_BF16 ? 2 : 4;

  for (int64_t b0 = 0; b0 < B; b0 += b_launch) {
    const int64_t bl = std::min<int64_t>(b_launch, B - b0);
    const int64_t R = bl * g1;
    spc::Params P{};
    P.q = static_cast<const char*>(q) + b0 * g1 * V * eb;
    P.p = static_cast<const char*>(p) + b0 * g1 * V * eb;
    P.draft = draft + b0 * gamma;
    P.uniforms = offset(uniforms, b0 * g1);
    P.B = (int32_t)bl;
    P.gamma = gamma;
    P.V = V;
    P.nt = (int32_t)nt;
    P.rule = rule;
    P.alpha = alpha;
    P.temp = force_greedy ? 0.0f : temperature;
    P.force_greedy = force_greedy ? 1 : 0;
    P.rule_mask = per_rule ? mask : 0u;
    P.rule_ps = per_rule ? ex->rule_per_seq + b0 : nullptr;
    P.alpha_ps = per_alpha ? ex->alpha_per_seq + b0 : nullptr;
    P.temp_ps = (per_temp && !force_greedy) ? ex->temp_per_seq + b0 : nullptr;
    P.out_accept = out_accept + b0;
    P.out_token = out_token + b0;
    P.out_defer = out_defer + b0 * g1;
    P.out_stats = ex ? offset(ex->out_row_stats, b0 * g1 * 8) : nullptr;
    P.out_argmax = ex ? offset(ex->out_argmax, b0 * g1 * 2) : nullptr;
    P.out_norm = ex ? offset(ex->out_sample_norm, b0) : nullptr;
    const Route route = choose_route(B, b_launch, R, g1, V, dtype, rules, per_rule, may_sample,
                                     force_greedy, cus);
    P.mom_set = route.mom_set;
    P.tv_self = route.tv_self ? 1 : 0;
    P.pair = route.pair ? 1 : 0;
    P.tv_jobs = route.tv_jobs ? 1 : 0;
    P.may_greedy = (force_greedy || per_temp) ? 1 : 0;
    P.wait_ticks = tv_wait_ticks();
    P.single_slots = R * nt * spc::kSlices;
    P.nsub = (int32_t)(nt * spc::tile_subchunks(dtype));
    // workgroups of the job pass: a wavefront per item of its largest
    // expected list (eta or TV slices of every tile), at most two workgroups per compute unit
    const int64_t np = nt * spc::kSlices;
    const int64_t items1 = np * (route.job_pass ? R : 0);
    constexpr int64_t kW = spc::kJobThreads / 64;
    const int job_groups = (int)std::max<int64_t>(
        1, std::min<int64_t>((items1 + kW - 1) / kW, 2 * (int64_t)cus));
    P.hdr = reinterpret_cast<uint32_t*>(ws + L.hdr);
    P.rowline = reinterpret_cast<uint32_t*>(ws + L.rowline);
    P.jobs = reinterpret_cast<uint64_t*>(ws + L.jobs);
    P.tiles = reinterpret_cast<spc::TilePart*>(ws + L.tiles);
    P.tvpart = reinterpret_cast<double*>(ws + L.tvpart);
    P.submass = reinterpret_cast<double*>(ws + L.submass);
    P.moms = reinterpret_cast<spc::TileMom*>(ws + L.moms);
    P.rowstat = reinterpret_cast<spc::RowStat*>(ws + L.rowstat);
    P.rowdec = reinterpret_cast<int32_t*>(ws + L.rowdec);
    P.etalist = reinterpret_cast<int32_t*>(ws + L.etalist);
    P.etacnt = reinterpret_cast<int32_t*>(ws + L.etacnt);
    const bool first = b0 == 0;
    hipEvent_t ev0 = first && ex ? ex->ev_tiles_begin : nullptr;
    hipEvent_t ev1 = first && ex ? ex->ev_tiles_end : nullptr;
    if (route.seq) {
      e = spc::launch_seq(P, dtype, ev0, ev1, stream);
    } else if (route.small) {
      // one launch: a workgroup per row holding the row in registers
      P.nsub = spc::kSmallSub;
      e = spc::launch_small(P, dtype, ev0, ev1, stream);
    } else {
      // sequences with a draw are drawn by the draw pass, the last kernel
      // (greedy ones write their token directly)
      e = spc::launch_step(P, dtype, may_sample, route.tv_pass, route.job_pass, job_groups, ev0, ev1,
                           stream);
    }
    if (e != hipSuccess) return fail(SPC_E_HIP, "kernel launch: %s", hipGetErrorString(e));
  }
  return SPC_OK;
}

spc_status draft_impl(const void* logits, int32_t dtype, int32_t B, int32_t V, float temperature,
                      const float* temp_per_seq, const float* uniforms, int32_t* out_token,
                      void* workspace, size_t workspace_bytes, hipStream_t stream) {
  g_err.clear();
  if (!logits || !out_token) return fail(SPC_E_NULL, "a required pointer is NULL");
  if (!temp_per_seq && !(isfinite(temperature) && temperature >= 0.0f))
    return fail(SPC_E_PARAM, "temperature must be finite and >= 0 (got %g)",
                (double)temperature);
  const bool greedy = !temp_per_seq && temperature == 0.0f;
  if (!greedy && !uniforms) return fail(SPC_E_NULL, "uniforms is NULL");
  if (B < 1 || V < 2) return fail(SPC_E_SHAPE, "bad shape B=%d V=%d (need B>=1, V>=2)", B, V);
  if (dtype != SPC_F32 && dtype != SPC_BF16) return fail(SPC_E_PARAM, "unknown dtype %d", dtype);
  if ((uintptr_t)logits % 16 != 0)
    return fail(SPC_E_ALIGN, "logit base pointer must be 16-byte aligned");
  // rows per launch, as a verify step of gamma = 1 with as many sequences
  const int64_t b_launch = seqs_per_launch(B, 1);
  const spc::WsLayout L = spc::ws_layout(b_launch, 1, V, dtype);
  // argument checks end here: no HIP call precedes them
  if (workspace && (workspace_bytes < L.total || ((uintptr_t)workspace % 256) != 0))
    return fail(SPC_E_WORKSPACE, "workspace of %zu bytes (need %zu, 256-byte aligned)",
                workspace_bytes, L.total);
  char* ws = static_cast<char*>(workspace);
  if (!ws) {
    const spc_status wst = internal_workspace(L.total, L.zero_end, stream, &ws);
    if (wst != SPC_OK) return wst;
  }
  const int64_t eb = dtype == SPC_BF16 ? 2 : 4;
  for (int64_t b0 = 0; b0 < B; b0 += b_launch) {
    const int64_t bl = std::min<int64_t>(b_launch, B - b0);
    spc::Params P{};
    P.q = static_cast<const char*>(logits) + b0 * V * eb;
    P.p = P.q;
    P.uniforms = offset(uniforms, b0);
    P.B = (int32_t)bl;
    P.gamma = 0;
    P.V = V;
    // Tiles twice as long as the statistics tiles once that still gives at
    // least 4 workgroups per CU; small batches take the statistics tile
    // length, for twice the workgroups (either way no more partials per row
    // than the workspace holds for this shape).
    const int64_t long_n = spc::draft_tile_elems(dtype, true);
    const bool long_tiles = bl * ((V + long_n - 1) / long_n) >= 1024;
    const int64_t tile_n = long_tiles ? long_n : spc::draft_tile_elems(dtype, false);
    P.nt = (int32_t)((V + tile_n - 1) / tile_n);
    P.rule = SPC_RULE_NEVER;
    P.temp = greedy ? 0.0f : temperature;
    P.force_greedy = greedy ? 1 : 0;
    P.temp_ps = offset(temp_per_seq, b0);
    P.out_token = out_token + b0;
    P.hdr = reinterpret_cast<uint32_t*>(ws + L.hdr);
    P.samp_cnt = reinterpret_cast<uint32_t*>(ws + L.rowline) + spc::kDraftArrive;
    P.tiles = reinterpret_cast<spc::TilePart*>(ws + L.tiles);
    const hipError_t e =
        spc::launch_draft(P, dtype, greedy || temp_per_seq, long_tiles, stream);
    if (e != hipSuccess) return fail(SPC_E_HIP, "kernel launch: %s", hipGetErrorString(e));
  }
  return SPC_OK;
}

}  // namespace

extern "C" {

spc_status spc_verify(const void* q_logits, const void* p_logits, int32_t dtype,
                      const int32_t* draft_tokens, const float* uniforms, int32_t B,
                      int32_t gamma, int32_t V, int32_t rule, float alpha, float temperature,
                      int32_t* out_accept_len, int32_t* out_next_token,
                      uint8_t* out_defer_mask, hipStream_t stream) {
  return verify_impl(q_logits, p_logits, dtype, draft_tokens, uniforms, B, gamma, V, rule, alpha,
                     temperature, false, out_accept_len, out_next_token, out_defer_mask,
                     nullptr, stream);
}

spc_status spc_greedy_verify(const void* q_logits, const void* p_logits, int32_t dtype,
                             const int32_t* draft_tokens, int32_t B, int32_t gamma, int32_t V,
                             int32_t rule, float alpha, int32_t* out_accept_len,
                             int32_t* out_next_token, uint8_t* out_defer_mask,
                             hipStream_t stream) {
  return verify_impl(q_logits, p_logits, dtype, draft_tokens, nullptr, B, gamma, V, rule, alpha,
                     0.0f, true, out_accept_len, out_next_token, out_defer_mask, nullptr, stream);
}

spc_status spc_verify_ex(const void* q_logits, const void* p_logits, int32_t dtype,
                         const int32_t* draft_tokens, const float* uniforms, int32_t B,
                         int32_t gamma, int32_t V, int32_t rule, float alpha, float temperature,
                         int32_t* out_accept_len, int32_t* out_next_token,
                         uint8_t* out_defer_mask, const spc_verify_ex_args* ex,
                         hipStream_t stream) {
  // a scalar temperature of exactly 0 (no per-sequence array) is the
  // batch-wide greedy step of spc_greedy_verify
  const bool greedy = !(ex && ex->temp_per_seq) && temperature == 0.0f;
  return verify_impl(q_logits, p_logits, dtype, draft_tokens, uniforms, B, gamma, V, rule, alpha,
                     temperature, greedy, out_accept_len, out_next_token, out_defer_mask, ex,
                     stream);
}

spc_status spc_verify_noalloc(const void* q_logits, const void* p_logits, int32_t dtype,
                              const int32_t* draft_tokens, const float* uniforms, int32_t B,
                              int32_t gamma, int32_t V, int32_t rule, float alpha,
                              float temperature, int32_t* out_accept_len,
                              int32_t* out_next_token, uint8_t* out_defer_mask,
                              const spc_verify_ex_args* ex, hipStream_t stream) {
  const bool greedy = !(ex && ex->temp_per_seq) && temperature == 0.0f;
  return verify_impl(q_logits, p_logits, dtype, draft_tokens, uniforms, B, gamma, V, rule, alpha,
                     temperature, greedy, out_accept_len, out_next_token, out_defer_mask, ex,
                     stream, true);
}

size_t spc_noalloc_scratch_bytes(void) { return kNoAllocBytes; }

spc_status spc_draft_sample(const void* logits, int32_t dtype, int32_t B, int32_t V,
                            float temperature, const float* temp_per_seq,
                            const float* uniforms, int32_t* out_token, hipStream_t stream) {
  return draft_impl(logits, dtype, B, V, temperature, temp_per_seq, uniforms, out_token, nullptr,
                    0, stream);
}

spc_status spc_draft_sample_ws(const void* logits, int32_t dtype, int32_t B, int32_t V,
                               float temperature, const float* temp_per_seq,
                               const float* uniforms, int32_t* out_token, void* workspace,
                               size_t workspace_bytes, hipStream_t stream) {
  return draft_impl(logits, dtype, B, V, temperature, temp_per_seq, uniforms, out_token,
                    workspace, workspace_bytes, stream);
}

size_t spc_workspace_bytes(int32_t B, int32_t gamma, int32_t V, int32_t dtype) {
  if (check_shape(B, gamma, V) != SPC_OK || (dtype != SPC_F32 && dtype != SPC_BF16)) return 0;
  return launch_layout(B, gamma, V, dtype).total;
}

size_t spc_workspace_zero_bytes(int32_t B, int32_t gamma, int32_t V, int32_t dtype) {
  if (check_shape(B, gamma, V) != SPC_OK || (dtype != SPC_F32 && dtype != SPC_BF16)) return 0;
  return launch_layout(B, gamma, V, dtype).zero_end;
}

size_t spc_draft_workspace_bytes(int32_t B, int32_t V, int32_t dtype) {
  if (B < 1 || V < 2 || (dtype != SPC_F32 && dtype != SPC_BF16)) return 0;
  return spc::ws_layout(seqs_per_launch(B, 1), 1, V, dtype).total;
}

const char* spc_last_error(void) { return g_err.c_str(); }

void spc_release(void) {
  std::lock_guard<std::mutex> lk(g_ws_mu);
  int cur = 0;
  if (hipGetDevice(&cur) != hipSuccess) cur = 0;
  for (auto& kv : g_ws) {
    if (hipSetDevice(kv.first) != hipSuccess) continue;
    if (kv.second.ptr) (void)hipFree(kv.second.ptr);
    for (void* r : kv.second.retired) (void)hipFree(r);
  }
  g_ws.clear();
  (void)hipSetDevice(cur);
}

int32_t spc_debug_route(int32_t B, int32_t gamma, int32_t V, int32_t dtype, uint32_t rules,
                        int32_t per_rule, int32_t greedy, int32_t cus) {
  if (check_shape(B, gamma, V) != SPC_OK || (dtype != SPC_F32 && dtype != SPC_BF16) || cus < 1)
    return 0;
  const int64_t g1 = (int64_t)gamma + 1, bl = seqs_per_launch(B, gamma);
  const Route t = choose_route(B, bl, bl * g1, g1, V, dtype, rules & kAllRules, per_rule != 0,
                               greedy == 0, greedy != 0, cus);
  return (t.seq ? spc::kRouteSeq : t.small ? spc::kRouteSmall : spc::kRouteTiles) |
         (t.tv_self ? spc::kRouteTvSelf : 0) | (t.tv_pass ? spc::kRouteTvPass : 0) |
         (t.tv_jobs ? spc::kRouteTvJobs : 0) | (t.job_pass ? spc::kRouteJobs : 0) |
         (t.pair ? spc::kRoutePair : 0);
}

const char* spc_version(void) { return "libspeccascade 0.2 (gfx950)"; }

}  // extern "C"

// C-ABI entry points of libdiffpower: contexts, designs, evals, forward and
// reverse sweeps.  The serving layer lives in dp_server.cpp.
#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <thread>

#include "dp_eval.h"

namespace dp {

static thread_local std::string g_err;

dp_status fail(dp_status st, const std::string &msg) {
  g_err = msg;
  return st;
}
void clear_error() { g_err.clear(); }

void ctx_retain(dp_ctx *c) { c->refs.fetch_add(1); }
void ctx_release(dp_ctx *c) {
  if (c->refs.fetch_sub(1) != 1) return;
  if (c->owned) {
    (void)hipStreamSynchronize(c->owned);
    (void)hipStreamDestroy(c->owned);
  }
  delete c;
}

constexpr size_t kReportPage = 4096;
ReportWords::~ReportWords() {
  for (uint32_t *p : pages_) (void)hipHostFree(p);
}
dp_status ReportWords::take(uint32_t **out) {
  std::lock_guard<std::mutex> lock(mu_);
  if (free_.empty()) {
    void *p = nullptr;
    DP_HIP_TRY(hipHostMalloc(&p, kReportPage));
    pages_.push_back(static_cast<uint32_t *>(p));
    for (size_t i = 0; i < kReportPage / sizeof(uint32_t); ++i) free_.push_back(pages_.back() + i);
  }
  *out = free_.back();
  free_.pop_back();
  **out = 0u;
  return DP_OK;
}
void ReportWords::give(uint32_t *word) {
  std::lock_guard<std::mutex> lock(mu_);
  free_.push_back(word);
}

void design_retain(dp_design *d) { d->refs.fetch_add(1); }
void design_release(dp_design *d) {
  if (d->refs.fetch_sub(1) != 1) return;
  dp_ctx *c = d->ctx;
  (void)hipStreamSynchronize(c->stream);
  delete d;
  ctx_release(c);
}

}  // namespace dp

using dp::DevBuf;
using dp::fail;

namespace {

constexpr int64_t kAutoWordBudget = 32ll << 30;  // bytes of simulation words in flight
// Largest forward sweep (kernel launches) captured into one HIP graph.  A graph
// pays off where a sweep is launch-bound; bigger sweeps run per level.
constexpr int64_t kMaxGraphLaunches = 1024;
const char *kVersion = "diffpower-mi355x 0.1 (gfx950)";
enum { SPAN_SIM = 0, SPAN_SP = 1, SPAN_BWD = 2, SPAN_STIM = 3 };

dp::GraphView view(const dp_design *d) { return dp::design_view(d); }
using dp::for_level_parts;
using dp::pairs_levels;

int32_t s_prime(const dp_eval *ev) { return (ev->S > 0 && !ev->paired_sizes) ? ev->S : 1; }
double kappa_of(const dp_params &p) { return p.energy_factor * p.vdd * p.vdd * p.fclk; }
int64_t n_words(const dp_params &p) { return p.n_sim / 64; }

dp_status check_params(const dp_params *p) {
  if (!p) return fail(DP_E_INVALID, "NULL params");
  if (p->mode < DP_MODELED || p->mode > DP_FROZEN_BETA)
    return fail(DP_E_INVALID, "params.mode must be DP_MODELED, DP_HYBRID or DP_FROZEN_BETA");
  if (p->beta_grad != DP_BETA_LOCAL && p->beta_grad != DP_BETA_STE)
    return fail(DP_E_INVALID, "params.beta_grad must be DP_BETA_LOCAL or DP_BETA_STE");
  if (!(p->beta_min > 0.0) || !(p->beta_max >= p->beta_min) || !std::isfinite(p->beta_max))
    return fail(DP_E_INVALID, "params: need 0 < beta_min <= beta_max < inf");
  const double k = kappa_of(*p);
  if (!std::isfinite(k) || k < 0.0) return fail(DP_E_INVALID, "params: bad vdd/fclk/energy_factor");
  if (p->mode == DP_HYBRID) {
    if (p->n_sim < 128 || p->n_sim % 64 != 0)
      return fail(DP_E_INVALID, "params.n_sim must be a multiple of 64 and >= 128 in DP_HYBRID");
    if (p->n_sim / 64 > (int64_t)INT32_MAX)
      return fail(DP_E_INVALID, "params.n_sim too large");
  }
  return DP_OK;
}

// The eval's pinned words, once.
dp_status ensure_reports(dp_eval *ev) {
  if (!ev->reports) ev->reports = ev->d->ctx->reports;
  if (!ev->flow_report) DP_TRY(ev->reports->take(&ev->flow_report));
  if (!ev->check_report) DP_TRY(ev->reports->take(&ev->check_report));
  return DP_OK;
}

// Refuse a float array (host or device) with values outside [lo, hi] or NaN.
// Device values are checked on the device; the kernel reports into a pinned word
// of the eval's (a device flag took a fill and a copy to the host more, 20 to 30
// us a call), and stores them in `copy` on its way where that is not null.
dp_status check_values(dp_eval *ev, const float *v, int64_t n, float lo, float hi, int on_device,
                       const char *what, float *copy = nullptr) {
  if (!v) return fail(DP_E_INVALID, std::string(what) + ": NULL pointer");
  if (!on_device) {
    for (int64_t i = 0; i < n; ++i)
      if (!(v[i] >= lo && v[i] <= hi))
        return fail(DP_E_INVALID, std::string(what) + ": value " + std::to_string(v[i]) +
                                      " at index " + std::to_string(i) + " out of range");
    return DP_OK;
  }
  hipStream_t s = ev->stream();
  DP_TRY(ensure_reports(ev));
  volatile uint32_t *bad = ev->check_report;
  *bad = 0u;
  DP_HIP_TRY(dp::launch_check_range(v, n, lo, hi, copy, ev->check_report, s));
  DP_HIP_TRY(hipStreamSynchronize(s));
  if (*bad) return fail(DP_E_INVALID, std::string(what) + ": a value is NaN or out of range");
  return DP_OK;
}

// Copy a caller array into a device staging buffer (device-to-device when on_device).
dp_status stage_in(DevBuf &buf, const void *src, size_t bytes, int on_device, hipStream_t s) {
  DP_TRY(buf.alloc(std::max<size_t>(bytes, 16)));
  if (bytes)
    DP_HIP_TRY(hipMemcpyAsync(buf.ptr, src, bytes,
                              on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, s));
  return DP_OK;
}

// What an import kernel reads: a device array as it is, a host one's copy in
// `stage`.
dp_status import_from(DevBuf &stage, const float *src, size_t bytes, int on_device, hipStream_t s,
                      const float **out) {
  *out = src;
  if (on_device) return DP_OK;
  DP_TRY(stage_in(stage, src, bytes, 0, s));
  *out = stage.as<float>();
  return DP_OK;
}

// --- profiling: events around launches, resolved after the stream drains
hipEvent_t take_event(dp_eval *ev) {
  if (ev->ev_used == ev->ev_pool.size()) {
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    ev->ev_pool.push_back(e);
  }
  return ev->ev_pool[ev->ev_used++];
}

struct SpanGuard {
  dp_eval *ev;
  size_t a = 0;
  int kind;
  double bytes;
  bool on;
  int64_t launches;
  hipStream_t st;
  SpanGuard(dp_eval *e, int k, double b, bool enabled, int64_t n_launch,
            hipStream_t stream = nullptr)
      : ev(e), kind(k), bytes(b), on(enabled), launches(n_launch),
        st(stream ? stream : e->stream()) {
    if (on) {
      a = ev->ev_used;
      hipEvent_t x = take_event(ev);
      if (!x) { on = false; return; }
      (void)hipEventRecord(x, st);
    }
  }
  ~SpanGuard() {
    if (!on) return;
    size_t b = ev->ev_used;
    hipEvent_t x = take_event(ev);
    if (!x) return;
    (void)hipEventRecord(x, st);
    ev->spans.push_back({a, b, kind, bytes, launches});
  }
};

dp_status resolve_profile(dp_eval *ev) {
  if (ev->spans.empty()) {
    ev->ev_used = 0;
    return DP_OK;
  }
  DP_HIP_TRY(hipStreamSynchronize(ev->stream()));
  for (const auto &sp : ev->spans) {
    float ms = 0.0f;
    DP_HIP_TRY(hipEventElapsedTime(&ms, ev->ev_pool[sp.a], ev->ev_pool[sp.b]));
    switch (sp.kind) {
      case SPAN_SIM: ev->prof.sim_ms += ms; ev->prof.sim_launches += sp.launches; ev->prof.sim_bytes += sp.bytes; break;
      case SPAN_SP: ev->prof.sp_ms += ms; ev->prof.sp_launches += sp.launches; ev->prof.sp_bytes += sp.bytes; break;
      case SPAN_BWD: ev->prof.bwd_ms += ms; ev->prof.bwd_launches += sp.launches; ev->prof.bwd_bytes += sp.bytes; break;
      default: ev->prof.stim_ms += ms; ev->prof.stim_launches += sp.launches; break;
    }
  }
  ev->spans.clear();
  ev->ev_used = 0;
  return DP_OK;
}

// --- chunking of the simulated words
// The simulation holds `cols` query columns' word buffers per stream (a
// column group, simulated by the same launches), each Tc words (plus a
// two-word halo when the run is cut into chunks) per net.
struct ChunkPlan {
  int64_t T = 0, Tc = 0, pitch = 0;
  int32_t halo = 0, n_chunks = 0;
  int32_t cols = 1;      // query columns per launch
  int32_t n_groups = 1;  // column groups, ceil(B / cols)
  // word tiles (launch_sim_flow) instead: words per tile (0: level launches),
  // tiles per column, teams' buffers
  int32_t tile = 0, n_tiles = 0, n_bufs = 0;
};

int32_t n_sim_streams(const dp_eval *ev) { return ev->sim_streams > 0 ? ev->sim_streams : 1; }

bool flow_ready(const dp_eval *ev, int32_t C);

// Whether the simulation runs in word tiles, and in which: with chunks, streams
// and columns left automatic.  Up to 24 tiles are a round of the teams; of the
// pitches that stay within it the narrowest (a level's turns grow with the
// pitch), and 64 words up to 32 tiles.  Beyond, and beyond 2^28 words over all
// nets and columns, the level launches' longer rows are the faster ones (forward,
// us, tiles against levels: 2K gates x 1280 words 105 / 123, x 5120 184 / 167;
// 117K x 257 271 / 424, x 1024 638 / 691; 300K x 1024 1516 / 1368; 1M x 257
// 1670 / 1966), as they are where fewer than 16 tiles leave XCDs without work
// in levels of more than 8192 gates (1M x 64: 899 / 817).  Half library cells,
// 300K x 256, with the reverse sweep: 1074 / 1914.  (Their kernel's registers
// leave room for 24 teams.)
// A level saves its launch, 3.4 us (11 with library cells); level launches read
// rows shorter than a wave's 128 words at 2 us more per million (net, column) and
// word short, and rows of an odd number of words at 1.5 us more per million words
// (117K gates x 3 levels: 256 words 150, 257 words 199).  A tile's rows cost 12 us
// per million words of one tile more, and what the columns' last tiles leave
// empty, beyond a sixteenth, 4 us per million words (300K gates x 20 levels, 5
// columns of 100 words: 935 / 828).  So with few levels of many gates level launches win (forward, us, tiles
// against levels: 117K gates x 3 levels x 1024 words 505 / 414, x 12 567 / 493, x 60
// 629 / 720; 1M x 256 words, 8 levels 1279 / 1065, 50 1383 / 1260, 100 1390 / 1461).
// Over 390 (design, columns, words) within the limits above the choice is at most
// 6 us slower than level launches (designs of two or three levels), or 2 %.
constexpr int64_t kTileMaxWords = 1ll << 28;
constexpr int32_t kTileTeams = 24, kTileWide = 8192;
bool tiles_pay(const dp_design *d, int32_t B, int64_t T, int64_t tiles, int32_t pitch) {
  const double n = d->n_nets * 1e-6, words = (double)(B * T), held = (double)(tiles * pitch);
  const double saved = 3.4 * d->depth + 8.0 * d->cell_levels +
                       2.0 * n * B * (double)std::max<int64_t>(0, 128 - T) +
                       (T % 2 != 0 ? 1.5 * n * words : 0.0);
  return saved > 8.0 + std::max(0.0, 12.0 * n * pitch - 25.0) +
                     4.0 * n * std::max(0.0, held * (15.0 / 16.0) - words);
}
void plan_tiles(const dp_eval *ev, ChunkPlan *c) {
  const dp_design *d = ev->d;
  if (ev->words_per_chunk > 0 || ev->sim_streams > 1 || ev->sim_cols > 0 ||
      std::chrono::steady_clock::now() < ev->tiles_retry || d->depth < 1 ||
      !flow_ready(ev, ev->B) || c->T > kTileMaxWords / d->n_nets / ev->B)
    return;
  for (int32_t pitch : {16, 32, 64}) {
    const int64_t tiles = (c->T + pitch - 1) / pitch * ev->B;
    if (tiles > (pitch < 64 ? kTileTeams : dp::kSimBufs)) continue;
    if (tiles < 16 && d->max_level_width > kTileWide) return;
    if (!dp::sim_fits(view(d), d->depth, ev->B, pitch, c->T)) return;
    if (!tiles_pay(d, ev->B, c->T, tiles, pitch)) return;
    c->n_chunks = 1;  // of the level launches in its place
    c->tile = pitch;
    c->n_tiles = (int32_t)(tiles / ev->B);
    c->n_bufs = std::min((int32_t)tiles, d->has_cell_gates ? kTileTeams : dp::kSimBufs);
    return;
  }
}

ChunkPlan plan_chunks(const dp_eval *ev) {
  ChunkPlan c;
  c.T = n_words(ev->prm);
  plan_tiles(ev, &c);
  if (c.tile) return c;
  // words per net that fit one stream's share of the budget, over all the
  // columns of its buffer
  const int64_t row_budget = std::max<int64_t>(
      kAutoWordBudget / (8 * (int64_t)ev->d->n_nets * n_sim_streams(ev)), 4);
  int64_t want = ev->words_per_chunk;
  if (want <= 0) want = c.T + (c.T & 1) <= row_budget ? c.T : row_budget - 2;
  want = std::max<int64_t>(2, want + (want & 1));
  if (want >= c.T) {
    c.Tc = c.T + (c.T & 1);
    c.halo = 0;
    c.n_chunks = 1;
  } else {
    c.Tc = want;
    c.halo = 2;
    c.n_chunks = (int32_t)((c.T + c.Tc - 1) / c.Tc);
  }
  c.pitch = c.halo + c.Tc;
  // as many columns per launch as the budget holds at this pitch
  c.cols = (int32_t)std::max<int64_t>(1, std::min<int64_t>(ev->B, row_budget / c.pitch));
  if (ev->sim_cols > 0) c.cols = std::min(c.cols, ev->sim_cols);
  c.n_groups = (ev->B + c.cols - 1) / c.cols;
  return c;
}

// Chunk k of column group `grp` on simulation stream `lane`.
dp::ChunkView chunk_view(const dp_eval *ev, const ChunkPlan &pl, int32_t k, int32_t lane,
                         int32_t grp) {
  dp::ChunkView v;
  const int64_t col_stride = (int64_t)ev->d->n_nets * pl.pitch;
  v.W = ev->words.as<uint64_t>() + (size_t)lane * pl.cols * col_stride;
  v.pitch = pl.pitch;
  v.col_stride = col_stride;
  const int64_t t0 = (int64_t)k * pl.Tc;
  const int64_t nw = std::min<int64_t>(pl.Tc, pl.T - t0);
  v.t_first = t0 - pl.halo;
  v.u_lo = pl.halo;
  v.u_hi = (int32_t)(pl.halo + nw);
  v.u_tog_lo = t0 == 0 ? pl.halo + 1 : pl.halo;
  v.pairs = (v.u_hi + 1) / 2;
  v.n_cols = std::min(pl.cols, ev->B - grp * pl.cols);
  return v;
}

int32_t pick_iters(const dp_eval *ev, const ChunkPlan &pl) {
  if (ev->sim_iters > 0) return ev->sim_iters;
  // about two waves per row: enough waves per level, few carry recomputes
  const int64_t pairs = pl.pitch / 2;
  if (pairs >= 1024) return 8;
  if (pairs >= 512) return 4;
  if (pairs >= 256) return 2;
  return 1;
}

bool hybrid(const dp_eval *ev) { return ev->prm.mode == DP_HYBRID; }

// A cooperative launch cannot be enqueued on the null stream; there it runs
// on a private stream that waits for the caller's stream and that the caller's
// stream then waits for.  Elsewhere it goes to `s` itself.
template <class F>
dp_status on_coop_stream(dp_eval *ev, hipStream_t s, F launch) {
  if (s) {
    DP_HIP_TRY(launch(s));
    return DP_OK;
  }
  if (!ev->coop_stream) {
    DP_HIP_TRY(hipStreamCreateWithFlags(&ev->coop_stream, hipStreamNonBlocking));
    for (hipEvent_t &e : ev->coop_events) DP_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  }
  DP_HIP_TRY(hipEventRecord(ev->coop_events[0], s));
  DP_HIP_TRY(hipStreamWaitEvent(ev->coop_stream, ev->coop_events[0], 0));
  DP_HIP_TRY(launch(ev->coop_stream));
  DP_HIP_TRY(hipEventRecord(ev->coop_events[1], ev->coop_stream));
  DP_HIP_TRY(hipStreamWaitEvent(s, ev->coop_events[1], 0));
  return DP_OK;
}

// The persistent sweeps' barrier words (allocated and zeroed when the
// schedule is chosen; the launcher zeroes all but the report word before
// each launch).
dp_status grid_barrier(dp_eval *ev, dp::GridBarrier *out) {
  if (!ev->barrier.ptr) return fail(DP_E_STATE, "persistent sweep without its barrier words");
  const double ticks = ev->barrier_limit_us * 100.0;  // the real-time counter runs at 100 MHz
  *out = dp::GridBarrier{ev->barrier.as<uint32_t>(), (uint64_t)std::max(ticks, 0.0)};
  ev->barrier_pending = true;
  return DP_OK;
}

// --- dataflow sweeps (launch_sp_flow, launch_bwd_flow)
// Allocate what the eval's dataflow sweeps need (once; before any capture).
dp_status ensure_flow(dp_eval *ev) {
  DP_TRY(ev->flow.alloc((dp::kFlowWords + dp::kSimWords) * sizeof(uint32_t)));
  return ensure_reports(ev);
}

// Whether a sweep over C columns of the eval can run as one dataflow launch
// (once ensure_flow has run).
bool flow_ready(const dp_eval *ev, int32_t C) {
  const dp_design *d = ev->d;
  return ev->flow.ptr && ev->schedule != DP_SCHED_PERSISTENT &&
         dp::flow_fits(view(d), d->depth, std::max(C, ev->B), d->n_edges);
}

// What a sweep takes, in us, of G million gates and N million (net, column)
// pairs over D levels: base + |(level D, gates G rounds + pairs N + far N log2 N)|
// + over N.  A level's latency and its work overlap, hence the root of squares.
// A dataflow sweep keeps a column in one XCD: its latency per level is a
// fraction of a launch's, its work goes by rounds of eight columns, and columns
// share lines that every XCD fetches; level launches have the whole chip for each
// level.  So few levels of many gates are faster in level launches (1M gates,
// one column, forward / gradient in us, levels against dataflow: 8 levels 46 /
// 117 against 71 / 153, 25 levels 83 / 144 against 80 / 143, 100 levels 233 / 401
// against 125 / 214; 117K gates, 16 columns: 3 levels 25 / 29 against 83 / 150, 60
// levels 128 / 245 against 84 / 124).  Fitted to 334 (design, columns) of 2K to
// 3.5M gates, 2 to 400 levels, 1 to 64 columns and 113 with 9 to 200 library
// cells in half of the gates or all (20K gates x 2 levels of nine cells, 32
// columns, 33 / 98 against 48 / 117; 117K x 12, one column, 107 / 367 against 66 /
// 67).  Dataflow is taken up to kFlowLean times the levels' fitted cost, as the
// fit errs that way in the middle (50K gates x 25 levels, 32 columns 62 us
// against 71, fitted 74 against 71; 20K x 20, 56 columns 61 against 69): over the
// 280 of the former that fit a dataflow sweep the choice is then 0.05 % (forward)
// and 0.3 % (gradient) slower than the better of the two on average and at most
// 5 % slower than level launches.
struct SweepCost {
  double base, level, gates, pairs, far, over;
};
constexpr double kFlowLean = 1.06;
constexpr SweepCost kSpFlow{20.5, 0.72, 31.6, 26.8, 0.0, 0.0}, kSpLevels{12.7, 1.82, 16.7, 0.0, 0.0, 7.9};
constexpr SweepCost kBwdFlow{13.4, 0.80, 118.6, 24.1, 7.3, 0.0}, kBwdLevels{5.1, 3.81, 123.0, 0.0, 0.0, 4.9};
// (level launches of one or two columns pull with whole waves)
constexpr SweepCost kBwdFlowFew{11.6, 0.74, 87.8, 61.4, 0.0, 0.0},
    kBwdLevelsFew{22.0, 2.80, 19.0, 0.0, 0.0, 71.5};
// every level with library cells
constexpr SweepCost kSpFlowCells{16.9, 3.79, 89.4, 25.5, 0.0, 0.0},
    kSpLevelsCells{10.6, 7.61, 24.1, 0.0, 0.0, 6.9};
constexpr SweepCost kBwdFlowCells{39.9, 1.64, 151.0, 92.4, 0.0, 0.0},
    kBwdLevelsCells{7.2, 34.9, 237.6, 0.0, 0.0, 39.9};
// gates: a column's, with the rounds of columns that follow one another; pairs:
// of all columns; both in millions.
double sweep_us(const SweepCost &c, double depth, double gates, double pairs) {
  const double work = c.gates * gates + c.pairs * pairs +
                      (pairs > 1.0 ? c.far * pairs * std::log2(pairs) : 0.0);
  return c.base + std::hypot(c.level * depth, work) + c.over * pairs;
}
// The same with library cells in `cells` of the levels.
double sweep_us(const SweepCost &fixed, const SweepCost &lib, const dp_design *d, double gates,
                double pairs) {
  const double us = sweep_us(fixed, d->depth, gates, pairs);
  if (d->cell_levels == 0) return us;
  const double part = (double)d->cell_levels / d->depth;
  return (1.0 - part) * us + part * sweep_us(lib, d->depth, gates, pairs);
}
bool flow_pays(const dp_design *d, int32_t C, bool reverse) {
  const double G = d->n_gates * 1e-6, N = (double)d->n_nets * C * 1e-6, rounds = (C + 7) / 8;
  if (!reverse)
    return sweep_us(kSpFlow, kSpFlowCells, d, G * rounds, N) <
           kFlowLean * sweep_us(kSpLevels, kSpLevelsCells, d, G, N);
  const bool few = C < 3;
  return sweep_us(few ? kBwdFlowFew : kBwdFlow, kBwdFlowCells, d, G * rounds, N) <
         kFlowLean * sweep_us(few ? kBwdLevelsFew : kBwdLevels, kBwdLevelsCells, d, G, N);
}

// Whether the eval's SP sweep, and a reverse sweep over C columns, run as one
// dataflow launch.
bool sp_flows(const dp_eval *ev) { return flow_ready(ev, ev->B) && flow_pays(ev->d, ev->B, false); }
bool bwd_flows(const dp_eval *ev, int32_t C) { return flow_ready(ev, C) && flow_pays(ev->d, C, true); }

// Whether the per-(b, s) reverse sweep over C columns runs in adjoints
// (launch_bwd_wide_level): from 16 size vectors, which then share an entry's
// partial derivative, and where there are pairs enough.  A wave of that sweep
// pulls a net's whole fan-out range, 0.9 us a strand in a row, so that a level
// takes its longest range's time however few its columns; contributions take 8
// us per million (gate, column), adjoints 2, and 33 us more a level with library
// cells.  Sweep by contributions / in adjoints, us: 117K gates, 4 x 32 columns
// 274 / 342, 16 x 16 422 / 361, 32 x 64 2077 / 812; 300K (ranges up to 220) 4 x 16
// 391 / 948, 20 x 16 1049 / 1387; 1M, 2 x 16 608 / 1587, 16 x 16 2427 / 2443, 32 x 16
// 4482 / 2864; 2M, 8 x 16 2572 / 2671, 16 x 16 4627 / 3519; half library cells, 117K,
// 2 x 40 2224 / 397.
constexpr int32_t kWideSizes = 16;
bool wide_reverse(const dp_eval *ev, int32_t C, int per_column) {
  const dp_design *d = ev->d;
  return per_column && s_prime(ev) >= kWideSizes && ev->schedule != DP_SCHED_PERSISTENT &&
         !bwd_flows(ev, C) &&
         (int64_t)d->n_gates * C + 5400000ll * d->cell_levels >= 130000 * d->pull_strands;
}

// What a dataflow reverse sweep over C columns takes besides contributions.
size_t seed_bytes(const dp_eval *ev, int32_t C) {
  return std::max<size_t>((size_t)ev->d->n_nets * C * sizeof(float), 16);
}
size_t part_bytes(const dp_eval *ev) {
  return std::max<size_t>((size_t)ev->B * ev->d->pins * ev->d->n_gates * sizeof(float), 16);
}
// (part alone may be there in another sweep's size)
bool have_flow_scratch(const dp_eval *ev, int32_t C) {
  return ev->seed.bytes >= seed_bytes(ev, C) && ev->part.bytes >= part_bytes(ev);
}
dp_status ensure_flow_scratch(dp_eval *ev, int32_t C) {
  if (have_flow_scratch(ev, C)) return DP_OK;
  if (std::chrono::steady_clock::now() < ev->scratch_retry) return DP_OK;
  dp_status st = ev->seed.alloc(seed_bytes(ev, C));
  if (st == DP_OK) st = ev->part.alloc(part_bytes(ev));
  if (st != DP_E_OOM) return st;
  // level by level where the device has no memory for it, and again in a second
  ev->seed.release();
  ev->part.release();
  ev->scratch_retry = std::chrono::steady_clock::now() + std::chrono::seconds(1);
  return DP_OK;
}
// Every buffer of a reverse sweep over C columns (before any capture).
dp_status ensure_reverse_buffers(dp_eval *ev, int32_t C, int per_column = 0) {
  const dp_design *d = ev->d;
  DP_TRY(ensure_flow(ev));
  if (wide_reverse(ev, C, per_column)) {  // contrib holds the adjoints
    DP_TRY(ev->contrib.alloc(std::max<size_t>((size_t)d->n_nets * C * sizeof(float), 16)));
    return ev->part.alloc(std::max<size_t>((size_t)d->n_edges * ev->B * sizeof(float), 16));
  }
  DP_TRY(ev->contrib.alloc(std::max<size_t>((size_t)d->n_edges * C * sizeof(float), 16)));
  return bwd_flows(ev, C) ? ensure_flow_scratch(ev, C) : DP_OK;
}

// Polls after which a wait of the eval's dataflow launches gives up: the
// default's share that dp_eval_set_barrier_timeout's limit is of its own.
uint32_t flow_limit(const dp_eval *ev) {
  return (uint32_t)(std::min(ev->barrier_limit_us / kBarrierLimitUs, 1.0) * dp::kFlowPolls);
}

dp::FlowCtl flow_ctl(const dp_eval *ev) {
  dp::FlowCtl ctl{ev->flow.as<uint32_t>(), ev->flow_report, 0, ev->d->ctx->n_cu};
  dp::flow_set_limit(ctl, flow_limit(ev));
  return ctl;
}

// At a host synchronization of the eval (its stream idle): whether a
// persistent or dataflow sweep since the last check had a wait give up.
// Reads and clears the report words, all of them.
dp_status barrier_status(dp_eval *ev) {
  const dp_status flow = dp::flow_status(ev);
  if (!ev->barrier_pending) return flow;
  uint32_t rep = 0;
  uint32_t *w = ev->barrier.as<uint32_t>() + dp::kBarrierReport;
  DP_HIP_TRY(hipMemcpy(&rep, w, sizeof(uint32_t), hipMemcpyDeviceToHost));
  ev->barrier_pending = false;
  if (rep == 0u) return flow;
  DP_HIP_TRY(dp::launch_fill_u32(w, 1, 0u, ev->stream()));
  DP_HIP_TRY(hipStreamSynchronize(ev->stream()));
  return fail(DP_E_HIP, "a persistent sweep's grid barrier gave up waiting (no progress for " +
                            std::to_string(ev->barrier_limit_us) +
                            " us); that sweep's outputs are NaN and not a result");
}

// Synchronize the eval's stream, then report a sweep of it that gave up
// (host-output calls end here).
dp_status sync_and_check(dp_eval *ev) {
  DP_HIP_TRY(hipStreamSynchronize(ev->stream()));
  return barrier_status(ev);
}

// Per-net beta [n_nets][B] of the last forward: the computed one (hybrid),
// the frozen one as given, or null in modeled mode (beta = 1).  (A frozen
// beta shared by every column is [n_nets]: see backward_args.)
float *beta_or_null(dp_eval *ev) {
  if (ev->prm.mode == DP_MODELED) return nullptr;
  return ev->prm.mode == DP_HYBRID ? ev->beta.as<float>() : ev->beta_frozen.as<float>();
}

// Whether the forward draws Markov stimulus words (a target transition rate
// per PI and no explicit stimulus).
bool markov(const dp_eval *ev) { return ev->have_tau && !ev->have_stim; }

// Launches of the modeled sweep's SP levels.
int64_t sp_sweep_launches(const dp_design *d, int32_t B) {
  int64_t n = 0;
  for (int32_t l = 1; l <= d->depth;) {
    if (pairs_levels(d, l, B)) {
      ++n;
      l += 2;
    } else {
      n += d->lvl_fixed[l] > 0 ? 1 : 0;
      n += d->lvl_fixed[l] < d->level_ptr[l + 1] - d->level_ptr[l] ? 1 : 0;
      ++l;
    }
  }
  return n;
}

// Kernel launches of one forward sweep in level launches (what a captured
// graph holds at most).
int64_t forward_launches(const dp_eval *ev, const ChunkPlan *pl) {
  const int64_t depth = ev->d->depth + ev->d->split_levels;
  if (!pl) return sp_sweep_launches(ev->d, ev->B) + 2;
  return (int64_t)pl->n_groups * pl->n_chunks * (depth + 1) + 4 + (markov(ev) ? 1 : 0) +
         ev->d->cell_levels;  // the library cells' SP launches
}

// Kernel launches of one reverse sweep in level launches, the measure of whether
// it is captured (a sweep in adjoints has two more, a dataflow sweep two in all).
int64_t reverse_launches(const dp_design *d) { return (int64_t)d->depth + d->split_levels + 1; }

// Allocate everything the forward sweep touches (before any capture).
dp_status ensure_forward_buffers(dp_eval *ev, const ChunkPlan *pl) {
  const dp_design *d = ev->d;
  const size_t nb = (size_t)d->n_nets * ev->B;
  DP_TRY(ensure_flow(ev));
  if (ev->prm.mode == DP_HYBRID) DP_TRY(ev->beta.alloc(nb * sizeof(float)));
  const int32_t cols = ev->B * s_prime(ev);
  DP_TRY(ev->power_partial.alloc(
      (size_t)dp::power_scratch(d->n_nets, ev->B, ev->S, ev->paired_sizes) * sizeof(double)));
  DP_TRY(ev->power.alloc((size_t)cols * sizeof(float)));
  if (pl) {
    DP_TRY(ev->ones.alloc(nb * sizeof(uint32_t)));
    DP_TRY(ev->tog.alloc(nb * sizeof(uint32_t)));
    if (pl->tile) {
      DP_TRY(ev->words.alloc((size_t)pl->n_bufs * d->n_nets * pl->tile * sizeof(uint64_t) +
                             (size_t)pl->n_tiles * nb * (2 * sizeof(uint64_t) + sizeof(uint32_t))));
      if (!ev->have_stim)
        DP_TRY(ev->mstim.alloc(std::max<size_t>((size_t)ev->B * d->n_pi * pl->T * sizeof(uint64_t), 16)));
      return DP_OK;
    }
    const int32_t L = n_sim_streams(ev);
    DP_TRY(ev->words.alloc((size_t)L * pl->cols * d->n_nets * pl->pitch * sizeof(uint64_t)));
    if (markov(ev))
      DP_TRY(ev->mstim.alloc(std::max<size_t>((size_t)ev->B * d->n_pi * pl->T * sizeof(uint64_t), 16)));
    while ((int32_t)ev->lane_streams.size() < L - 1) {
      hipStream_t st = nullptr;
      DP_HIP_TRY(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
      ev->lane_streams.push_back(st);
    }
    while ((int32_t)ev->lane_events.size() < L) {
      hipEvent_t e = nullptr;
      DP_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
      ev->lane_events.push_back(e);
    }
  }
  return DP_OK;
}

// Algorithmic bytes of one simulation launch of level l over `cols`
// columns of `words` words each (and the level's SP over B columns when
// fused).
double sim_level_bytes(const dp_design *d, int32_t l, int64_t words, int32_t cols, int32_t B,
                       bool fused) {
  const int64_t n = d->level_ptr[l + 1] - d->level_ptr[l];
  const int64_t pins = d->lvl_pins[l], read = d->lvl_read[l];
  // per column: fan-in words, output words of the nets that have readers (a
  // net without readers needs only its counts, so its words are not
  // stored), counters; per launch: indices, cell, fan-out range
  double b = (double)cols * ((double)(8 * pins + 8 * read) * (double)words + 8.0 * n)
             + (double)(4 * pins + n) + 8.0 * n;
  if (fused) b += (double)B * (4 * pins + 4 * n);  // SP gathers and writes
  return b;
}

double sp_level_bytes(const dp_design *d, int32_t l, int32_t B) {
  const int64_t n = d->level_ptr[l + 1] - d->level_ptr[l];
  const int64_t pins = d->lvl_pins[l];
  return (double)B * (4 * pins + 4 * n) + (double)(4 * pins + n);  // stored SP gathers, writes
}

double bwd_level_bytes(const dp_design *d, int32_t l, int32_t C) {
  const int64_t n = d->level_ptr[l + 1] - d->level_ptr[l];
  const int64_t pins = d->lvl_pins[l], fo = d->lvl_fanout[l];
  // per column: own SP (the seed), pulled contributions, fan-in SP gathers,
  // contribution writes
  const double per_col = 4.0 * n + 4.0 * fo + 4.0 * pins + 4.0 * pins;
  // structure: fan-out offsets and edge ids, fan-in indices, cell
  const double structure = 8.0 * n + 4.0 * fo + 4.0 * pins + n;
  return (double)C * per_col + structure;
}

// Plan a forward and make its buffers (*pl: null unless hybrid).  Tiles take up
// to a few times the words of the level launches in their place: where the device
// has no memory for them, level launches, and tiles again after a second.
dp_status plan_forward(dp_eval *ev, ChunkPlan *plan, const ChunkPlan **pl) {
  *pl = nullptr;
  DP_TRY(ensure_flow(ev));
  if (!hybrid(ev)) return ensure_forward_buffers(ev, nullptr);
  *pl = plan;
  *plan = plan_chunks(ev);
  const dp_status st = ensure_forward_buffers(ev, plan);
  if (st != DP_E_OOM || !plan->tile) return st;
  ev->words.release();
  if (!markov(ev)) ev->mstim.release();
  ev->tiles_retry = std::chrono::steady_clock::now() + std::chrono::seconds(1);
  *plan = plan_chunks(ev);
  return ensure_forward_buffers(ev, plan);
}

// Enqueue the whole forward sweep (no host sync, no allocation).
dp_status enqueue_forward_tail(dp_eval *ev, const ChunkPlan *pl);


dp_status enqueue_forward(dp_eval *ev, const ChunkPlan *pl) {
  const dp_design *d = ev->d;
  hipStream_t s = ev->stream();
  const dp::GraphView g = view(d);
  const bool prof = ev->profiling;
  float *sp = ev->sp.as<float>();
  const dp::SpFlow sweep{g, sp, d->level_dev.as<int32_t>(), ev->B, d->depth};
  const bool rides = pl && pl->tile && ev->B <= dp::kRideColumns;  // the SP sweep, with the tiles
  const auto sp_bytes = [&] {
    double bytes = 0.0;
    for (int32_t l = 1; l <= d->depth; ++l) bytes += sp_level_bytes(d, l, ev->B);
    return bytes;
  };
  if (rides) {
    DP_HIP_TRY(dp::launch_sp_arm(sweep, flow_ctl(ev), s));
  } else if (!pl || pl->tile) {  // modeled (or frozen-beta) sweep: one span over all level launches
    SpanGuard sg(ev, SPAN_SP, sp_bytes(), prof && d->depth > 0,
                 ev->schedule == DP_SCHED_PERSISTENT || sp_flows(ev)
                     ? 1
                     : sp_sweep_launches(d, ev->B));
    if (sp_flows(ev)) {
      DP_HIP_TRY(dp::launch_sp_flow(sweep, d->max_level_width, d->has_cell_gates, flow_ctl(ev), s));
    } else if (ev->schedule == DP_SCHED_PERSISTENT) {
      dp::SpLevel lv{sp, ev->B, 0, 0};
      dp::GridBarrier bar;
      DP_TRY(grid_barrier(ev, &bar));
      DP_TRY(on_coop_stream(ev, s, [&](hipStream_t cs) {
        return dp::launch_sp_persistent(g, lv, d->level_dev.as<int32_t>(), d->depth,
                                        (int64_t)d->max_level_width * ev->B, bar, cs);
      }));
    } else {
      for (int32_t l = 1; l <= d->depth;) {
        if (pairs_levels(d, l, ev->B)) {  // levels l and l + 1 in one launch
          const int32_t a0 = d->level_ptr[l], a1 = d->level_ptr[l + 1], b1 = d->level_ptr[l + 2];
          DP_HIP_TRY(dp::launch_sp_pair(g, dp::SpLevel{sp, ev->B, a0, a1 - a0},
                                        dp::SpLevel{sp, ev->B, a1, b1 - a1}, s));
          l += 2;
          continue;
        }
        DP_TRY(for_level_parts(d, l, [&](int32_t g0, int32_t n, bool cells) -> dp_status {
          DP_HIP_TRY(dp::launch_sp_level(g, dp::SpLevel{sp, ev->B, g0, n}, cells, s));
          return DP_OK;
        }));
        ++l;
      }
    }
  }
  if (pl && pl->tile) {
    const int32_t *streams = ev->have_streams ? ev->streams.as<int32_t>() : nullptr;
    const uint64_t *stim = ev->have_stim ? ev->stim.as<uint64_t>() : ev->mstim.as<uint64_t>();
    if (!ev->have_stim) {
      SpanGuard sg(ev, SPAN_STIM, 0.0, prof, 1);
      if (markov(ev))
        DP_HIP_TRY(dp::launch_markov_words(sp, ev->tau.as<float>(), streams, d->n_pi, ev->B, pl->T,
                                           ev->prm.seed, ev->mstim.as<uint64_t>(), s));
      else
        DP_HIP_TRY(dp::launch_stim_words(sp, streams, d->n_pi, ev->B, pl->T, ev->prm.seed,
                                         ev->mstim.as<uint64_t>(), s));
    }
    double bytes = rides ? sp_bytes() : 0.0;
    for (int32_t l = 1; l <= d->depth; ++l)
      bytes += sim_level_bytes(d, l, pl->T, ev->B, ev->B, false);
    SpanGuard sg(ev, SPAN_SIM, bytes, prof, 1);
    uint64_t *edge = ev->words.as<uint64_t>() + (size_t)pl->n_bufs * d->n_nets * pl->tile;
    const size_t n = (size_t)pl->n_tiles * d->n_nets * ev->B;
    const dp::SimFlow t{g, d->level_dev.as<int32_t>(), stim, ev->words.as<uint64_t>(),
                        reinterpret_cast<uint32_t *>(edge + 2 * n), edge, pl->T, d->depth, ev->B,
                        pl->tile, pl->n_tiles, pl->n_bufs};
    dp::FlowCtl ctl = flow_ctl(ev);
    ctl.words += dp::kFlowWords;
    DP_HIP_TRY(dp::launch_sim_flow(t, sweep, d->max_level_width, d->has_cell_gates, ctl, flow_ctl(ev),
                                   ev->ones.as<uint32_t>(), ev->tog.as<uint32_t>(), s));
  } else if (pl) {
    const size_t nb = (size_t)d->n_nets * ev->B;
    DP_HIP_TRY(dp::launch_fill_u32(ev->ones.as<uint32_t>(), (int64_t)nb, 0u, s));
    DP_HIP_TRY(dp::launch_fill_u32(ev->tog.as<uint32_t>(), (int64_t)nb, 0u, s));
    dp::SimTune tune{pick_iters(ev, *pl)};
    const int32_t *streams = ev->have_streams ? ev->streams.as<int32_t>() : nullptr;
    const uint64_t *stim_all = nullptr;  // [B][n_pi][T] words, or the generator
    if (ev->have_stim) {
      stim_all = ev->stim.as<uint64_t>();
    } else if (markov(ev)) {
      SpanGuard sg(ev, SPAN_STIM, 0.0, prof, 1);
      DP_HIP_TRY(dp::launch_markov_words(sp, ev->tau.as<float>(), streams, d->n_pi, ev->B, pl->T,
                                         ev->prm.seed, ev->mstim.as<uint64_t>(), s));
      stim_all = ev->mstim.as<uint64_t>();
    }
    // (column group, chunk) pieces are independent: piece j runs on stream
    // j % L with its own word buffers; the SP of each level is fused into
    // piece 0.
    const int32_t n_pieces = pl->n_groups * pl->n_chunks;
    // a capture records one stream only (multi-stream captures are off)
    const int32_t L = ev->capturing ? 1 : std::min<int32_t>(n_sim_streams(ev), n_pieces);
    if (L > 1) {
      DP_HIP_TRY(hipEventRecord(ev->lane_events[0], s));
      for (int32_t i = 1; i < L; ++i)
        DP_HIP_TRY(hipStreamWaitEvent(ev->lane_streams[i - 1], ev->lane_events[0], 0));
    }
    for (int32_t j = 0; j < n_pieces; ++j) {
      const int32_t grp = j / pl->n_chunks, k = j % pl->n_chunks, lane = j % L;
      const int32_t b = grp * pl->cols;  // first column of the group
      hipStream_t ls = lane == 0 ? s : ev->lane_streams[lane - 1];
      dp::CountView cnt{ev->ones.as<uint32_t>(), ev->tog.as<uint32_t>(), ev->B, b};
      const uint64_t *stim = stim_all ? stim_all + (size_t)b * d->n_pi * pl->T : nullptr;
      const dp::ChunkView cv = chunk_view(ev, *pl, k, lane, grp);
      {
        SpanGuard sg(ev, SPAN_STIM, 0.0, prof, 1, ls);
        DP_HIP_TRY(dp::launch_stimulus(g, cv, cnt, sp, stim, pl->T, streams, ev->prm.seed, tune,
                                       ls));
      }
      const bool fuse = (j == 0);
      const int64_t nw = cv.u_hi - cv.u_lo;
      double bytes = 0.0;
      for (int32_t l = 1; l <= d->depth; ++l)
        bytes += sim_level_bytes(d, l, nw, cv.n_cols, ev->B, fuse);
      // one span over the piece's level launches (their back-to-back time)
      SpanGuard sg(ev, SPAN_SIM, bytes, prof && d->depth > 0, d->depth + d->split_levels, ls);
      for (int32_t l = 1; l <= d->depth; ++l)
        DP_TRY(for_level_parts(d, l, [&](int32_t g0, int32_t n, bool cells) -> dp_status {
          const dp::SpLevel lv{sp, ev->B, g0, n};
          if (!cells) {
            DP_HIP_TRY(dp::launch_sim_level(g, cv, cnt, g0, n, fuse ? &lv : nullptr, false, tune,
                                            ls));
            return DP_OK;
          }
          // library cells: the narrow ones (sorted first) and the wider ones in
          // launches of their own; the range's SP rides with the first
          const int32_t ns = d->lvl_small_cells[l];
          if (ns > 0)
            DP_HIP_TRY(dp::launch_sim_level(g, cv, cnt, g0, ns, fuse ? &lv : nullptr, true, tune,
                                            ls, dp::kSmallCellInputs));
          if (ns < n)
            DP_HIP_TRY(dp::launch_sim_level(g, cv, cnt, g0 + ns, n - ns,
                                            fuse && ns == 0 ? &lv : nullptr, true, tune, ls));
          return DP_OK;
        }));
    }
    if (L > 1)
      for (int32_t i = 1; i < L; ++i) {
        DP_HIP_TRY(hipEventRecord(ev->lane_events[i], ev->lane_streams[i - 1]));
        DP_HIP_TRY(hipStreamWaitEvent(s, ev->lane_events[i], 0));
      }
  }
  return enqueue_forward_tail(ev, pl);
}

// Arguments of the power terms (TR, beta) and their sum over nets, after a
// forward sweep.
dp::PowerArgs power_args(dp_eval *ev, const ChunkPlan *pl) {
  const dp_design *d = ev->d;
  dp::PowerArgs pa{};
  pa.sp = ev->sp.as<float>();
  pa.tog = pl ? ev->tog.as<uint32_t>() : nullptr;
  pa.beta_frozen = ev->prm.mode == DP_FROZEN_BETA ? ev->beta_frozen.as<float>() : nullptr;
  pa.beta_shared = ev->beta_shared;
  pa.cap = ev->cap.as<float>();
  pa.size = ev->S > 0 ? ev->size.as<float>() : nullptr;
  pa.T = pl ? pl->T : 0;
  pa.kappa = (float)kappa_of(ev->prm);
  pa.beta_min = (float)ev->prm.beta_min;
  pa.beta_max = (float)ev->prm.beta_max;
  pa.mode = ev->prm.mode;
  pa.beta = hybrid(ev) ? ev->beta.as<float>() : nullptr;  // hybrid: stored on the way
  pa.n_pi = d->n_pi;
  pa.n_nets = d->n_nets;
  pa.G = d->n_gates;
  pa.B = ev->B;
  pa.S = ev->S;
  pa.paired = ev->paired_sizes;
  pa.partial = ev->power_partial.as<double>();
  pa.n_chunks = dp::power_chunks(d->n_nets);
  pa.power = ev->power.as<float>();
  return pa;
}
dp_status enqueue_forward_tail(dp_eval *ev, const ChunkPlan *pl) {
  DP_HIP_TRY(dp::launch_power(power_args(ev, pl), ev->stream()));
  return DP_OK;
}

// Output helper: a caller pointer, or a staging buffer copied out later.
struct OutMap {
  dp_eval *ev;
  int on_device;
  int slot = 0;
  struct Copy { void *dst; const void *src; size_t bytes; };
  std::vector<Copy> copies;
  template <class T>
  dp_status map(T *user, size_t count, T **dev) {
    *dev = nullptr;
    if (!user) return DP_OK;
    if (on_device) {
      *dev = user;
      return DP_OK;
    }
    DevBuf &b = ev->stage[slot++ % 8];
    DP_TRY(b.alloc(std::max<size_t>(count * sizeof(T), 16)));
    *dev = b.as<T>();
    copies.push_back({user, b.ptr, count * sizeof(T)});
    return DP_OK;
  }
  dp_status flush(hipStream_t s) {
    for (auto &c : copies)
      DP_HIP_TRY(hipMemcpyAsync(c.dst, c.src, c.bytes, hipMemcpyDeviceToHost, s));
    if (!on_device && !copies.empty()) DP_HIP_TRY(hipStreamSynchronize(s));
    return DP_OK;
  }
};

// Capture what `enqueue` puts on the eval's stream into *exec.  The capture
// runs on a private stream (the caller's stream may be the null stream,
// which cannot be captured); the graph is then launched on the caller's
// stream.  An older graph in *exec is destroyed once the stream drains.
template <class F>
dp_status capture_into(dp_eval *ev, hipGraphExec_t *exec, F &&enqueue) {
  if (!ev->capture_stream_owned)
    DP_HIP_TRY(hipStreamCreateWithFlags(&ev->capture_stream_owned, hipStreamNonBlocking));
  if (*exec) {
    DP_HIP_TRY(hipStreamSynchronize(ev->stream()));  // no launch of the old graph in flight
    (void)hipGraphExecDestroy(*exec);
    *exec = nullptr;
  }
  hipStream_t s = ev->capture_stream_owned;
  DP_HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  const bool prof = ev->profiling;
  ev->profiling = false;
  ev->capturing = true;  // stream() is the capture stream meanwhile
  dp_status st = enqueue();
  ev->capturing = false;
  ev->profiling = prof;
  hipGraph_t graph = nullptr;
  hipError_t e = hipStreamEndCapture(s, &graph);
  if (st != DP_OK) {
    if (graph) (void)hipGraphDestroy(graph);
    return st;
  }
  if (e != hipSuccess) return fail(DP_E_HIP, std::string("graph capture failed: ") + hipGetErrorString(e));
  e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) {
    *exec = nullptr;
    return fail(DP_E_HIP, std::string("graph instantiate failed: ") + hipGetErrorString(e));
  }
  return DP_OK;
}

// Capture the forward sweep into ev->graph_fwd.
dp_status capture_forward(dp_eval *ev, const ChunkPlan *pl, uint64_t key) {
  DP_TRY(capture_into(ev, &ev->graph_fwd, [&]() { return enqueue_forward(ev, pl); }));
  ev->graph_key = key;
  return DP_OK;
}

uint64_t graph_key(const dp_eval *ev, const ChunkPlan *pl) {
  uint64_t k = 1469598103934665603ull;
  auto mix = [&](uint64_t v) { k = (k ^ v) * 1099511628211ull; };
  mix((uint64_t)ev->prm.mode);
  mix((uint64_t)ev->prm.beta_grad);
  mix((uint64_t)ev->prm.n_sim);
  mix(ev->prm.seed);
  uint64_t bits;
  double kap = kappa_of(ev->prm);
  std::memcpy(&bits, &kap, 8); mix(bits);
  std::memcpy(&bits, &ev->prm.beta_min, 8); mix(bits);
  std::memcpy(&bits, &ev->prm.beta_max, 8); mix(bits);
  mix((uint64_t)ev->have_stim);
  mix((uint64_t)(uintptr_t)ev->stim.ptr);
  mix((uint64_t)markov(ev));
  mix((uint64_t)(uintptr_t)ev->mstim.ptr);
  mix((uint64_t)(uintptr_t)ev->tau.ptr);
  mix((uint64_t)ev->have_streams);
  mix((uint64_t)(uintptr_t)ev->streams.ptr);
  mix((uint64_t)(uintptr_t)ev->words.ptr);
  mix((uint64_t)(uintptr_t)ev->beta_frozen.ptr);
  mix((uint64_t)(uintptr_t)ev->size.ptr);
  mix((uint64_t)(uintptr_t)ev->stream());
  mix((uint64_t)ev->B);
  mix((uint64_t)ev->S);
  mix((uint64_t)ev->paired_sizes);
  mix((uint64_t)ev->beta_shared);
  mix(flow_limit(ev));
  if (pl) {
    mix((uint64_t)pl->Tc);
    mix((uint64_t)pl->tile);
    mix((uint64_t)pl->n_bufs);
    mix((uint64_t)pl->cols);
    mix((uint64_t)pick_iters(ev, *pl));
    mix((uint64_t)n_sim_streams(ev));
  }
  return k;
}

// Append a device copy to a list, which goes out when it is full.
dp_status list_copy(dp::CopyList *l, const float *src, float *dst, int64_t count, hipStream_t s) {
  if (l->add(src, dst, count)) return DP_OK;
  DP_HIP_TRY(dp::launch_copies(*l, s));
  *l = dp::CopyList{};
  if (l->add(src, dst, count)) return DP_OK;
  DP_HIP_TRY(hipMemcpyAsync(dst, src, (size_t)count * sizeof(float), hipMemcpyDeviceToDevice, s));
  return DP_OK;
}

// Copy the last forward's results out (caller numbering), on the eval's
// stream; host outputs are complete on return.  copies: where not null, takes
// the device copy of the powers instead.
dp_status export_forward(dp_eval *ev, const dp_fwd_out *out, const ChunkPlan *pl,
                         dp::CopyList *copies = nullptr) {
  const dp_design *d = ev->d;
  hipStream_t s = ev->stream();
  OutMap om{ev, out->on_device};
  const int64_t nb = (int64_t)d->n_nets * ev->B;
  dp::ExportArgs ea{};
  ea.sp = ev->sp.as<float>();
  ea.beta = beta_or_null(ev);
  ea.ones = pl ? ev->ones.as<uint32_t>() : nullptr;
  ea.tog = pl ? ev->tog.as<uint32_t>() : nullptr;
  ea.int2ext = d->int2ext.as<int32_t>();
  ea.T = pl ? pl->T : 0;
  ea.n_nets = d->n_nets;
  ea.B = ev->B;
  DP_TRY(om.map(out->sp, nb, &ea.o_sp));
  DP_TRY(om.map(out->tr, nb, &ea.o_tr));
  DP_TRY(om.map(out->sp_acc, nb, &ea.o_sp_acc));
  DP_TRY(om.map(out->tr_acc, nb, &ea.o_tr_acc));
  DP_TRY(om.map(out->beta, nb, &ea.o_beta));
  DP_TRY(om.map(out->tr_hyb, nb, &ea.o_tr_hyb));
  DP_TRY(om.map(out->ones, nb, &ea.o_ones));
  DP_TRY(om.map(out->toggles, nb, &ea.o_tog));
  if (ea.o_sp || ea.o_tr || ea.o_sp_acc || ea.o_tr_acc || ea.o_beta || ea.o_tr_hyb || ea.o_ones ||
      ea.o_tog)
    DP_HIP_TRY(dp::launch_export(ea, s));
  const size_t bytes = (size_t)ev->B * s_prime(ev) * sizeof(float);
  if (out->power && out->on_device && copies) {
    DP_TRY(list_copy(copies, ev->power.as<float>(), out->power, (int64_t)ev->B * s_prime(ev), s));
  } else if (out->power) {
    DP_HIP_TRY(hipMemcpyAsync(out->power, ev->power.ptr, bytes,
                              out->on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, s));
  }
  DP_TRY(om.flush(s));
  if (!out->on_device && out->power) DP_HIP_TRY(hipStreamSynchronize(s));
  return DP_OK;
}

// Arguments of the reverse sweep over C columns with upstream weights w
// (device, or null = 1).
dp::BwdArgs backward_args(dp_eval *ev, const float *w, int per_column, int32_t C) {
  const dp_design *d = ev->d;
  dp::BwdArgs ba{};
  ba.sp = ev->sp.as<float>();
  if (ev->beta_shared && ev->prm.mode == DP_FROZEN_BETA) {  // one beta per net (serving)
    ba.beta = ev->beta_frozen.as<float>();
    ba.beta_shared = 1;
  } else {
    ba.beta = beta_or_null(ev);
  }
  ba.cap = ev->cap.as<float>();
  ba.w = w;
  ba.size = ev->S > 0 ? ev->size.as<float>() : nullptr;
  ba.contrib = ev->contrib.as<float>();
  ba.kappa = (float)kappa_of(ev->prm);
  ba.n_pi = d->n_pi;
  ba.G = d->n_gates;
  ba.B = ev->B;
  ba.S = ev->S;
  ba.C = C;
  ba.cdiv = per_column ? s_prime(ev) : 1;
  ba.ste = ev->prm.beta_grad == DP_BETA_STE;
  ba.per_column = per_column;
  ba.paired = ev->paired_sizes;
  ba.fixed = ev->have_fixed ? ev->fixed.as<uint8_t>() : nullptr;
  return ba;
}

// Enqueue the reverse levels and the PI adjoints into dst [C][n_pi] (device)
// on the eval's stream; no allocation, no host synchronisation.
dp_status enqueue_backward(dp_eval *ev, const dp::BwdArgs &ba, float *dst) {
  const dp_design *d = ev->d;
  hipStream_t s = ev->stream();
  const dp::GraphView g = view(d);
  double bwd_bytes = 0.0;
  for (int32_t l = d->depth; l >= 1; --l) bwd_bytes += bwd_level_bytes(d, l, ba.C);
  if (bwd_flows(ev, ba.C) && have_flow_scratch(ev, ba.C)) {
    const dp::FlowCtl ctl = flow_ctl(ev);
    SpanGuard sg(ev, SPAN_BWD, bwd_bytes, ev->profiling && d->depth > 0, 1);
    DP_HIP_TRY(dp::launch_bwd_flow(
        dp::BwdFlow{g, ba, dst, ev->seed.as<float>(), ev->part.as<float>(),
                    d->level_dev.as<int32_t>(), d->n_edges, d->depth},
        std::max(d->max_level_width, d->n_pi), d->has_cell_gates, ctl, s));
    return DP_OK;
  }
  if (wide_reverse(ev, ba.C, ba.per_column) && !ba.lam) {
    float *lam = ev->contrib.as<float>(), *part = ev->part.as<float>();
    SpanGuard sg(ev, SPAN_BWD, bwd_bytes, ev->profiling && d->depth > 0, d->depth);
    DP_HIP_TRY(dp::launch_edge_partials(g, ba.sp, ba.B, d->has_cell_gates, part, s));
    for (int32_t l = d->depth; l >= 1; --l) {
      const int32_t g0 = d->level_ptr[l], n = d->level_ptr[l + 1] - g0;
      const dp::HeavySpan hs = dp::heavy_span(d, g0, n);
      DP_HIP_TRY(dp::launch_bwd_wide_level(g, ba, part, lam, d->n_pi + g0, n, s, hs.gates, hs.n));
    }
    const dp::HeavySpan hp = dp::heavy_pis(d);
    DP_HIP_TRY(dp::launch_bwd_wide_level(g, ba, part, lam, 0, d->n_pi, s, hp.gates, hp.n));
    DP_HIP_TRY(dp::launch_bwd_wide_out(lam, d->n_pi, ba.C, dst, s));
    return DP_OK;
  }
  if (ev->schedule == DP_SCHED_PERSISTENT) {
    dp::GridBarrier bar;
    DP_TRY(grid_barrier(ev, &bar));
    SpanGuard sg(ev, SPAN_BWD, bwd_bytes, ev->profiling && d->depth > 0, d->depth);
    return on_coop_stream(ev, s, [&](hipStream_t cs) {
      return dp::launch_bwd_persistent(g, ba, d->level_dev.as<int32_t>(), d->depth,
                                       (int64_t)d->max_level_width * ba.C, dst, bar, cs);
    });
  }
  {
    SpanGuard sg(ev, SPAN_BWD, bwd_bytes, ev->profiling && d->depth > 0, d->depth + d->split_levels);
    for (int32_t l = d->depth; l >= 1; --l)
      DP_TRY(for_level_parts(d, l, [&](int32_t g0, int32_t n, bool cells) -> dp_status {
        const dp::HeavySpan hs = dp::heavy_span(d, g0, n);
        DP_HIP_TRY(dp::launch_bwd_level(g, ba, g0, n, cells, s, hs.gates, hs.n));
        return DP_OK;
      }));
  }
  const dp::HeavySpan hp = dp::heavy_pis(d);
  DP_HIP_TRY(dp::launch_bwd_pi(g, ba, dst, s, hp.gates, hp.n));
  return DP_OK;
}

// Every argument the reverse sweep's launches take (a captured sweep is
// replayed only while all of them are unchanged).
uint64_t reverse_key(const dp_eval *ev, const dp::BwdArgs &ba, const float *dst) {
  uint64_t k = 1469598103934665603ull;
  auto mix = [&](uint64_t v) { k = (k ^ v) * 1099511628211ull; };
  for (const void *ptr : {(const void *)ba.sp, (const void *)ba.beta, (const void *)ba.cap,
                          (const void *)ba.w, (const void *)ba.size, (const void *)ba.contrib,
                          (const void *)ba.lam, (const void *)ba.fixed, (const void *)dst,
                          (const void *)ev->part.ptr, (const void *)ev->seed.ptr,
                          (const void *)ev->stream()})
    mix((uint64_t)(uintptr_t)ptr);
  mix((uint64_t)have_flow_scratch(ev, ba.C));
  uint32_t kb;
  std::memcpy(&kb, &ba.kappa, 4);
  mix(kb);
  mix(flow_limit(ev));
  for (int32_t v : {ba.n_pi, ba.G, ba.B, ba.S, ba.C, ba.cdiv, ba.ste, ba.per_column, ba.paired,
                    ba.beta_shared})
    mix((uint64_t)(uint32_t)v);
  return k;
}

// The reverse sweep of run_backward: under DP_SCHED_GRAPH captured once
// into ev->graph_bwd (re-captured when any launch argument changes) and
// replayed, otherwise enqueued launch by launch.
dp_status reverse_sweep(dp_eval *ev, const dp::BwdArgs &ba, float *dst) {
  const dp_design *d = ev->d;
  if (ev->schedule != DP_SCHED_GRAPH || ev->profiling || reverse_launches(d) > kMaxGraphLaunches)
    return enqueue_backward(ev, ba, dst);
  const uint64_t k = reverse_key(ev, ba, dst);
  if (!ev->graph_bwd || ev->graph_bwd_key != k) {
    DP_TRY(capture_into(ev, &ev->graph_bwd, [&]() { return enqueue_backward(ev, ba, dst); }));
    ev->graph_bwd_key = k;
  }
  DP_HIP_TRY(hipGraphLaunch(ev->graph_bwd, ev->stream()));
  return DP_OK;
}

}  // namespace

namespace dp {
// Takes note of failures that an eval's groups report and lets go of those
// that are gone; done_only: looks at these alone (nothing of theirs is running).
void note_shared(dp_eval *ev, bool done_only) {
  for (size_t i = 0; i < ev->shared_reports.size();) {
    dp_eval::Shared &r = ev->shared_reports[i];
    std::unique_lock<std::mutex> lock(r.report->mu);
    const bool done = r.report->done;
    if (done || !done_only) {
      const uint64_t n = r.report->count();
      ev->shared_failed = ev->shared_failed || n != r.seen;
      r.seen = n;
    }
    lock.unlock();
    if (done) ev->shared_reports.erase(ev->shared_reports.begin() + i);
    else ++i;
  }
}
// Launches that concern the eval report there from now on.
void join_shared(dp_eval *ev, const std::shared_ptr<SharedReport> &report) {
  for (const dp_eval::Shared &r : ev->shared_reports)
    if (r.report == report) return;
  note_shared(ev, true);
  std::lock_guard<std::mutex> lock(report->mu);
  ev->shared_reports.push_back({report, report->failures});
}
dp_status flow_status(dp_eval *ev) {
  note_shared(ev, false);
  bool bad = ev->shared_failed;
  ev->shared_failed = false;
  if (volatile uint32_t *own = ev->flow_report; own && *own != 0u) {
    *own = 0u;
    bad = true;
  }
  if (!bad) return DP_OK;
  return fail(DP_E_HIP, "a sweep's wait for its own results gave up; that sweep's outputs are NaN "
                        "and not a result");
}
dp_status params_ok(const dp_params *p) { return check_params(p); }
double kappa(const dp_params &p) { return kappa_of(p); }
}  // namespace dp

dp_eval::~dp_eval() {
  if (graph_fwd) (void)hipGraphExecDestroy(graph_fwd);
  if (graph_bwd) (void)hipGraphExecDestroy(graph_bwd);
  if (graph_fb) (void)hipGraphExecDestroy(graph_fb);
  if (capture_stream_owned) (void)hipStreamDestroy(capture_stream_owned);
  if (flow_report) reports->give(flow_report);
  if (check_report) reports->give(check_report);
  if (coop_stream) {
    (void)hipStreamSynchronize(coop_stream);
    (void)hipStreamDestroy(coop_stream);
  }
  for (auto e : coop_events)
    if (e) (void)hipEventDestroy(e);
  for (auto e : ev_pool) (void)hipEventDestroy(e);
  for (auto st : lane_streams) {
    (void)hipStreamSynchronize(st);
    (void)hipStreamDestroy(st);
  }
  for (auto e : lane_events) (void)hipEventDestroy(e);
}

// =========================================================================
extern "C" {

void dp_params_default(dp_params *p) {
  if (!p) return;
  p->vdd = 1.0;
  p->fclk = 1.0;
  p->energy_factor = 0.5;
  p->beta_min = 0.1;
  p->beta_max = 10.0;
  p->mode = DP_MODELED;
  p->beta_grad = DP_BETA_LOCAL;
  p->n_sim = 4096;
  p->seed = 1;
}

const char *dp_last_error(void) { return dp::g_err.c_str(); }
const char *dp_version(void) { return kVersion; }

dp_status dp_ctx_create(int32_t device, void *hip_stream, dp_ctx **out) {
  if (!out) return fail(DP_E_INVALID, "dp_ctx_create: NULL out");
  int n = 0;
  DP_HIP_TRY(hipGetDeviceCount(&n));
  if (device < 0 || device >= n)
    return fail(DP_E_INVALID, "dp_ctx_create: no device " + std::to_string(device));
  DP_HIP_TRY(hipSetDevice(device));
  DP_TRY(dp::static_scratch_init(device));  // once per device: dp_forward_static's scratch
  int n_cu = 0;
  DP_HIP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device));
  auto *c = new dp_ctx();
  c->device = device;
  c->n_cu = n_cu;
  if (hip_stream == (void *)hipStreamLegacy) {
    c->stream = nullptr;  // the null stream
  } else if (hip_stream) {
    c->stream = (hipStream_t)hip_stream;
  } else {
    hipError_t e = hipStreamCreateWithFlags(&c->owned, hipStreamNonBlocking);
    if (e != hipSuccess) {
      delete c;
      return fail(DP_E_HIP, std::string("hipStreamCreate failed: ") + hipGetErrorString(e));
    }
    c->stream = c->owned;
  }
  *out = c;
  return DP_OK;
}

dp_status dp_ctx_set_stream(dp_ctx *ctx, void *hip_stream) {
  if (!ctx) return fail(DP_E_INVALID, "dp_ctx_set_stream: NULL ctx");
  if (hip_stream == (void *)hipStreamLegacy) {
    ctx->stream = nullptr;  // the null stream
    return DP_OK;
  }
  if (!hip_stream && !ctx->owned) {
    DP_HIP_TRY(hipSetDevice(ctx->device));
    DP_HIP_TRY(hipStreamCreateWithFlags(&ctx->owned, hipStreamNonBlocking));
  }
  ctx->stream = hip_stream ? (hipStream_t)hip_stream : ctx->owned;
  return DP_OK;
}

dp_status dp_ctx_synchronize(dp_ctx *ctx) {
  if (!ctx) return fail(DP_E_INVALID, "dp_ctx_synchronize: NULL ctx");
  DP_HIP_TRY(hipStreamSynchronize(ctx->stream));
  return DP_OK;
}

void dp_ctx_destroy(dp_ctx *ctx) {
  if (ctx) dp::ctx_release(ctx);
}

dp_status dp_compile(dp_ctx *ctx, const dp_netlist *netlist, dp_design **out) {
  if (ctx) {
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return fail(DP_E_HIP, std::string("hipSetDevice: ") + hipGetErrorString(e));
  }
  return dp::compile_design(ctx, netlist, 0, nullptr, nullptr, out);
}

dp_status dp_compile_cells(dp_ctx *ctx, const dp_netlist *netlist, int32_t n_cells,
                           const char *const *cells, dp_design **out) {
  if (ctx) {
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return fail(DP_E_HIP, std::string("hipSetDevice: ") + hipGetErrorString(e));
  }
  return dp::compile_design(ctx, netlist, n_cells, cells, nullptr, out);
}

dp_status dp_compile_library(dp_ctx *ctx, const dp_netlist *netlist, int32_t n_cells,
                             const char *const *cells, const char *const *pins,
                             dp_design **out) {
  if (ctx) {
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return fail(DP_E_HIP, std::string("hipSetDevice: ") + hipGetErrorString(e));
  }
  return dp::compile_design(ctx, netlist, n_cells, cells, pins, out);
}

dp_status dp_design_cell_logic(const dp_design *d, int32_t *logic, int32_t *n_logic) {
  if (!d) return fail(DP_E_INVALID, "dp_design_cell_logic: NULL design");
  if (logic && !d->h_cell_logic.empty())
    std::memcpy(logic, d->h_cell_logic.data(), sizeof(int32_t) * d->h_cell_logic.size());
  if (n_logic) *n_logic = d->n_cells;
  return DP_OK;
}

dp_status dp_design_info(const dp_design *d, dp_design_info_t *out) {
  if (!d || !out) return fail(DP_E_INVALID, "dp_design_info: NULL argument");
  out->n_pi = d->n_pi;
  out->n_gates = d->n_gates;
  out->n_nets = d->n_nets;
  out->depth = d->depth;
  out->n_edges = d->n_edges;
  out->max_level_width = d->max_level_width;
  out->reserved = 0;
  out->device_bytes = d->device_bytes;
  return DP_OK;
}

dp_status dp_design_levels(const dp_design *d, int32_t *level) {
  if (!d || !level) return fail(DP_E_INVALID, "dp_design_levels: NULL argument");
  std::memcpy(level, d->h_level.data(), sizeof(int32_t) * d->n_nets);
  return DP_OK;
}

void dp_design_destroy(dp_design *d) {
  if (d) dp::design_release(d);
}

dp_status dp_eval_create(dp_design *d, int32_t n_cols, int32_t n_size, const dp_params *params,
                         dp_eval **out) {
  if (!d || !out) return fail(DP_E_INVALID, "dp_eval_create: NULL argument");
  if (n_cols < 1 || n_size < 0) return fail(DP_E_INVALID, "dp_eval_create: need B >= 1, S >= 0");
  DP_TRY(check_params(params));
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  auto *ev = new dp_eval();
  ev->d = d;
  ev->B = n_cols;
  ev->S = n_size;
  ev->prm = *params;
  dp_status st = ev->sp.alloc((size_t)d->n_nets * n_cols * sizeof(float));
  if (st == DP_OK) st = ev->cap.alloc((size_t)d->n_nets * sizeof(float));
  if (st == DP_OK && n_size > 0) st = ev->size.alloc((size_t)n_size * d->n_gates * sizeof(float));
  if (st != DP_OK) {
    delete ev;
    return st;
  }
  dp::design_retain(d);
  *out = ev;
  return DP_OK;
}

dp_status dp_eval_set_params(dp_eval *ev, const dp_params *params) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_set_params: NULL eval");
  DP_TRY(check_params(params));
  ev->prm = *params;
  ev->inputs_version++;
  return DP_OK;
}

void dp_eval_destroy(dp_eval *ev) {
  if (!ev) return;
  (void)hipStreamSynchronize(ev->stream());
  dp_design *d = ev->d;
  delete ev;
  dp::design_release(d);
}

dp_status dp_set_pi_prob(dp_eval *ev, const float *p, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_pi_prob: NULL eval");
  const dp_design *d = ev->d;
  const int64_t n = (int64_t)ev->B * d->n_pi;
  if (n == 0) {
    ev->have_pi = true;
    ev->inputs_version++;
    return DP_OK;
  }
  DP_TRY(check_values(ev, p, n, 0.0f, 1.0f, on_device, "dp_set_pi_prob"));
  hipStream_t s = ev->stream();
  const float *src;
  DP_TRY(import_from(ev->p_stage, p, n * sizeof(float), on_device, s, &src));
  DP_HIP_TRY(dp::launch_load_pi(src, ev->sp.as<float>(), d->n_pi, ev->B, s));
  if (!on_device) DP_HIP_TRY(hipStreamSynchronize(s));
  ev->have_pi = true;
  ev->inputs_version++;
  return DP_OK;
}

dp_status dp_set_caps(dp_eval *ev, const float *cap, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_caps: NULL eval");
  const dp_design *d = ev->d;
  DP_TRY(check_values(ev, cap, d->n_nets, 0.0f, 3.0e38f, on_device, "dp_set_caps"));
  hipStream_t s = ev->stream();
  const float *src;
  DP_TRY(import_from(ev->cap_stage, cap, (size_t)d->n_nets * sizeof(float), on_device, s, &src));
  DP_HIP_TRY(dp::launch_gather_nets_f32(src, d->int2ext.as<int32_t>(),
                                        ev->cap.as<float>(), d->n_nets, s));
  if (!on_device) DP_HIP_TRY(hipStreamSynchronize(s));
  ev->have_cap = true;
  ev->inputs_version++;
  return DP_OK;
}

dp_status dp_set_cell_sizes(dp_eval *ev, const float *size, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_cell_sizes: NULL eval");
  if (ev->S == 0) return fail(DP_E_INVALID, "dp_set_cell_sizes: eval was created with S = 0");
  const dp_design *d = ev->d;
  const int64_t n = (int64_t)ev->S * d->n_gates;
  DP_TRY(check_values(ev, size, n, 0.0f, 3.0e38f, on_device, "dp_set_cell_sizes"));
  hipStream_t s = ev->stream();
  const float *src;
  DP_TRY(import_from(ev->size_stage, size, n * sizeof(float), on_device, s, &src));
  DP_HIP_TRY(dp::launch_import_sizes(src, d->int2ext.as<int32_t>(), d->ext2int.as<int32_t>(),
                                     ev->size.as<float>(), d->n_pi, d->n_gates, ev->S, s));
  if (!on_device) DP_HIP_TRY(hipStreamSynchronize(s));
  ev->have_size = true;
  ev->inputs_version++;
  return DP_OK;
}

dp_status dp_set_beta(dp_eval *ev, const float *beta, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_beta: NULL eval");
  const dp_design *d = ev->d;
  const int64_t n = (int64_t)ev->B * d->n_nets;
  DP_TRY(check_values(ev, beta, n, 0.0f, 3.0e38f, on_device, "dp_set_beta"));
  hipStream_t s = ev->stream();
  DP_TRY(ev->beta_frozen.alloc(n * sizeof(float)));
  const float *src;
  DP_TRY(import_from(ev->beta_stage, beta, n * sizeof(float), on_device, s, &src));
  DP_HIP_TRY(dp::launch_import_cols_f32(src, d->int2ext.as<int32_t>(),
                                        ev->beta_frozen.as<float>(), d->n_nets, ev->B, s));
  if (!on_device) DP_HIP_TRY(hipStreamSynchronize(s));
  ev->have_beta = true;
  ev->inputs_version++;
  return DP_OK;
}

dp_status dp_set_stimulus(dp_eval *ev, const uint64_t *words, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_stimulus: NULL eval");
  ev->inputs_version++;
  if (!words) {
    ev->have_stim = false;
    return DP_OK;
  }
  const dp_design *d = ev->d;
  const int64_t T = n_words(ev->prm);
  if (T <= 0) return fail(DP_E_INVALID, "dp_set_stimulus: params.n_sim is 0");
  const size_t bytes = (size_t)ev->B * d->n_pi * T * sizeof(uint64_t);
  hipStream_t s = ev->stream();
  DP_TRY(stage_in(ev->stim, words, bytes, on_device, s));
  if (!on_device) DP_HIP_TRY(hipStreamSynchronize(s));
  ev->have_stim = true;
  return DP_OK;
}

dp_status dp_set_pi_rates(dp_eval *ev, const float *tau, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_pi_rates: NULL eval");
  ev->inputs_version++;
  if (!tau) {
    ev->have_tau = false;
    return DP_OK;
  }
  const int64_t n = (int64_t)ev->B * ev->d->n_pi;
  if (n > 0) {
    DP_TRY(check_values(ev, tau, n, 0.0f, 1.0f, on_device, "dp_set_pi_rates"));
    hipStream_t s = ev->stream();
    DP_TRY(stage_in(ev->tau, tau, (size_t)n * sizeof(float), on_device, s));
    if (!on_device) DP_HIP_TRY(hipStreamSynchronize(s));
  }
  ev->have_tau = true;
  return DP_OK;
}

dp_status dp_set_pi_streams(dp_eval *ev, const int32_t *stream) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_pi_streams: NULL eval");
  ev->inputs_version++;
  if (!stream) {
    ev->have_streams = false;
    return DP_OK;
  }
  const int32_t n_pi = ev->d->n_pi;
  for (int32_t i = 0; i < n_pi; ++i)
    if (stream[i] < 0 || stream[i] >= n_pi)
      return fail(DP_E_INVALID, "dp_set_pi_streams: stream " + std::to_string(stream[i]) +
                                    " of PI " + std::to_string(i) + " is not a PI");
  if (n_pi > 0) {
    hipStream_t s = ev->stream();
    DP_TRY(stage_in(ev->streams, stream, (size_t)n_pi * sizeof(int32_t), 0, s));
    DP_HIP_TRY(hipStreamSynchronize(s));
  }
  ev->have_streams = true;
  return DP_OK;
}

dp_status dp_set_pi_fixed(dp_eval *ev, const uint8_t *fixed) {
  if (!ev) return fail(DP_E_INVALID, "dp_set_pi_fixed: NULL eval");
  ev->have_fixed = false;  // read by the reverse sweep only: the forward stays valid
  const int32_t n_pi = ev->d->n_pi;
  if (!fixed || n_pi == 0) return DP_OK;
  hipStream_t s = ev->stream();
  DP_TRY(stage_in(ev->fixed, fixed, (size_t)n_pi, 0, s));
  DP_HIP_TRY(hipStreamSynchronize(s));
  ev->have_fixed = true;
  return DP_OK;
}

dp_status dp_eval_set_schedule(dp_eval *ev, int32_t schedule, int64_t words_per_chunk,
                               int32_t sim_pairs_per_lane) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_set_schedule: NULL eval");
  if (schedule < DP_SCHED_AUTO || schedule > DP_SCHED_PERSISTENT)
    return fail(DP_E_INVALID, "dp_eval_set_schedule: unknown schedule");
  if (words_per_chunk < 0 || (words_per_chunk > 0 && words_per_chunk < 2))
    return fail(DP_E_INVALID, "dp_eval_set_schedule: words_per_chunk must be 0 or >= 2");
  if (!(sim_pairs_per_lane == 0 || sim_pairs_per_lane == 1 || sim_pairs_per_lane == 2 ||
        sim_pairs_per_lane == 4 || sim_pairs_per_lane == 8))
    return fail(DP_E_INVALID, "dp_eval_set_schedule: sim_pairs_per_lane must be 0, 1, 2, 4 or 8");
  if (schedule == DP_SCHED_PERSISTENT && ev->d->has_cell_gates)
    return fail(DP_E_UNSUPPORTED,
                "dp_eval_set_schedule: the persistent schedule runs the fixed cells only");
  if (schedule == DP_SCHED_PERSISTENT && !ev->barrier.ptr) {
    DP_TRY(ev->barrier.alloc(dp::kBarrierAlloc * sizeof(uint32_t)));
    DP_HIP_TRY(dp::launch_fill_u32(ev->barrier.as<uint32_t>(), dp::kBarrierAlloc, 0u, ev->stream()));
  }
  ev->schedule = schedule;
  ev->words_per_chunk = words_per_chunk;
  ev->sim_iters = sim_pairs_per_lane;
  return DP_OK;
}

static dp_status run_backward(dp_eval *ev, const float *grad_power, int per_column,
                              float *dpi, float *dcap, float *dsize, int32_t on_device);

dp_status dp_eval_autotune(dp_eval *ev, int32_t reps, int32_t with_backward, double *best_ms) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_autotune: NULL eval");
  if (reps < 1) reps = 1;
  const int32_t s0 = ev->schedule, i0 = ev->sim_iters, l0 = ev->sim_streams;
  const int64_t c0 = ev->words_per_chunk;
  const bool prof = ev->profiling;
  ev->profiling = false;
  struct Cand { int32_t sched; int32_t iters; int64_t chunk; int32_t lanes; };
  std::vector<Cand> cands;
  const int64_t T = n_words(ev->prm);
  if (hybrid(ev)) {
    DP_TRY(ensure_flow(ev));
    // automatic chunks on one stream may be word tiles; whole rows in level
    // launches are then a chunk of T words
    ev->words_per_chunk = ev->sim_streams = 0;
    ev->schedule = DP_SCHED_LEVEL;  // (as the candidates': the persistent one has no tiles)
    const bool tiles = plan_chunks(ev).tile > 0;
    ev->schedule = s0;
    ev->words_per_chunk = c0;
    ev->sim_streams = l0;
    if (tiles)
      for (int32_t sc : {DP_SCHED_LEVEL, DP_SCHED_GRAPH}) cands.push_back({sc, 1, 0, 1});
    const int64_t chunks[3] = {tiles ? T : 0, (T / 2 + 1) & ~1ll, (T / 4 + 1) & ~1ll};
    for (int k = 0; k < 3; ++k) {
      if (k > 0 && chunks[k] < 128) continue;
      for (int32_t lanes : {1, 2, 4}) {
        const int64_t keep_chunk = ev->words_per_chunk;
        const int32_t keep_lanes = ev->sim_streams;
        ev->words_per_chunk = chunks[k];
        ev->sim_streams = lanes;
        const ChunkPlan cp = plan_chunks(ev);
        ev->words_per_chunk = keep_chunk;
        ev->sim_streams = keep_lanes;
        const int64_t pieces = (int64_t)cp.n_groups * cp.n_chunks;  // independent pieces
        if (lanes > 1 && lanes > pieces) continue;
        if ((int64_t)lanes * ev->d->n_nets * 8 * (k == 0 ? T : chunks[k] + 2) > kAutoWordBudget)
          continue;
        for (int32_t it : {1, 2, 4, 8})
          for (int32_t sc : {DP_SCHED_LEVEL, DP_SCHED_GRAPH}) cands.push_back({sc, it, chunks[k], lanes});
      }
    }
  } else {
    for (int32_t sc : {DP_SCHED_LEVEL, DP_SCHED_GRAPH}) cands.push_back({sc, 0, 0, 1});
  }
  DevBuf bwd_out;  // scratch for the timed reverse sweeps
  if (with_backward) DP_TRY(bwd_out.alloc((size_t)ev->B * std::max(ev->d->n_pi, 1) * 4));
  hipStream_t s = ev->stream();
  hipEvent_t e0 = nullptr, e1 = nullptr;
  DP_HIP_TRY(hipEventCreate(&e0));
  DP_HIP_TRY(hipEventCreate(&e1));
  double best = 1e300;
  Cand win{s0, i0, c0, l0};
  dp_status st = DP_OK;
  for (const Cand &c : cands) {
    ev->schedule = c.sched;
    ev->sim_iters = c.iters;
    ev->words_per_chunk = c.chunk;
    ev->sim_streams = c.lanes;
    if (c.sched == DP_SCHED_GRAPH) {
      if (c.lanes > 1) continue;  // a graph is captured on one stream: same as lanes = 1
      ChunkPlan cp;
      if (hybrid(ev)) cp = plan_chunks(ev);
      if (forward_launches(ev, hybrid(ev) ? &cp : nullptr) > kMaxGraphLaunches) continue;
    }
    auto once = [&]() -> dp_status {
      dp_status r = dp_forward(ev, nullptr);
      if (r == DP_OK && with_backward)
        r = run_backward(ev, nullptr, 0, bwd_out.as<float>(), nullptr, nullptr, 1);
      return r;
    };
    if ((st = once()) != DP_OK) break;  // warm-up, graph capture
    if (hipEventRecord(e0, s) != hipSuccess) { st = fail(DP_E_HIP, "autotune: event"); break; }
    for (int32_t r = 0; r < reps && st == DP_OK; ++r) st = once();
    if (st != DP_OK) break;
    float ms = 0.0f;
    if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
      st = fail(DP_E_HIP, "autotune: event timing failed");
      break;
    }
    if (ms / reps < best) {
      best = ms / reps;
      win = c;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  ev->profiling = prof;
  ev->schedule = win.sched;
  ev->sim_iters = win.iters;
  ev->words_per_chunk = win.chunk;
  ev->sim_streams = win.lanes;
  if (st != DP_OK) return st;
  if (best_ms) *best_ms = best;
  return DP_OK;
}

dp_status dp_eval_set_sim_streams(dp_eval *ev, int32_t sim_streams) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_set_sim_streams: NULL eval");
  if (sim_streams < 0 || sim_streams > 16)
    return fail(DP_E_INVALID, "dp_eval_set_sim_streams: need 0 <= sim_streams <= 16");
  ev->sim_streams = sim_streams;
  return DP_OK;
}

dp_status dp_eval_set_sim_columns(dp_eval *ev, int32_t columns) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_set_sim_columns: NULL eval");
  if (columns < 0) return fail(DP_E_INVALID, "dp_eval_set_sim_columns: need columns >= 0");
  ev->sim_cols = columns;
  return DP_OK;
}

dp_status dp_eval_get_schedule(const dp_eval *ev, int32_t *schedule, int64_t *words_per_chunk,
                               int32_t *sim_pairs_per_lane, int32_t *sim_streams) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_get_schedule: NULL eval");
  if (schedule) *schedule = ev->schedule;
  if (words_per_chunk) *words_per_chunk = ev->words_per_chunk;
  if (sim_pairs_per_lane) *sim_pairs_per_lane = ev->sim_iters;
  if (sim_streams) *sim_streams = n_sim_streams(ev);
  return DP_OK;
}

dp_status dp_eval_synchronize(dp_eval *ev) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_synchronize: NULL eval");
  DP_HIP_TRY(hipSetDevice(ev->d->ctx->device));
  DP_HIP_TRY(hipStreamSynchronize(ev->stream()));
  return barrier_status(ev);
}

dp_status dp_eval_set_barrier_timeout(dp_eval *ev, double microseconds) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_set_barrier_timeout: NULL eval");
  if (!(microseconds >= 0.0) || !std::isfinite(microseconds))
    return fail(DP_E_INVALID, "dp_eval_set_barrier_timeout: need a finite time >= 0");
  ev->barrier_limit_us = microseconds;
  return DP_OK;
}

dp_status dp_eval_profile(dp_eval *ev, int32_t enable) {
  if (!ev) return fail(DP_E_INVALID, "dp_eval_profile: NULL eval");
  ev->profiling = enable != 0;
  ev->prof = dp_profile{};
  return DP_OK;
}

dp_status dp_eval_get_profile(dp_eval *ev, dp_profile *out) {
  if (!ev || !out) return fail(DP_E_INVALID, "dp_eval_get_profile: NULL argument");
  DP_TRY(resolve_profile(ev));
  *out = ev->prof;
  return DP_OK;
}

dp_status dp_forward(dp_eval *ev, const dp_fwd_out *out) {
  if (!ev) return fail(DP_E_INVALID, "dp_forward: NULL eval");
  const dp_design *d = ev->d;
  if (!ev->have_pi) return fail(DP_E_STATE, "dp_forward: PI probabilities not set");
  if (!ev->have_cap) return fail(DP_E_STATE, "dp_forward: capacitances not set");
  if (ev->S > 0 && !ev->have_size) return fail(DP_E_STATE, "dp_forward: cell sizes not set");
  if (ev->prm.mode == DP_FROZEN_BETA && !ev->have_beta)
    return fail(DP_E_STATE, "dp_forward: DP_FROZEN_BETA needs dp_set_beta");
  const bool hyb = hybrid(ev);
  if (out && !hyb && (out->sp_acc || out->tr_acc || out->ones || out->toggles))
    return fail(DP_E_INVALID, "dp_forward: simulation outputs need DP_HYBRID");
  if (hyb && ev->have_stim &&
      ev->stim.bytes < (size_t)ev->B * d->n_pi * n_words(ev->prm) * sizeof(uint64_t))
    return fail(DP_E_STATE, "dp_forward: the explicit stimulus is shorter than n_sim/64 words");
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  hipStream_t s = ev->stream();
  ChunkPlan plan;
  const ChunkPlan *pl;
  DP_TRY(plan_forward(ev, &plan, &pl));
  if (ev->schedule == DP_SCHED_GRAPH && forward_launches(ev, pl) > kMaxGraphLaunches)
    return fail(DP_E_UNSUPPORTED, "dp_forward: the sweep has " +
                std::to_string(forward_launches(ev, pl)) + " launches, more than the " +
                std::to_string(kMaxGraphLaunches) + " a graph may hold; use DP_SCHED_LEVEL");
  const bool use_graph = ev->schedule == DP_SCHED_GRAPH && !ev->profiling;
  if (use_graph) {
    const uint64_t key = graph_key(ev, pl);
    if (!ev->graph_fwd || ev->graph_key != key) DP_TRY(capture_forward(ev, pl, key));
    DP_HIP_TRY(hipGraphLaunch(ev->graph_fwd, s));
  } else {
    DP_TRY(enqueue_forward(ev, pl));
  }
  ev->fwd_version = ev->inputs_version;
  if (out) DP_TRY(export_forward(ev, out, pl));
  if (out && !out->on_device) DP_TRY(sync_and_check(ev));
  return DP_OK;
}

static dp_status run_backward(dp_eval *ev, const float *grad_power, int per_column,
                              float *dpi, float *dcap, float *dsize, int32_t on_device) {
  const dp_design *d = ev->d;
  if (ev->fwd_version != ev->inputs_version || ev->fwd_version == 0)
    return fail(DP_E_STATE, "dp_backward: no completed forward for the current inputs");
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  hipStream_t s = ev->stream();
  const int32_t Sp = s_prime(ev);
  const int32_t cols = ev->B * Sp;
  const int32_t C = per_column ? cols : ev->B;
  const float *w = nullptr;
  if (grad_power) {
    DP_TRY(ev->w.alloc(std::max<size_t>((size_t)cols * sizeof(float), 16)));
    DP_TRY(check_values(ev, grad_power, cols, -3.0e38f, 3.0e38f, on_device, "dp_backward grad",
                        ev->w.as<float>()));
    if (!on_device)
      DP_TRY(stage_in(ev->w, grad_power, (size_t)cols * sizeof(float), 0, s));
    w = ev->w.as<float>();
  }
  if (dpi) {
    DP_TRY(ensure_reverse_buffers(ev, C, per_column));
    const dp::BwdArgs ba = backward_args(ev, w, per_column, C);
    float *dst = dpi;
    const size_t bytes = (size_t)C * d->n_pi * sizeof(float);
    if (!on_device) {
      DP_TRY(ev->pi_out.alloc(std::max<size_t>(bytes, 16)));
      dst = ev->pi_out.as<float>();
    }
    DP_TRY(reverse_sweep(ev, ba, dst));
    if (!on_device && bytes)
      DP_HIP_TRY(hipMemcpyAsync(dpi, dst, bytes, hipMemcpyDeviceToHost, s));
  }
  if (dcap || (dsize && ev->S > 0)) {
    OutMap om{ev, on_device};
    dp::GradExportArgs ga{};
    ga.sp = ev->sp.as<float>();
    ga.beta = beta_or_null(ev);
    ga.beta_shared = ev->beta_shared && ev->prm.mode == DP_FROZEN_BETA;
    if (ga.beta_shared) ga.beta = ev->beta_frozen.as<float>();
    ga.kappa = (float)kappa_of(ev->prm);
    ga.cap = ev->cap.as<float>();
    ga.w = w;
    ga.size = ev->S > 0 ? ev->size.as<float>() : nullptr;
    ga.int2ext = d->int2ext.as<int32_t>();
    ga.n_pi = d->n_pi;
    ga.n_nets = d->n_nets;
    ga.G = d->n_gates;
    ga.B = ev->B;
    ga.S = ev->S;
    ga.paired = ev->paired_sizes;
    DP_TRY(om.map(dcap, (size_t)d->n_nets, &ga.dcap));
    if (ev->S > 0) DP_TRY(om.map(dsize, (size_t)ev->S * d->n_gates, &ga.dsize));
    DP_HIP_TRY(dp::launch_grad_export(ga, s));
    DP_TRY(om.flush(s));
  }
  if (!on_device) DP_TRY(sync_and_check(ev));
  return DP_OK;
}

dp_status dp_backward(dp_eval *ev, const float *grad_power, float *dpower_dpi, float *dpower_dcap,
                      float *dpower_dsize, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_backward: NULL eval");
  if (dpower_dsize && ev->S == 0)
    return fail(DP_E_INVALID, "dp_backward: dpower_dsize needs cell sizes (S > 0)");
  return run_backward(ev, grad_power, 0, dpower_dpi, dpower_dcap, dpower_dsize, on_device);
}

dp_status dp_power_gradients(dp_eval *ev, float *dpower_dsp, float *score, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_power_gradients: NULL eval");
  const dp_design *d = ev->d;
  if (ev->fwd_version != ev->inputs_version || ev->fwd_version == 0)
    return fail(DP_E_STATE, "dp_power_gradients: no completed forward for the current inputs");
  if (!dpower_dsp && !score) return DP_OK;
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  hipStream_t s = ev->stream();
  const int32_t B = ev->B;
  DP_TRY(ensure_reverse_buffers(ev, B));
  DP_TRY(ev->pi_out.alloc(std::max<size_t>((size_t)B * d->n_pi * sizeof(float), 16)));
  DevBuf lam;
  DP_TRY(lam.alloc((size_t)B * d->n_nets * sizeof(float)));
  dp::BwdArgs ba = backward_args(ev, nullptr, 0, B);
  ba.lam = lam.as<float>();
  DP_TRY(enqueue_backward(ev, ba, ev->pi_out.as<float>()));
  OutMap om{ev, on_device};
  float *o_lam = nullptr, *o_score = nullptr;
  DP_TRY(om.map(dpower_dsp, (size_t)B * d->n_nets, &o_lam));
  DP_TRY(om.map(score, (size_t)B * d->n_gates, &o_score));
  DP_HIP_TRY(dp::launch_grad_lambda_export(lam.as<float>(), ev->sp.as<float>(),
                                           d->int2ext.as<int32_t>(), d->n_pi, d->n_nets, B, B, 1,
                                           0x1p-20f, o_lam, o_score, s));
  DP_TRY(om.flush(s));
  DP_HIP_TRY(hipStreamSynchronize(s));  // the adjoint buffer is freed on return
  return barrier_status(ev);
}

dp_status dp_power_virus(dp_eval *ev, int32_t steps, double eta, uint8_t *v0, float *p_final,
                         double *p_virus, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_power_virus: NULL eval");
  if (steps < 0 || !std::isfinite(eta))
    return fail(DP_E_INVALID, "dp_power_virus: need steps >= 0 and a finite eta");
  if (ev->prm.mode == DP_HYBRID)
    return fail(DP_E_UNSUPPORTED, "dp_power_virus: the ascent runs DP_MODELED or DP_FROZEN_BETA");
  if (ev->S > 0) return fail(DP_E_UNSUPPORTED, "dp_power_virus: size vectors are not supported");
  if (!ev->have_pi) return fail(DP_E_STATE, "dp_power_virus: start probabilities not set");
  if (!ev->have_cap) return fail(DP_E_STATE, "dp_power_virus: capacitances not set");
  if (ev->prm.mode == DP_FROZEN_BETA && !ev->have_beta)
    return fail(DP_E_STATE, "dp_power_virus: DP_FROZEN_BETA needs dp_set_beta");
  const dp_design *d = ev->d;
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  hipStream_t s = ev->stream();
  const int32_t B = ev->B;
  const size_t nb = (size_t)d->n_nets * B, pb = (size_t)d->n_pi * B;
  DP_TRY(ensure_forward_buffers(ev, nullptr));
  DP_TRY(ensure_reverse_buffers(ev, B));
  DP_TRY(ev->pi_out.alloc(std::max<size_t>(pb * sizeof(float), 16)));
  // the proxy is the power without kappa: upstream weight 1 / kappa per column
  DP_TRY(ev->w.alloc(std::max<size_t>((size_t)B * sizeof(float), 16)));
  DP_HIP_TRY(dp::launch_fill_f32(ev->w.as<float>(), B, (float)(1.0 / kappa_of(ev->prm)), s));
  const dp::BwdArgs ba = backward_args(ev, ev->w.as<float>(), 0, B);
  for (int32_t t = 0; t < steps; ++t) {
    DP_TRY(enqueue_forward(ev, nullptr));
    DP_TRY(enqueue_backward(ev, ba, ev->pi_out.as<float>()));
    DP_HIP_TRY(dp::launch_virus_step(ev->sp.as<float>(), ev->pi_out.as<float>(), (float)eta,
                                     d->n_pi, B, s));
  }
  // v0, v1 = 1 - v0 and a two-cycle bit-parallel simulation of the pair
  DevBuf stim, words, v0_dev, p_dev, pv;
  DP_TRY(stim.alloc(std::max<size_t>(pb * 2 * sizeof(uint64_t), 16)));
  DP_TRY(words.alloc((size_t)B * d->n_nets * 2 * sizeof(uint64_t)));
  DP_TRY(v0_dev.alloc(std::max<size_t>(pb, 16)));
  DP_TRY(p_dev.alloc(std::max<size_t>(pb * sizeof(float), 16)));
  DP_TRY(pv.alloc(std::max<size_t>((size_t)B * sizeof(double), 16)));
  DP_TRY(ev->ones.alloc(nb * sizeof(uint32_t)));
  DP_TRY(ev->tog.alloc(nb * sizeof(uint32_t)));
  DP_HIP_TRY(dp::launch_virus_vectors(ev->sp.as<float>(), stim.as<uint64_t>(), v0_dev.as<uint8_t>(),
                                      p_dev.as<float>(), d->n_pi, B, s));
  DP_HIP_TRY(dp::launch_fill_u32(ev->ones.as<uint32_t>(), (int64_t)nb, 0u, s));
  DP_HIP_TRY(dp::launch_fill_u32(ev->tog.as<uint32_t>(), (int64_t)nb, 0u, s));
  const dp::GraphView g = view(d);
  const dp::SimTune tune{1};
  dp::ChunkView cv{};  // every column's pair in one launch per level
  cv.W = words.as<uint64_t>();
  cv.pitch = 2;
  cv.col_stride = (int64_t)d->n_nets * 2;
  cv.t_first = 0;
  cv.pairs = 1;
  cv.u_lo = 0;
  cv.u_hi = 2;
  cv.u_tog_lo = 1;
  cv.n_cols = B;
  const dp::CountView cnt{ev->ones.as<uint32_t>(), ev->tog.as<uint32_t>(), B, 0};
  DP_HIP_TRY(dp::launch_stimulus(g, cv, cnt, ev->sp.as<float>(), stim.as<uint64_t>(), 2, nullptr,
                                 0, tune, s));
  for (int32_t l = 1; l <= d->depth; ++l)
    DP_TRY(for_level_parts(d, l, [&](int32_t g0, int32_t n, bool cells) -> dp_status {
      DP_HIP_TRY(dp::launch_sim_level(g, cv, cnt, g0, n, nullptr, cells, tune, s));
      return DP_OK;
    }));
  DP_HIP_TRY(dp::launch_virus_power(ev->tog.as<uint32_t>(), ev->cap.as<float>(), d->n_nets, B,
                                    pv.as<double>(), s));
  const hipMemcpyKind k = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  if (v0 && pb) DP_HIP_TRY(hipMemcpyAsync(v0, v0_dev.ptr, pb, k, s));
  if (p_final && pb) DP_HIP_TRY(hipMemcpyAsync(p_final, p_dev.ptr, pb * sizeof(float), k, s));
  if (p_virus) DP_HIP_TRY(hipMemcpyAsync(p_virus, pv.ptr, (size_t)B * sizeof(double), k, s));
  DP_HIP_TRY(hipStreamSynchronize(s));  // the scratch buffers are freed on return
  ev->inputs_version++;  // the PI probabilities are now the ascended ones
  const dp_status st = barrier_status(ev);
  if (st != DP_OK) ev->have_pi = false;  // or what NaN gradients made of them
  return st;
}

dp_status dp_backward_columns(dp_eval *ev, float *dpower_dpi, int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_backward_columns: NULL eval");
  if (!dpower_dpi) return fail(DP_E_INVALID, "dp_backward_columns: NULL output");
  return run_backward(ev, nullptr, 1, dpower_dpi, nullptr, nullptr, on_device);
}

dp_status dp_forward_backward_columns(dp_eval *ev, float *power, float *dpower_dpi,
                                      int32_t on_device) {
  if (!ev) return fail(DP_E_INVALID, "dp_forward_backward_columns: NULL eval");
  const dp_design *d = ev->d;
  // the schedules that capture: the whole pair of sweeps as one graph;
  // otherwise the two calls as they are
  const bool hyb = hybrid(ev);
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  DP_TRY(ensure_flow(ev));
  ChunkPlan plan;
  if (hyb) plan = plan_chunks(ev);
  const ChunkPlan *pl = hyb ? &plan : nullptr;
  const int64_t launches = forward_launches(ev, pl) + reverse_launches(d);
  if (ev->schedule != DP_SCHED_GRAPH || ev->profiling || launches > kMaxGraphLaunches) {
    DP_TRY(dp_forward(ev, nullptr));
    if (power) {
      const size_t bytes = (size_t)ev->B * s_prime(ev) * sizeof(float);
      DP_HIP_TRY(hipMemcpyAsync(power, ev->power.ptr, bytes,
                                on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                                ev->stream()));
    }
    if (dpower_dpi) return run_backward(ev, nullptr, 1, dpower_dpi, nullptr, nullptr, on_device);
    if (!on_device) DP_TRY(sync_and_check(ev));
    return DP_OK;
  }
  // the checks of dp_forward and dp_backward, then every buffer before the
  // capture
  if (!ev->have_pi) return fail(DP_E_STATE, "dp_forward_backward_columns: PI probabilities not set");
  if (!ev->have_cap) return fail(DP_E_STATE, "dp_forward_backward_columns: capacitances not set");
  if (ev->S > 0 && !ev->have_size)
    return fail(DP_E_STATE, "dp_forward_backward_columns: cell sizes not set");
  if (ev->prm.mode == DP_FROZEN_BETA && !ev->have_beta)
    return fail(DP_E_STATE, "dp_forward_backward_columns: DP_FROZEN_BETA needs dp_set_beta");
  if (hyb && ev->have_stim &&
      ev->stim.bytes < (size_t)ev->B * d->n_pi * n_words(ev->prm) * sizeof(uint64_t))
    return fail(DP_E_STATE, "dp_forward_backward_columns: the explicit stimulus is shorter than "
                            "n_sim/64 words");
  DP_HIP_TRY(hipSetDevice(d->ctx->device));
  hipStream_t s = ev->stream();
  DP_TRY(plan_forward(ev, &plan, &pl));
  const int32_t C = ev->B * s_prime(ev);
  DP_TRY(ensure_reverse_buffers(ev, C, 1));
  const size_t dpi_bytes = (size_t)C * d->n_pi * sizeof(float);
  float *dst = on_device ? dpower_dpi : nullptr;
  if (!dst) {  // host output, or none: the sweep writes the staging buffer
    DP_TRY(ev->pi_out.alloc(std::max<size_t>(dpi_bytes, 16)));
    dst = ev->pi_out.as<float>();
  }
  const dp::BwdArgs ba = backward_args(ev, nullptr, 1, C);
  // the forward's key and the reverse sweep's, combined
  const uint64_t key = graph_key(ev, pl) * 1099511628211ull ^ reverse_key(ev, ba, dst);
  if (!ev->graph_fb || ev->graph_fb_key != key) {
    DP_TRY(capture_into(ev, &ev->graph_fb, [&]() -> dp_status {
      DP_TRY(enqueue_forward(ev, pl));
      return enqueue_backward(ev, ba, dst);
    }));
    ev->graph_fb_key = key;
  }
  DP_HIP_TRY(hipGraphLaunch(ev->graph_fb, s));
  ev->fwd_version = ev->inputs_version;
  const hipMemcpyKind k = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  if (power)
    DP_HIP_TRY(hipMemcpyAsync(power, ev->power.ptr, (size_t)C * sizeof(float), k, s));
  if (dpower_dpi && !on_device && dpi_bytes)
    DP_HIP_TRY(hipMemcpyAsync(dpower_dpi, dst, dpi_bytes, hipMemcpyDeviceToHost, s));
  if (!on_device) {
    DP_TRY(sync_and_check(ev));
  }
  return DP_OK;
}

}  // extern "C"

// =========================================================================
// Design groups: the sweeps of several evals as one graph launch.
constexpr int32_t kGroupBranches = 4;  // streams beyond the hardware queues only queue

// Host threads that enqueue a group's branches side by side: a launch-bound
// sweep is limited by how fast one thread submits kernels, so each branch
// gets a thread of its own.  Workers live as long as the group.
namespace dp {

namespace {
// Range of level l of one kind: fixed cells first, then library cells.
void level_part(const dp_design *d, int32_t l, int k, int32_t *g0, int32_t *n) {
  const int32_t a = d->level_ptr[l], nl = d->level_ptr[l + 1] - a, nf = d->lvl_fixed[l];
  *g0 = k == 0 ? a : a + nf;
  *n = k == 0 ? nf : nl - nf;
}
}  // namespace

void MergedTables::build(const Lane *lanes, int32_t n, bool forward, bool reverse) {
  D = 0;
  for (int32_t j = 0; j < n; ++j) D = std::max(D, lanes[j].ev->d->depth);
  fs.clear();
  bs.clear();
  f_launch.clear();
  const size_t m = 2 * (size_t)(D + 1);
  b_off.assign(m, 0);
  b_cnt.assign(m, 0);
  b_blk.assign(m, 0);
  // forward: level indices l and l + 1 share a launch when every design that
  // has level l holds fixed cells only there and pairs it with l + 1 (or
  // ends at l)
  for (int32_t l = 1; forward && l <= D;) {
    bool pair = l + 1 <= D;
    for (int32_t j = 0; j < n && pair; ++j) {
      const dp_eval *ev = lanes[j].ev;
      const dp_design *d = ev->d;
      if (l > d->depth) continue;
      if (d->lvl_fixed[l] != d->level_ptr[l + 1] - d->level_ptr[l]) pair = false;
      else if (l + 1 <= d->depth && !pairs_levels(d, l, ev->B)) pair = false;
    }
    for (int k = 0; k < (pair ? 1 : 2); ++k) {
      FwdLaunch fl{(int32_t)fs.size(), 0, 0, k == 1};
      for (int32_t j = 0; j < n; ++j) {
        dp_eval *ev = lanes[j].ev;
        const dp_design *d = ev->d;
        if (l > d->depth) continue;
        int32_t g0, cnt;
        level_part(d, l, k, &g0, &cnt);
        if (cnt == 0) continue;
        SpLevel second{ev->sp.as<float>(), ev->B, 0, 0};
        if (pair && l + 1 <= d->depth) {
          second.g0 = d->level_ptr[l + 1];
          second.n = d->level_ptr[l + 2] - second.g0;
        }
        const uint32_t blocks =
            (uint32_t)(((int64_t)(cnt + second.n) * ev->B + kMergedBlock - 1) / kMergedBlock);
        fs.push_back({view(d), SpLevel{ev->sp.as<float>(), ev->B, g0, cnt}, second, fl.blocks});
        fl.blocks += blocks;
      }
      fl.cnt = (int32_t)fs.size() - fl.off;
      if (fl.cnt > 0) f_launch.push_back(fl);
    }
    l += pair ? 2 : 1;
  }
  for (int32_t l = 1; reverse && l <= D; ++l)
    for (int k = 0; k < 2; ++k) {
      const size_t i = 2 * (size_t)l + k;
      b_off[i] = (int32_t)bs.size();
      for (int32_t j = 0; j < n; ++j) {
        dp_eval *ev = lanes[j].ev;
        const dp_design *d = ev->d;
        if (l > d->depth || !lanes[j].backward) continue;
        int32_t g0, cnt;
        level_part(d, l, k, &g0, &cnt);
        if (cnt == 0) continue;
        const uint32_t blocks =
            (uint32_t)(((int64_t)cnt * ev->B + kMergedBlock - 1) / kMergedBlock);
        bs.push_back({view(d), backward_args(ev, nullptr, 0, ev->B), g0, cnt, b_blk[i]});
        b_blk[i] += blocks;
      }
      b_cnt[i] = (int32_t)bs.size() - b_off[i];
    }
}

int64_t MergedTables::level_launches(const Lane *lanes, int32_t n) {
  int32_t depth = 0;
  for (int32_t j = 0; j < n; ++j) depth = std::max(depth, lanes[j].ev->d->depth);
  int64_t c = 0;
  for (int32_t l = 1; l <= depth; ++l)
    for (int k = 0; k < 2; ++k) {
      bool any = false;
      for (int32_t j = 0; j < n && !any; ++j) {
        const dp_design *d = lanes[j].ev->d;
        int32_t g0, cnt = 0;
        if (l <= d->depth) level_part(d, l, k, &g0, &cnt);
        any = cnt > 0;
      }
      c += any;
    }
  return c;
}

dp_status MergedTables::launch_forward(const SpSeg *dev, hipStream_t s) const {
  for (const FwdLaunch &fl : f_launch)
    DP_HIP_TRY(launch_sp_multi(dev + fl.off, fl.cnt, fl.blocks, fl.cells, s));
  return DP_OK;
}

dp_status MergedTables::launch_reverse(const BwdSeg *dev, hipStream_t s) const {
  for (int32_t l = D; l >= 1; --l)
    for (int k = 0; k < 2; ++k) {
      const size_t i = 2 * (size_t)l + k;
      DP_HIP_TRY(launch_bwd_multi(dev + b_off[i], b_cnt[i], b_blk[i], k == 1, s));
    }
  return DP_OK;
}

void FlowTables::build(const MergedTables::Lane *lanes, int32_t n) {
  fs.clear();
  bs.clear();
  f_jobs = b_jobs = 0;
  f_blocks = b_blocks = 0;
  f_widest = b_widest = 1;
  f_cells = b_cells = false;
  ctl = flow_ctl(lanes[0].ev);
  for (int32_t j = 1; j < n; ++j)
    flow_set_limit(ctl, std::min(ctl.limit, flow_limit(lanes[j].ev)));
  std::vector<int32_t> order(n);
  for (int32_t j = 0; j < n; ++j) order[j] = j;
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
    return lanes[x].ev->d->n_nets > lanes[y].ev->d->n_nets;
  });
  for (int32_t j : order) {
    dp_eval *ev = lanes[j].ev;
    const dp_design *d = ev->d;
    f_cells = f_cells || d->has_cell_gates;
    SpFlowSeg f{};
    f.t = SpFlow{view(d), ev->sp.as<float>(), d->level_dev.as<int32_t>(), ev->B, d->depth};
    f.job0 = f_jobs;
    f.block0 = f_blocks;
    f_jobs += ev->B;
    f_blocks += flow_arm_blocks(f.t, fs.empty());
    f_widest = std::max<int64_t>(f_widest, d->max_level_width);
    fs.push_back(f);
    if (!lanes[j].backward) continue;
    b_cells = b_cells || d->has_cell_gates;
    BwdFlowSeg b{};
    b.t = BwdFlow{view(d), backward_args(ev, nullptr, 0, ev->B), ev->pi_out.as<float>(),
                  ev->seed.as<float>(), ev->part.as<float>(), d->level_dev.as<int32_t>(),
                  d->n_edges, d->depth};
    b.job0 = b_jobs;
    b.block0 = b_blocks;
    ctl.sized = ctl.sized || staged_sizes(b.t.a);
    b_jobs += ev->B;
    b_blocks += flow_arm_blocks(b.t, bs.empty(), &b.arm_blocks, &b.seed_blocks);
    b_widest = std::max<int64_t>(b_widest, std::max(d->max_level_width, d->n_pi));
    bs.push_back(b);
  }
}

dp_status FlowTables::launch_forward(const SpFlowSeg *dev, hipStream_t s) const {
  DP_HIP_TRY(launch_sp_flow_multi(dev, (int32_t)fs.size(), f_jobs, f_blocks, f_widest, f_cells, ctl, s));
  return DP_OK;
}
dp_status FlowTables::launch_reverse(const BwdFlowSeg *dev, hipStream_t s) const {
  DP_HIP_TRY(launch_bwd_flow_multi(dev, (int32_t)bs.size(), b_jobs, b_blocks, b_widest, b_cells, ctl, s));
  return DP_OK;
}

// The same choice for the sweeps of n evals together: depth is the deepest
// one's, pairs (net, column) pairs in millions, turns the gates that the fullest
// XCD's columns walk (all columns share the eight), gates the evals' gates times
// their rounds of eight columns, since the columns of a design share its lines.
//   us = base + |(level D, turns T + pairs N + gates G)| + over N + each n
// So one launch for many levels or for many designs of few columns, and launches
// level by level for few levels of many pairs (forward / reverse in us, levels
// against dataflow: 4 x 117K gates x 3 levels, 8 columns each 49 / 71 against 127 /
// 220; 8 x 50K x 12, 8 columns 70 / 146 against 97 / 105; 8 x 1M x 8, one column 188 /
// 863 against 102 / 369; 4 x 117K x 60, 4 columns 176 / 346 against 89 / 100).
// Fitted to 250 sets of 2 to 16 designs of 2K to 1M gates, 2 to 100 levels, 1 to 16
// columns, 30 of them with library cells: the choice is 0.5 % (forward) and 0.4 %
// (reverse) slower than the better of the two on average.  Level by level each
// eval's startpoints are a launch of their own, by whole waves and one after
// another with one or two columns (about 50 us each), where dataflow was faster
// in every set.
namespace {
struct MultiCost {
  double base, level, turns, pairs, gates, over, each;
};
constexpr MultiCost kSpFlowMulti{23.3, 0.60, 63.8, 13.5, -14.8, 0.0, 0.0},
    kSpLevelsMulti{20.6, 2.15, 0.0, 0.0, 17.9, 4.0, 0.0};
constexpr MultiCost kBwdFlowMulti{8.3, 0.98, 171.0, 16.9, -4.4, 0.0, 0.0},
    kBwdLevelsMulti{-6.0, 5.4, 0.0, 0.0, 0.0, 27.6, 2.0};
// library cells in one of the designs
constexpr MultiCost kSpFlowMultiCells{23.8, 3.47, 203.0, 15.1, -34.3, 0.0, 0.0},
    kSpLevelsMultiCells{11.2, 7.8, 0.0, 0.0, 0.0, 7.1, 0.0};
constexpr MultiCost kBwdFlowMultiCells{31.4, 1.13, 251.0, 71.5, -20.9, 0.0, 0.0},
    kBwdLevelsMultiCells{0.0, 34.7, 0.0, 0.0, 0.0, 69.4, 0.0};
struct MultiSize {
  double depth = 0, pairs = 0, largest = 0, gates = 0, n = 0;
  bool cells = false, few = false;
  void add(const dp_eval *ev) {
    const dp_design *d = ev->d;
    const double rounds = (ev->B + 7) / 8, g = d->n_gates * 1e-6 * rounds;
    depth = std::max(depth, (double)d->depth);
    pairs += (double)d->n_nets * ev->B * 1e-6;
    largest = std::max(largest, g);
    gates += g;
    n += 1;
    cells = cells || d->has_cell_gates;
    few = few || ev->B < 3;
  }
  double us(const MultiCost &c) const {
    const double work = c.turns * std::max(largest, pairs / 8) + c.pairs * pairs + c.gates * gates;
    return c.base + std::hypot(c.level * depth, std::max(work, 0.0)) + c.over * pairs + c.each * n;
  }
};
}  // namespace

void SweepTables::choose(const MergedTables::Lane *lanes, int32_t n) {
  int64_t jobs = 0, items = 0;
  MultiSize f, b;
  bool ready = n > 0, b_ready = true;
  for (int32_t j = 0; j < n; ++j) {
    const dp_eval *ev = lanes[j].ev;
    ready = ready && flow_ready(ev, ev->B);
    jobs += ev->B;
    items += (int64_t)ev->d->n_nets * ev->B;
    f.add(ev);
    if (!lanes[j].backward) continue;
    b_ready = b_ready && have_flow_scratch(ev, ev->B);
    b.add(ev);
  }
  ready = ready && jobs <= kFlowMaxJobs && items <= kFlowMultiItems;
  flow_forward = ready && (f.cells ? f.us(kSpFlowMultiCells) < f.us(kSpLevelsMultiCells)
                                   : f.us(kSpFlowMulti) < f.us(kSpLevelsMulti));
  flow_reverse = ready && b_ready &&
                 (b.few || (b.cells ? b.us(kBwdFlowMultiCells) < b.us(kBwdLevelsMultiCells)
                                    : b.us(kBwdFlowMulti) < b.us(kBwdLevelsMulti)));
}

void SweepTables::build(const MergedTables::Lane *lanes, int32_t n) {
  choose(lanes, n);
  if (!flow_forward || !flow_reverse) levels.build(lanes, n, !flow_forward, !flow_reverse);
  if (flow_forward || flow_reverse) flow.build(lanes, n);
}

namespace {
template <class T>
size_t bytes_of(const std::vector<T> &v) {
  return v.size() * sizeof(T);
}
template <class T>
void copy_to(void *dst, const std::vector<T> &v) {
  if (!v.empty()) std::memcpy(dst, v.data(), bytes_of(v));
}
}  // namespace

size_t SweepTables::bwd_offset() const {
  return ((flow_forward ? bytes_of(flow.fs) : bytes_of(levels.fs)) + 255) & ~(size_t)255;
}
size_t SweepTables::bytes() const {
  return std::max<size_t>(bwd_offset() + (flow_reverse ? bytes_of(flow.bs) : bytes_of(levels.bs)), 256);
}
void SweepTables::pack(void *host) const {
  flow_forward ? copy_to(host, flow.fs) : copy_to(host, levels.fs);
  char *bwd = (char *)host + bwd_offset();
  flow_reverse ? copy_to(bwd, flow.bs) : copy_to(bwd, levels.bs);
}
dp_status SweepTables::launch_forward(const void *dev, hipStream_t s) const {
  return flow_forward ? flow.launch_forward(static_cast<const SpFlowSeg *>(dev), s)
                      : levels.launch_forward(static_cast<const SpSeg *>(dev), s);
}
dp_status SweepTables::launch_reverse(const void *dev, const MergedTables::Lane *lanes, int32_t n,
                                      hipStream_t s) const {
  const void *bwd = static_cast<const char *>(dev) + bwd_offset();
  if (flow_reverse) return flow.launch_reverse(static_cast<const BwdFlowSeg *>(bwd), s);
  DP_TRY(levels.launch_reverse(static_cast<const BwdSeg *>(bwd), s));
  for (int32_t j = 0; j < n; ++j) {
    if (!lanes[j].backward) continue;
    dp_eval *ev = lanes[j].ev;
    const HeavySpan hp = heavy_pis(ev->d);
    DP_HIP_TRY(launch_bwd_pi(view(ev->d), backward_args(ev, nullptr, 0, ev->B),
                             ev->pi_out.as<float>(), s, hp.gates, hp.n));
  }
  return DP_OK;
}

bool PowerTable::add(dp_eval *ev, float *host) {
  const PowerArgs a = power_args(ev, nullptr);
  if (!power_merges(a)) return false;
  if ((int64_t)a.n_nets * a.B <= 0) return true;
  segs.push_back(PowerSeg{a, host, blocks, cols});
  blocks += power_blocks(a);
  cols += a.B;
  widest = std::max(widest, a.B);
  return true;
}
dp_status PowerTable::launch(const void *dev, hipStream_t s) const {
  DP_HIP_TRY(launch_power_multi(static_cast<const PowerSeg *>(dev), (int32_t)segs.size(), blocks, cols,
                                widest, s));
  return DP_OK;
}

}  // namespace dp

struct GroupPool {
  std::vector<std::thread> workers;
  std::mutex mu;
  std::condition_variable cv, done;
  std::function<void(int)> task;
  uint64_t gen = 0;
  int n_tasks = 0, pending = 0;
  bool stop = false;

  void start(int n, int device) {
    for (int k = 0; k < n; ++k)
      workers.emplace_back([this, k, device]() {
        (void)hipSetDevice(device);
        uint64_t seen = 0;
        for (;;) {
          std::unique_lock<std::mutex> lk(mu);
          cv.wait(lk, [&] { return stop || gen != seen; });
          if (stop) return;
          seen = gen;
          const bool mine = k < n_tasks;
          lk.unlock();
          if (mine) task(k);
          lk.lock();
          if (mine && --pending == 0) done.notify_all();
        }
      });
  }
  // Run f(0) .. f(n - 1) on the workers and wait for all of them.
  void run(int n, std::function<void(int)> f) {
    std::unique_lock<std::mutex> lk(mu);
    task = std::move(f);
    n_tasks = n;
    pending = n;
    ++gen;
    cv.notify_all();
    done.wait(lk, [&] { return pending == 0; });
  }
  ~GroupPool() {
    {
      std::lock_guard<std::mutex> lk(mu);
      stop = true;
    }
    cv.notify_all();
    for (auto &t : workers) t.join();
  }
};

struct dp_group {
  GroupPool pool;
  // Merged level launches of the group's modeled evals (one launch per level
  // index and kind covers that level of every such eval): host tables and
  // their device copy, the power's segments at tab_dev_power.
  std::vector<int32_t> merged;      // eval indices
  dp::SweepTables tab;
  dp::DevBuf tab_dev;
  size_t tab_dev_power = 0;
  dp::PowerTable power;  // empty: each eval's power by itself
  bool have_tables = false;
  uint64_t tables_key = 0;
  dp_ctx *ctx = nullptr;
  std::vector<dp_eval *> evs;
  std::vector<hipStream_t> branch;  // up to kGroupBranches
  std::vector<hipEvent_t> join;     // one per branch
  std::vector<int32_t> branch_of;   // eval -> branch
  int32_t max_branches = 0;         // 0 = automatic
  bool use_graph = true;
  hipEvent_t fork = nullptr;
  hipStream_t capture = nullptr;
  hipGraphExec_t exec = nullptr;
  uint64_t key = 0;
  std::shared_ptr<dp::SharedReport> report;  // of the merged dataflow sweeps
  ~dp_group() {
    if (report) {
      std::lock_guard<std::mutex> lock(report->mu);
      report->done = true;
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    for (auto st : branch) {
      (void)hipStreamSynchronize(st);
      (void)hipStreamDestroy(st);
    }
    for (auto e : join) (void)hipEventDestroy(e);
    if (fork) (void)hipEventDestroy(fork);
    if (capture) (void)hipStreamDestroy(capture);
  }
};

namespace {

// Assign evals to branches: longest first, each to the least loaded branch
// (load = kernel launches, the cost of a launch-bound sweep).
void assign_branches(dp_group *g, const std::vector<int64_t> &cost) {
  const int32_t nb = (int32_t)g->branch.size();
  std::vector<int32_t> order(g->evs.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int32_t)i;
  std::stable_sort(order.begin(), order.end(),
                   [&](int32_t a, int32_t b) { return cost[a] > cost[b]; });
  std::vector<int64_t> load(nb, 0);
  g->branch_of.assign(g->evs.size(), 0);
  for (int32_t i : order) {
    const int32_t k = (int32_t)(std::min_element(load.begin(), load.end()) - load.begin());
    g->branch_of[i] = k;
    load[k] += cost[i];
  }
}

// Fork from `origin` into the branches, enqueue each eval's forward (and
// reverse) sweep on its branch with per-level launches, join back.
// Segment tables of the merged level launches (host work, one upload).
dp_status build_merged_tables(dp_group *g, bool backward) {
  std::vector<dp::MergedTables::Lane> lanes;
  for (int32_t i : g->merged) lanes.push_back({g->evs[i], backward});
  std::vector<char> host;
  g->power = dp::PowerTable{};
  for (int32_t i : g->merged)
    if (!g->power.add(g->evs[i], nullptr)) {  // (several size vectors)
      g->power = dp::PowerTable{};
      break;
    }
  g->tab.build(lanes.data(), (int32_t)lanes.size());
  g->tab.flow.ctl.report = g->report->word;
  g->tab_dev_power = (g->tab.bytes() + 255) & ~(size_t)255;
  host.resize(g->tab_dev_power + std::max<size_t>(g->power.bytes(), 256));
  DP_TRY(g->tab_dev.alloc(host.size()));
  g->tab.pack(host.data());
  if (!g->power.segs.empty())
    std::memcpy(host.data() + g->tab_dev_power, g->power.segs.data(),
                g->power.segs.size() * sizeof(dp::PowerSeg));
  DP_HIP_TRY(hipMemcpy(g->tab_dev.ptr, host.data(), host.size(), hipMemcpyHostToDevice));
  g->have_tables = true;
  return DP_OK;
}

// The modeled evals as merged level launches on `origin`: SP levels, each
// eval's finalize and power, and with backward the reverse levels and each
// eval's PI adjoints.
dp_status enqueue_merged(dp_group *g, hipStream_t origin, bool backward) {
  if (g->merged.empty()) return DP_OK;
  DP_TRY(g->tab.launch_forward(g->tab_dev.ptr, origin));
  if (!g->power.segs.empty())
    DP_TRY(g->power.launch((const char *)g->tab_dev.ptr + g->tab_dev_power, origin));
  else
    for (int32_t i : g->merged) {
      dp_eval *ev = g->evs[i];
      ev->branch = origin;
      const dp_status st = enqueue_forward_tail(ev, nullptr);
      ev->branch = nullptr;
      DP_TRY(st);
    }
  if (!backward) return DP_OK;
  std::vector<dp::MergedTables::Lane> lanes;
  for (int32_t i : g->merged) lanes.push_back({g->evs[i], true});
  return g->tab.launch_reverse(g->tab_dev.ptr, lanes.data(), (int32_t)lanes.size(), origin);
}

// `threads`: enqueue the branches from the group's worker threads, one
// each.  `single`: everything on `origin` itself, no branches (captures
// record one stream only).
dp_status enqueue_group(dp_group *g, hipStream_t origin, bool backward,
                        const std::vector<ChunkPlan> &plans, bool threads, bool single) {
  if (single) {
    for (size_t i = 0; i < g->evs.size(); ++i) {
      if (std::find(g->merged.begin(), g->merged.end(), (int32_t)i) != g->merged.end()) continue;
      dp_eval *ev = g->evs[i];
      const int32_t sched = ev->schedule;
      const bool prof = ev->profiling;
      ev->branch = origin;
      ev->schedule = DP_SCHED_LEVEL;
      ev->profiling = false;
      dp_status st = enqueue_forward(ev, &plans[i]);
      if (st == DP_OK && backward)
        st = enqueue_backward(ev, backward_args(ev, nullptr, 0, ev->B), ev->pi_out.as<float>());
      ev->branch = nullptr;
      ev->schedule = sched;
      ev->profiling = prof;
      DP_TRY(st);
    }
    return enqueue_merged(g, origin, backward);
  }
  DP_HIP_TRY(hipEventRecord(g->fork, origin));
  for (hipStream_t b : g->branch) DP_HIP_TRY(hipStreamWaitEvent(b, g->fork, 0));
  std::vector<bool> is_merged(g->evs.size(), false);
  for (int32_t i : g->merged) is_merged[i] = true;
  auto branch_task = [&](int32_t k) -> dp_status {
    for (size_t i = 0; i < g->evs.size(); ++i) {
      if (g->branch_of[i] != k || is_merged[i]) continue;
      dp_eval *ev = g->evs[i];
      const int32_t sched = ev->schedule;
      const bool prof = ev->profiling;
      ev->branch = g->branch[k];
      ev->schedule = DP_SCHED_LEVEL;
      ev->profiling = false;
      dp_status st = enqueue_forward(ev, hybrid(ev) ? &plans[i] : nullptr);
      if (st == DP_OK && backward)
        st = enqueue_backward(ev, backward_args(ev, nullptr, 0, ev->B), ev->pi_out.as<float>());
      ev->branch = nullptr;
      ev->schedule = sched;
      ev->profiling = prof;
      if (st != DP_OK) return st;
    }
    return DP_OK;
  };
  const int32_t nb = (int32_t)g->branch.size();
  if (threads && nb > 1) {
    std::vector<dp_status> st(nb, DP_OK);
    std::vector<std::string> msg(nb);
    g->pool.run(nb, [&](int k) {
      st[k] = branch_task(k);
      if (st[k] != DP_OK) msg[k] = dp_last_error();
    });
    for (int32_t k = 0; k < nb; ++k)
      if (st[k] != DP_OK) return fail(st[k], msg[k]);
  } else {
    for (int32_t k = 0; k < nb; ++k) DP_TRY(branch_task(k));
  }
  DP_TRY(enqueue_merged(g, origin, backward));
  for (size_t k = 0; k < g->branch.size(); ++k) {
    DP_HIP_TRY(hipEventRecord(g->join[k], g->branch[k]));
    DP_HIP_TRY(hipStreamWaitEvent(origin, g->join[k], 0));
  }
  return DP_OK;
}

}  // namespace

extern "C" {

dp_status dp_group_create(dp_ctx *ctx, dp_eval *const *evals, int32_t n_evals, dp_group **out) {
  if (!ctx || !evals || !out) return fail(DP_E_INVALID, "dp_group_create: NULL argument");
  if (n_evals < 1) return fail(DP_E_INVALID, "dp_group_create: need at least one eval");
  for (int32_t i = 0; i < n_evals; ++i) {
    if (!evals[i]) return fail(DP_E_INVALID, "dp_group_create: NULL eval");
    if (evals[i]->d->ctx != ctx)
      return fail(DP_E_INVALID, "dp_group_create: every eval's design must belong to this context");
    if (evals[i]->own_stream) return fail(DP_E_INVALID, "dp_group_create: serving lanes cannot join");
    for (int32_t j = 0; j < i; ++j)
      if (evals[j] == evals[i]) return fail(DP_E_INVALID, "dp_group_create: an eval appears twice");
  }
  DP_HIP_TRY(hipSetDevice(ctx->device));
  auto *g = new dp_group();
  g->ctx = ctx;
  g->evs.assign(evals, evals + n_evals);
  hipError_t e = hipEventCreateWithFlags(&g->fork, hipEventDisableTiming);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&g->capture, hipStreamNonBlocking);
  for (int32_t i = 0; i < std::min(n_evals, kGroupBranches) && e == hipSuccess; ++i) {
    hipStream_t st = nullptr;
    hipEvent_t ev = nullptr;
    e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (e == hipSuccess) g->branch.push_back(st);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e == hipSuccess) g->join.push_back(ev);
  }
  if (e != hipSuccess) {
    delete g;
    return fail(DP_E_HIP, std::string("dp_group_create: ") + hipGetErrorString(e));
  }
  g->report = std::make_shared<dp::SharedReport>();
  g->report->words = ctx->reports;
  if (const dp_status st = ctx->reports->take(&g->report->word); st != DP_OK) {
    delete g;
    return st;
  }
  if (g->branch.size() > 1) g->pool.start((int)g->branch.size(), ctx->device);
  dp::ctx_retain(ctx);
  *out = g;
  return DP_OK;
}

dp_status dp_group_run(dp_group *g, int32_t backward, const dp_fwd_out *outs,
                       float *const *dpower_dpi, int32_t on_device) {
  if (!g) return fail(DP_E_INVALID, "dp_group_run: NULL group");
  DP_HIP_TRY(hipSetDevice(g->ctx->device));
  const size_t n = g->evs.size();
  std::vector<ChunkPlan> plans(n);
  std::vector<int64_t> cost(n, 0);
  int64_t launches = 0;
  uint64_t key = 1469598103934665603ull;
  auto mix = [&](uint64_t v) { key = (key ^ v) * 1099511628211ull; };
  mix((uint64_t)(backward != 0));
  for (size_t i = 0; i < n; ++i) {
    dp_eval *ev = g->evs[i];
    const dp_design *d = ev->d;
    if (!ev->have_pi || !ev->have_cap || (ev->S > 0 && !ev->have_size) ||
        (ev->prm.mode == DP_FROZEN_BETA && !ev->have_beta))
      return fail(DP_E_STATE, "dp_group_run: eval " + std::to_string(i) + " has inputs missing");
    if (outs && !hybrid(ev) &&
        (outs[i].sp_acc || outs[i].tr_acc || outs[i].ones || outs[i].toggles))
      return fail(DP_E_INVALID, "dp_group_run: simulation outputs need DP_HYBRID");
    if (hybrid(ev) && ev->have_stim &&
        ev->stim.bytes < (size_t)ev->B * d->n_pi * n_words(ev->prm) * sizeof(uint64_t))
      return fail(DP_E_STATE, "dp_group_run: an explicit stimulus is too short");
    // planned, and its buffers made, for the schedule that the group runs it in
    struct AsLevel {
      dp_eval *ev;
      const int32_t own = ev->schedule;
      explicit AsLevel(dp_eval *e) : ev(e) { ev->schedule = DP_SCHED_LEVEL; }
      ~AsLevel() { ev->schedule = own; }
    } as_level(ev);
    const ChunkPlan *pl;
    DP_TRY(plan_forward(ev, &plans[i], &pl));
    cost[i] = forward_launches(ev, hybrid(ev) ? &plans[i] : nullptr);
    if (backward) {
      DP_TRY(ensure_reverse_buffers(ev, ev->B));
      // (whatever its own route: a dataflow sweep is of every eval or of none)
      if (!hybrid(ev) && flow_ready(ev, ev->B)) DP_TRY(ensure_flow_scratch(ev, ev->B));
      DP_TRY(ev->pi_out.alloc(std::max<size_t>((size_t)ev->B * d->n_pi * sizeof(float), 16)));
      cost[i] += d->depth + d->split_levels + 1;
    }
    launches += cost[i];
    mix(graph_key(ev, hybrid(ev) ? &plans[i] : nullptr));
    mix((uint64_t)(uintptr_t)ev->contrib.ptr);
    mix((uint64_t)(uintptr_t)ev->part.ptr);
    mix((uint64_t)(uintptr_t)ev->seed.ptr);
    mix((uint64_t)(uintptr_t)ev->pi_out.ptr);
    mix((uint64_t)(uintptr_t)(ev->have_fixed ? ev->fixed.ptr : nullptr));
    mix((uint64_t)ev->B);
    mix((uint64_t)(uintptr_t)ev->sp.ptr);
    mix((uint64_t)(uintptr_t)ev->beta.ptr);
    mix((uint64_t)(uintptr_t)ev->cap.ptr);
    mix((uint64_t)(uintptr_t)ev->power.ptr);
    mix((uint64_t)(uintptr_t)ev->power_partial.ptr);
  }
  // modeled evals go into the merged level launches; the others (hybrid)
  // run on the branches
  g->merged.clear();
  for (size_t i = 0; i < n; ++i)
    if (!hybrid(g->evs[i])) {
      g->merged.push_back((int32_t)i);
      launches -= cost[i];
      cost[i] = 0;
    }
  if (!g->merged.empty()) {
    std::vector<dp::MergedTables::Lane> lanes;
    for (int32_t i : g->merged) lanes.push_back({g->evs[i], backward != 0});
    dp::SweepTables route;
    route.choose(lanes.data(), (int32_t)lanes.size());
    mix((uint64_t)route.flow_forward + 2 * (uint64_t)route.flow_reverse);
    if (route.flow_forward || route.flow_reverse)
      for (const auto &l : lanes) dp::join_shared(l.ev, g->report);
    const int64_t levels = dp::MergedTables::level_launches(lanes.data(), (int32_t)lanes.size());
    launches += (route.flow_forward ? 2 : levels) + (int64_t)g->merged.size() * (backward ? 4 : 3);
    if (backward) launches += route.flow_reverse ? 2 : levels;
  }
  const int32_t want = g->max_branches > 0 ? g->max_branches : kGroupBranches;
  const int32_t nb = std::max<int32_t>(1, std::min<int32_t>({want, (int32_t)g->branch.size(), (int32_t)n}));
  std::vector<hipStream_t> all = g->branch;
  g->branch.resize(nb);
  assign_branches(g, cost);
  for (size_t i = 0; i < n; ++i) mix((uint64_t)g->branch_of[i]);
  hipStream_t s = g->ctx->stream;
  struct Restore {
    dp_group *g;
    std::vector<hipStream_t> all;
    ~Restore() { g->branch = all; }
  } restore{g, all};
  if (g->tables_key != key || !g->have_tables) {
    DP_HIP_TRY(hipStreamSynchronize(s));  // no run reads the old tables
    DP_TRY(build_merged_tables(g, backward != 0));
    g->tables_key = key;
  }
  if (g->use_graph && launches <= kMaxGraphLaunches) {
    if (!g->exec || g->key != key) {
      if (g->exec) {
        DP_HIP_TRY(hipStreamSynchronize(s));
        (void)hipGraphExecDestroy(g->exec);
        g->exec = nullptr;
      }
      DP_HIP_TRY(hipStreamBeginCapture(g->capture, hipStreamCaptureModeThreadLocal));
      const dp_status st = enqueue_group(g, g->capture, backward != 0, plans, false, true);
      hipGraph_t graph = nullptr;
      const hipError_t e = hipStreamEndCapture(g->capture, &graph);
      if (st != DP_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return st;
      }
      if (e != hipSuccess) return fail(DP_E_HIP, std::string("group capture failed: ") + hipGetErrorString(e));
      const hipError_t ei = hipGraphInstantiate(&g->exec, graph, nullptr, nullptr, 0);
      (void)hipGraphDestroy(graph);
      if (ei != hipSuccess) {
        g->exec = nullptr;
        return fail(DP_E_HIP, std::string("group instantiate failed: ") + hipGetErrorString(ei));
      }
      g->key = key;
    }
    DP_HIP_TRY(hipGraphLaunch(g->exec, s));
  } else {
    DP_TRY(enqueue_group(g, s, backward != 0, plans, true, false));
  }
  bool host_out = false;
  dp::CopyList copies{};
  for (size_t i = 0; i < n; ++i) {
    dp_eval *ev = g->evs[i];
    ev->fwd_version = ev->inputs_version;
    if (outs) {
      DP_TRY(export_forward(ev, &outs[i], hybrid(ev) ? &plans[i] : nullptr, &copies));
      host_out = host_out || !outs[i].on_device;
    }
    if (backward && dpower_dpi && dpower_dpi[i] && ev->d->n_pi > 0) {
      const int64_t count = (int64_t)ev->B * ev->d->n_pi;
      if (on_device)
        DP_TRY(list_copy(&copies, ev->pi_out.as<float>(), dpower_dpi[i], count, s));
      else
        DP_HIP_TRY(hipMemcpyAsync(dpower_dpi[i], ev->pi_out.ptr, count * sizeof(float),
                                  hipMemcpyDeviceToHost, ev->stream()));
      host_out = host_out || !on_device;
    }
  }
  DP_HIP_TRY(dp::launch_copies(copies, s));
  if (host_out) {
    DP_HIP_TRY(hipStreamSynchronize(s));
    dp_status st = DP_OK;  // every eval's words are read, whichever fails first
    for (dp_eval *ev : g->evs) {
      const dp_status one = barrier_status(ev);
      if (st == DP_OK) st = one;
    }
    return st;
  }
  return DP_OK;
}

dp_status dp_group_configure(dp_group *g, int32_t use_graph, int32_t max_branches) {
  if (!g) return fail(DP_E_INVALID, "dp_group_configure: NULL group");
  if (max_branches < 0) return fail(DP_E_INVALID, "dp_group_configure: max_branches < 0");
  g->use_graph = use_graph != 0;
  g->max_branches = max_branches;
  return DP_OK;
}

void dp_group_destroy(dp_group *g) {
  if (!g) return;
  dp_ctx *c = g->ctx;
  (void)hipStreamSynchronize(c->stream);
  delete g;
  dp::ctx_release(c);
}

}  // extern "C"

// =========================================================================
// Serving lanes (internal).
namespace dp {

size_t lane_bytes(const dp_design *d, int32_t capacity) {
  const size_t nn = d->n_nets, G = d->n_gates, np = d->n_pi;
  // SP per net (the frozen beta is one per net, shared by the columns);
  // contributions per edge; sizes (and their staging) per gate;
  // probabilities and dP/dp
  const size_t per_col = 4 * (nn + (size_t)d->n_edges + 2 * G + 2 * np) +
                         8 * (size_t)power_chunks(d->n_nets) + 16;
  return (size_t)capacity * per_col + 8 * nn;
}

size_t lane_flow_bytes(const dp_design *d, int32_t capacity) {
  return (size_t)capacity * 4 * ((size_t)d->n_nets + (size_t)d->pins * d->n_gates) +
         (kFlowWords + kSimWords) * sizeof(uint32_t);
}

void lane_drop_flow(dp_eval *ev) {
  ev->seed.release();
  ev->part.release();
  ev->flow.release();
}

dp_status lane_add_flow(dp_eval *ev, int32_t capacity) {
  const dp_design *d = ev->d;
  dp_status st = ev->seed.alloc(std::max<size_t>((size_t)d->n_nets * capacity * 4, 16));
  if (st == DP_OK)
    st = ev->part.alloc(std::max<size_t>((size_t)capacity * d->pins * d->n_gates * 4, 16));
  if (st == DP_OK) st = ensure_flow(ev);
  if (st != DP_OK) lane_drop_flow(ev);
  return st;
}

dp_status lane_create(dp_design *d, int32_t capacity, const dp_params *prm, hipStream_t stream,
                      const float *cap_int, const float *beta_int, bool flow, dp_eval **out) {
  DP_TRY(check_params(prm));
  if (prm->mode == DP_HYBRID) return fail(DP_E_UNSUPPORTED, "serving lanes run DP_MODELED or DP_FROZEN_BETA");
  auto *ev = new dp_eval();
  ev->d = d;
  ev->B = capacity;
  ev->S = capacity;
  ev->paired_sizes = true;
  ev->prm = *prm;
  ev->own_stream = stream;
  ev->schedule = DP_SCHED_LEVEL;
  const size_t nn = d->n_nets;
  dp_status st = DP_OK;
  auto A = [&](DevBuf &b, size_t bytes) {
    if (st == DP_OK) st = b.alloc(std::max<size_t>(bytes, 16));
  };
  A(ev->sp, nn * capacity * 4);
  A(ev->cap, nn * 4);
  A(ev->size, (size_t)capacity * d->n_gates * 4);
  A(ev->size_stage, (size_t)capacity * d->n_gates * 4);
  if (prm->mode == DP_HYBRID) A(ev->beta, nn * capacity * 4);
  A(ev->power_partial, (size_t)power_chunks(d->n_nets) * capacity * 8);
  A(ev->power, (size_t)capacity * 4);
  A(ev->contrib, (size_t)d->n_edges * capacity * 4);
  A(ev->pi_out, (size_t)capacity * d->n_pi * 4);
  if (beta_int) A(ev->beta_frozen, nn * 4);
  if (flow && st == DP_OK) st = lane_add_flow(ev, capacity);
  if (st != DP_OK) {
    delete ev;
    return st;
  }
  hipError_t e = hipMemcpyAsync(ev->cap.ptr, cap_int, nn * 4, hipMemcpyDeviceToDevice, stream);
  if (e == hipSuccess && beta_int)
    e = hipMemcpyAsync(ev->beta_frozen.ptr, beta_int, nn * 4, hipMemcpyDeviceToDevice, stream);
  // steps run on streams of their own: the lane's inputs must be in place
  // before any of them reads the lane
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    delete ev;
    return fail(DP_E_HIP, std::string("lane_create: ") + hipGetErrorString(e));
  }
  ev->beta_shared = beta_int != nullptr;
  ev->have_cap = ev->have_pi = true;
  ev->have_beta = beta_int != nullptr;
  design_retain(d);
  *out = ev;
  return DP_OK;
}

StepScratch::~StepScratch() {
  if (host) (void)hipHostFree(host);
}

dp_status lanes_run_merged(const LaneJob *jobs, int32_t n_jobs, hipStream_t s,
                           StepScratch *sc) {
  std::vector<LaneSeg> segs(n_jobs);
  uint32_t stage = 0, import = 0, out = 0;
  PowerTable power;
  for (int32_t j = 0; j < n_jobs; ++j) {
    const LaneJob &job = jobs[j];
    dp_eval *ev = job.ev;
    const dp_design *d = ev->d;
    ev->B = job.n;
    ev->S = job.size ? job.n : 0;
    ev->paired_sizes = job.size != nullptr;
    LaneSeg &l = segs[j];
    l = LaneSeg{job.p, ev->sp.as<float>(), d->n_gates > 0 ? job.size : nullptr,
                ev->size_stage.as<float>(), ev->size.as<float>(), d->int2ext.as<int32_t>(),
                job.backward && job.dpi && d->n_pi > 0 ? ev->pi_out.as<float>() : nullptr, job.dpi,
                d->n_pi, job.n, d->n_gates, stage, 0, import, out};
    uint32_t n_stage, n_import, n_out;
    lane_seg_blocks(l, n_stage, n_import, n_out);
    stage += n_stage;
    import += n_import;
    out += n_out;
    if (!power.add(ev, job.power)) return fail(DP_E_UNSUPPORTED, "a lane with several size vectors");
  }
  // segment tables: forward over every lane, reverse over the lanes that
  // want gradients
  std::vector<MergedTables::Lane> lanes(n_jobs);
  bool any_backward = false;
  for (int32_t j = 0; j < n_jobs; ++j) {
    lanes[j] = {jobs[j].ev, jobs[j].backward};
    any_backward = any_backward || jobs[j].backward;
  }
  SweepTables tab;
  tab.build(lanes.data(), n_jobs);
  const size_t sweeps = (tab.bytes() + 255) & ~(size_t)255;
  const size_t lanes_at = sweeps + power.bytes(), bytes = lanes_at + segs.size() * sizeof(LaneSeg);
  if (bytes > sc->cap) {
    if (sc->host) (void)hipHostFree(sc->host);
    sc->host = nullptr;
    sc->cap = 0;
    DP_HIP_TRY(hipHostMalloc(&sc->host, bytes));
    DP_TRY(sc->dev.alloc(bytes));
    sc->cap = bytes;
  }
  char *host = static_cast<char *>(sc->host), *dev = static_cast<char *>(sc->dev.ptr);
  tab.pack(host);
  std::memcpy(host + sweeps, power.segs.data(), power.segs.size() * sizeof(PowerSeg));
  std::memcpy(host + lanes_at, segs.data(), segs.size() * sizeof(LaneSeg));
  const auto *lane_tab = reinterpret_cast<const LaneSeg *>(dev + lanes_at);
  DP_HIP_TRY(hipMemcpyAsync(sc->dev.ptr, sc->host, bytes, hipMemcpyHostToDevice, s));
  DP_HIP_TRY(launch_lanes_stage(lane_tab, n_jobs, stage, import, s));
  DP_TRY(tab.launch_forward(dev, s));
  DP_TRY(power.launch(dev + sweeps, s));
  if (!any_backward) return DP_OK;
  DP_TRY(tab.launch_reverse(dev, lanes.data(), n_jobs, s));
  DP_HIP_TRY(launch_lanes_out(lane_tab, n_jobs, out, s));
  return DP_OK;
}

dp_status calibrate_beta(dp_design *d, const float *cap_ext, const dp_params *prm, float p_all,
                         float *beta_int) {
  dp_params hp = *prm;
  hp.mode = DP_HYBRID;
  dp_eval *ev = nullptr;
  DP_TRY(dp_eval_create(d, 1, 0, &hp, &ev));
  std::vector<float> p(d->n_pi, p_all);
  dp_status st = dp_set_pi_prob(ev, p.data(), 0);
  if (st == DP_OK) st = dp_set_caps(ev, cap_ext, 0);
  if (st == DP_OK) st = dp_forward(ev, nullptr);
  if (st == DP_OK) {
    hipError_t e = hipMemcpyAsync(beta_int, ev->beta.ptr, (size_t)d->n_nets * 4,
                                  hipMemcpyDeviceToDevice, ev->stream());
    if (e == hipSuccess) e = hipStreamSynchronize(ev->stream());
    if (e != hipSuccess) st = fail(DP_E_HIP, std::string("calibrate_beta: ") + hipGetErrorString(e));
  }
  dp_eval_destroy(ev);
  return st;
}

}  // namespace dp


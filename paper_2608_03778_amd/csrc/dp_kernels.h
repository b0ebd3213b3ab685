// Launch interface of the gfx950 kernels (dp_kernels.hip).  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dp {

// Net-level graph arrays in internal numbering (see dp_design).
// Library cells: the host compiles each expression to post-order code for
// a stack machine that the kernels interpret.  An instruction is
// op | arg << 8; arg is the input index of kCellIn.
constexpr int kCellBase = 16;  // gate opcode of library cell c is kCellBase + c
constexpr int kCellMaxIn = 6;
constexpr int kCellMaxCode = 32;
constexpr int kCellMaxStack = 8;
enum : int { kCellIn = 0, kCellNot = 1, kCellAnd = 2, kCellOr = 3, kCellXor = 4,
             kCellZero = 5, kCellOne = 6 };
// The same code as steps for the SP sweeps, kCellRule words per cell: the
// number of steps, the most values that wait below the current one, two
// zeros, then the steps.  A step takes an input or a constant as the new
// current value, or combines the current value with an input, or the last
// waiting value with the current one; NOTs ride along.
constexpr int kCellRule = kCellMaxCode + 4;
enum : int { kRuleInput = 7, kRuleInputNot = 8,  // input index, and whether it is complemented
             kRuleOp = 4,                        // shift of the operation: kCellAnd.. less kCellAnd
             kRulePush = 0, kRuleWithInput = 1 << 6, kRuleWithLast = 2 << 6, kRuleConst = 3 << 6,
             kRuleKind = 3 << 6,
             kRuleNot = 1 << 8 };  // the result (of an operation) is complemented; a constant: one

struct GraphView {
  const uint8_t *op;        // [G]
  const int32_t *in;        // [pins][G] (unused pins alias pin 0)
  const int32_t *rev_ptr;   // [n_nets + 1]
  const int32_t *rev_net;   // [n_edges] reader's output net of each fan-out entry
  const int32_t *slot;      // [pins][G] fan-out position of each pin (-1: no such pin)
  const uint16_t *code;     // [n_cells][kCellMaxCode] library cells' stack code (op | arg << 8), padded
  const int32_t *cell;      // [n_cells][3]: code offset, length, inputs
  const uint16_t *rule;     // [n_cells][kCellRule] the code as steps
  const uint64_t *tt;       // [n_cells] truth tables: bit m = output for input pattern m
  const uint8_t *arity;     // [G] input count of each gate
  int32_t pins;             // rows of in and slot (3, or the widest cell)
  int32_t n_pi, G, n_nets;
};

// Simulation word buffers of the query columns a launch covers: column
// cnt.col + c has its own buffer at W + c * col_stride, whose row r (an
// internal net) holds words [t0 - halo, t0 - halo + pitch) of the current
// chunk at r * pitch.  Local word u counts ones when u in [u_lo, u_hi) and
// toggles (against word u - 1) when u in [u_tog_lo, u_hi).
struct ChunkView {
  uint64_t *W;
  int64_t pitch;       // words per row (even)
  int64_t col_stride;  // words between the buffers of consecutive columns
  int64_t t_first;     // global cycle of local word 0 (t0 - halo)
  int32_t pairs;       // word pairs per row to compute, ceil(u_hi / 2)
  int32_t u_lo, u_hi, u_tog_lo;
  int32_t n_cols;      // columns of the launch, cnt.col .. cnt.col + n_cols - 1
};

// Counter arrays [n_nets][B]; a launch adds into columns cnt.col onwards.
struct CountView {
  uint32_t *ones, *tog;
  int32_t B, col;
};

// Signal probabilities are stored as one float per net and column,
// [n_nets][B]: the smaller of p and q = 1 - p, negated when it is q.  The
// kernels work on the pair (p, q): every cell rule has a form without
// cancellation for both, so TR = 2 p q keeps its relative accuracy when p is
// near 0 or 1, and the larger of the two is always 1 minus the smaller, so
// the one float holds the pair exactly.

// SP of one level of B columns, optionally fused into a simulation launch.
struct SpLevel {
  float *sp;          // [n_nets][B]
  int32_t B;
  int32_t g0, n;      // level gate range (internal ids)
};

// Tunables of the simulation launch.
struct SimTune {
  int32_t iters;      // word pairs per lane per wave: 1, 2, 4 or 8
};

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s);
hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s);

// PI probabilities [B][n_pi] (caller layout) -> stored SP [n_pi][B].
hipError_t launch_load_pi(const float *p, float *sp, int32_t n_pi, int32_t B, hipStream_t s);
// Check values are finite and inside [lo, hi]; sets *bad = 1 otherwise (bad may
// be pinned host memory).  copy: where not null, the values are stored there.
hipError_t launch_check_range(const float *v, int64_t n, float lo, float hi, float *copy,
                              uint32_t *bad, hipStream_t s);
// Caller-numbered per-net array [n_nets] -> internal numbering.
hipError_t launch_gather_nets_f32(const float *src_ext, const int32_t *int2ext, float *dst_int,
                                  int32_t n_nets, hipStream_t s);
// [B][n_nets] caller numbering -> [n_nets][B] internal.
hipError_t launch_import_cols_f32(const float *src, const int32_t *int2ext, float *dst,
                                  int32_t n_nets, int32_t B, hipStream_t s);
// Sizes [S][G] caller gate numbering -> [G][S] internal gate order.
hipError_t launch_import_sizes(const float *src, const int32_t *int2ext, const int32_t *ext2int,
                               float *dst, int32_t n_pi, int32_t G, int32_t S, hipStream_t s);

// One SP level (modeled sweep).
// cells: the range holds library cells only (every launch below that takes
// the flag runs a range of one kind; a level's library cells follow its
// fixed cells).
hipError_t launch_sp_level(const GraphView &g, const SpLevel &lv, bool cells, hipStream_t s);
// Two consecutive levels of fixed cells in one launch (b starts where a
// ends; the same columns and SP array): level b's lanes recompute the pins
// level a drives instead of waiting for them, bit for bit as level a's
// lanes compute them.
hipError_t launch_sp_pair(const GraphView &g, const SpLevel &a, const SpLevel &b, hipStream_t s);

// PI rows of one chunk for the launch's columns: Philox stimulus (stim ==
// nullptr) or explicit words stim[c][i][T] (c counted from column cnt.col);
// counts ones/toggles of the PI nets.
// stream [n_pi]: the Philox stream of each PI (null = its own index).
hipError_t launch_stimulus(const GraphView &g, const ChunkView &c, const CountView &cnt,
                           const float *p_col /* stored SP [n_pi][B] */,
                           const uint64_t *stim, int64_t T, const int32_t *stream, uint64_t seed,
                           const SimTune &tune, hipStream_t s);
// Markov stimulus words out [B][n_pi][T] from the PI probabilities (stored
// SP [n_pi][B]), the target transition rates tau [B][n_pi] and the streams
// (null = own).
hipError_t launch_markov_words(const float *sp, const float *tau, const int32_t *stream,
                               int32_t n_pi, int32_t B, int64_t T, uint64_t seed, uint64_t *out,
                               hipStream_t s);

// Library cells with at most this many inputs run in simulation launches
// of their own, with more word pairs per lane than the wider cells.
constexpr int kSmallCellInputs = 3;

// One simulation level of one chunk for the launch's columns, with SP of
// the gates of sp (every column; gates of the launch's kind) fused in when
// sp != nullptr.  cell_inputs: the most inputs a library cell of the range
// has (kSmallCellInputs or fewer selects the narrow instance).
hipError_t launch_sim_level(const GraphView &g, const ChunkView &c, const CountView &cnt,
                            int32_t g0, int32_t n, const SpLevel *sp, bool cells,
                            const SimTune &tune, hipStream_t s, int cell_inputs = 6);

// Caller-numbered exports of forward quantities, [B][n_nets].
struct ExportArgs {
  const float *sp;            // [n_nets][B]
  const float *beta;
  const uint32_t *ones, *tog;
  const int32_t *int2ext;
  int64_t T;
  float *o_sp, *o_tr, *o_sp_acc, *o_tr_acc, *o_beta, *o_tr_hyb;
  uint32_t *o_ones, *o_tog;
  int32_t n_nets, B;
};
hipError_t launch_export(const ExportArgs &a, hipStream_t s);

// The per-net power terms and their sum (Eq. 1, 2, 5).  For net n and
// column b: TR_model = 2 P (1 - P); beta = 1 (modeled), the frozen beta,
// or in hybrid mode clip(TR_acc / TR_model) with TR_acc = toggles /
// (64 (T - 1)) (0/0 -> 1, x/0 -> beta_max), stored in `beta`; the term
// x = kappa beta TR_model, and P[b][s] = sum_n x[n][b] C_n s_s(drv n),
// accumulated in double in an order fixed by the net index alone.  No
// per-net term array is stored: whatever needs x again (the gradient with
// respect to C and s) recomputes it from SP and beta.
struct PowerArgs {
  const float *sp;                  // [n_nets][B]
  const uint32_t *tog;              // [n_nets][B] toggle counts (hybrid), or null
  const float *beta_frozen;         // [n_nets][B], [n_nets] when beta_shared, or null
  int32_t beta_shared;              // one frozen beta for every column
  const float *cap, *size;          // cap [n_nets] internal; size [G][S] internal or null
  int64_t T;                        // simulated words (hybrid)
  float kappa, beta_min, beta_max;
  int32_t mode;                     // DP_MODELED, DP_HYBRID, DP_FROZEN_BETA
  float *beta;                      // out [n_nets][B] (hybrid), or null
  int32_t n_pi, n_nets, G, B, S;    // S = 0: no sizes
  int32_t paired;                   // column b uses size row b; power is [B]
  double *partial;                  // scratch
  int32_t n_chunks;
  float *power;                     // [B][S'] (device)
};
int32_t power_chunks(int32_t n_nets);
// Nets of a slab of the (b, s) contraction: about 256 slabs (see k_power_mfma).
inline int32_t power_slab_nets(int32_t n_nets) {
  const int32_t n = (n_nets / 256 + 63) / 64 * 64;
  return n < 64 ? 64 : n > 2048 ? 2048 : n;
}
inline int32_t power_slabs(int32_t n_nets) {
  const int32_t len = power_slab_nets(n_nets);
  return (n_nets + len - 1) / len;
}
// The (b, s) results whose partials are held at once: the face in pieces of nb
// columns x ns size vectors.  A result's slabs depend on the net count alone
// (its bits do not depend on what shares the call), so the partials of a whole
// face would take up to 32 times what slabs of 2,048 nets do (16,448 nets,
// 4,096 x 4,096 results: 34 GB); a piece's take no more than those, or 64 MiB
// (from which on a piece has a thousand waves of work or more).  Sides are whole
// tiles of 32.
struct PowerPiece {
  int32_t nb, ns;
};
inline PowerPiece power_piece(int32_t n_nets, int32_t B, int32_t S) {
  const int64_t face = (int64_t)B * S, whole = ((int64_t)n_nets + 2047) / 2048 * face;
  const int64_t most = (whole > (1 << 23) ? whole : 1 << 23) / power_slabs(n_nets);
  if (face <= most) return PowerPiece{B, S};
  const auto side = [](int64_t fit, int32_t all) {
    fit = fit < 32 ? 32 : fit / 32 * 32;
    return fit < all ? (int32_t)fit : all;
  };
  const int32_t ns = side(most / (B < 32 ? B : 32), S);
  return PowerPiece{side(most / ns, B), ns};
}
// Doubles of PowerArgs::partial.
inline int64_t power_scratch(int32_t n_nets, int32_t B, int32_t S, int32_t paired) {
  if (S <= 0 || paired || n_nets <= 0) return (int64_t)power_chunks(n_nets) * B;
  const PowerPiece p = power_piece(n_nets, B, S);
  return (int64_t)power_slabs(n_nets) * p.nb * p.ns;
}
hipError_t launch_power(const PowerArgs &a, hipStream_t s);

// The power of several evals (design groups, serving steps) as one pair of
// launches: per column one sum, as launch_power's with one or paired sizes.
// A segment's blocks start at block0 (power_blocks each, a multiple of 8),
// its columns at col0; host, where not null, receives the powers too.
struct PowerSeg {
  PowerArgs a;
  float *host;
  uint32_t block0;
  int32_t col0;
};
inline bool power_merges(const PowerArgs &a) { return a.mode != 1 && (a.S == 0 || a.paired || !a.size); }
uint32_t power_blocks(const PowerArgs &a);
hipError_t launch_power_multi(const PowerSeg *segs /* device */, int32_t n_segs, uint32_t blocks,
                              int32_t cols, int32_t widest /* B */, hipStream_t s);

// Device copies of floats as one launch (a group's outputs: a copy each took
// 4.7 us of the device).
struct CopyList {
  static constexpr int kMax = 32;
  struct Item {
    const float *src;
    float *dst;
    uint32_t n, block0;
  } c[kMax];
  int32_t n = 0;
  uint32_t blocks = 0;
  bool add(const float *src, float *dst, int64_t count);  // false: no room
};
hipError_t launch_copies(const CopyList &l, hipStream_t s);

// A serving step's inputs out of its lanes' pinned host buffers, and their
// gradients into them, each as one launch over all lanes.
struct LaneSeg {
  const float *p;        // pinned [B][n_pi]
  float *sp;             // [n_nets][B]
  const float *size;     // pinned [B][G], or null
  float *size_stage;     // [B][G]
  float *size_dev;       // [G][B]
  const int32_t *int2ext;
  const float *dpi;      // [B][n_pi], or null
  float *dpi_host;       // pinned
  int32_t n_pi, B, G;
  uint32_t stage0, pi_blocks, import0, out0;  // first blocks of its three launches, and its PIs' share
};
// Blocks of a lane in the three launches (and of its PIs in the first).
void lane_seg_blocks(LaneSeg &l, uint32_t &stage, uint32_t &import, uint32_t &out);
hipError_t launch_lanes_stage(const LaneSeg *segs /* device */, int32_t n_segs, uint32_t stage_blocks,
                              uint32_t import_blocks, hipStream_t s);
hipError_t launch_lanes_out(const LaneSeg *segs /* device */, int32_t n_segs, uint32_t blocks,
                            hipStream_t s);

// Reverse sweep.  Columns c in [0, C); the SP column of c is c / cdiv.  The
// local seed of net n in column c is computed where it is used:
//   kappa C_n 2 (q - p) * (beta unless STE) * weight(n, c),
// with weight the upstream weight times the driver's size factor:
//   per_column: w[c] s_{c mod S'}(n);  paired: w[b] s_b(n);
//   otherwise (contracted): sum_s w[b][s] s_s(n).
struct BwdArgs {
  const float *sp;            // [n_nets][B]
  const float *beta;          // [n_nets][B], [n_nets] when beta_shared, or null (beta = 1)
  const float *cap;           // [n_nets] internal
  const float *w;             // [B][S'] (null = 1)
  const float *size;          // [G][S] internal, or null (all 1)
  float *contrib;             // [n_edges][C], in fan-out (reader) order
  float *lam;                 // [C][n_nets] internal: every net's adjoint, or null
  const uint8_t *fixed;       // [n_pi]: nonzero = excluded from the gradients (0), or null
  float kappa;
  int32_t n_pi, G, B, S, C, cdiv, ste, per_column, paired;
  int32_t beta_shared;        // one beta per net for every column
};
// Gates whose fan-out range has more than kHeavyPull entries are "heavy":
// with kSerialColumns columns or more, heavy[0, n_heavy) lists the launch
// range's heavy gates (internal ids, ascending; all of them, no others),
// which cooperative workgroups pull; fewer columns ignore the list.
constexpr int32_t kHeavyPull = 32;
hipError_t launch_bwd_level(const GraphView &g, const BwdArgs &a, int32_t g0, int32_t n,
                            bool cells, hipStream_t s, const int32_t *heavy = nullptr,
                            int32_t n_heavy = 0);
// The per-(b, s) reverse sweep with many size vectors, in adjoints instead of
// contributions: a net's adjoint is its seed plus, over its fan-out entries,
// the reader's adjoint times the entry's partial derivative, which the size
// vectors of one b share.  lam [n_nets][C]; part [n_edges][B].
// launch_edge_partials fills part; then launch_bwd_wide_level per level
// (net0: its first net; heavy: as launch_bwd_level) and for the PIs (net0 0),
// and launch_bwd_wide_out writes out [C][n_pi].
hipError_t launch_edge_partials(const GraphView &g, const float *sp, int32_t B, bool cells,
                                float *part, hipStream_t s);
hipError_t launch_bwd_wide_level(const GraphView &g, const BwdArgs &a, const float *part, float *lam,
                                 int32_t net0, int32_t n, hipStream_t s, const int32_t *heavy,
                                 int32_t n_heavy);
hipError_t launch_bwd_wide_out(const float *lam, int32_t n_pi, int32_t C, float *out, hipStream_t s);

// PI adjoints -> out[c][n_pi].
// heavy[0, n_heavy): every PI with more than kHeavyPull fan-out entries
// (ascending), pulled by cooperative workgroups at kSerialColumns columns or
// more; fewer columns ignore the list.
hipError_t launch_bwd_pi(const GraphView &g, const BwdArgs &a, float *out, hipStream_t s,
                         const int32_t *heavy = nullptr, int32_t n_heavy = 0);

// Several designs in one launch: one level index of every design of a group.
// Segment k owns the blocks [block0_k, block0_{k+1}) (block0 ascending, the
// first 0); its items are the (gate, column) pairs of its level range, column
// innermost, as in the single-design launches.
struct SpSeg {
  GraphView g;
  SpLevel lv;
  // the design's next level in the same launch (fixed cells, launch_sp_pair's
  // recomputation), or n = 0; the segment's items are then (lv.n + lv2.n) B
  SpLevel lv2;
  uint32_t block0;
};
struct BwdSeg {
  GraphView g;
  BwdArgs a;
  int32_t g0, n;
  uint32_t block0;
};
// Threads per workgroup of the merged launches; a segment's block0 and the
// launch's block count are in these units.  One wave: the launches are
// latency-bound gathers, and one-wave groups spread them over more CUs.
constexpr int kMergedBlock = 64;
// segs: device array of n_segs; blocks: total blocks of the launch.
hipError_t launch_sp_multi(const SpSeg *segs, int32_t n_segs, uint32_t blocks, bool cells,
                           hipStream_t s);
hipError_t launch_bwd_multi(const BwdSeg *segs, int32_t n_segs, uint32_t blocks, bool cells,
                            hipStream_t s);

// Every net's adjoint in caller numbering, lam_out [C][n_nets], and the
// Eq. 8 score of every gate from its output net, score [C][G] caller gate
// order: |lambda| P (1 - P) / max(|1 - 2P|, eps).  Either may be null.
hipError_t launch_grad_lambda_export(const float *lam, const float *sp, const int32_t *int2ext,
                                     int32_t n_pi, int32_t n_nets, int32_t B, int32_t C,
                                     int32_t cdiv, float eps, float *lam_out, float *score,
                                     hipStream_t s);

// Power-virus ascent (Alg. 4): P <- clip(P + eta * grad) on the PI rows of
// the stored SP [n_pi][B]; grad is [B][n_pi].
hipError_t launch_virus_step(float *sp, const float *grad, float eta, int32_t n_pi, int32_t B,
                             hipStream_t s);
// v0 = [P >= 1/2] ([B][n_pi] bytes), P ([B][n_pi] floats, or null) and the
// two-cycle stimulus [B][n_pi][2]: word 0 is v0 on every lane, word 1 its
// complement.
hipError_t launch_virus_vectors(const float *sp, uint64_t *stim, uint8_t *v0, float *p_out,
                                int32_t n_pi, int32_t B, hipStream_t s);
// P_virus[b] = sum_n cap[n] [net n toggled in column b] (toggles [n_nets][B]),
// accumulated in double in a fixed order.
hipError_t launch_virus_power(const uint32_t *tog, const float *cap, int32_t n_nets, int32_t B,
                              double *out, hipStream_t s);

// Persistent (cooperative) sweeps: all levels in one launch with a grid
// barrier between levels; fixed cells only.  level_ptr is the device copy of
// the design's level table; max_items the largest level's item count.
//
// The barrier's device words (kBarrierWords uint32, zeroed by the launcher
// on the stream before each launch): one arrival flag per block (block b
// stores the number of the barrier it reached to word b; a launch has at
// most kBarrierFlags blocks) and the timeout flag.  A wait that sees no new
// arrival for limit_ticks ticks of the 100 MHz real-time counter sets the
// timeout flag and stops, and every later wait of the launch stops at once;
// the sweep's outputs are then NaN and the report word (kBarrierReport) is
// set for the host to read.
constexpr int kBarrierFlags = 1024;
constexpr int kBarrierStride = 32;  // 128 bytes
constexpr int kBarrierTimeout = kBarrierFlags;
constexpr int kBarrierWords = kBarrierTimeout + kBarrierStride;
// One more word after them, not zeroed per launch: a wait that gives up also
// sets it, so it records that some sweep since the host last cleared it
// failed.
constexpr int kBarrierReport = kBarrierWords;
constexpr int kBarrierAlloc = kBarrierWords + kBarrierStride;
struct GridBarrier {
  uint32_t *words;       // [kBarrierAlloc]
  uint64_t limit_ticks;  // 100 MHz ticks without progress before a wait gives up
};
hipError_t launch_sp_persistent(const GraphView &g, const SpLevel &lv, const int32_t *level_ptr,
                                int32_t depth, int64_t max_items, GridBarrier bar,
                                hipStream_t s);
// Reverse levels depth..1 and then the PI adjoints into pi_out[c][n_pi].
hipError_t launch_bwd_persistent(const GraphView &g, const BwdArgs &a, const int32_t *level_ptr,
                                 int32_t depth, int64_t max_items, float *pi_out,
                                 GridBarrier bar, hipStream_t s);
// Dataflow sweeps (one launch per sweep, no level barrier; see the kernels):
// each column by a team of workgroups of one XCD, after a launch that arms
// the slots the sweep writes (the gate rows of sp; every entry of contrib)
// and clears the control words.
constexpr int kFlowDies = 8;       // XCDs that blocks are dealt to in turn
constexpr int kFlowXcds = 16;      // values of the XCD id register
constexpr int kFlowTeams = 8;      // teams per XCD at most
constexpr int kFlowMaxCols = 64;   // columns of a sweep at most
constexpr int kFlowLevels = 1024;  // depth + 2 of a design at most (the level table in LDS)
constexpr int kFlowSlots = kFlowMaxCols + 1;  // columns one team may claim, and "none left"
// control words: per team a line with its registration count and (16 words
// on) its closed member count; the columns each team claimed, in order; the
// next unclaimed column; the stop flag
constexpr int kFlowReg = 0;
constexpr int kFlowNext = kFlowReg + 32 * kFlowXcds * kFlowTeams;
constexpr int kFlowStop = kFlowNext + 32;
constexpr int kFlowClaims = kFlowStop + 32;
constexpr int kFlowWords = kFlowClaims + kFlowXcds * kFlowTeams * kFlowSlots;
struct FlowCtl {
  uint32_t *words;    // device, [kFlowWords]
  uint32_t *report;   // host-visible: set when a wait gave up
  uint32_t expected;  // workgroups a team's leader waits for (set by the launcher)
  int32_t n_cu;       // compute units of the device
  int32_t shifts;     // levels in which the waves take turns (set by the launcher)
  int32_t per_block;  // waves of a workgroup that take items (set by the launcher)
  // a wait counts its polls from start and gives up at limit; it looks at that
  // and at the stop flag once in kFlowRound polls
  uint32_t limit, start;
  int32_t sized;      // several designs: staged_sizes of one of them
};
// Polls (a tenth of a microsecond each, so seconds) after which a wait gives up
// by default.
constexpr uint32_t kFlowPolls = 1u << 26;
constexpr uint32_t kFlowRound = 64;
// Whether the seeds of a reverse sweep take several size vectors' weights
// through LDS (from this many on; fewer are read directly).
constexpr int32_t kStagedSizes = 4;
constexpr bool staged_sizes(const BwdArgs &a) {
  return a.size && !a.per_column && !a.paired && a.S >= kStagedSizes;
}
inline void flow_set_limit(FlowCtl &ctl, uint32_t polls) {
  ctl.limit = polls;
  ctl.start = polls < kFlowRound ? kFlowRound - 1 : 0;  // (a small one: at the first poll)
}
// The first block of level l that wave w of a team of `waves` takes, the next
// ones `waves` further each: over all waves every block once, whatever the
// team's size (it may close with fewer members than it was launched with), and
// from `shift` waves on by turns of the level (shifts: 1 or 2).
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int32_t flow_first_block(int32_t w, int32_t waves, int32_t shifts, int32_t l) {
  const int32_t b = w - (l & (shifts - 1)) * (waves / shifts);
  return b < 0 ? b + waves : b;
}
// Whether a sweep of C columns is one for these kernels: within their 32-bit
// offsets and tables, and few enough (net, column) pairs that its levels are
// bound by latency at the depths designs have (forward / reverse sweep by level
// launches against dataflow, in us: 1M gates x 100 levels, 4 columns 233 / 515
// against 183 / 301, 8 columns 238 / 526 against 243 / 521; 117K gates x 60
// levels, 32 columns 143 / 261 against 114 / 268, 64 columns 156 / 269 against
// 237 / 463).  Which of the two a sweep within these limits takes depends on
// its depth too (the eval's rule).
constexpr int64_t kFlowMaxItems = 1 << 22;
// Jobs and (net, column) pairs of a sweep over several designs.  The pairs' line
// is where the range measured first ended and not where level launches catch up:
// on deep designs dataflow is still ahead beyond it (300K gates x 75 levels, 4
// designs x 8 columns, 9.7M pairs, forward / reverse in us 209 / 540 against 235 /
// 976), and below it 1M x 100, 8 designs of one column, 8.1M pairs, 149 / 367
// against 386 / 780.
constexpr int32_t kFlowMaxJobs = kFlowMaxCols;
constexpr int64_t kFlowMultiItems = 2 * kFlowMaxItems;
inline bool flow_fits(const GraphView &g, int32_t depth, int32_t C, int64_t n_edges) {
  return C <= kFlowMaxCols && depth + 2 <= kFlowLevels && g.n_nets < (1 << 24) &&
         (int64_t)g.n_nets * C <= kFlowMaxItems && n_edges < (1ll << 29);
}
struct SpFlow {
  GraphView g;
  float *sp;                 // [n_nets][B]
  const int32_t *level_ptr;  // device copy of the level table
  int32_t B, depth;
};
struct BwdFlow {
  GraphView g;
  BwdArgs a;                 // contrib here: [C][n_edges], each in fan-out order
  float *pi_out;             // [C][n_pi]
  float *seed;               // scratch [C][n_nets]: the nets' seeds
  float *part;               // scratch [B][pins][G]: the gates' partial derivatives
  const int32_t *level_ptr;
  int64_t n_edges;
  int32_t depth;
};
// Several designs in one sweep: segment k's columns are the jobs [job0_k,
// job0_{k+1}) that the teams claim, and its arming takes the blocks from
// block0 on (both ascending, the first 0).
struct SpFlowSeg {
  SpFlow t;
  int32_t job0;
  uint32_t block0;
};
struct BwdFlowSeg {
  BwdFlow t;
  int32_t job0;
  uint32_t block0, arm_blocks, seed_blocks;  // arming: contributions, then seeds, then partials
};
// Blocks that arm a segment (clears: the one that also clears the control
// words, which is the first).
uint32_t flow_arm_blocks(const SpFlow &t, bool clears);
uint32_t flow_arm_blocks(const BwdFlow &t, bool clears, uint32_t *arm_blocks, uint32_t *seed_blocks);
// segs: device table of n_segs; jobs: columns of all segments; blocks: arming
// blocks of all segments; widest: over all segments.
hipError_t launch_sp_flow_multi(const SpFlowSeg *segs, int32_t n_segs, int32_t jobs,
                                uint32_t blocks, int64_t widest, bool cells, FlowCtl ctl,
                                hipStream_t s);
hipError_t launch_bwd_flow_multi(const BwdFlowSeg *segs, int32_t n_segs, int32_t jobs,
                                 uint32_t blocks, int64_t widest, bool cells, FlowCtl ctl,
                                 hipStream_t s);
// widest: gates of the widest level; cells: the design holds library cells.
// Arms the slots of an SP sweep and clears its control words (launch_sp_flow
// does so itself).
hipError_t launch_sp_arm(const SpFlow &t, FlowCtl ctl, hipStream_t s);
hipError_t launch_sp_flow(const SpFlow &t, int64_t widest, bool cells, FlowCtl ctl, hipStream_t s);
// The reverse levels and then the PI adjoints; widest also covers the PIs.
hipError_t launch_bwd_flow(const BwdFlow &t, int64_t widest, bool cells, FlowCtl ctl,
                           hipStream_t s);

// The simulation in word tiles (see the kernels): a tile is `pitch` words of
// one column, all levels by one team of workgroups of one XCD.  Control words: a line per (XCD, team) with its registration; the
// next team buffer, the next tile, the stop flag; per buffer a line with its
// team's claimed tile and one per member for the level flags.
constexpr int kSimTeams = 4;      // teams per XCD at most
constexpr int kSimMembers = 32;   // workgroups per team at most
constexpr int kSimBufs = kFlowDies * kSimTeams;
constexpr int kSimReg = 0;
constexpr int kSimNextBuf = kSimReg + 32 * kFlowXcds * kSimTeams;
constexpr int kSimNextTile = kSimNextBuf + 32;
constexpr int kSimStop = kSimNextTile + 32;
constexpr int kSimClaim = kSimStop + 32;
constexpr int kSimFlags = kSimClaim + 32 * kSimBufs;
constexpr int kSimWords = kSimFlags + 32 * kSimBufs * kSimMembers;
// In the counts of a simulation that gave up (a count is 64 T at most); rates
// and betas formed from it are NaN.
constexpr uint32_t kNoCount = 0xFFFFFFFFu;
struct SimFlow {
  GraphView g;
  const int32_t *level_ptr;
  const uint64_t *stim;  // [B][n_pi][T] the PIs' words
  uint64_t *W;           // [n_bufs][n_nets][pitch] the teams' rows
  uint32_t *cnt;         // [B][n_chunks][n_nets] counts, ones | toggles << 16
  uint64_t *edge;        // [B][n_chunks][n_nets][2] first and last word
  int64_t T;
  int32_t depth, B;
  int32_t pitch, n_chunks;  // words per tile (16, 32 or 64), tiles per column
  int32_t n_bufs;           // teams that work at once
};
// Whether a simulation is within the kernels' 32-bit offsets and tables.
inline bool sim_fits(const GraphView &g, int32_t depth, int32_t B, int32_t pitch, int64_t T) {
  return depth >= 1 && depth + 2 <= kFlowLevels && (pitch == 16 || pitch == 32 || pitch == 64) &&
         (int64_t)g.n_nets * pitch < (1ll << 29) && g.n_nets < (1 << 27) &&
         (T + pitch - 1) / pitch < 65535 / B;
}
hipError_t launch_stim_words(const float *sp /* stored SP [n_pi][B] */, const int32_t *stream,
                             int32_t n_pi, int32_t B, int64_t T, uint64_t seed, uint64_t *out,
                             hipStream_t s);
// Whether the SP sweep of the simulated columns goes out with the tiles: with
// one or two columns it holds one or two XCDs' CUs, and the other XCDs' teams
// take up the tiles (300K gates half library cells 1030 -> 785 us a pass, 117K
// gates x 257 words 416 -> 365).  Five columns gain nothing (50K gates x 64
// words: 140 us one after the other, 147 together).
constexpr int32_t kRideColumns = 2;
// The simulation, and with sp.B <= kRideColumns the SP sweep of the same columns
// (armed by launch_sp_arm), as one launch.  ctl.words: [kSimWords].  Writes ones
// and tog [n_nets][B]; a simulation that gives up leaves kNoCount
// there and NaN as the gates' probabilities.
hipError_t launch_sim_flow(const SimFlow &t, const SpFlow &sp, int64_t widest, bool cells,
                           FlowCtl ctl, FlowCtl sp_ctl, uint32_t *ones, uint32_t *tog,
                           hipStream_t s);

// dcap[ext n] = sum_{b,s} w[b][s] x[n][b] size_s(n) and dsize[s][ext g] =
// sum_b w[b][s] x[out g][b] C_out g, with x = kappa beta TR_model
// recomputed from SP and beta.
struct GradExportArgs {
  const float *sp;            // [n_nets][B]
  const float *beta;          // [n_nets][B], [n_nets] when beta_shared, or null (beta = 1)
  int32_t beta_shared;
  float kappa;
  const float *cap;           // [n_nets]
  const float *w;             // [B][S'] or null
  const float *size;          // [G][S] internal or null
  const int32_t *int2ext;
  int32_t n_pi, n_nets, G, B, S;
  int32_t paired;             // column b uses size row b
  float *dcap;                // [n_nets] caller numbering (sum over b, s) or null
  float *dsize;               // [S][G] caller gate numbering (sum over b) or null
};
hipError_t launch_grad_export(const GradExportArgs &a, hipStream_t s);

}  // namespace dp

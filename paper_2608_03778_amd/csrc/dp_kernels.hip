// gfx950 kernels of the DiffPower hot path.
//
// Layouts (internal net numbering, see dp_design):
//   SP (packed, see sp_load)       float  [n_nets][B]      (query column innermost)
//   beta                           float  [n_nets][B]      (hybrid; a frozen beta is read as given)
//   contrib                        float  [n_edges][C]     (fan-out order of the reader)
//   simulation words W             uint64 [n_nets][pitch]  (one chunk of cycles)
//   ones, toggles                  uint32 [n_nets][B]
//
// Work mapping: the SP and reverse kernels give one lane to each
// (gate or net, column).  The simulation kernel gives one 64-lane wave to a
// (gate, run of word pairs): the wave's cell is uniform, so the cell switch
// is a scalar branch outside the word loop; each lane moves 16-byte word
// pairs, so every fan-in row is read as contiguous 1 KiB wave-wide accesses.

#include <algorithm>
#include <type_traits>

#include "dp_kernels.h"

namespace dp {
namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / 64;
// The simulation level runs in smaller workgroups: finer grains fill the
// chip's last wave of blocks more evenly (0.5% per level on MI355X against
// 256 threads; 64 threads gained nothing further).
constexpr int kSimBlock = 128;
constexpr int kSimWaves = kSimBlock / 64;
// Per-level SP and reverse launches are latency-bound gathers with few items
// (one per gate and column): one-wave workgroups spread a level over as many
// CUs as it has waves, so no CU's address unit serialises several waves'
// gathers (the one-column reverse level 0.5 us faster than with 256 threads).
constexpr int kLevelBlock = 64;

// Two consecutive simulation words as one 16-byte vector (a single
// dwordx4 access per lane).
typedef uint64_t w2 __attribute__((ext_vector_type(2)));
// A signal probability and its complement (p, q = 1 - p), one 8-byte access.
typedef float f2 __attribute__((ext_vector_type(2)));

enum : int { INV = 0, BUF, AND2, OR2, NAND2, NOR2, XOR2, AOI21, MUX2 };

__device__ __forceinline__ int arity_of(int op) { return op < AND2 ? 1 : (op < AOI21 ? 2 : 3); }

__device__ __forceinline__ float clamp01(float v) { return fminf(fmaxf(v, 0.0f), 1.0f); }

// A net's probability is stored as one float: the smaller of p and q =
// 1 - p, negated when it is q (sign bit set: p is the larger, so p = 1 is
// -0.0).  The larger is always 1 minus the smaller (settle() makes it so for
// gate outputs, and for a startpoint p >= 1/2 the difference 1 - p is exact),
// so the (p, q) pair the rules work on comes back bit for bit from 4 bytes.
__device__ __forceinline__ f2 sp_load(float s) {
  const float m = fabsf(s);
  return (__float_as_uint(s) >> 31) ? f2{1.0f - m, m} : f2{m, 1.0f - m};
}

// A startpoint probability in the stored form.
__device__ __forceinline__ float sp_pack(float p) { return p <= 0.5f ? p : -(1.0f - p); }

// Clip to [0, 1] (Alg. 2) and re-tie the pair: the smaller of p and q comes
// from its own formula (full relative accuracy), the larger is 1 minus it.
// Without this, rounding drift of p + q - 1 adds up along reconvergent
// paths and grows with the number of paths.  Returns the stored form.
__device__ __forceinline__ float settle(f2 v) {
  const float p = clamp01(v.x), q = clamp01(v.y);
  return p <= q ? p : -q;
}

// Probability that the cell output is 1, and its complement, for
// independent inputs (Sec. II-B; Alg. 2 gives AND = a0 a1 and NAND =
// 1 - a0 a1).  Inputs and outputs are (p, q = 1 - p) pairs and every
// formula is a sum of products of p's and q's, so neither output loses
// relative accuracy when the probability is close to 0 or 1.
__device__ __forceinline__ f2 sp_rule(int op, f2 a, f2 b, f2 c) {
  const float pa = a.x, qa = a.y, pb = b.x, qb = b.y, pc = c.x, qc = c.y;
  f2 r;
  switch (op) {
    case INV: r = f2{qa, pa}; break;
    case BUF: r = a; break;
    case AND2: r = f2{pa * pb, fmaf(pa, qb, qa)}; break;
    case OR2: r = f2{fmaf(qa, pb, pa), qa * qb}; break;
    case NAND2: r = f2{fmaf(pa, qb, qa), pa * pb}; break;
    case NOR2: r = f2{qa * qb, fmaf(qa, pb, pa)}; break;
    case XOR2: r = f2{fmaf(pa, qb, qa * pb), fmaf(pa, pb, qa * qb)}; break;
    case AOI21: r = f2{fmaf(pa, qb, qa) * qc, fmaf(pa * pb, qc, pc)}; break;  // !((A1&A2)|B)
    default: r = f2{fmaf(qc, pa, pc * pb), fmaf(qc, qa, pc * qb)}; break;     // MUX2 S?I1:I0
  }
  return r;
}

// Partial derivatives of the output probability with respect to each input
// probability (Sec. III-E: dAND/da = b, dOR/da = 1 - b, dXOR/da = 1 - 2b,
// dNOT = -1; the compound cells by the product rule).
__device__ __forceinline__ void sp_partials(int op, f2 a, f2 b, f2 c, float &d0, float &d1,
                                            float &d2) {
  const float pa = a.x, qa = a.y, pb = b.x, qb = b.y, pc = c.x, qc = c.y;
  d1 = 0.0f;
  d2 = 0.0f;
  switch (op) {
    case INV: d0 = -1.0f; break;
    case BUF: d0 = 1.0f; break;
    case AND2: d0 = pb; d1 = pa; break;
    case OR2: d0 = qb; d1 = qa; break;
    case NAND2: d0 = -pb; d1 = -pa; break;
    case NOR2: d0 = -qb; d1 = -qa; break;
    case XOR2: d0 = qb - pb; d1 = qa - pa; break;
    case AOI21: d0 = -pb * qc; d1 = -pa * qc; d2 = -fmaf(pa, qb, qa); break;
    default: d0 = qc; d1 = pc; d2 = pb - pa; break;  // MUX2
  }
}

// ---------------------------------------------------------------- library cells
// A library cell is post-order stack code (Alg. 1), interpreted operation by
// operation: each binary operation applies its independent-input rule to its
// two operands (Sec. III-E: AND ab, OR a + b - ab, XOR a + b - 2ab, NOT 1 - a),
// in the same cancellation-free (p, q) form as the fixed cells.
// Each cell's code sits padded to kCellMaxCode words (64 bytes) at offset
// c * kCellMaxCode, so a lane loads its whole program with four 16-byte
// loads that depend only on the opcode, in flight with its input gathers,
// and interprets it from registers.
struct LaneCode {
  uint32_t w[kCellMaxCode / 2];  // two instructions per dword
  int len, nin;
};

__device__ __forceinline__ LaneCode lane_code(const GraphView &g, int op) {
  LaneCode lc;
  const int c = op - kCellBase;
  lc.len = g.cell[3 * c + 1];
  lc.nin = g.cell[3 * c + 2];
  const uint4 *src = reinterpret_cast<const uint4 *>(g.code + (int64_t)c * kCellMaxCode);
#pragma unroll
  for (int k = 0; k < kCellMaxCode / 8; ++k) {
    const uint4 v = src[k];
    lc.w[4 * k] = v.x;
    lc.w[4 * k + 1] = v.y;
    lc.w[4 * k + 2] = v.z;
    lc.w[4 * k + 3] = v.w;
  }
  return lc;
}

__device__ __forceinline__ int code_at(const LaneCode &lc, int i) {
  return (int)((lc.w[i >> 1] >> ((i & 1) * 16)) & 0xffffu);
}

__device__ __forceinline__ f2 pair_op(int op, f2 a, f2 b) {
  if (op == kCellAnd) return f2{a.x * b.x, fmaf(a.x, b.y, a.y)};
  if (op == kCellOr) return f2{fmaf(a.y, b.x, a.x), a.y * b.y};
  return f2{fmaf(a.x, b.y, a.y * b.x), fmaf(a.x, b.x, a.y * b.y)};  // XOR
}

// One cell's steps, the same cell for the wave: a step's form is a scalar
// branch, up to NS waiting values shift through registers, and the steps come
// four at a time, the next four on their way.  (The stack code interpreted
// lane by lane had stack and inputs in scratch memory: 0.5 us an instruction,
// 738 us for the SP sweep of 300K gates x 75 levels, half of them library
// cells; the code interpreted this way 347 us, its steps 267.)
template <int NS, class Src>
__device__ __forceinline__ f2 cell_steps(Src src, int n, uint64_t next, const f2 (&x)[kCellMaxIn]) {
  f2 st[NS];  // waiting, the last one first
#pragma unroll
  for (int j = 0; j < NS; ++j) st[j] = f2{0.0f, 1.0f};
  f2 top = st[0];
  for (int i = 0; i < n;) {
    uint64_t w = next;
    next = src[min(i / 4 + 2, kCellRule / 4 - 1)];
    for (const int end = min(i + 4, n); i < end; ++i, w >>= 16) {
      const int c = (int)w & 0xffff, kind = c & kRuleKind;
      f2 in = x[0];
#pragma unroll
      for (int j = 1; j < kCellMaxIn; ++j)
        if ((c & kRuleInput) == j) in = x[j];
      if (c & kRuleInputNot) in = f2{in.y, in.x};
      if (kind == kRulePush || kind == kRuleConst) {
#pragma unroll
        for (int j = NS - 1; j > 0; --j) st[j] = st[j - 1];
        st[0] = top;
        if (kind == kRuleConst) in = c & kRuleNot ? f2{1.0f, 0.0f} : f2{0.0f, 1.0f};
        top = in;
      } else {
        f2 a = top, b = in;
        if (kind == kRuleWithLast) {
          a = st[0];
          b = top;
#pragma unroll
          for (int j = 0; j + 1 < NS; ++j) st[j] = st[j + 1];
        }
        top = pair_op(((c >> kRuleOp) & 3) + kCellAnd, a, b);
        if (c & kRuleNot) top = f2{top.y, top.x};
      }
    }
  }
  return top;
}
__device__ __forceinline__ f2 cell_sp_uniform(const GraphView &g, int cell, const f2 (&x)[kCellMaxIn]) {
  const auto *src = (const __attribute__((address_space(4))) uint64_t *)(uintptr_t)(g.rule + (int64_t)cell * kCellRule);
  const uint64_t head = src[0], next = src[1];
  const int n = (int)head & 0xffff, most = (int)(head >> 16) & 0xffff;
  return most <= 2 ? cell_steps<2>(src, n, next, x) : cell_steps<kCellMaxStack - 1>(src, n, next, x);
}
// A wave of one cell takes its steps under scalar control; lanes of different
// cells go through their own together, masks in place of branches.  (A turn of
// the wave per cell, which gates sorted by cell keep to a few: forward of 2K
// gates x 20 levels of 200 different cells, one column, 1,038 us against 126; of
// nine cells 263 against 143; 300K gates x 75 levels of nine 637 against 617.
// Without the scalar form: 64 columns, 251 us against 267 for 20K gates.)
__device__ __forceinline__ f2 cell_sp(const GraphView &g, int op, const f2 (&x)[kCellMaxIn]) {
  const int first = __builtin_amdgcn_readfirstlane(op);
  if (__all(op == first)) return cell_sp_uniform(g, first - kCellBase, x);
  const auto *src = reinterpret_cast<const uint64_t *>(g.rule + (int64_t)(op - kCellBase) * kCellRule);
  const uint64_t head = src[0], next = src[1];
  return cell_steps<kCellMaxStack - 1>(src, (int)head & 0xffff, next, x);
}

// Partial derivatives of a cell's probability with respect to its inputs
// (Sec. III-E, Alg. 3), by reverse mode over the code read as a tape.  The
// forward pass gives every instruction its value and records, for each
// operation, which instructions produced its operands (the stack holds
// instruction indices).  Every value feeds exactly one later instruction
// (the code is a tree), so the backward pass visits the instructions from
// the last to the first and finds each adjoint set, once, by its consumer:
// an operation sets its operands' adjoints to its own times the local
// derivative (AND: the other operand; OR: its complement; XOR: q - p of the
// other operand; NOT: -1), and an input instruction adds its adjoint to the
// input's partial.
__device__ void cell_partials(const LaneCode &lc, const f2 *x, float *d) {
  f2 val[kCellMaxCode];
  float adj[kCellMaxCode];
  uint8_t lhs[kCellMaxCode], rhs[kCellMaxCode];
  uint8_t st[kCellMaxStack];
  int top = 0;
  for (int i = 0; i < lc.len; ++i) {
    const int w = code_at(lc, i), op = w & 0xff;
    if (op == kCellIn) {
      val[i] = x[w >> 8];
    } else if (op == kCellZero) {
      val[i] = f2{0.0f, 1.0f};
    } else if (op == kCellOne) {
      val[i] = f2{1.0f, 0.0f};
    } else if (op == kCellNot) {
      lhs[i] = st[--top];
      val[i] = f2{val[lhs[i]].y, val[lhs[i]].x};
    } else {
      rhs[i] = st[--top];
      lhs[i] = st[--top];
      val[i] = pair_op(op, val[lhs[i]], val[rhs[i]]);
    }
    st[top++] = (uint8_t)i;
  }
  for (int k = 0; k < lc.nin; ++k) d[k] = 0.0f;
  adj[lc.len - 1] = 1.0f;
  for (int i = lc.len - 1; i >= 0; --i) {
    const int w = code_at(lc, i), op = w & 0xff;
    const float a = adj[i];
    if (op == kCellIn) {
      d[w >> 8] += a;
    } else if (op == kCellNot) {
      adj[lhs[i]] = -a;
    } else if (op == kCellAnd || op == kCellOr || op == kCellXor) {
      const f2 u = val[lhs[i]], v = val[rhs[i]];
      const float du = op == kCellAnd ? v.x : (op == kCellOr ? v.y : v.y - v.x);
      const float dv = op == kCellAnd ? u.x : (op == kCellOr ? u.y : u.y - u.x);
      adj[lhs[i]] = a * du;
      adj[rhs[i]] = a * dv;
    }
  }
}

// Boolean function of a cell on 64 lanes (Sec. III-C).
template <int OP>
__device__ __forceinline__ uint64_t cell_bits(uint64_t a, uint64_t b, uint64_t c) {
  if constexpr (OP == INV) return ~a;
  else if constexpr (OP == BUF) return a;
  else if constexpr (OP == AND2) return a & b;
  else if constexpr (OP == OR2) return a | b;
  else if constexpr (OP == NAND2) return ~(a & b);
  else if constexpr (OP == NOR2) return ~(a | b);
  else if constexpr (OP == XOR2) return a ^ b;
  else if constexpr (OP == AOI21) return ~((a & b) | c);
  else return (a & ~c) | (b & c);  // MUX2
}

template <int OP>
constexpr int kArity = OP < AND2 ? 1 : (OP < AOI21 ? 2 : 3);

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__device__ __forceinline__ int64_t gidx() {
  return (int64_t)blockIdx.x * kBlock + threadIdx.x;
}

// Launches stay below 2^32 threads in total.
constexpr int64_t kMaxBlocks = (1ll << 32) / kBlock - 1;
inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }
inline unsigned level_blocks(int64_t n) { return (unsigned)((n + kLevelBlock - 1) / kLevelBlock); }
// SP level launches of many lanes take 256-thread workgroups: a dependent
// launch of 5,000 one-wave workgroups costs about 0.3 us more than one of
// 1,250 four-wave workgroups, while a few waves still spread over as many
// CUs as one-wave workgroups give them.
constexpr int kWideBlock = 256;
constexpr int64_t kWideLanes = 65536;
inline unsigned level_block(int64_t lanes) { return lanes >= kWideLanes ? kWideBlock : kLevelBlock; }
inline unsigned level_grid(int64_t lanes) {
  const int64_t bs = level_block(lanes);
  return (unsigned)((lanes + bs - 1) / bs);
}
inline bool too_big(int64_t items) { return (items + kBlock - 1) / kBlock > kMaxBlocks; }

// ---------------------------------------------------------------- plumbing
__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
  int64_t i = gidx();
  if (i < n) p[i] = v;
}
__global__ __launch_bounds__(kBlock) void k_fill_f32(float *p, int64_t n, float v) {
  int64_t i = gidx();
  if (i < n) p[i] = v;
}

__global__ __launch_bounds__(kBlock) void k_load_pi(const float *__restrict__ p,
                                                     float *__restrict__ sp, int32_t n_pi,
                                                     int32_t B) {
  int64_t idx = gidx();
  if (idx >= (int64_t)n_pi * B) return;
  int32_t i = (int32_t)(idx / B), b = (int32_t)(idx - (int64_t)i * B);
  sp[idx] = sp_pack(p[(int64_t)b * n_pi + i]);
}

__global__ __launch_bounds__(kBlock) void k_check_range(const float *__restrict__ v, int64_t n,
                                                         float lo, float hi, float *copy,
                                                         uint32_t *bad) {
  int64_t i = gidx();
  if (i >= n) return;
  float x = v[i];
  if (copy) copy[i] = x;
  if (!(x >= lo && x <= hi)) *bad = 1;  // NaN fails both comparisons
}

__global__ __launch_bounds__(kBlock) void k_gather_nets(const float *__restrict__ src,
                                                         const int32_t *__restrict__ int2ext,
                                                         float *__restrict__ dst, int32_t n) {
  int64_t i = gidx();
  if (i < n) dst[i] = src[int2ext[i]];
}

__global__ __launch_bounds__(kBlock) void k_import_cols(const float *__restrict__ src,
                                                         const int32_t *__restrict__ int2ext,
                                                         float *__restrict__ dst, int32_t n_nets,
                                                         int32_t B) {
  int64_t idx = gidx();
  if (idx >= (int64_t)n_nets * B) return;
  int32_t n = (int32_t)(idx / B), b = (int32_t)(idx - (int64_t)n * B);
  dst[idx] = src[(int64_t)b * n_nets + int2ext[n]];
}

// Sizes [S][G] in caller gate order -> [G][S] in internal order: the kernels
// that read them have a net's size vectors in consecutive lanes (with [S][G]
// the per-(b, s) reverse level read 64 lines per wave for its sizes alone).
// A block takes 64 gates x 8 size vectors through LDS: gathers along a row of
// the caller's array, stores along a row of the result.  With many vectors a
// group of eight stays with one XCD, whose L2 holds its rows while all gates
// gather from them (117K gates x 256: 368 us with groups of 32 anywhere).
constexpr int32_t kSizeGates = 64, kSizeVecs = 8;
constexpr int32_t kSizeXcds = 8;
__device__ __forceinline__ void import_sizes(const float *__restrict__ src,
                                             const int32_t *__restrict__ int2ext,
                                             float *__restrict__ dst, int32_t n_pi, int32_t G,
                                             int32_t S, int32_t block) {
  __shared__ float tile[kSizeGates][kSizeVecs + 1];
  const int32_t g_tiles = (G + kSizeGates - 1) / kSizeGates;
  const int32_t groups = (S + kSizeVecs - 1) / kSizeVecs;
  const int32_t ways = groups >= kSizeXcds ? kSizeXcds : 1;  // blocks go to the XCDs in turn
  const int32_t slot = block / ways;
  const int32_t g0 = (slot % g_tiles) * kSizeGates;
  const int32_t s0 = (slot / g_tiles * ways + block % ways) * kSizeVecs;
  if (s0 >= S) return;
  const int32_t gl = (int32_t)threadIdx.x & 63, sl = (int32_t)threadIdx.x >> 6;
  if (g0 + gl < G) {
    const int32_t e = int2ext[n_pi + g0 + gl] - n_pi;
#pragma unroll
    for (int k = 0; k < kSizeVecs / kWavesPerBlock; ++k) {
      const int32_t s = s0 + sl + k * kWavesPerBlock;
      if (s < S) tile[gl][sl + k * kWavesPerBlock] = src[(int64_t)s * G + e];
    }
  }
  __syncthreads();
  const int32_t ns = min(kSizeVecs, S - s0), ng = min(kSizeGates, G - g0);
  for (int32_t i = (int32_t)threadIdx.x; i < ng * ns; i += kBlock)
    dst[(int64_t)(g0 + i / ns) * S + s0 + i % ns] = tile[i / ns][i % ns];
}
__global__ __launch_bounds__(kBlock) void k_import_sizes(const float *__restrict__ src,
                                                          const int32_t *__restrict__ int2ext,
                                                          float *__restrict__ dst, int32_t n_pi,
                                                          int32_t G, int32_t S) {
  import_sizes(src, int2ext, dst, n_pi, G, S, (int32_t)blockIdx.x);
}

// The same from the caller's side: a block reads 64 of the caller's gates x 32
// size vectors, whole lines, and writes each gate's run of the result.  The
// gathers above fetch a line for every float once a row is past an L2
// (dp_set_cell_sizes, us, gathered / in runs: 117K gates x 32 43 / 25, x 256
// 209 / 89; 300K x 32 134 / 39; 1M x 2 35 / 30, x 8 144 / 39, x 32 562 / 87).
// One vector has runs of a single float (1M 25 / 28), and small arrays are the
// launches alone (117K x 4 16.6 / 17.5, x 6 17.6 / 17.7, x 8 19.4 / 17.7;
// 300K x 2 17.4 / 18.5, x 3 19.6 / 19.8, x 4 22.9 / 20.2; 50K x 12 17.5 / 17.1).
constexpr int32_t kSizeRuns = 32;
constexpr int64_t kSizeRunsMin = 800'000;
__global__ __launch_bounds__(kBlock) void k_import_size_runs(const float *__restrict__ src,
                                                              const int32_t *__restrict__ ext2int,
                                                              float *__restrict__ dst, int32_t n_pi,
                                                              int32_t G, int32_t S) {
  __shared__ float tile[kSizeGates][kSizeRuns + 1];
  __shared__ int32_t row[kSizeGates];
  const int32_t g_tiles = (G + kSizeGates - 1) / kSizeGates;
  const int32_t g0 = ((int32_t)blockIdx.x % g_tiles) * kSizeGates;
  const int32_t s0 = ((int32_t)blockIdx.x / g_tiles) * kSizeRuns;
  const int32_t gl = (int32_t)threadIdx.x & 63, sl = (int32_t)threadIdx.x >> 6;
  const int32_t ns = min(kSizeRuns, S - s0), ng = min(kSizeGates, G - g0);
  if (gl < ng) {
    if (sl == 0) row[gl] = ext2int[n_pi + g0 + gl] - n_pi;
#pragma unroll
    for (int k = 0; k < kSizeRuns / kWavesPerBlock; ++k) {
      const int32_t s = sl + k * kWavesPerBlock;
      if (s < ns) tile[gl][s] = src[(int64_t)(s0 + s) * G + g0 + gl];
    }
  }
  __syncthreads();
  for (int32_t i = (int32_t)threadIdx.x; i < ng * ns; i += kBlock)
    dst[(int64_t)row[i / ns] * S + s0 + i % ns] = tile[i / ns][i % ns];
}

// ---------------------------------------------------------------- serving steps
// A step's lanes staged by one launch that reads their pinned host buffers
// itself, and one that orders the sizes; the gradients go back the same way.
// (A copy and a launch per lane and array: with eight lanes of 10K to 117K
// gates a step spent 290 us before its sweeps, half of it the copy engine's
// latency.)
template <class Seg>
__device__ __forceinline__ int32_t seg_at(const Seg *segs, int32_t n, uint32_t Seg::*first) {
  int32_t k = 0;
  while (k + 1 < n && segs[k + 1].*first <= blockIdx.x) ++k;
  return k;
}
constexpr int32_t kLaneCopy = 4 * 4 * kBlock;  // floats a block copies
__device__ __forceinline__ void lane_copy(const float *src, float *dst, int64_t n, uint32_t block) {
  const int64_t i0 = (int64_t)block * kLaneCopy + 4 * threadIdx.x;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = i0 + 4 * kBlock * k;
    if (i + 4 <= n) {
      *reinterpret_cast<float4 *>(dst + i) = *reinterpret_cast<const float4 *>(src + i);
    } else {
      for (int64_t j = i; j < n; ++j) dst[j] = src[j];
    }
  }
}
constexpr int32_t kCopyPer = 4;  // floats a thread copies
__global__ __launch_bounds__(kBlock) void k_copies(CopyList l) {
  int32_t k = 0;
  while (k + 1 < l.n && l.c[k + 1].block0 <= blockIdx.x) ++k;
  const uint32_t i0 = (blockIdx.x - l.c[k].block0) * (kBlock * kCopyPer) + threadIdx.x;
#pragma unroll
  for (int j = 0; j < kCopyPer; ++j) {
    const uint32_t i = i0 + j * kBlock;
    if (i < l.c[k].n) l.c[k].dst[i] = l.c[k].src[i];
  }
}
__global__ __launch_bounds__(kBlock) void k_lanes_stage(const LaneSeg *__restrict__ segs, int32_t n_segs) {
  const LaneSeg l = segs[seg_at(segs, n_segs, &LaneSeg::stage0)];
  const uint32_t block = blockIdx.x - l.stage0;
  if (block >= l.pi_blocks) {
    lane_copy(l.size, l.size_stage, (int64_t)l.B * l.G, block - l.pi_blocks);
    return;
  }
  const int64_t i = (int64_t)block * kBlock + threadIdx.x;
  if (i >= (int64_t)l.n_pi * l.B) return;
  const int32_t b = (int32_t)(i / l.n_pi), pi = (int32_t)(i - (int64_t)b * l.n_pi);
  l.sp[(int64_t)pi * l.B + b] = sp_pack(l.p[i]);
}
__global__ __launch_bounds__(kBlock) void k_lanes_import(const LaneSeg *__restrict__ segs, int32_t n_segs) {
  const LaneSeg l = segs[seg_at(segs, n_segs, &LaneSeg::import0)];
  import_sizes(l.size_stage, l.int2ext, l.size_dev, l.n_pi, l.G, l.B, (int32_t)(blockIdx.x - l.import0));
}
__global__ __launch_bounds__(kBlock) void k_lanes_out(const LaneSeg *__restrict__ segs, int32_t n_segs) {
  const LaneSeg l = segs[seg_at(segs, n_segs, &LaneSeg::out0)];
  lane_copy(l.dpi, l.dpi_host, (int64_t)l.B * l.n_pi, blockIdx.x - l.out0);
}

// ---------------------------------------------------------------- SP level
// One lane per (gate, column) of level [g0, g0 + n): gather the fan-in
// probabilities, apply the cell rule, clip to [0, 1] (Alg. 2).
// CELLS: the range holds library cells only (their own kernel instances, so
// the fixed-cell kernels keep their register budget).
// Row j of a per-pin table ([pins][G]), or row 0 where the design's widest
// gate has fewer pins: a choice of address that is uniform across the
// launch, so a gather through it waits on no other load.  (In the fan-in
// table, pins a gate does not use alias its pin 0; callers ignore them.)
__device__ __forceinline__ const int32_t *pin_row(const int32_t *tab, const GraphView &g, int j) {
  return tab + (g.pins > j ? (int64_t)j * g.G : 0);
}

// Takes loaded values at this point: every load before it is then issued
// ahead of the first wait, and none can be moved into the branch of the one
// opcode that reads it or behind a use of another (each would add a
// dependent round trip).
template <typename T>
__device__ __forceinline__ void value_taken(T v) { asm volatile("" ::"v"(v)); }
template <typename... V>
__device__ __forceinline__ void gathers_done(V... v) {
  (value_taken(v), ...);
}

template <bool CELLS>
__device__ __forceinline__ void sp_item(const GraphView &g, const SpLevel &lv, uint32_t idx) {
  const int32_t B = lv.B;
  const uint32_t gl32 = idx / (uint32_t)B;
  const int32_t gl = (int32_t)gl32;
  const int32_t b = (int32_t)(idx - gl32 * (uint32_t)B);
  const int32_t gi = lv.g0 + gl;
  const int op = g.op[gi];
  float *sp = lv.sp;
  if constexpr (CELLS) {
    // every pin row (unused pins alias pin 0), so the gathers need no count;
    // the indices arrive with the opcode, the probabilities with the cell's
    // code, and no gather waits on another
    int32_t pin[kCellMaxIn];
#pragma unroll
    for (int k = 0; k < kCellMaxIn; ++k) pin[k] = k < g.pins ? g.in[k * g.G + gi] : 0;
    value_taken(op);
#pragma unroll
    for (int k = 0; k < kCellMaxIn; ++k) value_taken(pin[k]);
    float r[kCellMaxIn];
#pragma unroll
    for (int k = 0; k < kCellMaxIn; ++k) r[k] = k < g.pins ? sp[(int64_t)pin[k] * B + b] : 0.0f;
    f2 x[kCellMaxIn];
#pragma unroll
    for (int k = 0; k < kCellMaxIn; ++k) x[k] = k < g.pins ? sp_load(r[k]) : f2{0.0f, 1.0f};
    sp[(int64_t)(g.n_pi + gi) * B + b] = settle(cell_sp(g, op, x));
    return;
  }
  // the opcode and every pin's index arrive in one load round; the second
  // round gathers the probabilities of the pins the gate has
  const int32_t i0 = g.in[gi];
  const int32_t i1 = pin_row(g.in, g, 1)[gi];
  const int32_t i2 = pin_row(g.in, g, 2)[gi];
  gathers_done(op, i0, i1, i2);
  const int k = arity_of(op);
  const float sa = sp[(int64_t)i0 * B + b];
  float sb = 0.0f, sc = 0.0f;
  if (k > 1) sb = sp[(int64_t)i1 * B + b];
  if (k > 2) sc = sp[(int64_t)i2 * B + b];
  gathers_done(sa, sb, sc);
  const f2 z = f2{0.0f, 1.0f};
  sp[(int64_t)(g.n_pi + gi) * B + b] =
      settle(sp_rule(op, sp_load(sa), k > 1 ? sp_load(sb) : z, k > 2 ? sp_load(sc) : z));
}

__global__ __launch_bounds__(kWideBlock) void k_sp_level(GraphView g, SpLevel lv) {
  const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < (uint32_t)lv.n * (uint32_t)lv.B) sp_item<false>(g, lv, idx);
}

__global__ __launch_bounds__(kBlock) void k_sp_cells(GraphView g, SpLevel lv) {
  const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx < (uint32_t)lv.n * (uint32_t)lv.B) sp_item<true>(g, lv, idx);
}

// The same for an even column count, two columns per lane: one 8-byte
// access moves two stored probabilities, and half as many waves cover the
// level.

__global__ __launch_bounds__(kWideBlock) void k_sp_level_x2(GraphView g, SpLevel lv) {
  const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t half = (uint32_t)lv.B / 2;
  if (idx >= (uint32_t)lv.n * half) return;
  const uint32_t gl = idx / half;
  const int32_t b = 2 * (int32_t)(idx - gl * half);
  const int32_t gi = lv.g0 + (int32_t)gl;
  const int op = g.op[gi];
  const int k = arity_of(op);
  const f2 *sp2 = reinterpret_cast<const f2 *>(lv.sp);
  const int64_t B2 = lv.B / 2;
  const f2 z = f2{0.0f, 1.0f};
  const int32_t i0 = g.in[gi];
  const int32_t i1 = pin_row(g.in, g, 1)[gi];
  const int32_t i2 = pin_row(g.in, g, 2)[gi];
  gathers_done(op, i0, i1, i2);
  const f2 a = sp2[(int64_t)i0 * B2 + b / 2];
  f2 bl = f2{0.0f, 0.0f}, cl = f2{0.0f, 0.0f};
  if (k > 1) bl = sp2[(int64_t)i1 * B2 + b / 2];
  if (k > 2) cl = sp2[(int64_t)i2 * B2 + b / 2];
  gathers_done(a.x, a.y, bl.x, bl.y, cl.x, cl.y);
  const float r0 = settle(sp_rule(op, sp_load(a.x), k > 1 ? sp_load(bl.x) : z,
                                  k > 2 ? sp_load(cl.x) : z));
  const float r1 = settle(sp_rule(op, sp_load(a.y), k > 1 ? sp_load(bl.y) : z,
                                  k > 2 ? sp_load(cl.y) : z));
  reinterpret_cast<f2 *>(lv.sp)[(int64_t)(g.n_pi + gi) * B2 + b / 2] = f2{r0, r1};
}

// A column of a lane's four.
__device__ __forceinline__ float quad_elem(const float4 &v, int k) {
  return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w;
}
// f(integral_constant<OP>) of the fixed cell op.
template <class F>
__device__ __forceinline__ void with_cell(int op, const F &f) {
  switch (op) {
#define DP_CELL_CASE(OP) case OP: f(std::integral_constant<int, OP>{}); break
    DP_CELL_CASE(INV);
    DP_CELL_CASE(BUF);
    DP_CELL_CASE(AND2);
    DP_CELL_CASE(OR2);
    DP_CELL_CASE(NAND2);
    DP_CELL_CASE(NOR2);
    DP_CELL_CASE(XOR2);
    DP_CELL_CASE(AOI21);
#undef DP_CELL_CASE
    default: f(std::integral_constant<int, MUX2>{}); break;
  }
}
// And four columns a lane, from kQuadItems (gate, column) pairs of a level on,
// where there are waves enough all the same.  Forward and reverse, one column
// or two a lane against four, us: 1M gates x 100 levels, 32 columns (320K
// pairs a level) 914 / 984, 64 columns 1275 / 1197, 128 columns 2101 / 1618;
// 117K gates x 60 levels, 128 columns (250K pairs) 450 / 492, 256 columns 675 /
// 622.
constexpr int64_t kQuadItems = 400000;
__global__ __launch_bounds__(kWideBlock) void k_sp_level_x4(GraphView g, SpLevel lv) {
  const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t quads = (uint32_t)lv.B / 4;
  const uint32_t gl = idx / quads;
  if (gl >= (uint32_t)lv.n) return;
  const int32_t b = 4 * (int32_t)(idx - gl * quads), gi = lv.g0 + (int32_t)gl;
  const int op = g.op[gi];
  const int32_t i0 = g.in[gi], i1 = pin_row(g.in, g, 1)[gi], i2 = pin_row(g.in, g, 2)[gi];
  gathers_done(op, i0, i1, i2);
  const auto row = [&](int32_t r) {
    return reinterpret_cast<float4 *>(lv.sp + (int64_t)r * lv.B + b);
  };
  const int k = arity_of(op);
  const float4 x0 = *row(i0), x1 = *row(k > 1 ? i1 : i0), x2 = *row(k > 2 ? i2 : i0);
  const f2 z = f2{0.0f, 1.0f};
  float r[4];
  with_cell(op, [&](auto cell) {
    constexpr int OP = decltype(cell)::value;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      r[j] = settle(sp_rule(OP, sp_load(quad_elem(x0, j)), kArity<OP> > 1 ? sp_load(quad_elem(x1, j)) : z,
                            kArity<OP> > 2 ? sp_load(quad_elem(x2, j)) : z));
  });
  *row(g.n_pi + gi) = make_float4(r[0], r[1], r[2], r[3]);
}

// ---------------------------------------------------------------- simulation
// Count ones / toggles of one word pair computed by this lane.  `prev` is the
// word before the pair's first word.
__device__ __forceinline__ void count_pair(const ChunkView &c, int32_t p, w2 y, uint64_t prev,
                                           uint32_t &ones, uint32_t &togs) {
  const int32_t u0 = 2 * p, u1 = u0 + 1;
  if (u0 >= c.u_lo && u0 < c.u_hi) ones += __popcll(y.x);
  if (u1 >= c.u_lo && u1 < c.u_hi) ones += __popcll(y.y);
  if (u0 >= c.u_tog_lo && u0 < c.u_hi) togs += __popcll(y.x ^ prev);
  if (u1 >= c.u_tog_lo && u1 < c.u_hi) togs += __popcll(y.y ^ y.x);
}

// One gate's row over pairs [p_begin, p_begin + 64*ITERS): loads of all
// iterations are issued before any store so they overlap in flight.  Rows
// are addressed as 16-byte word pairs so each lane moves one pair per access.
template <int OP, int ITERS>
__device__ __forceinline__ void sim_gate_row(const w2 *__restrict__ r0,
                                             const w2 *__restrict__ r1,
                                             const w2 *__restrict__ r2,
                                             w2 *__restrict__ out, bool keep, int32_t p_begin,
                                             const ChunkView &c, int lane, uint32_t &ones,
                                             uint32_t &togs) {
  constexpr int K = kArity<OP>;
  uint64_t carry = 0;
  if (p_begin > 0) {  // word just before this run, recomputed from its inputs
    const int32_t q = p_begin - 1;
    carry = cell_bits<OP>(r0[q].y, K > 1 ? r1[q].y : 0, K > 2 ? r2[q].y : 0);
  }
  w2 x0[ITERS], x1[ITERS], x2[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int32_t p = p_begin + it * 64 + lane;
    const bool ok = p < c.pairs;
    const w2 z = w2{0, 0};
    x0[it] = ok ? r0[p] : z;
    x1[it] = (ok && K > 1) ? r1[p] : z;
    x2[it] = (ok && K > 2) ? r2[p] : z;
  }
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int32_t p = p_begin + it * 64 + lane;
    w2 y;
    y.x = cell_bits<OP>(x0[it].x, x1[it].x, x2[it].x);
    y.y = cell_bits<OP>(x0[it].y, x1[it].y, x2[it].y);
    uint64_t prev = __shfl_up(y.y, 1u);
    if (lane == 0) prev = carry;
    carry = __shfl(y.y, 63);
    if (p < c.pairs) {
      // streaming store: a row's readers run in later launches, mostly on
      // other XCDs, so the words gain nothing from this XCD's L2 (measured
      // 3% faster per level than a plain store on MI355X); a row nobody
      // reads is not stored at all
      if (keep) __builtin_nontemporal_store(y, out + p);
      count_pair(c, p, y, prev, ones, togs);
    }
  }
}

// A library cell's Boolean function from its truth table (bit m = output for
// the input pattern m, input k = bit k of m), by Shannon expansion depth
// first: f = x_{N-1} ? f(x_{N-1} = 1) : f(x_{N-1} = 0), one bit select per
// node, N + 1 words live.  The simulation needs exact bits only, which the
// table gives; probabilities and partials follow the code (op by op).
template <int N>
__device__ __forceinline__ uint64_t tt_eval(const uint64_t *x, uint64_t tt, int base) {
  if constexpr (N == 1) {
    const uint64_t m0 = 0ull - ((tt >> base) & 1ull), m1 = 0ull - ((tt >> (base + 1)) & 1ull);
    return (x[0] & m1) | (~x[0] & m0);
  } else {
    const uint64_t lo = tt_eval<N - 1>(x, tt, base);
    const uint64_t hi = tt_eval<N - 1>(x, tt, base + (1 << (N - 1)));
    return (x[N - 1] & hi) | (~x[N - 1] & lo);
  }
}

// A library cell's row with N inputs: sim_gate_row with the table in place
// of the fixed rule.
template <int N, int ITERS, int NMAX>
__device__ __forceinline__ void sim_tt_row(const int32_t (&ix)[NMAX], uint64_t tt,
                                           const w2 *__restrict__ W, int64_t pp,
                                           w2 *__restrict__ out, bool keep, int32_t p_begin,
                                           const ChunkView &c, int lane, uint32_t &ones,
                                           uint32_t &togs) {
  const w2 *r[N];
#pragma unroll
  for (int k = 0; k < N; ++k) r[k] = W + (int64_t)ix[k] * pp;
  uint64_t carry = 0;
  if (p_begin > 0) {  // word just before this run, recomputed from its inputs
    uint64_t x[N];
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = r[k][p_begin - 1].y;
    carry = tt_eval<N>(x, tt, 0);
  }
  w2 v[N][ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int32_t p = p_begin + it * 64 + lane;
    const bool ok = p < c.pairs;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k][it] = ok ? r[k][p] : w2{0, 0};
  }
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int32_t p = p_begin + it * 64 + lane;
    uint64_t xa[N], xb[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      xa[k] = v[k][it].x;
      xb[k] = v[k][it].y;
    }
    const w2 y = w2{tt_eval<N>(xa, tt, 0), tt_eval<N>(xb, tt, 0)};
    uint64_t prev = __shfl_up(y.y, 1u);
    if (lane == 0) prev = carry;
    carry = __shfl(y.y, 63);
    if (p < c.pairs) {
      if (keep) __builtin_nontemporal_store(y, out + p);  // see sim_gate_row
      count_pair(c, p, y, prev, ones, togs);
    }
  }
}

template <int ITERS, int NMAX>
__device__ __forceinline__ void sim_cell_row(const GraphView &g, int op, int32_t gi,
                                             const w2 *__restrict__ W, int64_t pp,
                                             w2 *__restrict__ out, bool keep, int32_t p_begin,
                                             const ChunkView &c, int lane, uint32_t &ones,
                                             uint32_t &togs) {
  // the gate's input count and every pin's input net go out with the
  // opcode (pin rows past the design's widest cell alias pin 0), so the
  // input rows load in the next round; the table rides along with them
  const int nin = __builtin_amdgcn_readfirstlane((int)g.arity[gi]);
  int32_t ix[NMAX];
#pragma unroll
  for (int k = 0; k < NMAX; ++k) ix[k] = __builtin_amdgcn_readfirstlane(pin_row(g.in, g, k)[gi]);
  const int cl = op - kCellBase;
  const uint64_t t = g.tt[cl];
  const uint64_t tt = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(t >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)t);
  // NMAX: the most inputs a cell of the launch has (the instance for narrow
  // cells keeps fewer registers, so more of its waves are resident)
  switch (nin) {
    case 1: sim_tt_row<1, ITERS>(ix, tt, W, pp, out, keep, p_begin, c, lane, ones, togs); break;
    case 2: sim_tt_row<2, ITERS>(ix, tt, W, pp, out, keep, p_begin, c, lane, ones, togs); break;
    case 3: sim_tt_row<3, ITERS>(ix, tt, W, pp, out, keep, p_begin, c, lane, ones, togs); break;
    default:
      if constexpr (NMAX > 3) {
        switch (nin) {
          case 4: sim_tt_row<4, ITERS>(ix, tt, W, pp, out, keep, p_begin, c, lane, ones, togs); break;
          case 5: sim_tt_row<5, ITERS>(ix, tt, W, pp, out, keep, p_begin, c, lane, ones, togs); break;
          default: sim_tt_row<6, ITERS>(ix, tt, W, pp, out, keep, p_begin, c, lane, ones, togs); break;
        }
      }
      break;
  }
}

// CELLS: 0 for fixed cells, else the most inputs a library cell of the
// launch has.
template <int ITERS, int CELLS>
__global__ __launch_bounds__(kSimBlock) void k_sim_level(GraphView g, ChunkView c, CountView cnt,
                                                      int32_t g0, int32_t n, int32_t waves_per_row,
                                                      int32_t sim_blocks, SpLevel sp) {
  if ((int32_t)blockIdx.x >= sim_blocks) {  // fused SP of the same level (and kind)
    const uint32_t idx = (blockIdx.x - (uint32_t)sim_blocks) * kSimBlock + threadIdx.x;
    if (idx < (uint32_t)sp.n * (uint32_t)sp.B) sp_item<(CELLS > 0)>(g, sp, idx);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t task = (int64_t)blockIdx.x * kSimWaves + wave;
  // tasks: (column, gate, run of word pairs), column outermost
  const int64_t per_col = (int64_t)n * waves_per_row;
  if (task >= per_col * c.n_cols) return;
  const int32_t lc = (int32_t)(task / per_col);
  const int64_t rest = task - (int64_t)lc * per_col;
  const int32_t gl = (int32_t)(rest / waves_per_row);
  const int32_t seg = (int32_t)(rest - (int64_t)gl * waves_per_row);
  const int32_t gi = g0 + gl;
  const int op = __builtin_amdgcn_readfirstlane((int)g.op[gi]);
  const int64_t pp = c.pitch / 2;  // pairs per row
  uint64_t *Wc = c.W + (int64_t)lc * c.col_stride;
  const w2 *W = reinterpret_cast<const w2 *>(Wc);
  const w2 *r0 = W + (int64_t)__builtin_amdgcn_readfirstlane(g.in[gi]) * pp;
  const w2 *r1 = W + (int64_t)__builtin_amdgcn_readfirstlane(g.in[g.G + gi]) * pp;
  const w2 *r2 = W + (int64_t)__builtin_amdgcn_readfirstlane(g.in[2 * g.G + gi]) * pp;
  w2 *out = reinterpret_cast<w2 *>(Wc) + (int64_t)(g.n_pi + gi) * pp;
  // a net with no readers needs its counts only: its words are not stored
  const int32_t on = g.n_pi + gi;
  const bool keep = __builtin_amdgcn_readfirstlane(g.rev_ptr[on + 1]) >
                    __builtin_amdgcn_readfirstlane(g.rev_ptr[on]);
  const int32_t p_begin = seg * 64 * ITERS;
  uint32_t ones = 0, togs = 0;
  if constexpr (CELLS > 0) {
    sim_cell_row<ITERS, CELLS>(g, op, gi, W, pp, out, keep, p_begin, c, lane, ones, togs);
  } else {
  switch (op) {
    case INV: sim_gate_row<INV, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case BUF: sim_gate_row<BUF, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case AND2: sim_gate_row<AND2, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case OR2: sim_gate_row<OR2, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case NAND2: sim_gate_row<NAND2, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case NOR2: sim_gate_row<NOR2, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case XOR2: sim_gate_row<XOR2, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    case AOI21: sim_gate_row<AOI21, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
    default: sim_gate_row<MUX2, ITERS>(r0, r1, r2, out, keep, p_begin, c, lane, ones, togs); break;
  }
  }
  ones = wave_sum(ones);
  togs = wave_sum(togs);
  if (lane == 0) {
    const int64_t o = (int64_t)(g.n_pi + gi) * cnt.B + cnt.col + lc;
    if (ones) atomicAdd(cnt.ones + o, ones);
    if (togs) atomicAdd(cnt.tog + o, togs);
  }
}

// ---------------------------------------------------------------- stimulus
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of
// (c0,c1,c2,c3) -> (hi(M1 c2)^c1^k0, lo(M1 c2), hi(M0 c0)^c3^k1, lo(M0 c0)),
// key bumped by the Weyl constants between rounds.  The words are bound by
// vector issue: a round is two full products and two three-operand xors
// (v_bitop3_b32, truth table 0x96; as pairs of v_xor_b32 a call is 60
// instructions in place of 40; with the shifts below the 1M-gate design's
// 8,192 x 1,024 words take 200 us, 253 before).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = make_uint4(xor3((uint32_t)(p1 >> 32), c.y, k0), (uint32_t)p1,
                   xor3((uint32_t)(p0 >> 32), c.w, k1), (uint32_t)p0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// floor(p * 2^32) of a float32 probability, exact in double.
__device__ __forceinline__ uint64_t prob_threshold(float p) {
  const double v = (double)p * 4294967296.0;
  if (!(v > 0.0)) return 0;
  if (v >= 4294967296.0) return 1ull << 32;
  return (uint64_t)v;
}

// A bit u < threshold for a threshold up to 2^32 (all, which 32 bits cannot
// hold, as a mask).
struct BitThreshold {
  uint32_t t;
  uint64_t all;  // ~0: every bit is one
};
__device__ __forceinline__ BitThreshold bit_threshold(uint64_t thr) {
  return BitThreshold{(uint32_t)thr, thr >> 32 ? ~0ull : 0ull};
}

// Shifts the bit u < t into h from below: a compare and an add with carry
// (left to the compiler it is a compare, a select, a shift and an or).
// UNI: t is wave-uniform.
template <bool UNI>
__device__ __forceinline__ void shift_in(uint32_t &h, uint32_t u, uint32_t t) {
  if constexpr (UNI)
    asm("v_cmp_gt_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
        : "+v"(h) : "v"(u), "s"(t) : "vcc");
  else
    asm("v_cmp_gt_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
        : "+v"(h) : "v"(u), "v"(t) : "vcc");
}

// Word t of PI i: i.i.d. Bernoulli(p) lanes, the temporal-independence case
// of the Markov stimulus of Sec. III-C; lane j = 4q + l is 1 iff lane l of
// Philox(t, i, q, 0; seed) is below the threshold.  The uniforms do not
// depend on the column, so one draw serves NT thresholds (query columns);
// the words are shifted in from their last lane on.
template <bool UNI, int NT>
__device__ __forceinline__ void stim_words(uint32_t pi, uint32_t t, const BitThreshold (&thr)[NT],
                                           uint32_t k0, uint32_t k1, uint64_t (&w)[NT]) {
#pragma unroll
  for (int half = 1; half >= 0; --half) {
    uint32_t h[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) h[c] = 0;
#pragma unroll 2
    for (int q = 7; q >= 0; --q) {
      const uint4 u = philox4x32_10(make_uint4(t, pi, (uint32_t)(8 * half + q), 0u), k0, k1);
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        shift_in<UNI>(h[c], u.w, thr[c].t);
        shift_in<UNI>(h[c], u.z, thr[c].t);
        shift_in<UNI>(h[c], u.y, thr[c].t);
        shift_in<UNI>(h[c], u.x, thr[c].t);
      }
    }
#pragma unroll
    for (int c = 0; c < NT; ++c)
      w[c] = half ? (uint64_t)h[c] << 32 : (w[c] | h[c]) | thr[c].all;
  }
}

// The same word with the wave's lanes in place of its bits: lane j draws bit
// j (one call where stim_words takes sixteen).
__device__ __forceinline__ uint32_t stim_lane(uint32_t pi, uint32_t t, uint32_t k0, uint32_t k1) {
  const uint32_t j = threadIdx.x & 63;
  const uint4 u = philox4x32_10(make_uint4(t, pi, j >> 2, 0u), k0, k1);
  return (j & 2) ? ((j & 1) ? u.w : u.z) : ((j & 1) ? u.y : u.x);
}

// ---------------------------------------------------------------- paired SP levels
// Two consecutive fixed-cell levels in one launch: lanes [0, a.n B) run
// level a as k_sp_level does; lanes [a.n B, (a.n + b.n) B) run level b, and
// a pin that level a drives is recomputed from that gate's own inputs (its
// structure in the second load round, its inputs in the third) with the
// arithmetic level a's lane performs, so the value is bit for bit the one
// that lane stores.  One dependent round more than a level launch, one
// launch boundary less: for a few columns, where a level's launch is
// latency-bound, two levels cost about what one did.
__device__ __forceinline__ f2 sp_recomputed(int op, float u0, float u1, float u2) {
  const int k = arity_of(op);
  const f2 z = f2{0.0f, 1.0f};
  return sp_load(settle(sp_rule(op, sp_load(u0), k > 1 ? sp_load(u1) : z, k > 2 ? sp_load(u2) : z)));
}

__device__ __forceinline__ void sp_pair_item(const GraphView &g, const SpLevel &a,
                                             const SpLevel &b, uint32_t idx) {
  const uint32_t na = (uint32_t)a.n * (uint32_t)a.B;
  if (idx < na) {
    sp_item<false>(g, a, idx);
    return;
  }
  const uint32_t t = idx - na;
  const int32_t B = b.B;
  if (t >= (uint32_t)b.n * (uint32_t)B) return;
  const uint32_t gl = t / (uint32_t)B;
  const int32_t col = (int32_t)(t - gl * (uint32_t)B);
  const int32_t gi = b.g0 + (int32_t)gl;
  float *sp = b.sp;
  // first load round: the gate's opcode and pins
  const int op = g.op[gi];
  const int32_t i0 = g.in[gi];
  const int32_t i1 = pin_row(g.in, g, 1)[gi];
  const int32_t i2 = pin_row(g.in, g, 2)[gi];
  gathers_done(op, i0, i1, i2);
  const int k = arity_of(op);
  const int32_t lo = g.n_pi + a.g0, hi = lo + a.n;  // the nets level a drives
  const bool r0 = i0 >= lo && i0 < hi, r1 = k > 1 && i1 >= lo && i1 < hi,
             r2 = k > 2 && i2 >= lo && i2 < hi;
  // second load round: a pin level a drives gives that gate's structure, any other
  // pin its stored probability
  int32_t po[3] = {0, 0, 0}, pj[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  float v[3] = {0.0f, 0.0f, 0.0f};
  const int32_t pin[3] = {i0, i1, i2};
  const bool rec[3] = {r0, r1, r2};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if (j >= k) continue;
    if (rec[j]) {
      const int32_t pg = pin[j] - g.n_pi;
      po[j] = g.op[pg];
      pj[j][0] = g.in[pg];
      pj[j][1] = pin_row(g.in, g, 1)[pg];
      pj[j][2] = pin_row(g.in, g, 2)[pg];
    } else {
      v[j] = sp[(int64_t)pin[j] * B + col];
    }
  }
  gathers_done(po[0], po[1], po[2], pj[0][0], pj[0][1], pj[0][2], pj[1][0], pj[1][1], pj[1][2],
               pj[2][0], pj[2][1], pj[2][2], v[0], v[1], v[2]);
  // third load round: the recomputed gates' inputs (levels below a: stored)
  float u[3][3] = {{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if (j >= k || !rec[j]) continue;
    const int kp = arity_of(po[j]);
    u[j][0] = sp[(int64_t)pj[j][0] * B + col];
    if (kp > 1) u[j][1] = sp[(int64_t)pj[j][1] * B + col];
    if (kp > 2) u[j][2] = sp[(int64_t)pj[j][2] * B + col];
  }
  f2 x[3];
  const f2 z = f2{0.0f, 1.0f};
#pragma unroll
  for (int j = 0; j < 3; ++j)
    x[j] = j >= k ? z : (rec[j] ? sp_recomputed(po[j], u[j][0], u[j][1], u[j][2]) : sp_load(v[j]));
  sp[(int64_t)(g.n_pi + gi) * B + col] = settle(sp_rule(op, x[0], x[1], x[2]));
}

__global__ __launch_bounds__(kWideBlock) void k_sp_pair(GraphView g, SpLevel a, SpLevel b) {
  sp_pair_item(g, a, b, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---------------------------------------------------------------- Markov stimulus
// Startpoints with a target transition rate tau (Sec. III-C): each lane is a
// two-state chain with stationary law Bernoulli(p); a lane at 1 stays with
// probability 1 - tau / (2p), a lane at 0 rises with probability
// tau / (2 (1 - p)), each cycle's draw being the same Philox uniform as the
// independent stimulus (counter (t, stream, lane / 4)); cycle 0 is the
// stationary draw.  Probabilities in double, clamped to [0, 1].
__device__ __forceinline__ uint64_t threshold_d(double x) {
  const double v = x * 4294967296.0;
  if (!(v > 0.0)) return 0;
  if (v >= 4294967296.0) return 1ull << 32;
  return (uint64_t)v;
}

__device__ __forceinline__ void markov_probs(float p, float tau, double &rise, double &stay) {
  const double pd = (double)p, td = (double)tau;
  if (pd <= 0.0) {
    rise = 0.0;
    stay = 0.0;
  } else if (pd >= 1.0) {
    rise = 1.0;
    stay = 1.0;
  } else {
    rise = td / (2.0 * (1.0 - pd));
    stay = 1.0 - td / (2.0 * pd);
  }
  if (rise > 1.0) rise = 1.0;
  if (stay < 0.0) stay = 0.0;
}

// A lane's next bit as a map of its previous bit: x -> (x & s) | (~x & u),
// 64 lanes at once.  Maps compose associatively.
struct BitMap {
  uint64_t s, u;
};
__device__ __forceinline__ BitMap bitmap_then(BitMap first, BitMap then) {
  return BitMap{(first.s & then.s) | (~first.s & then.u), (first.u & then.s) | (~first.u & then.u)};
}
__device__ __forceinline__ uint64_t bitmap_apply(BitMap m, uint64_t x) {
  return (x & m.s) | (~x & m.u);
}

constexpr int kMarkovK = 4;  // consecutive words per lane and tile

// Words [B][n_pi][T] of every (column, startpoint), one wave each.  A tile of
// 64 K words: each lane draws the maps of its K words and composes them, an
// inclusive scan over the lanes composes the prefixes, and each lane applies
// its exclusive prefix to the word carried in from the previous tile, then
// its own maps in order.
__global__ __launch_bounds__(kBlock) void k_markov_words(const float *__restrict__ sp,
                                                         const float *__restrict__ tau,
                                                         const int32_t *__restrict__ stream,
                                                         int32_t n_pi, int32_t B, int64_t T,
                                                         uint32_t k0, uint32_t k1,
                                                         uint64_t *__restrict__ out) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + wave;  // b * n_pi + i
  if (row >= (int64_t)B * n_pi) return;
  const int32_t b = (int32_t)(row / n_pi), i = (int32_t)(row - (int64_t)b * n_pi);
  const float p = sp_load(sp[(int64_t)i * B + b]).x;
  double rise, stay;
  markov_probs(p, tau[(int64_t)b * n_pi + i], rise, stay);
  const BitThreshold thr_p = bit_threshold(prob_threshold(p)),
                     thr_rise = bit_threshold(threshold_d(rise)),
                     thr_stay = bit_threshold(threshold_d(stay));
  const uint32_t si = stream ? (uint32_t)stream[i] : (uint32_t)i;
  uint64_t *orow = out + row * T;
  const BitMap id = BitMap{~0ull, 0ull};
  uint64_t carry = 0;  // cycle 0's map is constant, so the first carry is moot
  for (int64_t t0 = 0; t0 < T; t0 += 64 * kMarkovK) {
    BitMap m[kMarkovK];
    BitMap f = id;
#pragma unroll
    for (int k = 0; k < kMarkovK; ++k) {
      const int64_t t = t0 + (int64_t)lane * kMarkovK + k;
      m[k] = id;
      if (t < T) {
        const BitThreshold thr[2] = {t == 0 ? thr_p : thr_stay, t == 0 ? thr_p : thr_rise};
        uint64_t w[2];
        stim_words<false>(si, (uint32_t)t, thr, k0, k1, w);
        m[k] = BitMap{w[0], w[1]};
      }
      f = bitmap_then(f, m[k]);
    }
    for (int d = 1; d < 64; d <<= 1) {  // inclusive scan: earlier lanes' maps first
      const BitMap g = BitMap{__shfl_up(f.s, (unsigned)d), __shfl_up(f.u, (unsigned)d)};
      if (lane >= d) f = bitmap_then(g, f);
    }
    BitMap e = BitMap{__shfl_up(f.s, 1u), __shfl_up(f.u, 1u)};
    if (lane == 0) e = id;
    uint64_t x = bitmap_apply(e, carry);
#pragma unroll
    for (int k = 0; k < kMarkovK; ++k) {
      const int64_t t = t0 + (int64_t)lane * kMarkovK + k;
      x = bitmap_apply(m[k], x);
      if (t < T) orow[t] = x;
    }
    carry = __shfl(x, 63);
  }
}

// PI rows of NC query columns at a time: one draw of uniforms serves them all
// (32 columns of the 117K-gate sizing sweep, 2,048 PIs x 1,024 words: 1,775 us
// with a draw per column, 430 us with one per eight).
// STIM: explicit words (NC 1).
template <int ITERS, int NC, bool STIM>
__global__ __launch_bounds__(kBlock) void k_stimulus(int32_t n_pi, ChunkView c, CountView cnt,
                                                     const float *__restrict__ p_rows,
                                                     const uint64_t *__restrict__ stim, int64_t T,
                                                     const int32_t *__restrict__ stream,
                                                     uint32_t k0, uint32_t k1,
                                                     int32_t waves_per_row) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t task = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  // tasks: (column group, PI, run of word pairs), group outermost
  const int64_t per_grp = (int64_t)n_pi * waves_per_row;
  if (task >= per_grp * ((c.n_cols + NC - 1) / NC)) return;
  const int32_t grp = (int32_t)(task / per_grp);
  const int64_t rest = task - (int64_t)grp * per_grp;
  const int32_t i = (int32_t)(rest / waves_per_row);
  const int32_t seg = (int32_t)(rest - (int64_t)i * waves_per_row);
  const int32_t lc0 = grp * NC, cols = min(NC, c.n_cols - lc0);
  const uint32_t si = stream ? (uint32_t)stream[i] : (uint32_t)i;  // shared stream
  BitThreshold thr[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const BitThreshold b = bit_threshold(prob_threshold(
        sp_load(p_rows[(int64_t)i * cnt.B + cnt.col + lc0 + min(k, cols - 1)]).x));
    thr[k].t = (uint32_t)__builtin_amdgcn_readfirstlane((int)b.t);
    thr[k].all = __builtin_amdgcn_readfirstlane((int)b.all) ? ~0ull : 0ull;
  }
  const uint64_t *srow = STIM ? stim + ((int64_t)lc0 * n_pi + i) * T : nullptr;
  // every column's word u of the chunk (cycles outside the run: zero)
  auto words = [&](int64_t u, uint64_t (&w)[NC]) {
    const int64_t t = c.t_first + u;
    const bool in = t >= 0 && t < T;
    if constexpr (STIM) {
      w[0] = in ? srow[t] : 0;
    } else {
      stim_words<true>(si, (uint32_t)t, thr, k0, k1, w);
      if (!in)
#pragma unroll
        for (int k = 0; k < NC; ++k) w[k] = 0;
    }
  };
  uint64_t *out = c.W + (int64_t)lc0 * c.col_stride + (int64_t)i * c.pitch;
  const int32_t p_begin = seg * 64 * ITERS;
  uint64_t carry[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) carry[k] = 0;
  if (p_begin > 0) {  // the word before the run
    const int64_t t = c.t_first + 2 * (int64_t)p_begin - 1;
    if (t >= 0 && t < T) {
      if constexpr (STIM) {
        carry[0] = srow[t];
      } else {
        const uint32_t u = stim_lane(si, (uint32_t)t, k0, k1);
#pragma unroll
        for (int k = 0; k < NC; ++k) carry[k] = __ballot(u < thr[k].t) | thr[k].all;
      }
    }
  }
  uint32_t ones[NC], togs[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) ones[k] = togs[k] = 0;
  for (int it = 0; it < ITERS; ++it) {
    const int32_t p = p_begin + it * 64 + lane;
    uint64_t x[NC], y[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) x[k] = y[k] = 0;
    if (p < c.pairs) {
      words(2 * (int64_t)p, x);
      words(2 * (int64_t)p + 1, y);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      uint64_t prev = __shfl_up(y[k], 1u);
      if (lane == 0) prev = carry[k];
      carry[k] = __shfl(y[k], 63);
      if (p < c.pairs && k < cols) {
        const w2 v = w2{x[k], y[k]};
        reinterpret_cast<w2 *>(out + k * c.col_stride)[p] = v;
        count_pair(c, p, v, prev, ones[k], togs[k]);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const uint32_t o1 = wave_sum(ones[k]), t1 = wave_sum(togs[k]);
    if (lane == 0 && k < cols) {
      const int64_t o = (int64_t)i * cnt.B + cnt.col + lc0 + k;
      if (o1) atomicAdd(cnt.ones + o, o1);
      if (t1) atomicAdd(cnt.tog + o, t1);
    }
  }
}

// ---------------------------------------------------------------- beta and terms
// The hybrid beta of a net whose TR_model is tm and whose simulation counted
// tog toggles: clip(TR_acc / TR_model) with TR_acc = toggles / (64 (T - 1))
// (Eq. 4-5; 0/0 -> 1, x/0 -> beta_max).  NaN where a sweep that gave up left no
// count or no probability (the clip alone would make beta_min of it).
__device__ __forceinline__ float hybrid_beta(const PowerArgs &a, uint32_t tog, float tm) {
  if (tog == kNoCount || tm != tm) return __builtin_nanf("");
  const float ta = (float)((double)tog / (64.0 * (double)(a.T - 1)));
  const float beta = tm == 0.0f ? (ta == 0.0f ? 1.0f : a.beta_max) : ta / tm;
  return fminf(fmaxf(beta, a.beta_min), a.beta_max);
}

// beta of net n in column b (idx = n B + b) with TR_model = tm: 1 in modeled
// mode, the frozen value, or the hybrid value.
__device__ __forceinline__ float beta_of(const PowerArgs &a, int64_t idx, int32_t n, float tm) {
  if (a.mode == 1) return hybrid_beta(a, a.tog[idx], tm);
  if (a.mode == 2) return a.beta_shared ? a.beta_frozen[n] : a.beta_frozen[idx];
  return 1.0f;
}

// The hybrid beta of every (net, column), for the contraction with many
// size vectors (the sum over nets with one or paired sizes takes it in the
// same pass, k_power_sp).
__global__ __launch_bounds__(kBlock) void k_beta(PowerArgs a) {
  const int64_t idx = gidx();
  if (idx >= (int64_t)a.n_nets * a.B) return;
  const int32_t n = (int32_t)(idx / a.B);
  const f2 pq = sp_load(a.sp[idx]);
  a.beta[idx] = beta_of(a, idx, n, 2.0f * pq.x * pq.y);
}

__global__ __launch_bounds__(kBlock) void k_export(ExportArgs a) {
  const int64_t idx = gidx();
  if (idx >= (int64_t)a.n_nets * a.B) return;
  const int32_t n = (int32_t)(idx / a.B), b = (int32_t)(idx - (int64_t)n * a.B);
  const int64_t o = (int64_t)b * a.n_nets + a.int2ext[n];
  const f2 pq = sp_load(a.sp[idx]);
  const float tm = 2.0f * pq.x * pq.y;
  if (a.o_sp) a.o_sp[o] = pq.x;
  if (a.o_tr) a.o_tr[o] = tm;
  const float beta = a.beta ? a.beta[idx] : 1.0f;
  if (a.o_beta) a.o_beta[o] = beta;
  if (a.o_tr_hyb) a.o_tr_hyb[o] = beta * tm;
  const auto rate = [](uint32_t count, int64_t words) {
    return count == kNoCount ? __builtin_nanf("") : (float)((double)count / (64.0 * (double)words));
  };
  if (a.o_sp_acc) a.o_sp_acc[o] = rate(a.ones[idx], a.T);
  if (a.o_tr_acc) a.o_tr_acc[o] = rate(a.tog[idx], a.T - 1);
  if (a.o_ones) a.o_ones[o] = a.ones[idx];
  if (a.o_tog) a.o_tog[o] = a.tog[idx];
}

// ---------------------------------------------------------------- power
// P[b] = sum_n x[n][b] C_n s_b(drv n) with x = kappa beta TR_model, one or
// paired sizes, accumulated in double in an order fixed by the net index
// alone, so a column's power does not depend on the launch it rides in:
// nets in chunks of kPowerChunk; lane j of kPowerLanes sums the chunk's
// nets j, j + kPowerLanes, ... in increasing order; the lane sums are added
// by a fixed pairwise tree (stride 32, 16, ..., 1); the chunks by
// k_power_final.  A block takes one chunk for a tile of tb columns (tb a
// power of two up to 64), the column innermost, so a wave's SP loads are
// whole row segments of tb columns; with tb = 64 a thread keeps the sums
// of several lanes.  Each term is computed where it is summed, and in
// hybrid mode beta is stored on the way.  The column tiles of one chunk go
// to blocks of one XCD (blocks are dealt to the XCDs in turn), which then
// share the chunk's capacitance and size lines in their L2.
constexpr int32_t kPowerChunk = 2048;
constexpr int32_t kPowerLanes = 64;
constexpr int32_t kPowerCols = 64;       // columns per block at most
constexpr int32_t kPowerThreads = 1024;  // threads per block at most
constexpr int32_t kPowerBatch = 8;       // terms per thread whose loads go out together
constexpr int32_t kXcds = 8;

// NQ lanes per thread (1 for tb <= 16 columns, 2 for 32, 4 for 64); MODE
// is the beta mode (0 modeled, 1 hybrid, 2 frozen).  Every operand of a
// round's eight terms is loaded (at a clamped, valid address) before the
// first term is formed; a term past the chunk's end is dropped.
template <int NQ, int MODE>
__device__ __forceinline__ void power_block(const PowerArgs &a, int32_t tb, int32_t col_tiles,
                                            uint32_t block, double *lds) {
  constexpr int U = kPowerBatch / NQ;  // nets of each lane per round
  constexpr int32_t jper = kPowerLanes / NQ;
  const int32_t xcd = (int32_t)(block % kXcds), slot = (int32_t)(block / kXcds);
  const int32_t chunk = (slot / col_tiles) * kXcds + xcd;
  const int32_t tile = slot - (slot / col_tiles) * col_tiles;
  if (chunk >= a.n_chunks) return;  // the grid's round-up to whole XCD rounds
  const int32_t c = (int32_t)threadIdx.x % tb, j0 = (int32_t)threadIdx.x / tb;
  const int32_t b = tile * tb + c;
  const int32_t n_lo = chunk * kPowerChunk, n_hi = min(n_lo + kPowerChunk, a.n_nets);
  const bool sized = a.size && a.paired;
  double acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
  const bool mine = j0 < jper;  // (not in a workgroup sized for a wider segment)
  if (mine && b < a.B) {
    for (int32_t i0 = 0; n_lo + i0 * kPowerLanes < n_hi; i0 += U) {
      // aux: the toggle count (hybrid) or the frozen beta's bits
      float v[kPowerBatch], cv[kPowerBatch], sv[kPowerBatch];
      uint32_t aux[kPowerBatch];
#pragma unroll
      for (int k = 0; k < kPowerBatch; ++k) {
        const int32_t n = min(n_lo + j0 + (k / U) * jper + (i0 + k % U) * kPowerLanes, n_hi - 1);
        const int64_t idx = (int64_t)n * a.B + b;
        v[k] = a.sp[idx];
        cv[k] = a.cap[n];
        if constexpr (MODE == 1) aux[k] = a.tog[idx];
        if constexpr (MODE == 2)
          aux[k] = __float_as_uint(a.beta_frozen[a.beta_shared ? (int64_t)n : idx]);
        sv[k] = (sized && n >= a.n_pi) ? a.size[(int64_t)max(n - a.n_pi, 0) * a.S + b] : 1.0f;
      }
#pragma unroll
      for (int k = 0; k < kPowerBatch; ++k) {
        const int32_t n = n_lo + j0 + (k / U) * jper + (i0 + k % U) * kPowerLanes;
        if (n < n_hi) {
          const f2 pq = sp_load(v[k]);
          const float tm = 2.0f * pq.x * pq.y;
          float beta = 1.0f;
          if constexpr (MODE == 2) beta = __uint_as_float(aux[k]);
          if constexpr (MODE == 1) {
            beta = hybrid_beta(a, aux[k], tm);
            a.beta[(int64_t)n * a.B + b] = beta;
          }
          acc[k / U] += (double)(a.kappa * beta * tm) * (double)(cv[k] * sv[k]);
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    if (mine) lds[(j0 + q * jper) * tb + c] = acc[q];
  __syncthreads();
  for (int32_t stride = kPowerLanes / 2; stride > 0; stride >>= 1) {
    for (int32_t e = threadIdx.x; e < stride * tb; e += blockDim.x)
      lds[e] += lds[e + stride * tb];
    __syncthreads();
  }
  if ((int32_t)threadIdx.x < tb && b < a.B) a.partial[(int64_t)chunk * a.B + b] = lds[c];
}
template <int NQ, int MODE>
__global__ __launch_bounds__(kPowerThreads) void k_power_sp(PowerArgs a, int32_t tb,
                                                           int32_t col_tiles) {
  __shared__ double lds[kPowerLanes * kPowerCols];
  power_block<NQ, MODE>(a, tb, col_tiles, blockIdx.x, lds);
}
// Several evals' nets in one launch, tiles of up to kPowerMulti columns.
constexpr int32_t kPowerMulti = kPowerThreads / kPowerLanes;
__host__ __device__ inline int32_t power_tile(int32_t B) {
  int32_t tb = 1;
  while (tb < B && tb < kPowerMulti) tb *= 2;
  return tb;
}
__global__ __launch_bounds__(kPowerThreads) void k_power_multi(const PowerSeg *__restrict__ segs,
                                                              int32_t n_segs) {
  __shared__ double lds[kPowerLanes * kPowerMulti];
  const PowerSeg &sg = segs[seg_at(segs, n_segs, &PowerSeg::block0)];
  const int32_t tb = power_tile(sg.a.B), tiles = (sg.a.B + tb - 1) / tb;
  if (sg.a.mode == 2)
    power_block<1, 2>(sg.a, tb, tiles, blockIdx.x - sg.block0, lds);
  else
    power_block<1, 0>(sg.a, tb, tiles, blockIdx.x - sg.block0, lds);
}

__device__ __forceinline__ double block_sum_d(double v, double *lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kWavesPerBlock; ++i) r += lds[i];
  return r;
}

// Many size vectors (S > 0, not paired): P[b][s] = sum_n X[n][b] Y[n][s]
// with X[n][b] = kappa beta TR_model and Y[n][s] = C_n s_s(drv n), both
// float, their products and sums in double: a (B x N)(N x S) contraction on
// the FP64 matrix cores.  A wave takes a slab of nets and MB x MS tiles of 16
// columns b and 16 size vectors s; it loads both operands straight from
// memory (16 consecutive b, or s, of four consecutive nets per load), sixteen
// nets' loads in flight, so the operands need no LDS.  Partials
// [slab][b][s] are summed over slabs in a fixed order, a piece of the (b, s)
// face (power_piece: b0, s0 on, whole tiles) at a time.  The slab's length
// depends on the net count alone: about 256 slabs, so that a small (b, s)
// face still fills the chip (50K nets, 8 x 4: 330 us on 25 blocks of a 32 x 64
// tile staged through LDS, vector FP64).
typedef double d4 __attribute__((ext_vector_type(4)));

template <int MB, int MS>
__global__ __launch_bounds__(kBlock) void k_power_mfma(PowerArgs a, const float *beta,
                                                       int32_t beta_shared, int32_t n_slabs,
                                                       int32_t slab_nets, int32_t b0, int32_t s0,
                                                       PowerPiece pc) {
  constexpr int U = 4;  // steps of four nets in flight
  const int32_t tiles_s = (pc.ns + 16 * MS - 1) / (16 * MS);
  const int32_t tiles_b = (pc.nb + 16 * MB - 1) / (16 * MB);
  const int32_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t task = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  if (task >= (int64_t)n_slabs * tiles_b * tiles_s) return;
  const int32_t ts = (int32_t)(task % tiles_s);
  const int32_t rest = (int32_t)(task / tiles_s);
  const int32_t tb = rest % tiles_b, slab = rest / tiles_b;
  const int32_t n_lo = slab * slab_nets, n_hi = min(n_lo + slab_nets, a.n_nets);
  const int32_t i = (int32_t)threadIdx.x & 15, kk = ((int32_t)threadIdx.x >> 4) & 3;
  int32_t b[MB], s[MS];
#pragma unroll
  for (int m = 0; m < MB; ++m) b[m] = b0 + tb * 16 * MB + 16 * m + i;
#pragma unroll
  for (int m = 0; m < MS; ++m) s[m] = s0 + ts * 16 * MS + 16 * m + i;
  const bool gates = a.G > 0;
  d4 acc[MB][MS];
#pragma unroll
  for (int p = 0; p < MB; ++p)
#pragma unroll
    for (int q = 0; q < MS; ++q) acc[p][q] = d4{0.0, 0.0, 0.0, 0.0};
  for (int32_t base = n_lo; base < n_hi; base += 4 * U) {
    float v[U][MB], bt[U][MB], sz[U][MS], cap[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // every load at a valid address
      const int32_t n = min(base + 4 * u + kk, n_hi - 1);
      cap[u] = a.cap[n];
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const int64_t idx = (int64_t)n * a.B + min(b[m], a.B - 1);
        v[u][m] = a.sp[idx];
        bt[u][m] = beta ? beta[beta_shared ? (int64_t)n : idx] : 1.0f;
      }
#pragma unroll
      for (int m = 0; m < MS; ++m)
        sz[u][m] = gates ? a.size[(int64_t)max(n - a.n_pi, 0) * a.S + min(s[m], a.S - 1)] : 1.0f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t n = base + 4 * u + kk;
      double x[MB], y[MS];
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const f2 pq = sp_load(v[u][m]);
        const float tm = 2.0f * pq.x * pq.y;
        x[m] = n < n_hi && b[m] < a.B ? (double)(a.kappa * bt[u][m] * tm) : 0.0;
      }
#pragma unroll
      for (int m = 0; m < MS; ++m)
        y[m] = n < n_hi && s[m] < a.S ? (double)(cap[u] * (n >= a.n_pi ? sz[u][m] : 1.0f)) : 0.0;
#pragma unroll
      for (int p = 0; p < MB; ++p)
#pragma unroll
        for (int q = 0; q < MS; ++q)
          acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[p], y[q], acc[p][q], 0, 0, 0);
    }
  }
  // register r of a tile holds row 4 r + lane / 16, column lane % 16
#pragma unroll
  for (int p = 0; p < MB; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int32_t bb = tb * 16 * MB + 16 * p + 4 * r + kk;
#pragma unroll
      for (int q = 0; q < MS; ++q)
        if (bb < pc.nb && s[q] - s0 < pc.ns)
          a.partial[((int64_t)slab * pc.nb + bb) * pc.ns + s[q] - s0] = acc[p][q][r];
    }
}

// The slabs' partials of 16 (b, s) results of a piece per block: thread (k, c)
// sums slabs k, k + 16, ... of result c in order, then a fixed order over k.
// power: the piece's first result in rows of S.
__global__ __launch_bounds__(kBlock) void k_power_slabs(const double *__restrict__ partial,
                                                        int32_t n_slabs, int32_t n_cols,
                                                        int32_t ns, int32_t S, float *power) {
  __shared__ double lds[16][16];
  const int32_t c = (int32_t)threadIdx.x & 15, k = (int32_t)threadIdx.x >> 4;
  const int32_t col = min((int32_t)blockIdx.x * 16 + c, n_cols - 1);
  double acc = 0.0;
#pragma unroll 4
  for (int32_t j = k; j < n_slabs; j += 16) acc += partial[(int64_t)j * n_cols + col];
  lds[k][c] = acc;
  __syncthreads();
  if (k != 0 || (int32_t)blockIdx.x * 16 + c >= n_cols) return;
  double r = lds[0][c];
  for (int32_t j = 1; j < 16; ++j) r += lds[j][c];
  power[(int64_t)(col / ns) * S + col % ns] = (float)r;
}

// One block per column: thread t sums chunks t, t + 256, ... in order, then
// a fixed tree over the block.
__device__ __forceinline__ float power_column(const double *partial, int32_t n_chunks, int32_t n_cols,
                                              int32_t col) {
  __shared__ double lds[kWavesPerBlock];
  double acc = 0.0;
  for (int32_t k = threadIdx.x; k < n_chunks; k += kBlock) acc += partial[(int64_t)k * n_cols + col];
  return (float)block_sum_d(acc, lds);
}
__global__ __launch_bounds__(kBlock) void k_power_final(PowerArgs a, int32_t n_cols) {
  const float r = power_column(a.partial, a.n_chunks, n_cols, (int32_t)blockIdx.x);
  if (threadIdx.x == 0) a.power[blockIdx.x] = r;
}
__global__ __launch_bounds__(kBlock) void k_power_final_multi(const PowerSeg *__restrict__ segs,
                                                             int32_t n_segs) {
  int32_t k = 0;
  while (k + 1 < n_segs && segs[k + 1].col0 <= (int32_t)blockIdx.x) ++k;
  const PowerSeg &sg = segs[k];
  const int32_t col = (int32_t)blockIdx.x - sg.col0;
  const float r = power_column(sg.a.partial, sg.a.n_chunks, sg.a.B, col);
  if (threadIdx.x != 0) return;
  sg.a.power[col] = r;
  if (sg.host) sg.host[col] = r;
}

// ---------------------------------------------------------------- reverse sweep
// The weights of a net over several size vectors, ws[k] = sum over s of
// w[k][s] size_s(n) in order of s (a PI's sizes are 1) for cols columns' rows
// w, for one net per thread of the workgroup.  Sizes come through LDS
// kSizeChunk vectors at a time: neighbouring nets' rows are one run of memory,
// while a wave's threads, each along its own row, read 64 lines an instruction
// (dP/dC of 1M gates x 4 columns x 32 vectors: 2,197 us read directly).
// net_of(thread): its net, or -1.  Every thread of the workgroup calls it;
// fresh: the chunk in LDS is not this one's.
constexpr int32_t kSizeChunk = 16;
template <int ROWS, int COLS, class NetOf>
__device__ __forceinline__ void staged_weights(const float *size, int32_t n_pi, int32_t S, const float *w,
                                               int32_t cols, float (&lds)[ROWS][kSizeChunk + 1],
                                               const NetOf &net_of, bool fresh, float (&ws)[COLS]) {
#pragma unroll
  for (int k = 0; k < COLS; ++k) ws[k] = 0.0f;
  for (int32_t s0 = 0; s0 < S; s0 += kSizeChunk) {
    const int32_t m = min(kSizeChunk, S - s0);
    if (fresh || S > kSizeChunk) {
      __syncthreads();
      float v[kSizeChunk];
#pragma unroll
      for (int k = 0; k < kSizeChunk; ++k) {
        const int32_t e = (int32_t)threadIdx.x + k * ROWS, row = e / kSizeChunk, col = e % kSizeChunk;
        const int32_t net = net_of(row);
        v[k] = 1.0f;
        if (net >= n_pi && col < m) v[k] = size[(int64_t)(net - n_pi) * S + s0 + col];
      }
#pragma unroll
      for (int k = 0; k < kSizeChunk; ++k) {
        const int32_t e = (int32_t)threadIdx.x + k * ROWS;
        lds[e / kSizeChunk][e % kSizeChunk] = v[k];
      }
      __syncthreads();
    }
    for (int32_t s = 0; s < m; ++s) {
      const float sz = lds[threadIdx.x][s];
#pragma unroll
      for (int k = 0; k < COLS; ++k)
        if (k < cols) ws[k] = fmaf(w ? w[(int64_t)k * S + s0 + s] : 1.0f, sz, ws[k]);
    }
  }
}

// Local adjoint seed of net n in reverse column c (SP column b): the
// derivative of the net's own power term, kappa C 2 (1 - 2P) (Eq. 2 and
// Eq. 7), times beta (unless STE), the upstream weight and the driver's size
// factor (per column, paired, or summed over the size vectors).  Rounded as it
// stands (no product of it is fused into the sum that the caller adds it to),
// so that a sweep which stores seeds has the same bits.
// staged: ws is the net's weight over the size vectors, from staged_weights.
__device__ __forceinline__ float seed_of(const BwdArgs &a, int32_t n, int32_t c, int32_t b,
                                         f2 pq, float beta, float cap, bool staged = false,
                                         float ws = 0.0f) {
#pragma clang fp contract(off)
  const float local = a.kappa * cap * 2.0f * (pq.y - pq.x);
  const float base = a.ste ? local : beta * local;
  const bool gate = n >= a.n_pi && a.size;
  const int64_t g = (int64_t)(n - a.n_pi);
  if (a.per_column) {
    const int32_t s = c - b * a.cdiv;
    const float w = a.w ? a.w[c] : 1.0f;
    const float sz = gate ? a.size[g * a.S + s] : 1.0f;
    return base * w * sz;
  }
  if (a.paired) {
    const float w = a.w ? a.w[b] : 1.0f;
    const float sz = gate ? a.size[g * a.S + b] : 1.0f;
    return base * (w * sz);
  }
  const int32_t Sp = a.S > 0 ? a.S : 1;
  if (!staged) {
    ws = 0.0f;
    for (int32_t s = 0; s < Sp; ++s) {
      const float w = a.w ? a.w[(int64_t)b * Sp + s] : 1.0f;
      const float sz = gate ? a.size[g * a.S + s] : 1.0f;
      ws = fmaf(w, sz, ws);
    }
  }
  return base * ws;
}

// Sum of the contributions the readers of a net left for it.  Readers write
// into the net's own contiguous range [e0, e1) of the contribution buffer
// (fan-out order), so the sum needs no index indirection.  Its order is fixed
// by the graph alone (not by the column, its lane or the batch): the range is
// cut into strands of kStrand consecutive entries, each strand is summed
// serially, and the strand sums are added in strand order.  Two ways reach
// that same sum bit for bit:
//  * lane-serial: a lane walks its own (net, column) strands.  With many
//    columns the wave's lanes are the columns of one net, so every load is a
//    contiguous row;
//  * wave-cooperative, for nets with more than one strand when columns are
//    few: lane j sums strand j of one (net, column) and the strand sums are
//    then added in order through lane shuffles.
// Every lane of the wave must call this (inactive lanes pass e0 == e1 and
// active == false); `serial` must be uniform across the wave.
constexpr int32_t kStrand = 8;
// C at which every pull is lane-serial (nets with more than kHeavyPull entries
// pulled by whole workgroups); below it a wave's lanes share its nets' long
// ranges.  Measured on the 1M-gate design (modeled fwd+bwd): the shared pull
// wins at 1 and 2 columns (0.65 against 0.81 ms, 0.71 against 0.82 ms), the
// lane-serial one from 3 (0.83 against 0.88 ms; 0.83 against 1.06 ms at 4, and
// 3.2x at 16).
constexpr int32_t kSerialColumns = 3;
// The same switch for launches without heavy-net workgroups (library cells,
// merged launches of several designs, the persistent kernel), where a
// lane-serial pull of a long range costs one lane several dependent rounds.
constexpr int32_t kSerialColumnsNoHeavy = 32;

// The entries [e, min(e + kStrand, e1)) of one strand into v (zeros past e1).
__device__ __forceinline__ void strand_load(const float *__restrict__ contrib, int32_t e,
                                            int32_t e1, int32_t C, int32_t c,
                                            float (&v)[kStrand]) {
#pragma unroll
  for (int i = 0; i < kStrand; ++i) v[i] = e + i < e1 ? contrib[(int64_t)(e + i) * C + c] : 0.0f;
}

// A strand's sum in entry order; m = entries left from the strand's start.
__device__ __forceinline__ float strand_fold(const float (&v)[kStrand], int32_t m) {
  float acc = v[0];
#pragma unroll
  for (int i = 1; i < kStrand; ++i)
    if (i < m) acc += v[i];
  return acc;
}

__device__ __forceinline__ float strand_sum(const float *__restrict__ contrib, int32_t e,
                                            int32_t e1, int32_t C, int32_t c) {
  float v[kStrand];
  strand_load(contrib, e, e1, C, c, v);
  return strand_fold(v, e1 - e);
}

// The canonical sum by one lane: a single strand directly; longer ranges four
// strands (32 loads in flight) at a time, their sums folded in strand order.
__device__ __forceinline__ float serial_pull(const float *__restrict__ contrib, int32_t e0,
                                             int32_t e1, int32_t C, int32_t c) {
  if (e1 - e0 <= kStrand) return e1 > e0 ? strand_sum(contrib, e0, e1, C, c) : 0.0f;
  float acc = 0.0f;
  for (int32_t e = e0; e < e1; e += 4 * kStrand) {
    float v[4 * kStrand];
#pragma unroll
    for (int i = 0; i < 4 * kStrand; ++i) v[i] = e + i < e1 ? contrib[(int64_t)(e + i) * C + c] : 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t es = e + q * kStrand;
      if (es < e1) {
        float sum = v[q * kStrand];
#pragma unroll
        for (int i = 1; i < kStrand; ++i)
          if (es + i < e1) sum += v[q * kStrand + i];
        acc = (es == e0) ? sum : acc + sum;
      }
    }
  }
  return acc;
}

__device__ __forceinline__ float pull_sum(const float *__restrict__ contrib, int32_t e0,
                                          int32_t e1, int32_t C, int32_t c, bool active,
                                          int lane, bool serial) {
  if (serial) return active ? serial_pull(contrib, e0, e1, C, c) : 0.0f;
  const bool light = active && e1 - e0 <= kStrand;
  // the light ranges' loads go out before the heavy batching's shuffles
  float lv[kStrand];
  if (light) strand_load(contrib, e0, e1, C, c, lv);
  uint64_t heavy = __ballot(active && !light);
  // the wave's heavy nets take consecutive strand positions (lane order);
  // when they fit in 64, their strands load in the same round as the light
  // ranges
  // (A wave holds few heavy nets, so their offsets are a short uniform loop
  // over the heavy lanes; lane values are read with readlane, a register
  // read, rather than cross-lane shuffles through LDS.)
  bool batched = false;
  int32_t cnt = 0, my_h = -1, my_j = 0;
  if (heavy) {
    cnt = ((heavy >> lane) & 1) ? (e1 - e0 + kStrand - 1) / kStrand : 0;
    int32_t run = 0;
    for (uint64_t hh = heavy; hh; hh &= hh - 1) {
      const int h = __builtin_ctzll(hh);
      const int32_t hc = __builtin_amdgcn_readlane(cnt, h);
      if (lane >= run && lane < run + hc) {
        my_h = h;
        my_j = lane - run;
      }
      run += hc;
    }
    batched = run <= 64;
    if (!batched) my_h = -1;
  }
  int32_t hbeg = 0, hend = 0, hcol = 0;
  if (batched) {
    const int src = my_h < 0 ? lane : my_h;
    hbeg = __shfl(e0, src) + my_j * kStrand;
    hend = __shfl(e1, src);
    hcol = __shfl(c, src);
  }
  float hv[kStrand];
  if (my_h >= 0) strand_load(contrib, hbeg, hend, C, hcol, hv);
  float acc = light ? strand_fold(lv, e1 - e0) : 0.0f;
  if (!heavy) return acc;
  if (batched) {
    const float v = my_h >= 0 ? strand_fold(hv, hend - hbeg) : 0.0f;
    const int32_t vbits = __float_as_int(v);
    // each heavy net folds its strand sums in strand order
    int32_t run = 0;
    for (uint64_t hh = heavy; hh; hh &= hh - 1) {
      const int h = __builtin_ctzll(hh);
      const int32_t hc = __builtin_amdgcn_readlane(cnt, h);
      float total = __int_as_float(__builtin_amdgcn_readlane(vbits, run));
      for (int32_t t = 1; t < hc; ++t)
        total = total + __int_as_float(__builtin_amdgcn_readlane(vbits, run + t));
      if (lane == h) acc = total;
      run += hc;
    }
    return acc;
  }
  while (heavy) {
    const int src = __builtin_ctzll(heavy);
    heavy &= heavy - 1;
    const int32_t h0 = __shfl(e0, src), h1 = __shfl(e1, src), hc = __shfl(c, src);
    const int32_t strands = (h1 - h0 + kStrand - 1) / kStrand;
    float total = 0.0f;
    for (int32_t base = 0; base < strands; base += 64) {
      const int32_t j = base + lane;
      const float v = j < strands ? strand_sum(contrib, h0 + j * kStrand, h1, C, hc) : 0.0f;
      const int32_t m = min(64, strands - base);
      for (int32_t t = 0; t < m; ++t) {
        const float u = __shfl(v, t);
        total = (base == 0 && t == 0) ? u : total + u;
      }
    }
    if (lane == src) acc = total;
  }
  return acc;
}

// Eq. 7 for one level: a gate's output adjoint is its seed plus the
// contributions its readers left on their fan-in slots (pulled in a fixed
// order, so the sum is deterministic); it then leaves lambda * dR/dx_j on
// each of its own fan-in slots.  Items are (gate, column) pairs, column
// innermost; item counts stay below 2^31.
// One (gate, column) item of a reverse level; every lane of the wave calls
// it (pull_sum needs the whole wave), lanes past the end pass active = false.
// WIDE (fixed cells): the launch's column count is at least kSerialColumns
// (pulls are lane-serial); a choice per launch, so each form keeps its own
// registers.  Library cells decide the pull per launch at run time.
// skip_heavy (WIDE only): items of gates with more than kHeavyPull fan-out
// entries are left to the launch's cooperative blocks (bwd_heavy).
// UNI (WIDE, a multiple of 64 columns): every wave holds one gate, so the
// gate's values are made wave-uniform once loaded (scalar branches, scalar
// row addresses, loops with scalar bounds).
template <bool CELLS, bool WIDE, bool UNI = false>
__device__ __forceinline__ void bwd_item(const GraphView &g, const BwdArgs &a, int32_t g0,
                                         int32_t n, uint32_t idx, int lane,
                                         bool skip_heavy = false) {
  const bool active = idx < (uint32_t)n * (uint32_t)a.C;
  // lanes past the end read row g0 (a level has at least one gate) and
  // store nothing, so no load needs a guard for them
  const uint32_t gl = active ? idx / (uint32_t)a.C : 0;
  const int32_t c = active ? (int32_t)(idx - gl * (uint32_t)a.C) : 0;
  const int32_t gi = g0 + (int32_t)gl;
  const int32_t out = g.n_pi + gi;
  const int32_t b = c / a.cdiv;
  const float *sp = a.sp;
  const f2 z = f2{0.0f, 1.0f};
  // first round: the item's structure and its own net's values; nothing here
  // waits on another load
  int32_t e0 = g.rev_ptr[out];
  int32_t e1r = g.rev_ptr[out + 1];
  int op = g.op[gi];
  const float sp_out = sp[(int64_t)out * a.B + b];
  const float beta = a.beta ? a.beta[a.beta_shared ? (int64_t)out : (int64_t)out * a.B + b] : 1.0f;
  const float cap = a.cap[out];
  if constexpr (CELLS) {  // library cell: partials over its code
    // the first round also takes every pin's index and slot; the second
    // every pin's probability, the cell's code and the pull, none of them
    // waiting on another
    int32_t pin[kCellMaxIn], sl[kCellMaxIn];
#pragma unroll
    for (int j = 0; j < kCellMaxIn; ++j) {
      pin[j] = j < g.pins ? g.in[j * g.G + gi] : 0;
      sl[j] = j < g.pins ? g.slot[j * g.G + gi] : 0;
    }
#pragma unroll
    for (int j = 0; j < kCellMaxIn; ++j) value_taken(pin[j]);
    float r[kCellMaxIn];
#pragma unroll
    for (int j = 0; j < kCellMaxIn; ++j) r[j] = j < g.pins ? sp[(int64_t)pin[j] * a.B + b] : 0.0f;
    const LaneCode lc = lane_code(g, op);
    const int32_t e1 = active ? e1r : e0;  // lanes past the end pull nothing
    const float pulled =
        pull_sum(a.contrib, e0, e1, a.C, c, active, lane, a.C >= kSerialColumnsNoHeavy);
    if (!active) return;
    float lam = seed_of(a, out, c, b, sp_load(sp_out), beta, cap) + pulled;
    if (a.ste) lam *= beta;
    if (a.lam) a.lam[(int64_t)c * (a.n_pi + a.G) + out] = lam;
    f2 x[kCellMaxIn];
    float d[kCellMaxIn];
#pragma unroll
    for (int j = 0; j < kCellMaxIn; ++j) x[j] = j < g.pins ? sp_load(r[j]) : z;
    cell_partials(lc, x, d);
#pragma unroll
    for (int j = 0; j < kCellMaxIn; ++j)
      if (j < lc.nin) a.contrib[(int64_t)sl[j] * a.C + c] = lam * d[j];
    return;
  }
  // every pin's index and slot go out with the opcode and the fan-out range
  // (unused pin rows alias pin 0); taken here, so none of them is moved
  // into the branch of the arity that reads it (each would add a dependent
  // round trip)
  int32_t i0 = g.in[gi];
  int32_t i1 = pin_row(g.in, g, 1)[gi];
  int32_t i2 = pin_row(g.in, g, 2)[gi];
  int32_t s0 = g.slot[gi];
  int32_t s1 = pin_row(g.slot, g, 1)[gi];
  int32_t s2 = pin_row(g.slot, g, 2)[gi];
  gathers_done(op, e0, e1r, i0, i1, i2, s0, s1, s2);
  if constexpr (UNI) {
    e0 = __builtin_amdgcn_readfirstlane(e0);
    e1r = __builtin_amdgcn_readfirstlane(e1r);
    op = __builtin_amdgcn_readfirstlane(op);
    i0 = __builtin_amdgcn_readfirstlane(i0);
    i1 = __builtin_amdgcn_readfirstlane(i1);
    i2 = __builtin_amdgcn_readfirstlane(i2);
    s0 = __builtin_amdgcn_readfirstlane(s0);
    s1 = __builtin_amdgcn_readfirstlane(s1);
    s2 = __builtin_amdgcn_readfirstlane(s2);
  }
  // second round: every pin's probability, whatever the opcode (a pin the
  // gate lacks reads pin 0's row again, a cache hit), beside the pull's
  // loads; the values are unpacked only after the pull, so no load waits
  // on another
  const float r0 = sp[(int64_t)i0 * a.B + b];
  const float r1 = sp[(int64_t)i1 * a.B + b];
  const float r2 = sp[(int64_t)i2 * a.B + b];
  if (WIDE && skip_heavy && e1r - e0 > kHeavyPull) return;
  const int32_t e1 = active ? e1r : e0;  // lanes past the end pull nothing
  const float pulled = pull_sum(a.contrib, e0, e1, a.C, c, active, lane, WIDE);
  if (!active) return;
  float lam = seed_of(a, out, c, b, sp_load(sp_out), beta, cap) + pulled;
  if (a.ste) lam *= beta;
  if (a.lam) a.lam[(int64_t)c * (a.n_pi + a.G) + out] = lam;
  const int k = arity_of(op);
  float d0, d1, d2;
  sp_partials(op, sp_load(r0), k > 1 ? sp_load(r1) : z, k > 2 ? sp_load(r2) : z, d0, d1, d2);
  a.contrib[(int64_t)s0 * a.C + c] = lam * d0;
  if (k > 1) a.contrib[(int64_t)s1 * a.C + c] = lam * d1;
  if (k > 2) a.contrib[(int64_t)s2 * a.C + c] = lam * d2;
}

// One gate with a long fan-out range, for 64 columns of a many-column
// reverse level, by a whole workgroup.  Lane-serially, one lane would pull a
// net's entries 32 at a time, one dependent round each (a 200-reader net:
// seven rounds, the level's critical path).  Here the waves share the
// strands: wave w sums strand groups w, w + waves, ... (four strands, 32
// loads, per group) into LDS, and wave 0 folds the strand sums in strand
// order: the canonical sum, bit for bit.  Wave 0 then finishes the item as
// bwd_item does; its own values and fan-in gathers go out before the pull.
constexpr int32_t kHeavyPass = 64;  // strand sums held in LDS at a time

// The canonical sum of [e0, e1) for column c by the whole workgroup; the
// result is meaningful in wave 0 (every thread must call it).
__device__ __forceinline__ float heavy_pull(const float *__restrict__ contrib, int32_t e0,
                                            int32_t e1, int32_t C, int32_t c) {
  __shared__ float ss[kHeavyPass][64];
  const int w = (int)(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6), lane = threadIdx.x & 63;
  const int32_t strands = (e1 - e0 + kStrand - 1) / kStrand;
  float pulled = 0.0f;
  for (int32_t p0 = 0; p0 < strands; p0 += kHeavyPass) {
    const int32_t np = min(kHeavyPass, strands - p0);
    for (int32_t q = 4 * w; q < np; q += 4 * nw) {
      const int32_t es = e0 + (p0 + q) * kStrand;
      float v[4 * kStrand];
#pragma unroll
      for (int i = 0; i < 4 * kStrand; ++i)
        v[i] = es + i < e1 ? contrib[(int64_t)(es + i) * C + c] : 0.0f;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int32_t st = es + t * kStrand;
        if (q + t < np) {
          float sum = v[t * kStrand];
#pragma unroll
          for (int i = 1; i < kStrand; ++i)
            if (st + i < e1) sum += v[t * kStrand + i];
          ss[q + t][lane] = sum;
        }
      }
    }
    __syncthreads();
    if (w == 0)
      for (int32_t t = 0; t < np; ++t) pulled = (p0 == 0 && t == 0) ? ss[0][lane] : pulled + ss[t][lane];
    __syncthreads();
  }
  return pulled;
}

__device__ __forceinline__ void bwd_heavy(const GraphView &g, const BwdArgs &a,
                                          const int32_t *__restrict__ heavy, uint32_t hb) {
  const int32_t cgroups = (a.C + 63) / 64;
  const int32_t gi = heavy[hb / (uint32_t)cgroups];
  const int32_t cg = (int32_t)(hb % (uint32_t)cgroups);
  const int w = (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const bool active = cg * 64 + lane < a.C;
  const int32_t c = active ? cg * 64 + lane : cg * 64;  // idle lanes load in-row
  const int32_t out = g.n_pi + gi;
  const int32_t b = c / a.cdiv;
  const float *sp = a.sp;
  const f2 z = f2{0.0f, 1.0f};
  const int32_t e0 = g.rev_ptr[out], e1 = g.rev_ptr[out + 1];
  const int op = g.op[gi];
  const int k = arity_of(op);
  const f2 pq = sp_load(sp[(int64_t)out * a.B + b]);
  const float beta = a.beta ? a.beta[a.beta_shared ? (int64_t)out : (int64_t)out * a.B + b] : 1.0f;
  const float cap = a.cap[out];
  // every pin's index and slot in the first round (unused pin rows alias
  // pin 0), every pin's probability beside the pull's first loads
  const int32_t i0 = g.in[gi], s0 = g.slot[gi];
  const int32_t i1 = pin_row(g.in, g, 1)[gi], s1 = pin_row(g.slot, g, 1)[gi];
  const int32_t i2 = pin_row(g.in, g, 2)[gi], s2 = pin_row(g.slot, g, 2)[gi];
  gathers_done(i0, i1, i2);
  const float r0 = sp[(int64_t)i0 * a.B + b];
  const float r1 = sp[(int64_t)i1 * a.B + b];
  const float r2 = sp[(int64_t)i2 * a.B + b];
  const float pulled = heavy_pull(a.contrib, e0, e1, a.C, c);
  if (w != 0 || !active) return;
  float lam = seed_of(a, out, c, b, pq, beta, cap) + pulled;
  if (a.ste) lam *= beta;
  if (a.lam) a.lam[(int64_t)c * (a.n_pi + a.G) + out] = lam;
  float d0, d1, d2;
  sp_partials(op, sp_load(r0), k > 1 ? sp_load(r1) : z, k > 2 ? sp_load(r2) : z, d0, d1, d2);
  a.contrib[(int64_t)s0 * a.C + c] = lam * d0;
  if (k > 1) a.contrib[(int64_t)s1 * a.C + c] = lam * d1;
  if (k > 2) a.contrib[(int64_t)s2 * a.C + c] = lam * d2;
}

// With many columns the first heavy_blocks blocks take the level's heavy
// gates (heavy[0, n_heavy), in groups of 64 columns; first, so their longer
// pulls start first), and the blocks after them the (gate, column) items,
// skipping the heavy gates.
template <bool CELLS, bool WIDE, bool UNI = false>
__global__ __launch_bounds__(kWideBlock) void k_bwd_level(GraphView g, BwdArgs a, int32_t g0,
                                                           int32_t n, const int32_t *heavy,
                                                           int32_t n_heavy, uint32_t heavy_blocks) {
  if constexpr (WIDE && !CELLS) {
    if (blockIdx.x < heavy_blocks) {
      bwd_heavy(g, a, heavy, blockIdx.x);
      return;
    }
  }
  bwd_item<CELLS, WIDE, UNI>(g, a, g0, n, (blockIdx.x - heavy_blocks) * blockDim.x + threadIdx.x,
                             threadIdx.x & 63, n_heavy > 0);
}

// A reverse level of many columns, four columns a lane (a multiple of four
// columns, each its own SP column): a level is bound by its instructions, of
// which a lane's structure loads and addresses are most, and four columns
// share them and move 16 bytes a load (from kQuadItems on).  A level of 10K
// gates x 64 columns 8.3 -> 7.7 us, x 128 14 -> 10.
// The sum is the canonical one: an entry that is not there adds -0, which
// changes no bit.
__global__ __launch_bounds__(kWideBlock) void k_bwd_quad(GraphView g, BwdArgs a, int32_t g0,
                                                          int32_t n, const int32_t *heavy,
                                                          int32_t n_heavy, uint32_t heavy_blocks) {
  if (blockIdx.x < heavy_blocks) {
    bwd_heavy(g, a, heavy, blockIdx.x);
    return;
  }
  const uint32_t idx = (blockIdx.x - heavy_blocks) * blockDim.x + threadIdx.x;
  const uint32_t quads = (uint32_t)a.C / 4;
  const uint32_t gl = idx / quads;
  if (gl >= (uint32_t)n) return;
  const int32_t c = 4 * (int32_t)(idx - gl * quads), gi = g0 + (int32_t)gl, out = g.n_pi + gi;
  const auto row = [&](const float *p, int32_t r) {
    return *reinterpret_cast<const float4 *>(p + (int64_t)r * a.C + c);
  };
  const int32_t e0 = g.rev_ptr[out], e1 = g.rev_ptr[out + 1];
  const int op = g.op[gi];
  const int32_t i0 = g.in[gi], i1 = pin_row(g.in, g, 1)[gi], i2 = pin_row(g.in, g, 2)[gi];
  const int32_t s0 = g.slot[gi], s1 = pin_row(g.slot, g, 1)[gi], s2 = pin_row(g.slot, g, 2)[gi];
  const float4 own = row(a.sp, out);
  float4 beta = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
  if (a.beta) {
    if (a.beta_shared) {
      const float x = a.beta[out];
      beta = make_float4(x, x, x, x);
    } else {
      beta = row(a.beta, out);
    }
  }
  const float cap = a.cap[out];
  gathers_done(op, e0, e1, i0, i1, i2, s0, s1, s2);
  if (n_heavy > 0 && e1 - e0 > kHeavyPull) return;
  const float4 r0 = row(a.sp, i0), r1 = row(a.sp, i1), r2 = row(a.sp, i2);
  const int32_t cnt = e1 - e0, last = max(e1 - 1, 0);
  float acc[4], sum[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = sum[k] = -0.0f;
  for (int32_t s = 0; __any(s < cnt); s += 4) {  // half a strand at a time
    float4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = row(a.contrib, min(e0 + s + i, last));
    if (s % kStrand == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc[k] += sum[k];
        sum[k] = -0.0f;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) sum[k] += s + i < cnt ? quad_elem(v[i], k) : -0.0f;
  }
  float lam[4], d[3][4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float pulled = cnt > 0 ? acc[k] + sum[k] : 0.0f, bk = quad_elem(beta, k);
    lam[k] = seed_of(a, out, c + k, c + k, sp_load(quad_elem(own, k)), bk, cap) + pulled;
    if (a.ste) lam[k] *= bk;
    if (a.lam) a.lam[(int64_t)(c + k) * (a.n_pi + a.G) + out] = lam[k];
  }
  const f2 z = f2{0.0f, 1.0f};
  with_cell(op, [&](auto cell) {
    constexpr int OP = decltype(cell)::value;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      sp_partials(OP, sp_load(quad_elem(r0, k)), kArity<OP> > 1 ? sp_load(quad_elem(r1, k)) : z,
                  kArity<OP> > 2 ? sp_load(quad_elem(r2, k)) : z, d[0][k], d[1][k], d[2][k]);
  });
  const int arity = arity_of(op);
  const int32_t slot[3] = {s0, s1, s2};
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (j < arity)
      *reinterpret_cast<float4 *>(a.contrib + (int64_t)slot[j] * a.C + c) =
          make_float4(lam[0] * d[j][0], lam[1] * d[j][1], lam[2] * d[j][2], lam[3] * d[j][3]);
}

// skip_heavy: PIs with more than kHeavyPull fan-out entries are left to the
// launch's cooperative blocks (bwd_pi_heavy).
// serial_cols: the column count from which pulls are lane-serial (the
// launch's choice: with or without heavy-PI workgroups).
__device__ __forceinline__ void bwd_pi_item(const GraphView &g, const BwdArgs &a, float *out,
                                            uint32_t idx, int lane, bool skip_heavy = false,
                                            int32_t serial_cols = kSerialColumns) {
  const bool active = idx < (uint32_t)g.n_pi * (uint32_t)a.C;
  const uint32_t i = active ? idx / (uint32_t)a.C : 0;
  const int32_t c = active ? (int32_t)(idx - i * (uint32_t)a.C) : 0;
  const int32_t e0 = g.rev_ptr[i];  // lanes past the end read PI 0 and store nothing
  const int32_t e1r = g.rev_ptr[i + 1];
  const int32_t e1 = active ? e1r : e0;
  const int32_t b = c / a.cdiv;
  const f2 pq = sp_load(a.sp[(int64_t)i * a.B + b]);
  const float beta = a.beta ? a.beta[a.beta_shared ? (int64_t)i : (int64_t)i * a.B + b] : 1.0f;
  const float cap = a.cap[i];
  const bool serial = a.C >= serial_cols;
  if (serial && skip_heavy && e1r - e0 > kHeavyPull) return;  // (lane-serial pulls only)
  const float pulled = pull_sum(a.contrib, e0, e1, a.C, c, active, lane, serial);
  if (!active) return;
  float lam = seed_of(a, (int32_t)i, c, b, pq, beta, cap) + pulled;
  if (a.ste) lam *= beta;
  if (a.fixed && a.fixed[i]) lam = 0.0f;  // excluded from the gradients
  out[(int64_t)c * g.n_pi + i] = lam;
  if (a.lam) a.lam[(int64_t)c * (a.n_pi + a.G) + i] = lam;
}

// A PI with a long fan-out range, for 64 columns, by a whole workgroup (as
// bwd_heavy for gates).
__device__ __forceinline__ void bwd_pi_heavy(const GraphView &g, const BwdArgs &a, float *out,
                                             const int32_t *__restrict__ heavy, uint32_t hb) {
  const int32_t cgroups = (a.C + 63) / 64;
  const int32_t i = heavy[hb / (uint32_t)cgroups];
  const int32_t cg = (int32_t)(hb % (uint32_t)cgroups);
  const int w = (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const bool active = cg * 64 + lane < a.C;
  const int32_t c = active ? cg * 64 + lane : cg * 64;
  const int32_t b = c / a.cdiv;
  const int32_t e0 = g.rev_ptr[i], e1 = g.rev_ptr[i + 1];
  const f2 pq = sp_load(a.sp[(int64_t)i * a.B + b]);
  const float beta = a.beta ? a.beta[a.beta_shared ? (int64_t)i : (int64_t)i * a.B + b] : 1.0f;
  const float cap = a.cap[i];
  const float pulled = heavy_pull(a.contrib, e0, e1, a.C, c);
  if (w != 0 || !active) return;
  float lam = seed_of(a, i, c, b, pq, beta, cap) + pulled;
  if (a.ste) lam *= beta;
  if (a.fixed && a.fixed[i]) lam = 0.0f;
  out[(int64_t)c * g.n_pi + i] = lam;
  if (a.lam) a.lam[(int64_t)c * (a.n_pi + a.G) + i] = lam;
}

// The first heavy_blocks blocks take the heavy PIs (many columns only).
__global__ __launch_bounds__(kBlock) void k_bwd_pi(GraphView g, BwdArgs a, float *out,
                                                   const int32_t *heavy, int32_t n_heavy,
                                                   uint32_t heavy_blocks) {
  if (blockIdx.x < heavy_blocks) {
    bwd_pi_heavy(g, a, out, heavy, blockIdx.x);
    return;
  }
  bwd_pi_item(g, a, out, (blockIdx.x - heavy_blocks) * kBlock + threadIdx.x, threadIdx.x & 63,
              n_heavy > 0);
}

// ---------------------------------------------------------------- many size vectors
// The per-(b, s) reverse sweep in adjoints: lam[n][c] = seed + sum over the
// net's fan-out entries of lam[reader][c] part[entry][b], the products rounded
// before the sum and summed as pull_sum does, so the results are those of the
// contributions bit for bit.  At 8,192 columns the contribution form was bound
// by vector issue (a lane per (gate, column) took some 250 instructions: 129 us
// per level of 1,950 gates for 255 MB); here a wave has one net, so its
// structure and branches are scalar, a lane has VEC columns, and a net's row
// is written once instead of once per pin.
//
// Partial derivative of every fan-out entry, [n_edges][B].
template <bool CELLS>
__global__ __launch_bounds__(kBlock) void k_edge_partials(GraphView g, const float *__restrict__ sp,
                                                          int32_t B, float *__restrict__ part) {
  const int64_t idx = gidx();
  if (idx >= (int64_t)g.G * B) return;
  const int32_t gi = (int32_t)(idx / B), b = (int32_t)(idx - (int64_t)gi * B);
  constexpr int N = CELLS ? kCellMaxIn : 3;
  const int op = g.op[gi];
  int32_t pin[N], slot[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    pin[j] = pin_row(g.in, g, j)[gi];
    slot[j] = pin_row(g.slot, g, j)[gi];
  }
  f2 x[N];
#pragma unroll
  for (int j = 0; j < N; ++j) x[j] = sp_load(sp[(int64_t)pin[j] * B + b]);
  if constexpr (CELLS) {
    if (op >= kCellBase) {
      const LaneCode lc = lane_code(g, op);
      float d[kCellMaxIn];
      cell_partials(lc, x, d);
#pragma unroll
      for (int j = 0; j < kCellMaxIn; ++j)
        if (j < lc.nin) part[(int64_t)slot[j] * B + b] = d[j];
      return;
    }
  }
  const int k = arity_of(op);
  const f2 z = f2{0.0f, 1.0f};
  float d0, d1, d2;
  sp_partials(op, x[0], k > 1 ? x[1] : z, k > 2 ? x[2] : z, d0, d1, d2);
  part[(int64_t)slot[0] * B + b] = d0;
  if (k > 1) part[(int64_t)slot[1] * B + b] = d1;
  if (k > 2) part[(int64_t)slot[2] * B + b] = d2;
}

// A product that is rounded before whatever is added to it.
__device__ __forceinline__ float mul_rounded(float x, float y) {
#pragma clang fp contract(off)
  return x * y;
}

// VEC consecutive columns of a row.
template <int VEC>
struct RowPart {
  float v[VEC];
};
template <int VEC>
__device__ __forceinline__ RowPart<VEC> row_load(const float *p) {
  RowPart<VEC> r;
  if constexpr (VEC == 4) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 x = *reinterpret_cast<const f4 *>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) r.v[k] = x[k];
  } else {
    r.v[0] = *p;
  }
  return r;
}
template <int VEC>
__device__ __forceinline__ void row_store(float *p, const RowPart<VEC> &r) {
  if constexpr (VEC == 4) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    *reinterpret_cast<f4 *>(p) = f4{r.v[0], r.v[1], r.v[2], r.v[3]};
  } else {
    *p = r.v[0];
  }
}

// One wave per (net, 64 VEC columns), the column segments innermost.  The
// first heavy_waves waves take the level's nets of long fan-out ranges, whose
// rows take many load rounds, so that they start first.
template <int VEC>
__global__ __launch_bounds__(kBlock) void k_bwd_wide(GraphView g, BwdArgs a,
                                                     const float *__restrict__ part, float *lam,
                                                     int32_t net0, int32_t n, int32_t segs,
                                                     const int32_t *__restrict__ heavy,
                                                     int32_t n_heavy) {
  const int32_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t task = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  const int32_t at = (int32_t)(task / segs), seg = (int32_t)(task - (int64_t)at * segs);
  if (at >= n_heavy + n) return;
  const bool is_heavy = at < n_heavy;
  int32_t net = net0 + (at - n_heavy);
  if (is_heavy) net = (net0 ? g.n_pi : 0) + heavy[at];
  net = __builtin_amdgcn_readfirstlane(net);
  const int32_t e0 = __builtin_amdgcn_readfirstlane(g.rev_ptr[net]);
  const int32_t len = __builtin_amdgcn_readfirstlane(g.rev_ptr[net + 1]) - e0;
  if (!is_heavy && n_heavy > 0 && len > kHeavyPull) return;
  const int32_t c0 = (seg * 64 + ((int32_t)threadIdx.x & 63)) * VEC;
  const bool active = c0 < a.C;  // (VEC divides C)
  const int32_t c = active ? c0 : 0, b = c / a.cdiv, s = c - b * a.cdiv;
  // the seed's values, and the pull's first strand, go out together
  const f2 pq = sp_load(a.sp[(int64_t)net * a.B + b]);
  const float beta = a.beta ? a.beta[a.beta_shared ? (int64_t)net : (int64_t)net * a.B + b] : 1.0f;
  const float cap = a.cap[net];
  const bool gate = net >= a.n_pi && a.size;
  RowPart<VEC> sz, w;
#pragma unroll
  for (int k = 0; k < VEC; ++k) sz.v[k] = w.v[k] = 1.0f;
  if (gate) sz = row_load<VEC>(a.size + (int64_t)(net - a.n_pi) * a.S + s);
  if (a.w) w = row_load<VEC>(a.w + c);
  RowPart<VEC> acc;
#pragma unroll
  for (int k = 0; k < VEC; ++k) acc.v[k] = 0.0f;
  for (int32_t st = 0; st < len; st += kStrand) {
    const int32_t m = min(kStrand, len - st), e = e0 + st;
    RowPart<VEC> x[kStrand];
    float d[kStrand];
#pragma unroll
    for (int i = 0; i < kStrand; ++i) {
      if (i < m) {  // (uniform)
        const int32_t r = __builtin_amdgcn_readfirstlane(g.rev_net[e + i]);
        x[i] = row_load<VEC>(lam + (int64_t)r * a.C + c);
        d[i] = part[(int64_t)(e + i) * a.B + b];
      }
    }
    RowPart<VEC> sum;
#pragma unroll
    for (int k = 0; k < VEC; ++k) sum.v[k] = mul_rounded(x[0].v[k], d[0]);
#pragma unroll
    for (int i = 1; i < kStrand; ++i) {
      if (i < m) {
#pragma unroll
        for (int k = 0; k < VEC; ++k) sum.v[k] += mul_rounded(x[i].v[k], d[i]);
      }
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k) acc.v[k] = st == 0 ? sum.v[k] : acc.v[k] + sum.v[k];
  }
  // the seed as seed_of forms it
  const float local = a.kappa * cap * 2.0f * (pq.y - pq.x);
  const float base = a.ste ? local : beta * local;
  const bool fixed = net < a.n_pi && a.fixed && a.fixed[net];
  RowPart<VEC> out;
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    float l = mul_rounded(mul_rounded(base, w.v[k]), sz.v[k]) + acc.v[k];
    if (a.ste) l *= beta;
    out.v[k] = fixed ? 0.0f : l;  // excluded from the gradients
  }
  if (active) row_store<VEC>(lam + (int64_t)net * a.C + c, out);
}

// lam rows of the PIs [n_pi][C] -> out [C][n_pi], 64 x 64 through LDS (written
// straight, a wave's 64 values go to 64 lines).
__global__ __launch_bounds__(kBlock) void k_bwd_wide_out(const float *__restrict__ lam, int32_t n_pi,
                                                         int32_t C, float *__restrict__ out) {
  __shared__ float tile[64][65];
  const int32_t ct = (C + 63) / 64;
  const int32_t c0 = (int32_t)(blockIdx.x % ct) * 64, i0 = (int32_t)(blockIdx.x / ct) * 64;
  const int32_t x = (int32_t)threadIdx.x & 63, y = (int32_t)threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int32_t i = i0 + y + 4 * k;
    if (i < n_pi && c0 + x < C) tile[y + 4 * k][x] = lam[(int64_t)i * C + c0 + x];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int32_t cc = c0 + y + 4 * k;
    if (cc < C && i0 + x < n_pi) out[(int64_t)cc * n_pi + i0 + x] = tile[x][y + 4 * k];
  }
}

// ---------------------------------------------------------------- adjoints and scores
__global__ __launch_bounds__(kBlock) void k_grad_lambda_export(
    const float *__restrict__ lam, const float *__restrict__ sp, const int32_t *__restrict__ int2ext,
    int32_t n_pi, int32_t n_nets, int32_t B, int32_t C, int32_t cdiv, float eps, float *lam_out,
    float *score) {
  const int64_t idx = gidx();
  if (idx >= (int64_t)n_nets * C) return;
  const int32_t c = (int32_t)(idx / n_nets), n = (int32_t)(idx - (int64_t)c * n_nets);
  const float l = lam[idx];
  const int32_t e = int2ext[n];
  if (lam_out) lam_out[(int64_t)c * n_nets + e] = l;
  if (score && n >= n_pi) {
    const f2 pq = sp_load(sp[(int64_t)n * B + c / cdiv]);
    const float slope = fmaxf(fabsf(pq.y - pq.x), eps);  // |1 - 2P| from the pair
    score[(int64_t)c * (n_nets - n_pi) + (e - n_pi)] = fabsf(l) * (pq.x * pq.y) / slope;
  }
}

// ---------------------------------------------------------------- power virus
// One ascent step of Alg. 4 on the startpoints, kept as (p, 1 - p) pairs.
__global__ __launch_bounds__(kBlock) void k_virus_step(float *sp, const float *__restrict__ grad,
                                                       float eta, int32_t n_pi, int32_t B) {
  const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx >= (uint32_t)n_pi * (uint32_t)B) return;
  const int32_t i = (int32_t)(idx / (uint32_t)B), b = (int32_t)(idx - (uint32_t)i * B);
  const float p = clamp01(fmaf(eta, grad[(int64_t)b * n_pi + i], sp_load(sp[idx]).x));
  sp[idx] = sp_pack(p);
}

// Threshold at 1/2 and spell out the two-cycle stimulus (v0, 1 - v0).
__global__ __launch_bounds__(kBlock) void k_virus_vectors(const float *__restrict__ sp,
                                                          uint64_t *stim, uint8_t *v0,
                                                          float *p_out, int32_t n_pi, int32_t B) {
  const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx >= (uint32_t)n_pi * (uint32_t)B) return;
  const int32_t b = (int32_t)(idx / (uint32_t)n_pi), i = (int32_t)(idx - (uint32_t)b * n_pi);
  const float p = sp_load(sp[(int64_t)i * B + b]).x;
  const bool one = p >= 0.5f;
  v0[idx] = one ? 1 : 0;
  if (p_out) p_out[idx] = p;
  const uint64_t w0 = one ? ~0ull : 0ull;
  stim[2 * (int64_t)idx] = w0;
  stim[2 * (int64_t)idx + 1] = ~w0;
}

// One block per column: thread t adds nets t, t + 256, ... in order, then a
// fixed tree over the block.
__global__ __launch_bounds__(kBlock) void k_virus_power(const uint32_t *__restrict__ tog,
                                                        const float *__restrict__ cap,
                                                        int32_t n_nets, int32_t B, double *out) {
  __shared__ double lds[kWavesPerBlock];
  const int32_t b = blockIdx.x;
  double acc = 0.0;
  for (int32_t n = threadIdx.x; n < n_nets; n += kBlock)
    if (tog[(int64_t)n * B + b] != 0u) acc += (double)cap[n];
  const double r = block_sum_d(acc, lds);
  if (threadIdx.x == 0) out[b] = r;
}

// ---------------------------------------------------------------- several designs
// The segment of this block (uniform over the block: a short scalar scan).
template <class Seg>
__device__ __forceinline__ int32_t seg_of(const Seg *__restrict__ segs, int32_t n_segs) {
  int32_t k = 0;
  while (k + 1 < n_segs && segs[k + 1].block0 <= blockIdx.x) ++k;
  return k;
}

template <bool CELLS>
__global__ __launch_bounds__(kMergedBlock) void k_sp_multi(const SpSeg *__restrict__ segs,
                                                           int32_t n_segs) {
  const SpSeg sg = segs[seg_of(segs, n_segs)];
  const uint32_t idx = (blockIdx.x - sg.block0) * kMergedBlock + threadIdx.x;
  if (!CELLS && sg.lv2.n > 0) {  // two levels of this design: launch_sp_pair's items
    sp_pair_item(sg.g, sg.lv, sg.lv2, idx);
    return;
  }
  if (idx < (uint32_t)sg.lv.n * (uint32_t)sg.lv.B) sp_item<CELLS>(sg.g, sg.lv, idx);
}

template <bool CELLS>
__global__ __launch_bounds__(kMergedBlock) void k_bwd_multi(const BwdSeg *__restrict__ segs,
                                                            int32_t n_segs) {
  const BwdSeg sg = segs[seg_of(segs, n_segs)];
  const uint32_t idx = (blockIdx.x - sg.block0) * kMergedBlock + threadIdx.x;
  if (!CELLS && sg.a.C >= kSerialColumnsNoHeavy)  // segments differ in width: chosen per block
    bwd_item<CELLS, true>(sg.g, sg.a, sg.g0, sg.n, idx, threadIdx.x & 63);
  else
    bwd_item<CELLS, false>(sg.g, sg.a, sg.g0, sg.n, idx, threadIdx.x & 63);
}

// ---------------------------------------------------------------- persistent sweeps
// One cooperative launch runs every level: a grid-stride loop over the
// level's items, then a grid barrier.  Whole waves step together so the
// wave-wide pull of the reverse sweep sees all its lanes.
//
// The barrier: at barrier k every block, once all its threads have stored
// their results, publishes k in its own arrival flag (a release store at
// device scope, which makes the block's stores visible beyond its XCD's L2);
// then the block's first wave reads all the flags, 64 at a time (lane i
// reads flags i, i + 64, ...), until every flag reads k or more, and takes
// one acquire fence.  No block waits on another's atomic: a barrier costs
// one release, the store's trip and the reads that see the last one.
// Cooperative launch keeps every block resident, so every wait ends; as a
// guard, a wait that sees no new arrival for limit_ticks ticks of the
// 100 MHz real-time counter sets the timeout flag and stops, a wait that
// finds the flag set stops at once, and the sweep's outputs are then written
// as NaN.  The wait that gives up also sets the report word, which the host
// reads at its next synchronization, so a broken sweep is reported and
// cannot pass for a result.
__device__ __forceinline__ bool barrier_timed_out(const GridBarrier &bar) {
  return __hip_atomic_load(bar.words + kBarrierTimeout, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT) != 0u;
}

__device__ __forceinline__ void grid_barrier(const GridBarrier &bar, uint32_t k) {
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint32_t lane = threadIdx.x, blocks = gridDim.x;
    if (lane == 0)
      __hip_atomic_store(bar.words + blockIdx.x, k, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t seen = 0;
    uint64_t since = __builtin_amdgcn_s_memrealtime();
    for (uint32_t it = 0;; ++it) {
      uint32_t arrived = 0;
      for (uint32_t b = lane; b < blocks; b += 64)
        arrived += __hip_atomic_load(bar.words + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= k;
      arrived = wave_sum(arrived);
      if (arrived == blocks) break;
      if ((it & 15u) == 0u && barrier_timed_out(bar)) break;
      const uint64_t now = __builtin_amdgcn_s_memrealtime();
      if (arrived != seen) {  // a new arrival restarts the clock
        seen = arrived;
        since = now;
      }
      if (now - since >= bar.limit_ticks) {  // at a limit of 0: the first poll that waits
        if (lane == 0) {
          __hip_atomic_store(bar.words + kBarrierTimeout, 1u, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(bar.words + kBarrierReport, 1u, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        }
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// A level item's structure (opcode and pin indices), loaded apart from its
// gathers so the persistent sweep can fetch the next level's before it
// waits at the barrier: the indices do not depend on any level's results.
struct SpFetch {
  int32_t op, i0, i1, i2;
};

__device__ __forceinline__ SpFetch sp_fetch(const GraphView &g, int32_t gi) {
  SpFetch f;
  f.op = g.op[gi];
  f.i0 = g.in[gi];
  f.i1 = pin_row(g.in, g, 1)[gi];
  f.i2 = pin_row(g.in, g, 2)[gi];
  return f;
}

__device__ __forceinline__ void sp_finish(const GraphView &g, const SpLevel &lv, int32_t gi,
                                          int32_t b, const SpFetch &f) {
  const int32_t B = lv.B;
  float *sp = lv.sp;
  const int k = arity_of(f.op);
  const float sa = sp[(int64_t)f.i0 * B + b];
  float sb = 0.0f, sc = 0.0f;
  if (k > 1) sb = sp[(int64_t)f.i1 * B + b];
  if (k > 2) sc = sp[(int64_t)f.i2 * B + b];
  gathers_done(sa, sb, sc);
  const f2 z = f2{0.0f, 1.0f};
  sp[(int64_t)(g.n_pi + gi) * B + b] =
      settle(sp_rule(f.op, sp_load(sa), k > 1 ? sp_load(sb) : z, k > 2 ? sp_load(sc) : z));
}

__global__ __launch_bounds__(kBlock) void k_sp_persistent(GraphView g, SpLevel lv,
                                                          const int32_t *__restrict__ level_ptr,
                                                          int32_t depth, GridBarrier bar) {
  const uint32_t stride = gridDim.x * kBlock;
  const uint32_t first = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t B = (uint32_t)lv.B;
  // this thread's first item of the coming level, fetched ahead
  int32_t g0 = level_ptr[1], n = level_ptr[2] - g0;
  SpFetch ahead{};
  if (first < (uint32_t)n * B) ahead = sp_fetch(g, g0 + (int32_t)(first / B));
  for (int32_t l = 1; l <= depth; ++l) {
    SpLevel cur = lv;
    cur.g0 = g0;
    cur.n = n;
    const uint32_t items = (uint32_t)n * B;
    for (uint32_t idx = first; idx < items; idx += stride) {
      const uint32_t gl = idx / B;
      const int32_t gi = g0 + (int32_t)gl;
      const SpFetch f = idx == first ? ahead : sp_fetch(g, gi);
      if (idx != first) gathers_done(f.op, f.i0, f.i1, f.i2);
      sp_finish(g, cur, gi, (int32_t)(idx - gl * B), f);
    }
    if (l < depth) {  // the next level's structure loads go out before the wait
      g0 = level_ptr[l + 1];
      n = level_ptr[l + 2] - g0;
      if (first < (uint32_t)n * B) ahead = sp_fetch(g, g0 + (int32_t)(first / B));
    }
    grid_barrier(bar, (uint32_t)l);
  }
  if (barrier_timed_out(bar)) {  // every gate's probability becomes NaN
    const int64_t nn = (int64_t)g.G * lv.B;
    float *out = lv.sp + (int64_t)g.n_pi * lv.B;
    for (int64_t i = first; i < nn; i += stride) out[i] = __builtin_nanf("");
  }
}

template <bool WIDE>
__global__ __launch_bounds__(kBlock) void k_bwd_persistent(GraphView g, BwdArgs a,
                                                           const int32_t *__restrict__ level_ptr,
                                                           int32_t depth, float *pi_out,
                                                           GridBarrier bar) {
  const uint32_t stride = gridDim.x * kBlock;
  const int lane = threadIdx.x & 63;
  const uint32_t first = blockIdx.x * kBlock + threadIdx.x;
  for (int32_t l = depth; l >= 1; --l) {
    const int32_t g0 = level_ptr[l], n = level_ptr[l + 1] - g0;
    const uint32_t items = (uint32_t)n * (uint32_t)a.C;
    // round the trip count up to whole waves
    for (uint32_t base = first - lane; base < items; base += stride)
      bwd_item<false, WIDE>(g, a, g0, n, base + lane, lane);
    grid_barrier(bar, (uint32_t)(depth - l + 1));
  }
  const uint32_t items = (uint32_t)g.n_pi * (uint32_t)a.C;
  if (barrier_timed_out(bar)) {  // the gradient becomes NaN
    for (uint32_t i = first; i < items; i += stride) pi_out[i] = __builtin_nanf("");
    return;
  }
  for (uint32_t base = first - lane; base < items; base += stride)
    bwd_pi_item(g, a, pi_out, base + lane, lane, false, kSerialColumnsNoHeavy);
}

// ---------------------------------------------------------------- dataflow sweeps
// A whole SP or reverse sweep in one launch and without a level barrier, each
// query column by a team of workgroups of one XCD: every array slot that the
// sweep will write holds kArmed (a NaN that no arithmetic here produces)
// before the launch, a consumer polls the very slots that it reads until none
// of them is armed, and a producer's store is all the signal there is.
//
// What bounds a sweep of few columns is the dependent chain of its levels.  A
// level launch pays the launch boundary and, with the L2 dropped there, each
// load round from beyond it: 2.3 us per SP level (two per launch) and 3.4 to
// 4.3 us per reverse level.  Inside one XCD a value goes from a store to a
// poll through the one L2 that its CUs share in 180 ns (measured; across XCDs
// 520 ns, and only with stores that write through).  So a column never leaves
// its XCD; further columns go to other teams.  SP and reverse sweep of one
// column, in us: 2K gates 36 and 72 by level launches, 17 and 21 (with 2 and 5
// for arming) here; 117K gates 132 and 235 against 47 and 64 (2 and 6); 1M
// gates 234 and 439 against 113 and 202 (5 and 15).
//
// Membership: the workgroups of a team register; the first (the leader)
// waits until the expected number has come, or briefly, and closes the list;
// whoever registers later leaves.  Items are dealt to the members' waves by
// rank, every wave takes its items in level order, and only running
// workgroups are members, so each wait is for work that a running wave will
// reach: nothing depends on how many workgroups fit on the device beside
// other streams' work.  As a guard a wait that polls ctl.limit times (seconds,
// unless the host set less) gives up: it raises the launch's stop flag, which
// ends every other wait at once, and the host-visible report word, and what it
// could not compute stays NaN.
//
// Polls are agent-scope loads: they go past the L1, which other CUs' stores
// do not reach, to the L2, where plain stores of the same XCD land.
//
// A level is one short turn of a lone wave per SIMD, so its instructions
// count as much as its latencies: addresses are 32-bit offsets from uniform
// bases (launch_*_flow refuses larger arrays), and a column's seeds and
// contributions are contiguous arrays of their own.
constexpr uint32_t kArmed = 0xFFFFFFFFu;
constexpr uint32_t kFlowClosed = 1u << 31;
constexpr uint64_t kFlowJoinTicks = 500;  // 5 us of the 100 MHz counter
constexpr int kFlowThreads = 512;         // threads per workgroup at most

__device__ __forceinline__ bool is_armed(float v) { return __float_as_uint(v) == kArmed; }
__device__ __forceinline__ float armed() { return __uint_as_float(kArmed); }
__device__ __forceinline__ uint32_t flow_load(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Element access by a 32-bit byte offset from a uniform base.
template <typename T>
__device__ __forceinline__ T *flow_at(T *base, uint32_t bytes) {
  using B = std::conditional_t<std::is_const_v<T>, const char, char>;
  return reinterpret_cast<T *>(reinterpret_cast<B *>(base) + bytes);
}
__device__ __forceinline__ float flow_poll(const float *base, uint32_t bytes) {
  return __hip_atomic_load(flow_at(base, bytes), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A plain store that the compiler may not split, widen or move past a poll.
__device__ __forceinline__ void flow_store(float *base, uint32_t bytes, float v) {
  __hip_atomic_store(flow_at(base, bytes), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One more poll of a wait: false when the wait has to end.
__device__ __forceinline__ bool flow_again(const FlowCtl &ctl, int stop, uint32_t &polls) {
  if ((++polls & (kFlowRound - 1)) != 0u) return true;
  if (flow_load(ctl.words + stop) != 0u) return false;
  if (polls < ctl.limit) return true;
  __hip_atomic_store(ctl.words + stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(ctl.report, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return false;
}

// This workgroup's place in its team.
struct FlowSeat {
  uint32_t team, rank, members;  // members == 0: not a member
};

// Blocks are dealt to the XCDs in turn, so block / kFlowDies counts an XCD's
// blocks, `expected` of them to a team.  (Were they dealt otherwise, teams
// would be smaller or larger, and still of one XCD each.)
__device__ __forceinline__ FlowSeat flow_join(const FlowCtl &ctl) {
  __shared__ FlowSeat seat;
  if (threadIdx.x == 0) {
    uint32_t x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    const uint32_t sub = min(blockIdx.x / kFlowDies / ctl.expected, (uint32_t)kFlowTeams - 1);
    const uint32_t team = (x & (kFlowXcds - 1)) * kFlowTeams + sub;
    uint32_t *reg = ctl.words + kFlowReg + team * 32, *open = reg + 16;
    const uint32_t r = __hip_atomic_fetch_add(reg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t n = 0;
    if (r == 0) {
      const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
      while (flow_load(reg) < ctl.expected && __builtin_amdgcn_s_memrealtime() - t0 < kFlowJoinTicks) {
      }
      n = __hip_atomic_fetch_or(reg, kFlowClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(open, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (!(r & kFlowClosed)) {
      uint32_t polls = ctl.start;
      while ((n = flow_load(open)) == 0u && flow_again(ctl, kFlowStop, polls)) {
      }
    }
    seat = FlowSeat{team, r, n};
  }
  __syncthreads();
  return FlowSeat{(uint32_t)__builtin_amdgcn_readfirstlane((int)seat.team),
                  (uint32_t)__builtin_amdgcn_readfirstlane((int)seat.rank),
                  (uint32_t)__builtin_amdgcn_readfirstlane((int)seat.members)};
}

// The k-th column of this team (claimed by its leader from the launch's
// list), or -1 when the list is used up.  Uniform over the workgroup.
__device__ __forceinline__ int32_t flow_claim(const FlowCtl &ctl, const FlowSeat &st, int32_t k,
                                              int32_t n_cols) {
  __shared__ int32_t col;
  __syncthreads();  // every wave has read the previous one
  if (threadIdx.x == 0) {
    uint32_t *slot = ctl.words + kFlowClaims + st.team * kFlowSlots + k;
    uint32_t v = 0;
    if (st.rank == 0) {
      const uint32_t t = __hip_atomic_fetch_add(ctl.words + kFlowNext, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      v = t < (uint32_t)n_cols ? t + 2u : 1u;  // 1: none left
      __hip_atomic_store(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      uint32_t polls = ctl.start;
      while ((v = flow_load(slot)) == 0u && flow_again(ctl, kFlowStop, polls)) {
      }
    }
    col = (int32_t)v - 2;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(col);
}

// A wave's walk over the 64-item blocks of a column's levels: block w, w + W,
// ... of each level in turn, w counted across the members first, so a
// level's blocks spread over as many CUs as there are, and from the shift on
// whose turn the level is.  The level table sits
// in LDS.
__shared__ int32_t flow_lv[kFlowLevels];

struct FlowWalk {
  int32_t w, waves;  // this wave's index, the team's waves
  int32_t n_pi, depth, shifts;
};

// A block of the walk: its first item is `base` of the n of level l, whose
// first net is `net` (level 0: the PIs).  n == 0: past the end.
struct FlowBlock {
  int32_t l, net, n, base;
};

// Loads the level table into LDS; every thread calls it, before any claim.
__device__ __forceinline__ FlowWalk flow_walk(const FlowSeat &st, const int32_t *level_ptr,
                                              int32_t depth, int32_t n_pi, const FlowCtl &ctl) {
  for (int32_t i = (int32_t)threadIdx.x; i < depth + 2; i += (int32_t)blockDim.x)
    flow_lv[i] = level_ptr[i];
  __syncthreads();
  const int32_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return FlowWalk{wave * (int32_t)st.members + (int32_t)st.rank,
                  ctl.per_block * (int32_t)st.members, n_pi, depth, ctl.shifts};
}

// The first block at or after `q` that has items, levels ascending (DIR 1,
// up to depth) or descending (DIR -1, down to the PIs).
template <int DIR>
__device__ __forceinline__ FlowBlock flow_settle(const FlowWalk &k, FlowBlock q) {
  while (q.base >= q.n) {
    if (q.l == (DIR > 0 ? k.depth : 0)) {
      q.n = 0;
      return q;
    }
    q.l += DIR;
    const int32_t a = __builtin_amdgcn_readfirstlane(flow_lv[q.l]);  // (entry 0 is 0)
    const int32_t b = __builtin_amdgcn_readfirstlane(flow_lv[q.l + 1]);
    q.net = q.l > 0 ? k.n_pi + a : 0;
    q.n = q.l > 0 ? b - a : k.n_pi;
    q.base = 64 * flow_first_block(k.w, k.waves, k.shifts, q.l);
  }
  return q;
}
template <int DIR>
__device__ __forceinline__ FlowBlock flow_next(const FlowWalk &k, FlowBlock q) {
  q.base += 64 * k.waves;
  return flow_settle<DIR>(k, q);
}

// A lane's net of a block; lanes past the level's end get its last net, so
// that what they load is in range, and are not active.
struct FlowItem {
  uint32_t net;
  int32_t active;
};
__device__ __forceinline__ FlowItem flow_item(const FlowBlock &q) {
  const int32_t at = q.base + (int32_t)(threadIdx.x & 63);
  return FlowItem{(uint32_t)(q.net + min(at, q.n - 1)), at < q.n ? 1 : 0};
}

// The rows of a per-pin table at gate gi; rows past the design's widest gate
// read its last row (a design has three rows at least).  Addresses without a
// branch: a fetch must leave no value to be merged, or the wave would wait
// for it on the spot.
template <int N>
__device__ __forceinline__ void flow_pins(const int32_t *tab, const GraphView &g, uint32_t gi,
                                          uint32_t (&out)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j)
    out[j] = (uint32_t)*flow_at(tab + (int64_t)(j < 3 ? j : min(j, g.pins - 1)) * g.G, 4 * gi);
}

template <bool CELLS>
constexpr int kFlowPins = CELLS ? kCellMaxIn : 3;

// Byte offset of net's entry in an [n_nets][B] array, column col (both
// below 2^24).
__device__ __forceinline__ uint32_t flow_off(uint32_t net, int32_t B, int32_t col) {
  return 4 * (__umul24(net, (uint32_t)B) + (uint32_t)col);
}

// ---- SP
template <bool CELLS>
struct SpFlowFetch {
  int32_t op;
  uint32_t pin[kFlowPins<CELLS>];
};
template <bool CELLS>
__device__ __forceinline__ SpFlowFetch<CELLS> sp_flow_fetch(const GraphView &g, uint32_t gi) {
  SpFlowFetch<CELLS> f;
  f.op = *flow_at(g.op, gi);
  flow_pins(g.in, g, gi, f.pin);
  return f;
}

// What an item's rule reads: its pins' probabilities, polled until none is
// armed.
template <bool CELLS>
struct SpFlowIn {
  int32_t op;
  int32_t ok;  // 0: the wait gave up
  float v[kFlowPins<CELLS>];
};
template <bool CELLS>
__device__ __forceinline__ SpFlowIn<CELLS> sp_flow_poll(const FlowCtl &ctl, const SpFlow &t,
                                                        int32_t col, const FlowItem &it,
                                                        const SpFlowFetch<CELLS> &f) {
  constexpr int N = kFlowPins<CELLS>;
  SpFlowIn<CELLS> x;
  x.op = f.op;
  x.ok = 1;
  int n = arity_of(f.op);
  if (CELLS && f.op >= kCellBase) n = t.g.cell[3 * (f.op - kCellBase) + 2];
  if (!it.active) n = 0;
  uint32_t at[N];
#pragma unroll
  for (int j = 0; j < N; ++j) at[j] = flow_off(f.pin[j], t.B, col);
#pragma unroll
  for (int j = 0; j < N; ++j) x.v[j] = j < n ? flow_poll(t.sp, at[j]) : 0.0f;
  uint32_t polls = ctl.start;
  for (;;) {
    bool wait = false;
#pragma unroll
    for (int j = 0; j < N; ++j) wait = wait || is_armed(x.v[j]);
    if (!wait) break;
    if (!flow_again(ctl, kFlowStop, polls)) {
      x.ok = 0;
      break;
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (is_armed(x.v[j])) x.v[j] = flow_poll(t.sp, at[j]);
  }
  return x;
}

template <bool CELLS>
__device__ __forceinline__ void sp_flow_store(const SpFlow &t, int32_t col, const FlowItem &it,
                                              const SpFlowIn<CELLS> &x) {
  if (!it.active) return;
  const uint32_t out = flow_off(it.net, t.B, col);
  if constexpr (CELLS) {
    if (x.op >= kCellBase) {
      f2 in[kCellMaxIn];
#pragma unroll
      for (int j = 0; j < kCellMaxIn; ++j) in[j] = sp_load(x.v[j]);
      const float r = settle(cell_sp(t.g, x.op, in));
      flow_store(t.sp, out, x.ok ? r : armed());
      return;
    }
  }
  const int k = arity_of(x.op);
  const f2 z = f2{0.0f, 1.0f};
  const float r = settle(sp_rule(x.op, sp_load(x.v[0]), k > 1 ? sp_load(x.v[1]) : z,
                                 k > 2 ? sp_load(x.v[2]) : z));
  flow_store(t.sp, out, x.ok ? r : armed());
}

// Two blocks of the wave's walk are in hand at a time.  Vector loads return
// in order, so a poll waits for whatever was issued before it: the fetch of
// the next but one block goes out between this block's poll and its store,
// where it overlaps the time the store takes to reach the next level.
template <bool CELLS>
__device__ __forceinline__ void sp_flow_column(const FlowCtl &ctl, const SpFlow &t,
                                               const FlowWalk &k, int32_t col) {
  const uint32_t n_pi = (uint32_t)t.g.n_pi;
  using Fetch = SpFlowFetch<CELLS>;
  FlowBlock q = flow_settle<1>(k, FlowBlock{0, 0, 0, 0});
  if (q.n == 0) return;
  FlowItem ia = flow_item(q);
  Fetch fa = sp_flow_fetch<CELLS>(t.g, ia.net - n_pi);
  q = flow_next<1>(k, q);
  int left = q.n;  // nonzero: a block is in hand after the current one
  FlowItem ib = q.n ? flow_item(q) : ia;
  Fetch fb = sp_flow_fetch<CELLS>(t.g, ib.net - n_pi);
  if (q.n) q = flow_next<1>(k, q);
  auto turn = [&](FlowItem &i, Fetch &f) {  // false: that was the last block
    const SpFlowIn<CELLS> x = sp_flow_poll<CELLS>(ctl, t, col, i, f);
    const FlowItem it = i;
    const bool more = left != 0;
    sp_flow_store<CELLS>(t, col, it, x);
    i = q.n ? flow_item(q) : i;  // (past the end: the same block again)
    f = sp_flow_fetch<CELLS>(t.g, i.net - n_pi);
    left = q.n;
    if (q.n) q = flow_next<1>(k, q);
    return more;
  };
  while (turn(ia, fa) && turn(ib, fb)) {
  }
}

template <bool CELLS>
__device__ __forceinline__ void sp_flow_team(const FlowCtl &ctl, const SpFlow &t) {
  const FlowSeat st = flow_join(ctl);
  if (st.members == 0) return;
  const FlowWalk k = flow_walk(st, t.level_ptr, t.depth, t.g.n_pi, ctl);
  const bool takes = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) < ctl.per_block;
  for (int32_t i = 0; i < kFlowSlots; ++i) {
    const int32_t col = flow_claim(ctl, st, i, t.B);
    if (col < 0) return;
    if (takes) sp_flow_column<CELLS>(ctl, t, k, col);
  }
}
template <bool CELLS>
__global__ __launch_bounds__(kFlowThreads) void k_sp_flow(FlowCtl ctl, SpFlow t) {
  sp_flow_team<CELLS>(ctl, t);
}

// A pointer read from a table, as one to global memory (loads through it are
// then global loads, not flat ones, whose waits also cover LDS).
template <typename T>
__device__ __forceinline__ T *global_ptr(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}
__device__ __forceinline__ GraphView global_view(GraphView g) {
  g.op = global_ptr(g.op);
  g.in = global_ptr(g.in);
  g.rev_ptr = global_ptr(g.rev_ptr);
  g.slot = global_ptr(g.slot);
  g.code = global_ptr(g.code);
  g.cell = global_ptr(g.cell);
  return g;
}
__device__ __forceinline__ SpFlow global_view(SpFlow t) {
  t.g = global_view(t.g);
  t.sp = global_ptr(t.sp);
  t.level_ptr = global_ptr(t.level_ptr);
  return t;
}
__device__ __forceinline__ BwdFlow global_view(BwdFlow t) {
  t.g = global_view(t.g);
  t.a.sp = global_ptr(t.a.sp);
  t.a.beta = global_ptr(t.a.beta);
  t.a.cap = global_ptr(t.a.cap);
  t.a.w = global_ptr(t.a.w);
  t.a.size = global_ptr(t.a.size);
  t.a.contrib = global_ptr(t.a.contrib);
  t.a.lam = global_ptr(t.a.lam);
  t.a.fixed = global_ptr(t.a.fixed);
  t.pi_out = global_ptr(t.pi_out);
  t.seed = global_ptr(t.seed);
  t.part = global_ptr(t.part);
  t.level_ptr = global_ptr(t.level_ptr);
  return t;
}
// The segment of a job, and of an arming block (uniform: a short scalar scan).
template <class Seg>
__device__ __forceinline__ int32_t seg_of_job(const Seg *__restrict__ segs, int32_t n, int32_t job) {
  int32_t k = 0;
  while (k + 1 < n && segs[k + 1].job0 <= job) ++k;
  return k;
}

template <bool CELLS>
__global__ __launch_bounds__(kFlowThreads) void k_sp_flow_multi(FlowCtl ctl,
                                                                const SpFlowSeg *__restrict__ segs,
                                                                int32_t n_segs, int32_t jobs) {
  const FlowSeat st = flow_join(ctl);
  if (st.members == 0) return;
  for (int32_t i = 0; i < kFlowSlots; ++i) {
    const int32_t job = flow_claim(ctl, st, i, jobs);
    if (job < 0) return;
    const int32_t k = seg_of_job(segs, n_segs, job);
    const SpFlow t = global_view(segs[k].t);
    const FlowWalk w = flow_walk(st, t.level_ptr, t.depth, t.g.n_pi, ctl);
    if (t.depth > 0) sp_flow_column<CELLS>(ctl, t, w, job - segs[k].job0);
  }
}

// ---- reverse: levels depth .. 1, then the PIs (level 0)
// The sweep's chain takes only what has to wait: a launch of the whole chip
// before it (k_bwd_arm) forms every net's seed and every gate's partial
// derivatives, which no level waits for, so an item loads one run of values
// in place of its net's probability, beta, capacitance and sizes and its
// fan-in's probabilities (random lines that one XCD would fetch alone) and
// takes no cell rule.
template <int N>
struct BwdFlowFetch {
  uint32_t e0, e1;  // the net's fan-out range
  int32_t slot[N];  // -1: no such pin
  float d[N];       // partial derivatives
  float seed, beta;
};

// What is uniform over a column.
struct BwdFlowCol {
  int32_t c, b;             // reverse column and its SP column
  const float *seed;        // [n_nets]
  const float *part;        // [pins][G]
  float *contrib;           // [n_edges]
  __amdgpu_buffer_rsrc_t contrib_rsrc;
};

template <int N>
__device__ __forceinline__ BwdFlowFetch<N> bwd_flow_fetch(const BwdFlow &t, const BwdFlowCol &u,
                                                          const FlowItem &i) {
  const GraphView &g = t.g;
  const BwdArgs &a = t.a;
  BwdFlowFetch<N> f;
  // a PI reads gate 0's rows and ignores them
  const uint32_t g4 = 4 * (uint32_t)max((int32_t)i.net - g.n_pi, 0), n4 = 4 * i.net;
  f.e0 = (uint32_t)*flow_at(g.rev_ptr, n4);
  f.e1 = (uint32_t)*flow_at(g.rev_ptr + 1, n4);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int64_t row = (int64_t)(j < 3 ? j : min(j, g.pins - 1)) * g.G;
    f.slot[j] = *flow_at(g.slot + row, g4);
    f.d[j] = *flow_at(u.part + row, g4);
  }
  f.seed = *flow_at(u.seed, n4);
  // STE alone takes the net's beta here; otherwise the seed again, unused
  const bool ste = a.ste && a.beta;
  f.beta = *flow_at(ste ? a.beta : u.seed,
                    ste && !a.beta_shared ? flow_off(i.net, a.B, u.b) : n4);
  return f;
}

// The K strands of eight entries from e on, in 16-byte loads past the L1, until
// none is armed; then the sum of the first m entries' strand sums in order, as
// strand_fold (any m <= 8 K, or more for all).  A strand beyond m reads
// nothing and entries beyond the array read as zero; the others' entries
// belong to later nets, of this level or a deeper one, so that waiting for them
// too, which takes half an instruction an entry in place of three, waits for
// no net that waits for this one.
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
constexpr int kBufferSc1 = 16;  // cache policy of a buffer load: agent scope
constexpr uint32_t kBeyond = ~15u;  // an offset past the end of every buffer
template <int K>
__device__ __forceinline__ float flow_strands(const FlowCtl &ctl, const BwdFlowCol &u, uint32_t e,
                                              int32_t m, int32_t &ok) {
  float v[K][kStrand];
  uint32_t polls = ctl.start;
  for (;;) {
    u4 w[K][2];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t at = 4 * e + 32u * k + 16u * h;
        w[k][h] = __builtin_amdgcn_raw_buffer_load_b128(
            u.contrib_rsrc, (int)(k == 0 || kStrand * k < m ? at : kBeyond), 0, kBufferSc1);
      }
    asm volatile("" ::: "memory");  // each round loads again
    uint32_t worst = 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < kStrand; ++i) {
        const uint32_t b = w[k][i / 4][i % 4];
        v[k][i] = __uint_as_float(b);
        worst = max(worst, b);  // kArmed is the largest
      }
    if (worst != kArmed) break;
    if (!flow_again(ctl, kFlowStop, polls)) {
      ok = 0;
      break;
    }
  }
  // (x + -0 is x, bit for bit: an entry or a strand that is not there)
  float acc = 0.0f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    float sum = k == 0 || kStrand * k < m ? v[k][0] : -0.0f;
#pragma unroll
    for (int i = 1; i < kStrand; ++i) sum += kStrand * k + i < m ? v[k][i] : -0.0f;
    acc = k == 0 ? sum : acc + sum;
  }
  return acc;
}

// The canonical sum of a net's contributions (strands of kStrand, their sums
// in order).  Lane by lane up to kFlowSerial entries, all of them polled in
// one round (a strand after another, a wave took as many rounds as its
// longest net has strands: reverse sweep of 1M gates 231 us against 222); the
// longer ranges (one net in a thousand) take the whole wave, one strand per
// lane.  Every lane of the wave calls it.
constexpr int32_t kFlowSerial = 4 * kStrand;
__device__ __forceinline__ float flow_pull(const FlowCtl &ctl, const BwdFlowCol &u, uint32_t e0,
                                           int32_t n, int lane, int32_t &ok) {
  float acc = 0.0f;
  const bool heavy = n > kFlowSerial;
  const int32_t mine = heavy ? 0 : n;
  if (__ballot(mine > 2 * kStrand)) {
    if (mine > 0) acc = flow_strands<4>(ctl, u, e0, mine, ok);
  } else if (__ballot(mine > kStrand)) {
    if (mine > 0) acc = flow_strands<2>(ctl, u, e0, mine, ok);
  } else if (mine > 0) {
    acc = flow_strands<1>(ctl, u, e0, mine, ok);
  }
  for (uint64_t hh = __ballot(heavy); hh; hh &= hh - 1) {
    const int h = __builtin_ctzll(hh);
    const uint32_t h0 = (uint32_t)__builtin_amdgcn_readlane((int)e0, h);
    const int32_t hn = __builtin_amdgcn_readlane(n, h);
    const int32_t strands = (hn + kStrand - 1) / kStrand;
    float total = 0.0f;
    for (int32_t base = 0; base < strands; base += 64) {
      const int32_t j = base + lane;
      float v = 0.0f;
      if (j < strands)
        v = flow_strands<1>(ctl, u, h0 + (uint32_t)(j * kStrand), hn - j * kStrand, ok);
      const int32_t vb = __float_as_int(v), m = min(64, strands - base);
      for (int32_t t = 0; t < m; ++t) {
        const float x = __int_as_float(__builtin_amdgcn_readlane(vb, t));
        total = (base == 0 && t == 0) ? x : total + x;
      }
    }
    if (lane == h) acc = total;
  }
  return acc;
}

// The end of an item whose contributions are summed: its adjoint, and what
// it leaves on its fan-in slots (a gate) or the gradient (a PI).
template <int N>
__device__ __forceinline__ void bwd_flow_store(const BwdFlow &t, const BwdFlowCol &u, bool gate,
                                               int32_t ok, const FlowItem &it,
                                               const BwdFlowFetch<N> &f, float pulled) {
  const BwdArgs &a = t.a;
  if (!it.active) return;
  float lam = f.seed + pulled;
  if (a.ste && a.beta) lam *= f.beta;
  if (!ok) lam = armed();
  if (!gate && a.fixed && a.fixed[it.net]) lam = 0.0f;  // excluded from the gradients
  if (a.lam) a.lam[(int64_t)u.c * (a.n_pi + a.G) + it.net] = lam;
  if (!gate) {
    t.pi_out[(int64_t)u.c * a.n_pi + it.net] = lam;
    return;
  }
#pragma unroll
  for (int j = 0; j < N; ++j)
    if ((j < 3 || j < t.g.pins) && f.slot[j] >= 0)
      flow_store(u.contrib, 4 * (uint32_t)f.slot[j], lam * f.d[j]);
}

// As sp_flow_column: the fetch of the next but one block goes out between a
// block's pull and its stores.
template <int N>
__device__ __forceinline__ void bwd_flow_column(const FlowCtl &ctl, const BwdFlow &t,
                                                const FlowWalk &k, int32_t c) {
  using Fetch = BwdFlowFetch<N>;
  BwdFlowCol u;
  u.c = c;
  u.b = c / t.a.cdiv;
  u.seed = t.seed + (int64_t)c * t.g.n_nets;
  u.part = t.part + (int64_t)u.b * t.g.pins * t.g.G;
  u.contrib = t.a.contrib + (int64_t)c * t.n_edges;
  u.contrib_rsrc = __builtin_amdgcn_make_buffer_rsrc(u.contrib, 0, (int)(4 * t.n_edges), 0x00020000);
  FlowBlock q = flow_settle<-1>(k, FlowBlock{t.depth + 1, 0, 0, 0});
  if (q.n == 0) return;
  // (a level holds gates only, or the PIs only: the kind is uniform)
  bool ga = q.l > 0;
  FlowItem ia = flow_item(q);
  Fetch fa = bwd_flow_fetch<N>(t, u, ia);
  q = flow_next<-1>(k, q);
  int left = q.n;  // nonzero: a block is in hand after the current one
  bool gb = q.n ? q.l > 0 : ga;
  FlowItem ib = q.n ? flow_item(q) : ia;
  Fetch fb = bwd_flow_fetch<N>(t, u, ib);
  if (q.n) q = flow_next<-1>(k, q);
  const int lane = (int)(threadIdx.x & 63);
  int32_t ok = 1;
  auto turn = [&](bool &gate_, FlowItem &i, Fetch &fetched) {
    const float pulled = flow_pull(ctl, u, fetched.e0,
                                   i.active ? (int32_t)(fetched.e1 - fetched.e0) : 0, lane, ok);
    const bool gate = gate_, more = left != 0;
    const FlowItem it = i;
    const Fetch f = fetched;
    bwd_flow_store<N>(t, u, gate, ok, it, f, pulled);
    gate_ = q.n ? q.l > 0 : gate_;
    i = q.n ? flow_item(q) : i;  // (past the end: the same block again)
    fetched = bwd_flow_fetch<N>(t, u, i);
    left = q.n;
    if (q.n) q = flow_next<-1>(k, q);
    return more;
  };
  while (turn(ga, ia, fa) && turn(gb, ib, fb)) {
  }
}

template <bool CELLS>
__global__ __launch_bounds__(kFlowThreads) void k_bwd_flow(FlowCtl ctl, BwdFlow t) {
  const FlowSeat st = flow_join(ctl);
  if (st.members == 0) return;
  const FlowWalk k = flow_walk(st, t.level_ptr, t.depth, t.g.n_pi, ctl);
  for (int32_t i = 0; i < kFlowSlots; ++i) {
    const int32_t c = flow_claim(ctl, st, i, t.a.C);
    if (c < 0) return;
    bwd_flow_column<kFlowPins<CELLS>>(ctl, t, k, c);
  }
}

template <bool CELLS>
__global__ __launch_bounds__(kFlowThreads) void k_bwd_flow_multi(
    FlowCtl ctl, const BwdFlowSeg *__restrict__ segs, int32_t n_segs, int32_t jobs) {
  const FlowSeat st = flow_join(ctl);
  if (st.members == 0) return;
  for (int32_t i = 0; i < kFlowSlots; ++i) {
    const int32_t job = flow_claim(ctl, st, i, jobs);
    if (job < 0) return;
    const int32_t k = seg_of_job(segs, n_segs, job);
    const BwdFlow t = global_view(segs[k].t);
    const FlowWalk w = flow_walk(st, t.level_ptr, t.depth, t.g.n_pi, ctl);
    bwd_flow_column<kFlowPins<CELLS>>(ctl, t, w, job - segs[k].job0);
  }
}

// Arms the n slots a sweep will write and clears its control words.  Four
// dwords per thread, each wave-wide store one contiguous run.
constexpr int kArmPer = 4;
__device__ __forceinline__ void flow_arm(uint32_t *p, int64_t n, uint32_t *words, int32_t n_words,
                                         uint32_t block) {
  const int64_t i0 = (int64_t)block * (kBlock * kArmPer) + threadIdx.x;
#pragma unroll
  for (int k = 0; k < kArmPer; ++k) {
    const int64_t i = i0 + k * kBlock;
    if (i < n)
      p[i] = kArmed;
    else if (i - n < n_words)
      words[i - n] = 0u;
  }
}
__global__ __launch_bounds__(kBlock) void k_flow_arm(uint32_t *p, int64_t n, uint32_t *words) {
  flow_arm(p, n, words, kFlowWords, blockIdx.x);
}

// Before a reverse sweep, in three runs of blocks: arms the contributions,
// writes every net's seed [C][n_nets], and every gate's partial derivatives
// [B][pins][G].  With the seeds the sweep's results become NaN, so that what a
// sweep that gives up does not reach is no earlier sweep's.  A NaN among the
// seeds and partials gets other bits than kArmed: the probabilities of an SP
// sweep that gave up are kArmed, whose bits a product may hand on, and a
// contribution of these bits would be waited for.
__device__ __forceinline__ float disarmed(float v) { return v == v ? v : __builtin_nanf(""); }
template <bool CELLS, bool SIZED>
__device__ __forceinline__ void bwd_arm(const BwdFlow &t, uint32_t *words, int32_t n_words,
                                        uint32_t block, uint32_t arm_blocks, uint32_t seed_blocks) {
  const GraphView &g = t.g;
  const BwdArgs &a = t.a;
  if (block < arm_blocks) {
    flow_arm(reinterpret_cast<uint32_t *>(a.contrib), t.n_edges * a.C, words, n_words, block);
    return;
  }
  if (block < arm_blocks + seed_blocks) {
    const int64_t first = (int64_t)(block - arm_blocks) * kBlock, idx = first + threadIdx.x;
    const int32_t c = (int32_t)(idx / g.n_nets), net = (int32_t)(idx - (int64_t)c * g.n_nets);
    const int32_t b = c / a.cdiv;
    const bool in = idx < (int64_t)g.n_nets * a.C;
    const bool staged = SIZED && staged_sizes(a);
    float ws[1] = {0.0f};
    if constexpr (SIZED)
      if (staged) {
        __shared__ float lds[kBlock][kSizeChunk + 1];
        const int32_t net0 = (int32_t)(first % g.n_nets);
        staged_weights<kBlock>(
            a.size, g.n_pi, a.S, a.w && in ? a.w + (int64_t)b * a.S : nullptr, 1, lds,
            [&](int32_t row) {  // (on into the next columns)
              const uint32_t n = (uint32_t)(net0 + row), all = (uint32_t)g.n_nets;
              return (int32_t)(n < all ? n : n % all);
            },
            true, ws);
      }
    if (!in) return;
    const float beta = a.beta ? a.beta[a.beta_shared ? (int64_t)net : (int64_t)net * a.B + b] : 1.0f;
    t.seed[idx] =
        disarmed(seed_of(a, net, c, b, sp_load(a.sp[(int64_t)net * a.B + b]), beta, a.cap[net],
                         staged, ws[0]));
    if (a.lam) a.lam[idx] = __builtin_nanf("");
    if (net < g.n_pi) t.pi_out[(int64_t)c * g.n_pi + net] = __builtin_nanf("");
    return;
  }
  const int64_t idx = (int64_t)(block - arm_blocks - seed_blocks) * kBlock + threadIdx.x;
  if (idx >= (int64_t)g.G * a.B) return;
  const int32_t b = (int32_t)(idx / g.G), gi = (int32_t)(idx - (int64_t)b * g.G);
  constexpr int N = kFlowPins<CELLS>;
  const int op = g.op[gi];
  int32_t pin[N];
#pragma unroll
  for (int j = 0; j < N; ++j) pin[j] = pin_row(g.in, g, j)[gi];
  float *part = t.part + (int64_t)b * g.pins * g.G + gi;
  f2 x[N];
#pragma unroll
  for (int j = 0; j < N; ++j) x[j] = sp_load(a.sp[(int64_t)pin[j] * a.B + b]);
  if constexpr (CELLS) {
    if (op >= kCellBase) {
      const LaneCode lc = lane_code(g, op);
      float d[kCellMaxIn];
      cell_partials(lc, x, d);
#pragma unroll
      for (int j = 0; j < kCellMaxIn; ++j)
        if (j < lc.nin) part[(int64_t)j * g.G] = disarmed(d[j]);
      return;
    }
  }
  const int k = arity_of(op);
  const f2 z = f2{0.0f, 1.0f};
  float d0, d1, d2;
  sp_partials(op, x[0], k > 1 ? x[1] : z, k > 2 ? x[2] : z, d0, d1, d2);
  part[0] = disarmed(d0);
  if (k > 1) part[g.G] = disarmed(d1);
  if (k > 2) part[2 * (int64_t)g.G] = disarmed(d2);
}
template <bool CELLS, bool SIZED>
__global__ __launch_bounds__(kBlock) void k_bwd_arm(BwdFlow t, uint32_t *words, uint32_t arm_blocks,
                                                    uint32_t seed_blocks) {
  bwd_arm<CELLS, SIZED>(t, words, kFlowWords, blockIdx.x, arm_blocks, seed_blocks);
}

// The same for the segments of a sweep over several designs; the first
// segment's blocks clear the control words.
__global__ __launch_bounds__(kBlock) void k_flow_arm_multi(const SpFlowSeg *__restrict__ segs,
                                                           int32_t n_segs, uint32_t *words) {
  const int32_t k = seg_of(segs, n_segs);
  const SpFlow t = global_view(segs[k].t);
  flow_arm(reinterpret_cast<uint32_t *>(t.sp + (int64_t)t.g.n_pi * t.B), (int64_t)t.g.G * t.B, words,
           k == 0 ? kFlowWords : 0, blockIdx.x - segs[k].block0);
}
template <bool CELLS, bool SIZED>
__global__ __launch_bounds__(kBlock) void k_bwd_arm_multi(const BwdFlowSeg *__restrict__ segs,
                                                          int32_t n_segs, uint32_t *words) {
  const int32_t k = seg_of(segs, n_segs);
  const BwdFlow t = global_view(segs[k].t);
  bwd_arm<CELLS, SIZED>(t, words, k == 0 ? kFlowWords : 0, blockIdx.x - segs[k].block0,
                 segs[k].arm_blocks, segs[k].seed_blocks);
}

// ---------------------------------------------------------------- word tiles
// The simulation of one query column's `pitch` consecutive words of cycles (a
// tile), all levels in one launch, by a team of one XCD: cycles are
// independent, so a tile needs nothing from another but the word before it,
// whose toggle the count kernel adds at the end.  Short simulations were
// bound by their chain of level launches (5.5 to 6.8 us each for a level of
// 0.3 to 4 MB); inside an XCD a level costs its barrier (0.7 us), the drain
// of its stores and a turn of row loads, pin 0's from the XCD's own L2, and
// other teams' tiles fill the waits.  50K gates x 45 levels, 5 columns of 64
// words: 277 -> 110 us; 117K gates x 60 levels, 257 words: 408 -> 190 us
// (3.2 us a level, about half of it the fabric's: half of the row reads are of
// older levels and miss the L2, and every row is evicted).
//
// Rows are [net][pitch] words of the team's own buffer, whole cache lines:
// 16 words (2 * LPG) while that gives no more tiles than teams, as a turn of
// the workgroup then covers the most gates.  LPG lanes take one gate's row, a
// pair of words each, so a wave takes 64 / LPG consecutive gates (sorted by
// cell: mostly one cell).  Row loads go past the L1, which other CUs' stores
// do not reach.  Rows are stored before the workgroup's flag; a level's last
// counts are left for the wait after it.  Loading older levels' rows before
// the wait, or the next turn's during a turn, was slower (432 to 510 against
// 438 us for the second case's whole pass): the waits are of the memory.
//
// A tile leaves per net its counts (packed, ones low) and its first and last
// word; k_sim_counts adds them up over the chunks with the toggles between
// chunks.
struct SimSeat {
  uint32_t buf, rank, members;  // members == 0: not a member
};

__device__ __forceinline__ SimSeat sim_join(const FlowCtl &ctl, uint32_t n_bufs, uint32_t block) {
  __shared__ SimSeat seat;
  if (threadIdx.x == 0) {
    uint32_t x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    const uint32_t sub = min(block / kFlowDies / ctl.expected, (uint32_t)kSimTeams - 1);
    uint32_t *reg = ctl.words + kSimReg + ((x & (kFlowXcds - 1)) * kSimTeams + sub) * 32;
    uint32_t *open = reg + 16;
    const uint32_t r = __hip_atomic_fetch_add(reg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t v = 0;  // members | (buffer + 1) << 8
    if (r == 0) {
      const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
      while (flow_load(reg) < ctl.expected && __builtin_amdgcn_s_memrealtime() - t0 < kFlowJoinTicks) {
      }
      const uint32_t n = min(__hip_atomic_fetch_or(reg, kFlowClosed, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT),
                             (uint32_t)kSimMembers);
      // a team that is far from whole (its CUs are taken) would hold a tile for
      // many times a whole team's time: it leaves its tiles to the others; an
      // XCD's first team always works
      uint32_t buf = ~0u - 1;
      if (sub == 0 || 4 * n >= 3 * ctl.expected)
        buf = __hip_atomic_fetch_add(ctl.words + kSimNextBuf, 1u, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
      v = n | min(buf + 1, 0xffffffu) << 8;
      __hip_atomic_store(open, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (!(r & kFlowClosed)) {
      uint32_t polls = ctl.start;
      while ((v = flow_load(open)) == 0u && flow_again(ctl, kSimStop, polls)) {
      }
    }
    const uint32_t buf = (v >> 8) - 1, members = v & 255u;
    // a team without a buffer, or a workgroup beyond a team's flags, leaves
    seat = SimSeat{buf, r, v != 0u && buf < n_bufs && r < members ? members : 0u};
  }
  __syncthreads();
  return SimSeat{(uint32_t)__builtin_amdgcn_readfirstlane((int)seat.buf),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)seat.rank),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)seat.members)};
}

// The team's barrier in two halves.  Arrive: this workgroup's stores so far
// are in the L2, which its flag (a line of its own) tells.
__device__ __forceinline__ void sim_arrive(const FlowCtl &ctl, const SimSeat &st, uint32_t epoch) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(ctl.words + kSimFlags + (st.buf * kSimMembers + st.rank) * 32, epoch,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Wait: every member has arrived.  The first wave reads all flags.  False (in
// the whole workgroup) when the wait gave up.
__device__ __forceinline__ bool sim_wait(const FlowCtl &ctl, const SimSeat &st, uint32_t epoch) {
  __shared__ int32_t go;
  if (threadIdx.x < 64) {
    const uint32_t *flags = ctl.words + kSimFlags + st.buf * kSimMembers * 32;
    uint32_t polls = ctl.start;
    int32_t ok = 1;
    for (;;) {
      const uint32_t v = threadIdx.x < st.members ? flow_load(flags + threadIdx.x * 32) : epoch;
      if (__all((int32_t)(v - epoch) >= 0)) break;
      if (!__any(flow_again(ctl, kSimStop, polls))) {
        ok = 0;
        break;
      }
    }
    if (threadIdx.x == 0) go = ok;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(go) != 0;
}

// The team's k-th tile, or -1 when the list is used up.  (One word: a member
// that has not read it yet is still before the next level's barrier, which
// the leader cannot pass.)
__device__ __forceinline__ int32_t sim_claim(const FlowCtl &ctl, const SimSeat &st, uint32_t k,
                                             int32_t n_tiles) {
  __shared__ int32_t tile;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t *slot = ctl.words + kSimClaim + st.buf * 32;  // sequence k + 1, tile + 1 (0: none left)
    uint32_t v = 0;
    if (st.rank == 0) {
      const uint32_t t = __hip_atomic_fetch_add(ctl.words + kSimNextTile, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      v = (k + 1) << 16 | (t < (uint32_t)n_tiles ? t + 1 : 0u);
      __hip_atomic_store(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      uint32_t polls = ctl.start;
      while ((v = flow_load(slot)) >> 16 != k + 1)
        if (!flow_again(ctl, kSimStop, polls)) {
          v = 0;
          break;
        }
    }
    tile = (int32_t)(v & 0xffffu) - 1;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(tile);
}

// Sum over the LPG lanes of a gate; the gate's last lane has it.
template <int LPG>
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
  if constexpr (LPG > 8) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
  if constexpr (LPG > 16) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
  return v;
}

// The previous lane's value (a gate's first lane does not use it).
template <int LPG>
__device__ __forceinline__ uint64_t prev_lane(uint64_t v) {
  constexpr int ctrl = LPG <= 16 ? 0x111 : 0x138;  // row_shr:1, wave_shr:1
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, ctrl, 0xf, 0xf, true);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), ctrl, 0xf, 0xf, true);
  return (uint64_t)hi << 32 | lo;
}

// What is uniform over a tile.
struct SimTile {
  __amdgpu_buffer_rsrc_t rows;  // the team's buffer
  uint32_t *cnt;                // [n_nets]
  uint64_t *edge;               // [n_nets][2]
  int32_t nw;                   // words of the chunk
};

// A gate's (or PI's) words, two per lane.
struct SimWords {
  uint64_t y0, y1;
  uint32_t net;
  bool valid;
};
template <int LPG>
__device__ __forceinline__ void sim_store(const SimTile &t, const SimWords &w, bool keep) {
  const uint32_t l = threadIdx.x & (LPG - 1);
  if (w.valid && keep && 2 * (int32_t)l < t.nw) {
    const u4 v = u4{(uint32_t)w.y0, (uint32_t)(w.y0 >> 32), (uint32_t)w.y1, (uint32_t)(w.y1 >> 32)};
    __builtin_amdgcn_raw_buffer_store_b128(v, t.rows, (int)(w.net * (LPG * 16u) + 16u * l), 0, 0);
  }
}
// Its counts and its first and last word.
template <int LPG>
__device__ __forceinline__ void sim_count(const SimTile &t, const SimWords &w) {
  const uint64_t y0 = w.y0, y1 = w.y1;
  const uint32_t net = w.net;
  const int32_t l = (int32_t)threadIdx.x & (LPG - 1), u0 = 2 * l;
  const bool in0 = u0 < t.nw, in1 = u0 + 1 < t.nw;
  const uint64_t prev = prev_lane<LPG>(y1);
  uint32_t ones = 0, togs = 0;
  if (in0) {
    ones = __popcll(y0);
    if (l) togs = __popcll(y0 ^ prev);
  }
  if (in1) {
    ones += __popcll(y1);
    togs += __popcll(y0 ^ y1);
  }
  const uint32_t sum = row_sum<LPG>(togs << 16 | ones);
  if (!w.valid) return;
  if (l == LPG - 1) *flow_at(t.cnt, 4 * net) = sum;
  if (l == 0) *flow_at(t.edge, 16 * net) = y0;
  if (u0 == ((t.nw - 1) & ~1)) *flow_at(t.edge + 1, 16 * net) = in1 ? y1 : y0;
}

template <bool CELLS>
struct SimFlowFetch {
  int32_t op, k;  // cell, its inputs
  uint32_t pin[kFlowPins<CELLS>];
  int32_t e0, e1;
};
template <bool CELLS>
__device__ __forceinline__ SimFlowFetch<CELLS> sim_flow_fetch(const GraphView &g, uint32_t gi) {
  SimFlowFetch<CELLS> f;
  f.op = *flow_at(g.op, gi);
  if constexpr (CELLS) f.k = *flow_at(g.arity, gi);
  else f.k = arity_of(f.op);
  flow_pins(g.in, g, gi, f.pin);
  f.e0 = *flow_at(g.rev_ptr + g.n_pi, 4 * gi);
  f.e1 = *flow_at(g.rev_ptr + g.n_pi + 1, 4 * gi);
  return f;
}

template <int LPG>
__device__ __forceinline__ w2 sim_row(const SimTile &t, uint32_t net, uint32_t l16) {
  const u4 v = __builtin_amdgcn_raw_buffer_load_b128(t.rows, (int)(net * (LPG * 16u) + l16), 0, kBufferSc1);
  return w2{(uint64_t)v[1] << 32 | v[0], (uint64_t)v[3] << 32 | v[2]};
}
// A library cell's function from its truth table, as tt_eval, with a table
// per lane: a leaf's mask is one sign-extending bit extract.
template <int N>
__device__ __forceinline__ w2 tt_lane(const w2 *x, uint32_t lo, uint32_t hi, int base) {
  if constexpr (N == 0) {
    const int32_t m = __builtin_amdgcn_sbfe((int32_t)(base < 32 ? lo : hi), base & 31, 1);
    const uint64_t v = (uint64_t)(uint32_t)m << 32 | (uint32_t)m;
    return w2{v, v};
  } else {
    const w2 a = tt_lane<N - 1>(x, lo, hi, base), b = tt_lane<N - 1>(x, lo, hi, base + (1 << (N - 1)));
    return w2{(x[N - 1].x & b.x) | (~x[N - 1].x & a.x), (x[N - 1].y & b.y) | (~x[N - 1].y & a.y)};
  }
}
template <int N>
__device__ __forceinline__ w2 sim_cell(const w2 (&x)[N], const SimFlowFetch<N == kCellMaxIn> &f, uint64_t tt) {
  switch (f.op) {
#define DP_SIM_CASE(OP) \
  case OP: return w2{cell_bits<OP>(x[0].x, x[1].x, x[2].x), cell_bits<OP>(x[0].y, x[1].y, x[2].y)}
    DP_SIM_CASE(INV);
    DP_SIM_CASE(BUF);
    DP_SIM_CASE(AND2);
    DP_SIM_CASE(OR2);
    DP_SIM_CASE(NAND2);
    DP_SIM_CASE(NOR2);
    DP_SIM_CASE(XOR2);
    DP_SIM_CASE(AOI21);
    default: break;
  }
  if constexpr (N == kCellMaxIn)
    if (f.op >= kCellBase) {
      const uint32_t lo = (uint32_t)tt, hi = (uint32_t)(tt >> 32);
      switch (f.k) {
        case 1: return tt_lane<1>(x, lo, hi, 0);
        case 2: return tt_lane<2>(x, lo, hi, 0);
        case 3: return tt_lane<3>(x, lo, hi, 0);
        case 4: return tt_lane<4>(x, lo, hi, 0);
        case 5: return tt_lane<5>(x, lo, hi, 0);
        default: return tt_lane<6>(x, lo, hi, 0);
      }
    }
  switch (MUX2) {
    DP_SIM_CASE(MUX2);
#undef DP_SIM_CASE
  }
}

// The first sp_blocks workgroups take the SP sweep of the same columns, which
// has few waves and long waits, beside the tiles.  Registers for six waves a
// SIMD: two or three teams of tiles and the sweep's (library cells spill one of
// them, 8 bytes of scratch).
template <int LPG, bool CELLS>
__global__ __launch_bounds__(kFlowThreads, 6) void k_sim_flow(FlowCtl ctl, SimFlow t, FlowCtl sp_ctl,
                                                              SpFlow sp, uint32_t sp_blocks) {
  if (blockIdx.x < sp_blocks) {
    sp_flow_team<CELLS>(sp_ctl, sp);
    return;
  }
  const SimSeat st = sim_join(ctl, (uint32_t)t.n_bufs, blockIdx.x - sp_blocks);
  if (st.members == 0) return;
  for (int32_t i = (int32_t)threadIdx.x; i < t.depth + 2; i += (int32_t)blockDim.x)
    flow_lv[i] = t.level_ptr[i];
  __syncthreads();
  constexpr int GP = 64 / LPG;  // gates of a wave
  constexpr int32_t pitch = 2 * LPG;
  const GraphView &g = t.g;
  const int32_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int32_t first = GP * (wave * (int32_t)st.members + (int32_t)st.rank);
  const int32_t step = GP * (int32_t)((blockDim.x >> 6) * st.members);
  const int32_t sub = ((int32_t)threadIdx.x & 63) / LPG;
  const uint32_t l = threadIdx.x & (LPG - 1), l16 = 16 * l;
  SimTile tile;
  tile.rows = __builtin_amdgcn_make_buffer_rsrc(t.W + (int64_t)st.buf * g.n_nets * pitch, 0,
                                                (int)((uint32_t)g.n_nets * (pitch * 8u)), 0x00020000);
  uint32_t epoch = 0;
  for (uint32_t k = 0;; ++k) {
    const int32_t id = sim_claim(ctl, st, k, t.n_chunks * t.B);
    if (id < 0) return;
    const int32_t b = id / t.n_chunks;
    const int64_t t0 = (int64_t)(id - b * t.n_chunks) * pitch;
    tile.nw = (int32_t)min<int64_t>(pitch, t.T - t0);
    tile.cnt = t.cnt + (int64_t)id * g.n_nets;
    tile.edge = t.edge + (int64_t)id * g.n_nets * 2;
    // the PIs' rows
    for (int32_t base = first; base < g.n_pi; base += step) {
      const int32_t i = min(base + sub, g.n_pi - 1);
      const uint64_t *row = t.stim + ((int64_t)b * g.n_pi + i) * t.T + t0;
      const int32_t u0 = 2 * (int32_t)l;
      const SimWords w{u0 < tile.nw ? row[u0] : 0, u0 + 1 < tile.nw ? row[u0 + 1] : 0, (uint32_t)i,
                       base + sub < g.n_pi};
      sim_store<LPG>(tile, w, true);
      sim_count<LPG>(tile, w);
    }
    sim_arrive(ctl, st, ++epoch);
    SimWords last{0, 0, 0, false};
    for (int32_t lv = 1; lv <= t.depth; ++lv) {
      const int32_t g0 = __builtin_amdgcn_readfirstlane(flow_lv[lv]);
      const int32_t n = __builtin_amdgcn_readfirstlane(flow_lv[lv + 1]) - g0;
      // while the other members arrive: the first gates' structure, and the
      // counts of the level before's last ones
      SimFlowFetch<CELLS> f = sim_flow_fetch<CELLS>(g, (uint32_t)(g0 + min(first + sub, n - 1)));
      sim_count<LPG>(tile, last);
      last.valid = false;
      if (!sim_wait(ctl, st, epoch)) return;
      for (int32_t base = first; base < n; base += step) {
        if (base != first) sim_count<LPG>(tile, last);
        const SimFlowFetch<CELLS> c = f;
        last.net = (uint32_t)(g.n_pi + g0 + min(base + sub, n - 1));
        last.valid = base + sub < n;
        w2 x[kFlowPins<CELLS>];
        x[0] = sim_row<LPG>(tile, c.pin[0], l16);
#pragma unroll
        for (int j = 1; j < kFlowPins<CELLS>; ++j)
          x[j] = c.k > j ? sim_row<LPG>(tile, c.pin[j], l16) : w2{0, 0};
        uint64_t tt = 0;
        if constexpr (CELLS) tt = *flow_at(g.tt, 8 * (uint32_t)max(c.op - kCellBase, 0));
        if (base + step < n) f = sim_flow_fetch<CELLS>(g, (uint32_t)(g0 + min(base + step + sub, n - 1)));
        const w2 y = sim_cell(x, c, tt);
        last.y0 = y.x;
        last.y1 = y.y;
        sim_store<LPG>(tile, last, c.e1 > c.e0);
      }
      sim_arrive(ctl, st, ++epoch);
    }
    sim_count<LPG>(tile, last);
    // the next tile rewrites the rows that this one's last levels read
    if (!sim_wait(ctl, st, epoch)) return;
  }
}

// Counts [n_nets][B] of all chunks, the toggles between chunks among them.  A
// simulation that gave up (stop) leaves kNoCount and the gates' probabilities as
// NaN, so that nothing computed from its counts can pass for a result; the PIs'
// are inputs and stay.
__global__ __launch_bounds__(kBlock) void k_sim_counts(SimFlow t, const uint32_t *stop, float *sp,
                                                       uint32_t *ones, uint32_t *tog) {
  const int64_t idx = gidx();
  if (idx >= (int64_t)t.g.n_nets * t.B) return;
  const int32_t b = (int32_t)(idx / t.g.n_nets), net = (int32_t)(idx - (int64_t)b * t.g.n_nets);
  const int64_t o = (int64_t)net * t.B + b;
  uint32_t n1 = 0, nt = 0;
  uint64_t last = 0;
#pragma unroll 4
  for (int32_t k = 0; k < t.n_chunks; ++k) {
    const int64_t at = ((int64_t)b * t.n_chunks + k) * t.g.n_nets + net;
    const uint32_t v = t.cnt[at];
    const w2 e = reinterpret_cast<const w2 *>(t.edge)[at];
    n1 += v & 0xffffu;
    nt += v >> 16;
    if (k) nt += __popcll(last ^ e.x);
    last = e.y;
  }
  const bool bad = *stop != 0u;
  ones[o] = bad ? kNoCount : n1;
  tog[o] = bad ? kNoCount : nt;
  if (bad && net >= t.g.n_pi) sp[o] = __builtin_nanf("");
}

// Words [B][n_pi][T] of the independent stimulus: a wave takes 64 cycles of one
// PI for NC columns.
template <int NC>
__global__ __launch_bounds__(kBlock) void k_stim_words(const float *__restrict__ sp,
                                                       const int32_t *__restrict__ stream,
                                                       int32_t n_pi, int32_t B, int64_t T,
                                                       uint32_t k0, uint32_t k1,
                                                       uint64_t *__restrict__ out) {
  const int32_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t task = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  const int64_t runs = (T + 63) / 64, per_grp = runs * n_pi;
  if (task >= per_grp * ((B + NC - 1) / NC)) return;
  const int32_t grp = (int32_t)(task / per_grp);
  const int64_t rest = task - grp * per_grp;
  const int32_t i = (int32_t)(rest / runs);
  const int64_t t = (rest - (int64_t)i * runs) * 64 + (threadIdx.x & 63);
  const int32_t b0 = grp * NC, cols = min(NC, B - b0);
  BitThreshold thr[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const BitThreshold x = bit_threshold(prob_threshold(
        sp_load(sp[(int64_t)i * B + b0 + min(k, cols - 1)]).x));
    thr[k].t = (uint32_t)__builtin_amdgcn_readfirstlane((int)x.t);
    thr[k].all = __builtin_amdgcn_readfirstlane((int)x.all) ? ~0ull : 0ull;
  }
  uint64_t w[NC];
  stim_words<true>(stream ? (uint32_t)stream[i] : (uint32_t)i, (uint32_t)t, thr, k0, k1, w);
  if (t < T)
#pragma unroll
    for (int k = 0; k < NC; ++k)
      if (k < cols) out[((int64_t)(b0 + k) * n_pi + i) * T + t] = w[k];
}

// dP/dC_n = sum_{b,s} w[b][s] kappa beta TR_model s_s(drv n);
// dP/ds[s][g] = sum_b w[b][s] kappa beta TR_model C of g's output net.
// x = kappa beta TR_model of net n in column b, recomputed as the forward's
// power sum computed it.
__device__ __forceinline__ float x_of(const GradExportArgs &a, int64_t n, int32_t b) {
  const int64_t idx = n * a.B + b;
  const f2 pq = sp_load(a.sp[idx]);
  const float tm = 2.0f * pq.x * pq.y;
  const float beta = a.beta ? a.beta[a.beta_shared ? n : idx] : 1.0f;
  return a.kappa * beta * tm;
}

// One wave per 64 nets.  The x values of the nets' rows are staged through
// LDS a tile of up to 32 columns at a time (consecutive lanes read
// consecutive (net, column) entries, so the loads are whole row segments;
// sixteen go out before the first store), then lane r sums its net's
// columns in order.
constexpr int32_t kCapRows = 64, kCapCols = 32, kCapBatch = 16;
constexpr int32_t kCapSized = 4;  // columns whose weights one pass over the sizes forms

template <bool BETA, bool SIZED>  // BETA: a beta array is present; SIZED: weights through LDS
__global__ __launch_bounds__(kCapRows) void k_grad_cap(GradExportArgs a) {
  __shared__ float xs[kCapRows][kCapCols + 1];
  __shared__ float wcol[kCapCols];  // without sizes a column's weight is the net's
  const int32_t r = (int32_t)threadIdx.x;
  const int64_t n0 = (int64_t)blockIdx.x * kCapRows;
  const int64_t n = n0 + r;
  const int32_t rows = (int32_t)min<int64_t>(kCapRows, a.n_nets - n0);
  const int32_t Sp = (a.S > 0 && !a.paired) ? a.S : 1;
  const bool gate = n >= a.n_pi && a.size;
  auto weight = [&](int32_t b) {
    float ws = 0.0f;
    for (int32_t s = 0; s < Sp; ++s) {
      const int32_t row = a.paired ? b : s;
      const float w = a.w ? a.w[(int64_t)b * Sp + s] : 1.0f;
      const float sz = gate ? a.size[(n - a.n_pi) * a.S + row] : 1.0f;
      ws = fmaf(w, sz, ws);
    }
    return ws;
  };
  __shared__ float lds[SIZED ? kCapRows : 1][kSizeChunk + 1];
  const auto net_of = [&](int32_t row) { return row < rows ? (int32_t)(n0 + row) : -1; };
  double acc = 0.0;
  for (int32_t b0 = 0; b0 < a.B; b0 += kCapCols) {
    const int32_t tw = min(kCapCols, a.B - b0), total = rows * tw;
    for (int32_t e0 = r; e0 < total; e0 += kCapBatch * kCapRows) {
      float v[kCapBatch];
      float bt[kCapBatch];
      // (row, column) of entry e: shifts for a whole tile, else a division
      const bool full = tw == kCapCols;
#pragma unroll
      for (int u = 0; u < kCapBatch; ++u) {  // clamped: every load is valid
        const int32_t e = min(e0 + u * kCapRows, total - 1);
        const int32_t rr = full ? e / kCapCols : e / tw;
        const int64_t nn = n0 + rr, idx = nn * a.B + b0 + (e - rr * tw);
        v[u] = a.sp[idx];
        bt[u] = BETA ? a.beta[a.beta_shared ? nn : idx] : 1.0f;
      }
#pragma unroll
      for (int u = 0; u < kCapBatch; ++u) {  // x as x_of forms it
        const f2 pq = sp_load(v[u]);
        v[u] = a.kappa * bt[u] * (2.0f * pq.x * pq.y);
      }
#pragma unroll
      for (int u = 0; u < kCapBatch; ++u) {
        const int32_t e = e0 + u * kCapRows, rr = full ? e / kCapCols : e / tw;
        if (e < total) xs[rr][e - rr * tw] = v[u];
      }
    }
    // without sizes the weight of column b is the same for every net: one
    // lane per column forms it (as weight() would), the row loop reads it
    if (!a.size && r < tw) wcol[r] = weight(b0 + r);
    __syncthreads();
    if constexpr (SIZED) {
      for (int32_t cc = 0; cc < tw; cc += kCapSized) {
        const float *w = a.w ? a.w + (int64_t)(b0 + cc) * Sp : nullptr;
        const int32_t cols = min(kCapSized, tw - cc);
        float ws[kCapSized];
        staged_weights(a.size, a.n_pi, Sp, w, cols, lds, net_of, b0 + cc == 0, ws);
#pragma unroll
        for (int k = 0; k < kCapSized; ++k)
          if (r < rows && k < cols) acc += (double)xs[r][cc + k] * (double)ws[k];
      }
    } else if (r < rows) {
      if (!a.size)
        for (int32_t cc = 0; cc < tw; ++cc) acc += (double)xs[r][cc] * (double)wcol[cc];
      else
        for (int32_t cc = 0; cc < tw; ++cc) acc += (double)xs[r][cc] * (double)weight(b0 + cc);
    }
    __syncthreads();
  }
  if (r < rows) a.dcap[a.int2ext[n]] = (float)acc;
}

// Few columns: one thread per net, its columns in order (the same sum as
// k_grad_cap); consecutive threads read consecutive rows, which at few
// columns are already whole lines, and no LDS pass is needed.
constexpr int32_t kCapRowsMinCols = 16;  // from this many columns k_grad_cap stages rows

template <bool SIZED>
__global__ __launch_bounds__(kBlock) void k_grad_cap_narrow(GradExportArgs a) {
  const int64_t n = gidx();
  const int32_t Sp = (a.S > 0 && !a.paired) ? a.S : 1;
  const bool gate = n >= a.n_pi && a.size;
  double acc = 0.0;
  if constexpr (SIZED) {
    __shared__ float lds[kBlock][kSizeChunk + 1];
    const auto net_of = [&](int32_t row) {
      const int64_t m = (int64_t)blockIdx.x * kBlock + row;
      return m < a.n_nets ? (int32_t)m : -1;
    };
    for (int32_t b = 0; b < a.B; b += kCapSized) {
      const int32_t cols = min(kCapSized, a.B - b);
      float ws[kCapSized];
      staged_weights(a.size, a.n_pi, Sp, a.w ? a.w + (int64_t)b * Sp : nullptr, cols, lds, net_of,
                     b == 0, ws);
#pragma unroll
      for (int k = 0; k < kCapSized; ++k)
        if (n < a.n_nets && k < cols) acc += (double)x_of(a, n, b + k) * (double)ws[k];
    }
    if (n < a.n_nets) a.dcap[a.int2ext[n]] = (float)acc;
    return;
  }
  if (n >= a.n_nets) return;
  for (int32_t b = 0; b < a.B; ++b) {
    float ws = 0.0f;
    for (int32_t s = 0; s < Sp; ++s) {
      const int32_t row = a.paired ? b : s;
      const float w = a.w ? a.w[(int64_t)b * Sp + s] : 1.0f;
      const float sz = gate ? a.size[(n - a.n_pi) * a.S + row] : 1.0f;
      ws = fmaf(w, sz, ws);
    }
    acc += (double)x_of(a, n, b) * (double)ws;
  }
  a.dcap[a.int2ext[n]] = (float)acc;
}

__global__ __launch_bounds__(kBlock) void k_grad_size(GradExportArgs a) {
  const int64_t idx = gidx();
  if (idx >= (int64_t)a.G * a.S) return;
  const int32_t s = (int32_t)(idx / a.G), g = (int32_t)(idx - (int64_t)s * a.G);
  const int32_t n = a.n_pi + g;
  double acc = 0.0;
  if (a.paired) {  // size row s belongs to column s only
    acc = (double)x_of(a, n, s) * (double)(a.w ? a.w[s] : 1.0f);
  } else {
    for (int32_t b = 0; b < a.B; ++b) {
      const float w = a.w ? a.w[(int64_t)b * a.S + s] : 1.0f;
      acc += (double)x_of(a, n, b) * (double)w;
    }
  }
  a.dsize[(int64_t)s * a.G + (a.int2ext[n] - a.n_pi)] = (float)(acc * (double)a.cap[n]);
}

}  // namespace

// ==================================================================== launchers
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_fill_u32<<<blocks_for(n), kBlock, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_fill_f32<<<blocks_for(n), kBlock, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_load_pi(const float *p, float *sp, int32_t n_pi, int32_t B, hipStream_t s) {
  const int64_t n = (int64_t)n_pi * B;
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_load_pi<<<blocks_for(n), kBlock, 0, s>>>(p, sp, n_pi, B);
  return hipGetLastError();
}

hipError_t launch_check_range(const float *v, int64_t n, float lo, float hi, float *copy,
                              uint32_t *bad, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_check_range<<<blocks_for(n), kBlock, 0, s>>>(v, n, lo, hi, copy, bad);
  return hipGetLastError();
}

hipError_t launch_gather_nets_f32(const float *src_ext, const int32_t *int2ext, float *dst_int,
                                  int32_t n_nets, hipStream_t s) {
  if (n_nets <= 0) return hipSuccess;
  k_gather_nets<<<blocks_for(n_nets), kBlock, 0, s>>>(src_ext, int2ext, dst_int, n_nets);
  return hipGetLastError();
}

hipError_t launch_import_cols_f32(const float *src, const int32_t *int2ext, float *dst,
                                  int32_t n_nets, int32_t B, hipStream_t s) {
  const int64_t n = (int64_t)n_nets * B;
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_import_cols<<<blocks_for(n), kBlock, 0, s>>>(src, int2ext, dst, n_nets, B);
  return hipGetLastError();
}

hipError_t launch_import_sizes(const float *src, const int32_t *int2ext, const int32_t *ext2int,
                               float *dst, int32_t n_pi, int32_t G, int32_t S, hipStream_t s) {
  if ((int64_t)G * S <= 0) return hipSuccess;
  if (S >= 2 && (int64_t)G * S >= kSizeRunsMin) {
    const int64_t blocks = (int64_t)((G + kSizeGates - 1) / kSizeGates) * ((S + kSizeRuns - 1) / kSizeRuns);
    if (blocks > kMaxBlocks) return hipErrorInvalidValue;
    k_import_size_runs<<<(unsigned)blocks, kBlock, 0, s>>>(src, ext2int, dst, n_pi, G, S);
    return hipGetLastError();
  }
  const int64_t groups = (S + kSizeVecs - 1) / kSizeVecs;
  const int64_t rounds = groups >= kSizeXcds ? (groups + kSizeXcds - 1) / kSizeXcds * kSizeXcds : groups;
  const int64_t blocks = (int64_t)((G + kSizeGates - 1) / kSizeGates) * rounds;
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  k_import_sizes<<<(unsigned)blocks, kBlock, 0, s>>>(src, int2ext, dst, n_pi, G, S);
  return hipGetLastError();
}

bool CopyList::add(const float *src, float *dst, int64_t count) {
  if (n == kMax || count > (1ll << 30)) return false;
  c[n++] = Item{src, dst, (uint32_t)count, blocks};
  blocks += (uint32_t)((count + kBlock * kCopyPer - 1) / (kBlock * kCopyPer));
  return true;
}
hipError_t launch_copies(const CopyList &l, hipStream_t s) {
  if (l.blocks) k_copies<<<l.blocks, kBlock, 0, s>>>(l);
  return hipGetLastError();
}
void lane_seg_blocks(LaneSeg &l, uint32_t &stage, uint32_t &import, uint32_t &out) {
  const int64_t sizes = l.size ? (int64_t)l.B * l.G : 0;
  l.pi_blocks = blocks_for((int64_t)l.n_pi * l.B);
  stage = l.pi_blocks + (uint32_t)((sizes + kLaneCopy - 1) / kLaneCopy);
  const int64_t groups = (l.B + kSizeVecs - 1) / kSizeVecs;
  const int64_t rounds = groups >= kSizeXcds ? (groups + kSizeXcds - 1) / kSizeXcds * kSizeXcds : groups;
  import = sizes ? (uint32_t)(((l.G + kSizeGates - 1) / kSizeGates) * rounds) : 0u;
  out = l.dpi ? (uint32_t)(((int64_t)l.B * l.n_pi + kLaneCopy - 1) / kLaneCopy) : 0u;
}
hipError_t launch_lanes_stage(const LaneSeg *segs, int32_t n_segs, uint32_t stage_blocks,
                              uint32_t import_blocks, hipStream_t s) {
  if (stage_blocks) k_lanes_stage<<<stage_blocks, kBlock, 0, s>>>(segs, n_segs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !import_blocks) return e;
  k_lanes_import<<<import_blocks, kBlock, 0, s>>>(segs, n_segs);
  return hipGetLastError();
}
hipError_t launch_lanes_out(const LaneSeg *segs, int32_t n_segs, uint32_t blocks, hipStream_t s) {
  if (blocks) k_lanes_out<<<blocks, kBlock, 0, s>>>(segs, n_segs);
  return hipGetLastError();
}

hipError_t launch_grad_lambda_export(const float *lam, const float *sp, const int32_t *int2ext,
                                     int32_t n_pi, int32_t n_nets, int32_t B, int32_t C,
                                     int32_t cdiv, float eps, float *lam_out, float *score,
                                     hipStream_t s) {
  const int64_t n = (int64_t)n_nets * C;
  if (n <= 0 || (!lam_out && !score)) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_grad_lambda_export<<<blocks_for(n), kBlock, 0, s>>>(lam, sp, int2ext, n_pi, n_nets, B, C,
                                                        cdiv, eps, lam_out, score);
  return hipGetLastError();
}

hipError_t launch_virus_step(float *sp, const float *grad, float eta, int32_t n_pi, int32_t B,
                             hipStream_t s) {
  const int64_t n = (int64_t)n_pi * B;
  if (n <= 0) return hipSuccess;
  if (n >= (1ll << 31)) return hipErrorInvalidValue;
  k_virus_step<<<blocks_for(n), kBlock, 0, s>>>(sp, grad, eta, n_pi, B);
  return hipGetLastError();
}

hipError_t launch_virus_vectors(const float *sp, uint64_t *stim, uint8_t *v0, float *p_out,
                                int32_t n_pi, int32_t B, hipStream_t s) {
  const int64_t n = (int64_t)n_pi * B;
  if (n <= 0) return hipSuccess;
  if (n >= (1ll << 31)) return hipErrorInvalidValue;
  k_virus_vectors<<<blocks_for(n), kBlock, 0, s>>>(sp, stim, v0, p_out, n_pi, B);
  return hipGetLastError();
}

hipError_t launch_virus_power(const uint32_t *tog, const float *cap, int32_t n_nets, int32_t B,
                              double *out, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  k_virus_power<<<(unsigned)B, kBlock, 0, s>>>(tog, cap, n_nets, B, out);
  return hipGetLastError();
}

hipError_t launch_sp_multi(const SpSeg *segs, int32_t n_segs, uint32_t blocks, bool cells,
                           hipStream_t s) {
  if (n_segs <= 0 || blocks == 0) return hipSuccess;
  if (cells)
    k_sp_multi<true><<<blocks, kMergedBlock, 0, s>>>(segs, n_segs);
  else
    k_sp_multi<false><<<blocks, kMergedBlock, 0, s>>>(segs, n_segs);
  return hipGetLastError();
}

hipError_t launch_bwd_multi(const BwdSeg *segs, int32_t n_segs, uint32_t blocks, bool cells,
                            hipStream_t s) {
  if (n_segs <= 0 || blocks == 0) return hipSuccess;
  if (cells)
    k_bwd_multi<true><<<blocks, kMergedBlock, 0, s>>>(segs, n_segs);
  else
    k_bwd_multi<false><<<blocks, kMergedBlock, 0, s>>>(segs, n_segs);
  return hipGetLastError();
}

hipError_t launch_sp_pair(const GraphView &g, const SpLevel &a, const SpLevel &b, hipStream_t s) {
  const int64_t n = ((int64_t)a.n + b.n) * a.B;
  if (n <= 0) return hipSuccess;
  if (n >= (1ll << 31) || a.B != b.B || a.sp != b.sp || b.g0 != a.g0 + a.n)
    return hipErrorInvalidValue;
  k_sp_pair<<<level_grid(n), level_block(n), 0, s>>>(g, a, b);
  return hipGetLastError();
}

hipError_t launch_sp_level(const GraphView &g, const SpLevel &lv, bool cells, hipStream_t s) {
  const int64_t n = (int64_t)lv.n * lv.B;
  if (n <= 0) return hipSuccess;
  if (n >= (1ll << 31)) return hipErrorInvalidValue;
  if (cells)
    k_sp_cells<<<blocks_for(n), kBlock, 0, s>>>(g, lv);
  else if (lv.B % 4 == 0 && n >= kQuadItems)
    k_sp_level_x4<<<level_grid(n / 4), level_block(n / 4), 0, s>>>(g, lv);
  else if (lv.B % 2 == 0)
    k_sp_level_x2<<<level_grid(n / 2), level_block(n / 2), 0, s>>>(g, lv);
  else
    k_sp_level<<<level_grid(n), level_block(n), 0, s>>>(g, lv);
  return hipGetLastError();
}

static int32_t waves_per_row(const ChunkView &c, int iters) {
  return (c.pairs + 64 * iters - 1) / (64 * iters);
}

hipError_t launch_stimulus(const GraphView &g, const ChunkView &c, const CountView &cnt,
                           const float *p_col, const uint64_t *stim, int64_t T,
                           const int32_t *stream, uint64_t seed, const SimTune &tune,
                           hipStream_t s) {
  if (g.n_pi <= 0 || c.pairs <= 0) return hipSuccess;
  if (c.n_cols <= 0) return hipSuccess;
  const int iters = tune.iters;
  const int32_t wpr = waves_per_row(c, iters);
  // columns per draw: as many as there are, up to eight (a lane's registers:
  // 101 at eight, four waves a SIMD)
  const int nc = stim || c.n_cols == 1 ? 1 : c.n_cols == 2 ? 2 : c.n_cols <= 4 ? 4 : 8;
  const int64_t tasks = (int64_t)g.n_pi * wpr * ((c.n_cols + nc - 1) / nc);
  if ((tasks + kWavesPerBlock - 1) / kWavesPerBlock > kMaxBlocks) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((tasks + kWavesPerBlock - 1) / kWavesPerBlock);
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  using K = void (*)(int32_t, ChunkView, CountView, const float *, const uint64_t *, int64_t,
                     const int32_t *, uint32_t, uint32_t, int32_t);
#define DP_STIM_ROW(NC, STIM) \
  { k_stimulus<1, NC, STIM>, k_stimulus<2, NC, STIM>, k_stimulus<4, NC, STIM>, k_stimulus<8, NC, STIM> }
  static const K table[5][4] = {DP_STIM_ROW(1, true), DP_STIM_ROW(1, false), DP_STIM_ROW(2, false),
                                DP_STIM_ROW(4, false), DP_STIM_ROW(8, false)};
#undef DP_STIM_ROW
  const int row = stim ? 0 : nc == 1 ? 1 : nc == 2 ? 2 : nc == 4 ? 3 : 4;
  const int col = iters == 1 ? 0 : iters == 2 ? 1 : iters == 4 ? 2 : 3;
  hipLaunchKernelGGL(table[row][col], dim3(grid), dim3(kBlock), 0, s, g.n_pi, c, cnt, p_col, stim,
                     T, stream, k0, k1, wpr);
  return hipGetLastError();
}

hipError_t launch_markov_words(const float *sp, const float *tau, const int32_t *stream,
                               int32_t n_pi, int32_t B, int64_t T, uint64_t seed, uint64_t *out,
                               hipStream_t s) {
  const int64_t rows = (int64_t)n_pi * B;
  if (rows <= 0 || T <= 0) return hipSuccess;
  const int64_t blocks = (rows + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  k_markov_words<<<(unsigned)blocks, kBlock, 0, s>>>(sp, tau, stream, n_pi, B, T, (uint32_t)seed,
                                                     (uint32_t)(seed >> 32), out);
  return hipGetLastError();
}

hipError_t launch_sim_level(const GraphView &g, const ChunkView &c, const CountView &cnt,
                            int32_t g0, int32_t n, const SpLevel *sp, bool cells,
                            const SimTune &tune, hipStream_t s, int cell_inputs) {
  if (n <= 0 || c.n_cols <= 0) return hipSuccess;
  const bool narrow = cells && cell_inputs <= kSmallCellInputs;
  // cells: up to 2 pairs per lane (up to 6 input rows each), narrow cells up to 4
  const int iters = cells ? min(tune.iters, narrow ? 4 : 2) : tune.iters;
  const int32_t wpr = waves_per_row(c, iters);
  const int64_t tasks = (int64_t)n * wpr * c.n_cols;
  const int64_t sim_blocks64 = (tasks + kSimWaves - 1) / kSimWaves;
  SpLevel spl{};
  int64_t sp_blocks = 0;
  if (sp) {
    spl = *sp;
    if ((int64_t)spl.n * spl.B >= (1ll << 31)) return hipErrorInvalidValue;
    sp_blocks = ((int64_t)spl.n * spl.B + kSimBlock - 1) / kSimBlock;
  }
  if (sim_blocks64 + sp_blocks > kMaxBlocks || sim_blocks64 > INT32_MAX) return hipErrorInvalidValue;
  const int32_t sim_blocks = (int32_t)sim_blocks64;
  const unsigned grid = (unsigned)(sim_blocks + sp_blocks);
  if (narrow) {
    switch (iters) {
      case 1: k_sim_level<1, 3><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
      case 2: k_sim_level<2, 3><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
      default: k_sim_level<4, 3><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
    }
    return hipGetLastError();
  }
  if (cells) {
    if (iters == 1)
      k_sim_level<1, 6><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl);
    else
      k_sim_level<2, 6><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl);
    return hipGetLastError();
  }
  switch (iters) {
    case 1: k_sim_level<1, 0><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
    case 2: k_sim_level<2, 0><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
    case 4: k_sim_level<4, 0><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
    default: k_sim_level<8, 0><<<grid, kSimBlock, 0, s>>>(g, c, cnt, g0, n, wpr, sim_blocks, spl); break;
  }
  return hipGetLastError();
}

hipError_t launch_export(const ExportArgs &a, hipStream_t s) {
  const int64_t n = (int64_t)a.n_nets * a.B;
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  k_export<<<blocks_for(n), kBlock, 0, s>>>(a);
  return hipGetLastError();
}

int32_t power_chunks(int32_t n_nets) {
  return n_nets <= 0 ? 1 : (n_nets + kPowerChunk - 1) / kPowerChunk;
}

uint32_t power_blocks(const PowerArgs &a) {
  const int32_t tb = power_tile(a.B);
  return (uint32_t)(kXcds * ((a.B + tb - 1) / tb) * ((a.n_chunks + kXcds - 1) / kXcds));
}
hipError_t launch_power_multi(const PowerSeg *segs, int32_t n_segs, uint32_t blocks, int32_t cols,
                              int32_t widest, hipStream_t s) {
  if (n_segs <= 0 || blocks == 0 || cols <= 0) return hipSuccess;
  k_power_multi<<<blocks, (unsigned)(kPowerLanes * power_tile(widest)), 0, s>>>(segs, n_segs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_power_final_multi<<<(unsigned)cols, kBlock, 0, s>>>(segs, n_segs);
  return hipGetLastError();
}
hipError_t launch_power(const PowerArgs &a, hipStream_t s) {
  const int32_t Sp = (a.S > 0 && !a.paired) ? a.S : 1;
  const int32_t n_cols = a.B * Sp;
  if ((int64_t)a.n_nets * a.B <= 0) return hipSuccess;
  if (a.S > 0 && !a.paired && a.size) {
    if (a.mode == 1) {  // the hybrid beta first: the contraction reads it
      if (!a.beta || too_big((int64_t)a.n_nets * a.B)) return hipErrorInvalidValue;
      k_beta<<<blocks_for((int64_t)a.n_nets * a.B), kBlock, 0, s>>>(a);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    const int32_t len = power_slab_nets(a.n_nets), n_slabs = power_slabs(a.n_nets);
    const float *beta = a.mode == 1 ? a.beta : a.mode == 2 ? a.beta_frozen : nullptr;
    const int32_t shared = a.mode == 2 ? a.beta_shared : 0;
    // two tiles a side where there are that many columns: each operand loaded
    // feeds two products
    const int mb = a.B > 16 ? 2 : 1, ms = a.S > 16 ? 2 : 1;
    using K = void (*)(PowerArgs, const float *, int32_t, int32_t, int32_t, int32_t, int32_t, PowerPiece);
    static const K table[2][2] = {{k_power_mfma<1, 1>, k_power_mfma<1, 2>},
                                  {k_power_mfma<2, 1>, k_power_mfma<2, 2>}};
    const PowerPiece piece = power_piece(a.n_nets, a.B, a.S);
    for (int32_t b0 = 0; b0 < a.B; b0 += piece.nb)
      for (int32_t s0 = 0; s0 < a.S; s0 += piece.ns) {
        const PowerPiece pc{std::min(piece.nb, a.B - b0), std::min(piece.ns, a.S - s0)};
        const int64_t tasks = (int64_t)n_slabs * ((pc.nb + 16 * mb - 1) / (16 * mb)) *
                              ((pc.ns + 16 * ms - 1) / (16 * ms));
        const int64_t blocks = (tasks + kWavesPerBlock - 1) / kWavesPerBlock;
        if (blocks > kMaxBlocks) return hipErrorInvalidValue;
        hipLaunchKernelGGL(table[mb - 1][ms - 1], dim3((unsigned)blocks), dim3(kBlock), 0, s, a,
                           beta, shared, n_slabs, len, b0, s0, pc);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const int32_t n = pc.nb * pc.ns;
        k_power_slabs<<<(unsigned)((n + 15) / 16), kBlock, 0, s>>>(
            a.partial, n_slabs, n, pc.ns, a.S, a.power + (int64_t)b0 * a.S + s0);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
    return hipSuccess;
  }
  if (a.mode == 1 && !a.beta) return hipErrorInvalidValue;
  if (a.n_chunks != power_chunks(a.n_nets)) return hipErrorInvalidValue;
  int32_t tb = 1;
  while (tb < a.B && tb < kPowerCols) tb *= 2;
  const int32_t col_tiles = (a.B + tb - 1) / tb;
  const int64_t blocks = (int64_t)kXcds * col_tiles * ((a.n_chunks + kXcds - 1) / kXcds);
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  if (a.mode < 0 || a.mode > 2) return hipErrorInvalidValue;
  const unsigned threads = (unsigned)std::min(kPowerLanes * tb, kPowerThreads);
  using K = void (*)(PowerArgs, int32_t, int32_t);
  static const K table[3][3] = {{k_power_sp<1, 0>, k_power_sp<1, 1>, k_power_sp<1, 2>},
                                {k_power_sp<2, 0>, k_power_sp<2, 1>, k_power_sp<2, 2>},
                                {k_power_sp<4, 0>, k_power_sp<4, 1>, k_power_sp<4, 2>}};
  const K kern = table[tb == 64 ? 2 : tb == 32 ? 1 : 0][a.mode];
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), 0, s, a, tb, col_tiles);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_power_final<<<(unsigned)n_cols, kBlock, 0, s>>>(a, n_cols);
  return hipGetLastError();
}


hipError_t launch_bwd_level(const GraphView &g, const BwdArgs &a, int32_t g0, int32_t n,
                            bool cells, hipStream_t s, const int32_t *heavy, int32_t n_heavy) {
  const int64_t items = (int64_t)n * a.C;
  if (items <= 0) return hipSuccess;
  if (items >= (1ll << 31)) return hipErrorInvalidValue;
  if (cells) {
    k_bwd_level<true, false><<<level_blocks(items), kLevelBlock, 0, s>>>(g, a, g0, n, nullptr,
                                                                          0, 0);
  } else if (a.C >= kSerialColumns) {
    if (n_heavy < 0 || (n_heavy > 0 && !heavy)) return hipErrorInvalidValue;
    // 256-thread workgroups at every size: the instance holds 16 KiB of LDS
    // for its heavy-net blocks, so one-wave workgroups would leave a CU ten
    // waves (8 columns: 0.87 ms fwd+bwd against 1.18 ms at 6 with one-wave
    // groups on the 1M-gate design)
    const int64_t hb = (int64_t)n_heavy * ((a.C + 63) / 64);
    const int64_t blocks = hb + blocks_for(items);
    if (blocks > kMaxBlocks) return hipErrorInvalidValue;
    if (a.C % 4 == 0 && a.C == a.B && a.cdiv == 1 && items >= kQuadItems)
      k_bwd_quad<<<(unsigned)(hb + blocks_for(items / 4)), kWideBlock, 0, s>>>(
          g, a, g0, n, heavy, n_heavy, (uint32_t)hb);
    else if (a.C % 64 == 0)  // one gate per wave
      k_bwd_level<false, true, true><<<(unsigned)blocks, kWideBlock, 0, s>>>(
          g, a, g0, n, heavy, n_heavy, (uint32_t)hb);
    else
      k_bwd_level<false, true><<<(unsigned)blocks, kWideBlock, 0, s>>>(
          g, a, g0, n, heavy, n_heavy, (uint32_t)hb);
  } else {
    k_bwd_level<false, false><<<level_grid(items), level_block(items), 0, s>>>(g, a, g0, n,
                                                                              nullptr, 0, 0);
  }
  return hipGetLastError();
}

hipError_t launch_edge_partials(const GraphView &g, const float *sp, int32_t B, bool cells,
                                float *part, hipStream_t s) {
  const int64_t n = (int64_t)g.G * B;
  if (n <= 0) return hipSuccess;
  if (too_big(n)) return hipErrorInvalidValue;
  if (cells)
    k_edge_partials<true><<<blocks_for(n), kBlock, 0, s>>>(g, sp, B, part);
  else
    k_edge_partials<false><<<blocks_for(n), kBlock, 0, s>>>(g, sp, B, part);
  return hipGetLastError();
}

hipError_t launch_bwd_wide_level(const GraphView &g, const BwdArgs &a, const float *part, float *lam,
                                 int32_t net0, int32_t n, hipStream_t s, const int32_t *heavy,
                                 int32_t n_heavy) {
  if (n <= 0 || a.C <= 0) return hipSuccess;
  if (n_heavy < 0 || (n_heavy > 0 && !heavy) || !part || !lam || !a.per_column || a.lam)
    return hipErrorInvalidValue;
  // four columns a lane where their rows are whole 16-byte pieces of one b
  const bool vec = a.C >= 256 && a.C % 4 == 0 && a.cdiv % 4 == 0;
  const int32_t span = vec ? 256 : 64, segs = (a.C + span - 1) / span;
  const int64_t blocks = ((int64_t)(n + n_heavy) * segs + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  if (vec)
    k_bwd_wide<4><<<(unsigned)blocks, kBlock, 0, s>>>(g, a, part, lam, net0, n, segs, heavy, n_heavy);
  else
    k_bwd_wide<1><<<(unsigned)blocks, kBlock, 0, s>>>(g, a, part, lam, net0, n, segs, heavy, n_heavy);
  return hipGetLastError();
}

hipError_t launch_bwd_wide_out(const float *lam, int32_t n_pi, int32_t C, float *out, hipStream_t s) {
  if (n_pi <= 0 || C <= 0) return hipSuccess;
  const int64_t blocks = (int64_t)((n_pi + 63) / 64) * ((C + 63) / 64);
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  k_bwd_wide_out<<<(unsigned)blocks, kBlock, 0, s>>>(lam, n_pi, C, out);
  return hipGetLastError();
}

hipError_t launch_bwd_pi(const GraphView &g, const BwdArgs &a, float *out, hipStream_t s,
                         const int32_t *heavy, int32_t n_heavy) {
  const int64_t items = (int64_t)g.n_pi * a.C;
  if (items <= 0) return hipSuccess;
  if (items >= (1ll << 31)) return hipErrorInvalidValue;
  if (n_heavy < 0 || (n_heavy > 0 && !heavy)) return hipErrorInvalidValue;
  if (a.C < kSerialColumns) n_heavy = 0;
  const int64_t hb = (int64_t)n_heavy * ((a.C + 63) / 64);
  const int64_t blocks = hb + blocks_for(items);
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  k_bwd_pi<<<(unsigned)blocks, kBlock, 0, s>>>(g, a, out, heavy, n_heavy, (uint32_t)hb);
  return hipGetLastError();
}

// Blocks of a cooperative launch: enough for the widest level, at most what
// stays resident on the device.
// One block per compute unit at most (and never more than stays resident):
// the barrier's cost grows with its block count, and a wider level is
// covered by the grid-stride loop.
static hipError_t persistent_grid(const void *kernel, int64_t max_items, unsigned *grid) {
  int dev = 0, ncu = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0);
  if (e != hipSuccess) return e;
  // one block per CU at most, and no more blocks than the barrier has flags
  const int64_t resident = std::min<int64_t>({(int64_t)per_cu * ncu, ncu, kBarrierFlags});
  if (resident < 1) return hipErrorInvalidValue;
  const int64_t want = std::max<int64_t>(1, (max_items + kBlock - 1) / kBlock);
  *grid = (unsigned)std::min(resident, want);
  return hipSuccess;
}

hipError_t launch_sp_persistent(const GraphView &g, const SpLevel &lv, const int32_t *level_ptr,
                                int32_t depth, int64_t max_items, GridBarrier bar,
                                hipStream_t s) {
  if (depth <= 0) return hipSuccess;
  if (max_items >= (1ll << 31) || !bar.words) return hipErrorInvalidValue;
  unsigned grid = 0;
  hipError_t e = persistent_grid(reinterpret_cast<const void *>(&k_sp_persistent), max_items, &grid);
  if (e != hipSuccess) return e;
  k_fill_u32<<<blocks_for(kBarrierWords), kBlock, 0, s>>>(bar.words, kBarrierWords, 0u);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  GraphView gv = g;
  SpLevel l = lv;
  const int32_t *lp = level_ptr;
  int32_t d = depth;
  GridBarrier gb = bar;
  void *args[] = {&gv, &l, &lp, &d, &gb};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(&k_sp_persistent), dim3(grid),
                                    dim3(kBlock), args, 0, s);
}

hipError_t launch_bwd_persistent(const GraphView &g, const BwdArgs &a, const int32_t *level_ptr,
                                 int32_t depth, int64_t max_items, float *pi_out,
                                 GridBarrier bar, hipStream_t s) {
  max_items = std::max<int64_t>(max_items, (int64_t)g.n_pi * a.C);
  if (max_items >= (1ll << 31) || !bar.words) return hipErrorInvalidValue;
  const void *kernel = a.C >= kSerialColumnsNoHeavy
                           ? reinterpret_cast<const void *>(&k_bwd_persistent<true>)
                           : reinterpret_cast<const void *>(&k_bwd_persistent<false>);
  unsigned grid = 0;
  hipError_t e = persistent_grid(kernel, max_items, &grid);
  if (e != hipSuccess) return e;
  k_fill_u32<<<blocks_for(kBarrierWords), kBlock, 0, s>>>(bar.words, kBarrierWords, 0u);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  GraphView gv = g;
  BwdArgs ba = a;
  const int32_t *lp = level_ptr;
  int32_t d = depth;
  float *po = pi_out;
  GridBarrier gb = bar;
  void *args[] = {&gv, &ba, &lp, &d, &po, &gb};
  return hipLaunchCooperativeKernel(kernel, dim3(grid), dim3(kBlock), args, 0, s);
}

// Workgroups of a dataflow sweep over C columns: a team gets enough waves for
// the widest level (64 items each) on as many of an XCD's CUs as there are
// waves, then more waves per workgroup; columns beyond one per XCD get teams
// of their own while the waves stay resident together, and queue after that.
// Blocks go to the XCDs in turn.
constexpr int64_t kFlowWavesPerCu = 16;
// The waves of two shifts take the levels in turn: a wave alone on its SIMD is
// bound by its instructions (a turn of the reverse sweep has some 400), and of
// these only a poll that succeeds, the sum and the stores are on the way from
// level to level; with one shift the next block's addresses and fetch were
// too.  Reverse sweep, one column, us, by shifts 1 / 2 / 4: 2K gates 24 / 21 /
// 24, 117K 78 / 64 / 73, 1M 209 / 202 / -; a whole pass with eight shifts is
// slower than with one.  The SP sweep gains 2 us, and with library cells
// loses (300K gates 274 / 292): one shift there, and where several teams fill
// a CU's SIMDs (forward, 117K gates x 32 columns 114 / 146, 50K x 64 100 / 129).
constexpr int32_t kFlowShifts = 2;
static void flow_shape(FlowCtl *ctl, int64_t widest, int32_t C, int32_t shifts, unsigned *grid,
                       unsigned *threads) {
  const int64_t cus = std::max<int64_t>(1, ctl->n_cu / kFlowDies);
  const int64_t waves = std::max<int64_t>(1, (widest + 63) / 64);
  int64_t m = std::min(waves, cus);
  int64_t wpb = (waves + m - 1) / m;
  if (wpb > kFlowThreads / 64) {  // a second workgroup per CU
    wpb = kFlowThreads / 64;
    m = std::min((waves + wpb - 1) / wpb, 2 * cus);
  }
  const int64_t fit = std::max<int64_t>(1, cus * kFlowWavesPerCu / (m * wpb));
  const int64_t teams = std::min<int64_t>({fit, kFlowTeams, (C + kFlowDies - 1) / kFlowDies});
  // (with several teams a CU's SIMDs have a wave each already)
  if (m * wpb * shifts * teams > cus * kFlowWavesPerCu || (teams > 2 && m * wpb * teams > 3 * cus))
    shifts = 1;
  if (wpb * shifts <= kFlowThreads / 64) wpb *= shifts;
  else m *= shifts;
  ctl->shifts = shifts;
  ctl->expected = (uint32_t)m;
  *grid = (unsigned)(m * kFlowDies * teams);
  *threads = (unsigned)(64 * wpb);
  ctl->per_block = (int32_t)wpb;
}

static int64_t fill_blocks(int64_t slots, bool clears) {
  return (slots + (clears ? kFlowWords : 0) + kBlock * kArmPer - 1) / (kBlock * kArmPer);
}
uint32_t flow_arm_blocks(const SpFlow &t, bool clears) {
  return (uint32_t)fill_blocks((int64_t)t.g.G * t.B, clears);
}
uint32_t flow_arm_blocks(const BwdFlow &t, bool clears, uint32_t *arm_blocks,
                         uint32_t *seed_blocks) {
  *arm_blocks = (uint32_t)fill_blocks(t.n_edges * t.a.C, clears);
  *seed_blocks = blocks_for((int64_t)t.g.n_nets * t.a.C);
  return *arm_blocks + *seed_blocks + blocks_for((int64_t)t.g.G * t.a.B);
}

hipError_t launch_sp_arm(const SpFlow &t, FlowCtl ctl, hipStream_t s) {
  if (!ctl.words || !ctl.report || !flow_fits(t.g, t.depth, t.B, 0)) return hipErrorInvalidValue;
  k_flow_arm<<<flow_arm_blocks(t, true), kBlock, 0, s>>>(
      reinterpret_cast<uint32_t *>(t.sp + (int64_t)t.g.n_pi * t.B), (int64_t)t.g.G * t.B, ctl.words);
  return hipGetLastError();
}
hipError_t launch_sp_flow(const SpFlow &t, int64_t widest, bool cells, FlowCtl ctl, hipStream_t s) {
  if (t.depth <= 0 || t.B <= 0) return hipSuccess;
  hipError_t e = launch_sp_arm(t, ctl, s);
  if (e != hipSuccess) return e;
  unsigned grid, threads;
  flow_shape(&ctl, widest, t.B, cells ? 1 : kFlowShifts, &grid, &threads);
  if (cells)
    k_sp_flow<true><<<grid, threads, 0, s>>>(ctl, t);
  else
    k_sp_flow<false><<<grid, threads, 0, s>>>(ctl, t);
  return hipGetLastError();
}

hipError_t launch_bwd_flow(const BwdFlow &t, int64_t widest, bool cells, FlowCtl ctl,
                           hipStream_t s) {
  if (t.a.C <= 0 || t.g.n_nets <= 0) return hipSuccess;
  if (!ctl.words || !ctl.report || !t.seed || !t.part || !flow_fits(t.g, t.depth, t.a.C, t.n_edges))
    return hipErrorInvalidValue;
  uint32_t ab, sb;
  const uint32_t blocks = flow_arm_blocks(t, true, &ab, &sb);
  const bool sized = staged_sizes(t.a);
  const auto arm = cells ? (sized ? k_bwd_arm<true, true> : k_bwd_arm<true, false>)
                         : (sized ? k_bwd_arm<false, true> : k_bwd_arm<false, false>);
  hipLaunchKernelGGL(arm, dim3(blocks), dim3(kBlock), 0, s, t, ctl.words, ab, sb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  unsigned grid, threads;
  flow_shape(&ctl, widest, t.a.C, kFlowShifts, &grid, &threads);
  if (cells)
    k_bwd_flow<true><<<grid, threads, 0, s>>>(ctl, t);
  else
    k_bwd_flow<false><<<grid, threads, 0, s>>>(ctl, t);
  return hipGetLastError();
}

hipError_t launch_sp_flow_multi(const SpFlowSeg *segs, int32_t n_segs, int32_t jobs,
                                uint32_t blocks, int64_t widest, bool cells, FlowCtl ctl,
                                hipStream_t s) {
  if (n_segs <= 0 || jobs <= 0) return hipSuccess;
  if (!ctl.words || !ctl.report || jobs > kFlowMaxJobs || blocks == 0) return hipErrorInvalidValue;
  k_flow_arm_multi<<<blocks, kBlock, 0, s>>>(segs, n_segs, ctl.words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  unsigned grid, threads;
  flow_shape(&ctl, widest, jobs, cells ? 1 : kFlowShifts, &grid, &threads);
  if (cells)
    k_sp_flow_multi<true><<<grid, threads, 0, s>>>(ctl, segs, n_segs, jobs);
  else
    k_sp_flow_multi<false><<<grid, threads, 0, s>>>(ctl, segs, n_segs, jobs);
  return hipGetLastError();
}

hipError_t launch_bwd_flow_multi(const BwdFlowSeg *segs, int32_t n_segs, int32_t jobs,
                                 uint32_t blocks, int64_t widest, bool cells, FlowCtl ctl,
                                 hipStream_t s) {
  if (n_segs <= 0 || jobs <= 0) return hipSuccess;
  if (!ctl.words || !ctl.report || jobs > kFlowMaxJobs || blocks == 0) return hipErrorInvalidValue;
  const auto arm = cells ? (ctl.sized ? k_bwd_arm_multi<true, true> : k_bwd_arm_multi<true, false>)
                         : (ctl.sized ? k_bwd_arm_multi<false, true> : k_bwd_arm_multi<false, false>);
  hipLaunchKernelGGL(arm, dim3(blocks), dim3(kBlock), 0, s, segs, n_segs, ctl.words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  unsigned grid, threads;
  flow_shape(&ctl, widest, jobs, kFlowShifts, &grid, &threads);
  if (cells)
    k_bwd_flow_multi<true><<<grid, threads, 0, s>>>(ctl, segs, n_segs, jobs);
  else
    k_bwd_flow_multi<false><<<grid, threads, 0, s>>>(ctl, segs, n_segs, jobs);
  return hipGetLastError();
}

hipError_t launch_stim_words(const float *sp, const int32_t *stream, int32_t n_pi, int32_t B,
                             int64_t T, uint64_t seed, uint64_t *out, hipStream_t s) {
  if (n_pi <= 0 || B <= 0 || T <= 0) return hipSuccess;
  const int nc = B == 1 ? 1 : B == 2 ? 2 : B <= 4 ? 4 : 8;
  const int64_t tasks = (T + 63) / 64 * n_pi * ((B + nc - 1) / nc);
  const int64_t blocks = (tasks + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks > kMaxBlocks) return hipErrorInvalidValue;
  using K = void (*)(const float *, const int32_t *, int32_t, int32_t, int64_t, uint32_t, uint32_t,
                     uint64_t *);
  const K kern = nc == 1 ? k_stim_words<1> : nc == 2 ? k_stim_words<2>
                 : nc == 4 ? k_stim_words<4> : k_stim_words<8>;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kBlock), 0, s, sp, stream, n_pi, B, T,
                     (uint32_t)seed, (uint32_t)(seed >> 32), out);
  return hipGetLastError();
}

hipError_t launch_sim_flow(const SimFlow &t, const SpFlow &sp, int64_t widest, bool cells,
                           FlowCtl ctl, FlowCtl sp_ctl, uint32_t *ones, uint32_t *tog,
                           hipStream_t s) {
  const int64_t nb = (int64_t)t.g.n_nets * t.B;
  if (nb <= 0 || t.T <= 0) return hipSuccess;
  if (!ctl.words || !ctl.report || !sp_ctl.words || !sp_ctl.report ||
      !flow_fits(sp.g, sp.depth, sp.B, 0) || !sim_fits(t.g, t.depth, t.B, t.pitch, t.T) ||
      t.n_chunks != (t.T + t.pitch - 1) / t.pitch || t.n_bufs < 1 || t.n_bufs > kSimBufs)
    return hipErrorInvalidValue;
  k_fill_u32<<<blocks_for(kSimWords), kBlock, 0, s>>>(ctl.words, kSimWords, 0u);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t cus = std::min<int64_t>(kSimMembers, std::max<int64_t>(1, ctl.n_cu / kFlowDies));
  ctl.expected = (uint32_t)cus;
  const unsigned grid = (unsigned)(cus * kFlowDies * ((t.n_bufs + kFlowDies - 1) / kFlowDies));
  // the sweep's workgroups: one a CU at most, so that the tiles' teams fit beside
  unsigned sp_blocks = 0, sp_threads;
  const int64_t sweep_widest = std::min<int64_t>(widest, cus * kFlowThreads);
  const bool ride = sp.B <= kRideColumns;
  if (ride) flow_shape(&sp_ctl, sweep_widest, sp.B, cells ? 1 : kFlowShifts, &sp_blocks, &sp_threads);
  if (ride && (int64_t)sp_ctl.expected > cus)
    flow_shape(&sp_ctl, sweep_widest, sp.B, 1, &sp_blocks, &sp_threads);
  using K = void (*)(FlowCtl, SimFlow, FlowCtl, SpFlow, uint32_t);
  K kern = cells ? k_sim_flow<32, true> : k_sim_flow<32, false>;
  if (t.pitch == 16) kern = cells ? k_sim_flow<8, true> : k_sim_flow<8, false>;
  if (t.pitch == 32) kern = cells ? k_sim_flow<16, true> : k_sim_flow<16, false>;
  hipLaunchKernelGGL(kern, dim3(sp_blocks + grid), dim3(kFlowThreads), 0, s, ctl, t, sp_ctl, sp, sp_blocks);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_sim_counts<<<blocks_for(nb), kBlock, 0, s>>>(t, ctl.words + kSimStop, sp.sp, ones, tog);
  return hipGetLastError();
}

hipError_t launch_grad_export(const GradExportArgs &a, hipStream_t s) {
  if (a.dcap && a.n_nets > 0) {
    const unsigned blocks = (unsigned)((a.n_nets + kCapRows - 1) / kCapRows);
    const bool sized = a.size && !a.paired && a.S >= kStagedSizes;
    if (a.B < kCapRowsMinCols) {
      const auto kern = sized ? k_grad_cap_narrow<true> : k_grad_cap_narrow<false>;
      hipLaunchKernelGGL(kern, dim3(blocks_for(a.n_nets)), dim3(kBlock), 0, s, a);
    } else {
      const auto kern = a.beta ? (sized ? k_grad_cap<true, true> : k_grad_cap<true, false>)
                               : (sized ? k_grad_cap<false, true> : k_grad_cap<false, false>);
      hipLaunchKernelGGL(kern, dim3(blocks), dim3(kCapRows), 0, s, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.dsize && a.S > 0 && a.G > 0) {
    k_grad_size<<<blocks_for((int64_t)a.G * a.S), kBlock, 0, s>>>(a);
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace dp

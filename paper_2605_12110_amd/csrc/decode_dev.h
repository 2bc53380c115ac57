// Attention over the selected blocks, device side (Sec. 3.4, kernel 3; Eq. (1) restricted to the selection).
//
// A selected logical block j of KV head h covers tokens [j*B_h, (j+1)*B_h); token t sits in
// physical page page_table[b][t / P] at slot t % P.  The kernel walks the selection as a virtual
// token sequence (position -> block list entry -> token -> page/slot) and reads K and V rows in
// place: no gather, no per-head page list, any mix of block sizes in one launch.
//
// Split-K flash decoding in one kernel: work-group (split, segment) handles `split_tokens`
// consecutive positions of its segment's selection and produces an unnormalised partial (m, l, o~)
// for the G query heads of the group.  A segment with one split normalises and writes its output
// rows directly; otherwise the partial goes to the workspace, the work-group draws a ticket from
// the segment's counter, and the one that draws the last ticket merges the segment's partials with
// the log-sum-exp rule.  No work-group ever waits for another, so the grid drains whatever the
// counters hold; they must be zero at launch (the selection kernel of the fused step clears them,
// the stand-alone entry point runs a clearing kernel first).
//
// Data path of one wave step (16 rows), without LDS:
//   * K rows are loaded in the layout of the matrix operand itself: lane (token = lane % 16, group = lane / 16)
//     loads the 16-byte pieces 4c + group, c = 0..3, of its token's row (a contraction may take the channels in any
//     order that Q follows too);  S = K Q^T is four 16x16x32 products;
//   * V rows are loaded one row per instruction, a lane two channels, at scalar addresses; byte permutes put four
//     rows of a channel side by side, which is the operand of the 4x4x4 product of 16 blocks: 4 query heads x
//     64 channels per instruction, so O of four heads takes 8 registers a lane (16x16 tiles, mostly padding
//     at G <= 8 query rows, took 32);
//   * Q's columns are repeated over the tile (head = column % 4, or % 8 for G > 4), so the logits of every head
//     come out in all lanes, the softmax runs in place, and the weights only have to cross between the four
//     groups of 16 lanes (register swaps);
//   * K of the next step is requested once the S product has consumed this step's, V four rows at a time behind the
//     product that consumed them: a work-group has 32 KB of rows in flight nearly always, and with at most 128
//     registers a lane (114-122 in the stand-alone kernel) four work-groups fit a compute unit.
// The addresses of a wave's steps come from its lanes: lane j looks up the block and page of eight consecutive
// tokens (half j % 2 of step j / 2; B >= 8 and P >= 8, so they lie in one block and one page), for 32 steps at once.
#pragma once
#include <type_traits>

#include "common.h"

namespace absb {

struct DecodeParams {
  // (what a work-group reads first comes first: the arguments are a few cold lines of memory)
  int32_t sel_stride, split_tokens, max_splits;
  int32_t some_dense;   // LISTED: some budgets cover their context; nobody selects for those requests
  int32_t stream_rows;  // 1: V rows pass the caches by
  float scale_log2;     // sm_scale * log2(e)
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const int32_t* sel_idx;
  const int32_t* sel_cnt;
  float* part_o;   // [nseg][max_splits][G][128]
  float* part_ml;  // [nseg][max_splits][G][4]  (running max in log2 units, sum of the rounded weights, exact sum, -)
  int32_t* tickets;  // [nseg], zero when the kernel starts
  // one-launch step only: the list is produced by another work-group of the same launch
  const int32_t* budget;    // [Bt]
  const int32_t* cent_off;  // [nseg+1]
  int32_t* flags;    // [nseg] (ABSB_TICKET_STRIDE apart): non-zero once the segment's list is complete
  int32_t* status;   // one word: set non-zero when a wait ran into its time limit
  void* out;       // [Bt][Hq][128]
  float* lse;      // [Bt][Hq] or null
  Geometry g;
};

inline DecodeParams make_decode_params(const Geometry& g, const Plan& pl, float sm_scale, const void* q,
                                       const void* k_cache, const void* v_cache, const int32_t* page_table,
                                       const int32_t* seq_lens, const int32_t* sel_idx, const int32_t* sel_cnt,
                                       int32_t sel_stride, void* out, float* lse, char* ws) {
  DecodeParams p;
  p.q = static_cast<const uint16_t*>(q);
  p.k = static_cast<const uint16_t*>(k_cache);
  p.v = static_cast<const uint16_t*>(v_cache);
  p.page_table = page_table;
  p.seq_lens = seq_lens;
  p.sel_idx = sel_idx;
  p.sel_cnt = sel_cnt;
  p.part_o = reinterpret_cast<float*>(ws + pl.ws_part_o);
  p.part_ml = reinterpret_cast<float*>(ws + pl.ws_part_ml);
  p.tickets = reinterpret_cast<int32_t*>(ws + pl.ws_tickets);
  p.budget = nullptr;
  p.cent_off = nullptr;
  p.flags = nullptr;
  p.status = nullptr;
  p.out = out;
  p.lse = lse;
  p.sel_stride = sel_stride;
  p.split_tokens = pl.split_tokens;
  p.max_splits = pl.max_splits;
  p.some_dense = 0;
  p.stream_rows = pl.stream_rows;
  p.scale_log2 = sm_scale * 1.4426950408889634f;
  p.g = g;
  return p;
}

constexpr float M_INIT = -1.0e30f;  // finite stand-in for "no token seen yet"
constexpr int DEC_THREADS = 256;
constexpr int DEC_WAVES = DEC_THREADS / 64;
constexpr int ROWS_PER_WAVE_STEP = 16;        // two halves of eight consecutive rows
constexpr int DEC_STEP = DEC_WAVES * ROWS_PER_WAVE_STEP;  // positions per work-group step
constexpr int MRG_UNROLL = 8;                 // splits a thread merges per memory round trip (half as many for few splits)
// LDS of one work-group, all of it for the epilogue: the waves' outputs, per-wave maxima and the two sums per
// head, two words for work-group broadcasts
constexpr int DEC_LDS_STATE = DEC_WAVES * ABSB_MAX_GROUP * ABSB_HEAD_DIM * 4;
constexpr int DEC_LDS_ML = 8 * DEC_THREADS * 4;  // of the merge: behind what its split lanes are folded in
static_assert(DEC_LDS_ML + DEC_THREADS * 16 <= DEC_LDS_STATE, "epilogue LDS");
constexpr int DEC_LDS_BYTES = DEC_LDS_STATE + 3 * ABSB_MAX_GROUP * DEC_WAVES * 4 + 16;
// a work-group that waits for its segment's list gives up after this long (100 MHz ticks): the
// wait cannot outlast the launch whatever the rest of the grid does
constexpr uint64_t DEC_WAIT_LIMIT_TICKS = 25u * 1000u * 1000u;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// D(16x16) += A(16x32) B(32x16), operands as eight 16-bit values per lane:
// A[m = lane%16][k = 8*(lane/16)+i], B[k = 8*(lane/16)+i][n = lane%16], D[m = 4*(lane/16)+i][n = lane%16].
template <int DT>
__device__ __forceinline__ float4_t mma_16x16x32(u32x4 a, u32x4 b, float4_t c) {
  if (DT == ABSB_F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8_t>(a), bitcast<half8_t>(b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(bitcast<bf16x8_t>(a), bitcast<bf16x8_t>(b), c, 0, 0, 0);
}
// 16 independent D(4x4) += A(4x4) B(4x4), one per block of four lanes, operands as four 16-bit values per lane:
// A[m = lane%4][k = i], B[k = i][n = lane%4], D[m = i][n = lane%4].
template <int DT>
__device__ __forceinline__ float4_t mma_4x4x4(u32x2 a, u32x2 b, float4_t c) {
  if (DT == ABSB_F16) return __builtin_amdgcn_mfma_f32_4x4x4f16(bitcast<half4_t>(a), bitcast<half4_t>(b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(bitcast<short4_t>(a), bitcast<short4_t>(b), c, 0, 0, 0);
}

// Exchanges between the four rows of 16 lanes by register swaps (no LDS crossbar round trip).
// The value of row `t` in every row, t = 0..3.
struct RowsOf {
  uint32_t of[4];
};
__device__ __forceinline__ RowsOf spread_rows(uint32_t x) {
  const auto h = __builtin_amdgcn_permlane16_swap(x, x, false, false);        // rows (0, 0, 2, 2) and (1, 1, 3, 3)
  const auto e = __builtin_amdgcn_permlane32_swap(h[0], h[0], false, false);  // rows (0, 0, 0, 0) and (2, 2, 2, 2)
  const auto o = __builtin_amdgcn_permlane32_swap(h[1], h[1], false, false);
  return RowsOf{{e[0], o[0], e[1], o[1]}};
}
template <typename Op>
__device__ __forceinline__ float across_rows(float x, Op op) {
  const auto h = __builtin_amdgcn_permlane16_swap(bitcast<uint32_t>(x), bitcast<uint32_t>(x), false, false);
  const float y = op(bitcast<float>(h[0]), bitcast<float>(h[1]));
  const auto e = __builtin_amdgcn_permlane32_swap(bitcast<uint32_t>(y), bitcast<uint32_t>(y), false, false);
  return op(bitcast<float>(e[0]), bitcast<float>(e[1]));
}
struct FAdd {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct FMax {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};

// Where the attention loop takes a segment's block list from.
enum : int {
  LIST_PLAIN = 0,     // device memory, complete before the launch
  LIST_COHERENT = 1,  // device memory, written by another work-group of this launch: device-coherent loads
  LIST_LOCAL = 2      // this work-group's LDS
};

// A block list: entry i is a block index of the segment (i itself where there is no list: everything is
// selected).  Indices beyond `last` read entry `last`
// (the loop prefetches ahead of the range it works on; the clamp keeps every read inside the storage).
template <int SRC>
struct ListRef {
  const int32_t* ptr;
  int last;
  __device__ __forceinline__ int at(int i) const {
    i = min(i, last);
    if (SRC != LIST_LOCAL && !ptr) return i;
    if (SRC == LIST_COHERENT) return ld_i32<true>(ptr + i);
    return ptr[i];
  }
};

// Entries [first, last] of a list, the work-group's LDS holding those; later ones read the last.
struct StretchRef {
  const int32_t* ptr;
  int first, last;
  __device__ __forceinline__ int at(int i) const { return ptr[min(i, last) - first]; }
};

// Query heads are taken in sets of four (the rows of a 4x4x4 product).
constexpr int head_sets(int G) { return (G + 3) / 4; }

// Running state of the online softmax of one wave.  Lane l works for head l % 4 (l % 8 with two sets): the running
// maximum, common to the wave's four row groups; partial sums over the group's rows of the weights as rounded
// for the P V product (the output's normaliser: the output stays a convex combination of value rows) and of the
// weights before rounding (the log-sum-exp: rounding to bf16 would bias it by up to 2^-8 when all weights
// round the same way); o[set][j][i] = O[head 4*set + i][channel 2*l + j].
template <int G>
struct AttnState {
  float m, l, lx;
  float4_t o[head_sets(G)][2];
  __device__ __forceinline__ void reset() {
    m = M_INIT;
    l = 0.0f;
    lx = 0.0f;
#pragma unroll
    for (int s = 0; s < head_sets(G); ++s) o[s][0] = o[s][1] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
  }
};

// What a work-group needs to know about its segment.
struct SplitCtx {
  int b, hs, hk, lb, L, lP;
};

// Q (the group's rows, from the first head's on) as the B operand of S = K Q^T: lane (column = lane % 16, group) holds the 16-byte pieces 4c + group of its head's
// row; columns repeat the heads, and heads beyond G are zero.
template <int G>
__device__ __forceinline__ void load_q(const uint16_t* rows, u32x4 (&qb)[4]) {
  const int lane = threadIdx.x & 63, grp = lane >> 4, head = lane & (4 * head_sets(G) - 1);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    qb[c] = u32x4{0u, 0u, 0u, 0u};
    if (head < G)
      qb[c] = *reinterpret_cast<const u32x4*>(rows + head * ABSB_HEAD_DIM + (4 * c + grp) * 8);
  }
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32);
}

// Attention of this wave over positions [pos_begin, pos_end) of the virtual token sequence of a block
// list (position -> list entry pos >> lb -> token -> page/slot), folded into `st`.  A work-group step
// covers DEC_STEP consecutive positions, 16 per wave; pos_begin must be a multiple of eight.
// `pages`: the request's row of the page table.
template <int DT, int G, bool STREAM, class List>
__device__ __forceinline__ void attend_rows(const DecodeParams& p, const SplitCtx& c, const List& list, const int32_t* pages,
                                            int pos_begin, int pos_end, const u32x4 (&qb)[4], AttnState<G>& st) {
  constexpr int SETS = head_sets(G);
  const int tid = threadIdx.x, lane = tid & 63, grp = lane >> 4, li = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lb = c.lb, L = c.L, lP = c.lP;
  const int wave_pos = pos_begin + wave * ROWS_PER_WAVE_STEP;
  const int nsteps = pos_end > wave_pos ? (pos_end - wave_pos + DEC_STEP - 1) / DEC_STEP : 0;
  const size_t head_off = (size_t)c.hk * p.g.s_head * 2;
  const char* kbase = reinterpret_cast<const char*>(p.k) + head_off + grp * 16;
  const char* vbase = reinterpret_cast<const char*>(p.v) + head_off;
  const uint32_t lane4 = lane * 4;
  const uint64_t pitch = (uint64_t)p.g.s_tok * 2;  // (any stride that fits the card: eight rows can span more than 4 GB)

  // ---- lane j: half j % 2 of step j / 2 of the current 32 steps.  `off`: byte offset of its first row (of a
  // legal token, whatever the list holds), `most`: which of its eight rows is the last that exists; `nv`: how
  // many of them count
  uint64_t off = 0;
  int most = 0, nv = 0;
  auto look_up = [&](int step0) __attribute__((always_inline)) {
    const int pos8 = wave_pos + (step0 + (lane >> 1)) * DEC_STEP + (lane & 1) * 8;
    const int t8 = (list.at(pos8 >> lb) << lb) + (pos8 & ((1 << lb) - 1));
    const int tc = max(0, min(t8, L - 1)) & ~7;
    off = ((uint64_t)pages[tc >> lP] * (uint64_t)p.g.s_page + (uint64_t)(tc & ((1 << lP) - 1)) * (uint64_t)p.g.s_tok) * 2;
    nv = min(8, min(pos_end - pos8, L - t8));
    most = nv > 0 ? min(7, L - 1 - tc) : 0;  // rows nobody needs: one line, not eight
  };
  u32x4 k[4];
  uint32_t v[16];
  int nv0 = 0, nv1 = 0;      // rows of the two halves that count, of the step being computed
  // of row `li` of the step whose rows are being requested, for V read back lane by lane (a 64-bit product per row
  // on the scalar unit: 43.4 -> 43.6 us a step on 16 x 8K-128K)
  uint64_t row_off = 0;
  auto issue_k = [&](int j) __attribute__((always_inline)) {  // j: even lane of the step's pair
    const uint64_t o0 = readlane_u64(off, j), o1 = readlane_u64(off, j + 1);
    const uint32_t m0 = (uint32_t)__builtin_amdgcn_readlane(most, j), m1 = (uint32_t)__builtin_amdgcn_readlane(most, j + 1);
    row_off = (li < 8 ? o0 : o1) + min((uint32_t)(li & 7), li < 8 ? m0 : m1) * pitch;
    const char* row = kbase + row_off;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4* piece = reinterpret_cast<const u32x4*>(row + 64 * i);
      k[i] = *piece;  // cached even when V passes by: half a line a token, the other half is the next piece's
    }
  };
  auto issue_v = [&](int t) __attribute__((always_inline)) {  // rows 4t .. 4t+3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* row = vbase + readlane_u64(row_off, 4 * t + i);  // a scalar
      const uint32_t* pair = reinterpret_cast<const uint32_t*>(row + lane4);
      v[4 * t + i] = STREAM ? __builtin_nontemporal_load(pair) : *pair;
    }
  };

  look_up(0);
  if (nsteps > 0) {
    issue_k(0);
    __builtin_amdgcn_sched_barrier(0);  // rows arrive in the order they are asked for: K first
#pragma unroll
    for (int t = 0; t < 4; ++t) issue_v(t);
  }
  float m = st.m, l = st.l, lx = st.lx;
  // One step from the rows in registers; MORE: the next step's rows are requested as registers come free.  (The last
  // step is a copy of its own: requests under a condition would be copied into place, after a wait for them.)
  auto compute = [&](int step, auto more) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(more)::value;
    const int j = 2 * (step & 31);
    nv0 = __builtin_amdgcn_readlane(nv, j);
    nv1 = __builtin_amdgcn_readlane(nv, j + 1);
    // ---- S[row][head] = K Q^T over the 128 channels (two accumulators: shorter dependent chain)
    float4_t s0 = {0.0f, 0.0f, 0.0f, 0.0f}, s1 = {0.0f, 0.0f, 0.0f, 0.0f};
    s0 = mma_16x16x32<DT>(k[0], qb[0], s0);
    s1 = mma_16x16x32<DT>(k[1], qb[1], s1);
    s0 = mma_16x16x32<DT>(k[2], qb[2], s0);
    s1 = mma_16x16x32<DT>(k[3], qb[3], s1);
    if (MORE) {
      if (j == 62) look_up(step + 1);
      issue_k(2 * ((step + 1) & 31));
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- online softmax in place: this lane holds rows 4*grp..4*grp+3 of its head
    float sc[4];
    const int live_rows = (grp < 2 ? nv0 : nv1) - 4 * (grp & 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[i] = i < live_rows ? (s0[i] + s1[i]) * p.scale_log2 : -__builtin_inff();
    const float mx = across_rows(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), FMax());
    const float mn = fmaxf(m, mx);
    const float alpha = fast_exp2(m - mn);
    m = mn;
    uint32_t pb[4];
    float psum = 0.0f, esum = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = fast_exp2(sc[i] - mn);
      const uint16_t ph = Elem<DT>::narrow(e);  // the weight as the product will see it
      psum += Elem<DT>::widen(ph);
      esum += e;
      pb[i] = ph;
    }
    l = __builtin_fmaf(l, alpha, psum);
    lx = __builtin_fmaf(lx, alpha, esum);
    // ---- rescale O when some head's maximum moved (rare once the maxima have settled)
    if (__any(alpha != 1.0f)) {
#pragma unroll
      for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = bitcast<float>(__builtin_amdgcn_readlane(bitcast<int>(alpha), 4 * s + i));
          st.o[s][0][i] *= a;
          st.o[s][1][i] *= a;
        }
    }
    // ---- the weights of rows 4t..4t+3 (group t's) for head 4*set + lane % 4, in every lane
    uint32_t w[SETS][2];
    const uint32_t own[2] = {pb[0] | (pb[1] << 16), pb[2] | (pb[3] << 16)};
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      if (SETS == 1) {
        w[0][x] = own[x];
      } else {  // lanes l and l ^ 4 hold heads l % 8 and (l ^ 4) % 8: each needs both
        const uint32_t other = (uint32_t)dpp_i<0x1B>(dpp_i<DPP_ROW_HALF_MIRROR>((int)own[x]));  // quad_perm [3,2,1,0]
        w[0][x] = (lane & 4) ? other : own[x];
        w[SETS - 1][x] = (lane & 4) ? own[x] : other;
      }
    }
    RowsOf wt[SETS][2];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x) wt[s][x] = spread_rows(w[s][x]);
    // ---- O[head][channel] += P V, four rows at a time: four rows of a channel side by side in two registers
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x2 ev = {__builtin_amdgcn_perm(v[4 * t + 1], v[4 * t], 0x05040100u),       // low halves: channel 2l
                        __builtin_amdgcn_perm(v[4 * t + 3], v[4 * t + 2], 0x05040100u)};
      const u32x2 od = {__builtin_amdgcn_perm(v[4 * t + 1], v[4 * t], 0x07060302u),       // high halves: channel 2l + 1
                        __builtin_amdgcn_perm(v[4 * t + 3], v[4 * t + 2], 0x07060302u)};
      if (MORE) issue_v(t);
#pragma unroll
      for (int s = 0; s < SETS; ++s) {
        const u32x2 a = {wt[s][0].of[t], wt[s][1].of[t]};
        st.o[s][0] = mma_4x4x4<DT>(a, ev, st.o[s][0]);
        st.o[s][1] = mma_4x4x4<DT>(a, od, st.o[s][1]);
      }
    }
  };
  // trip counts depend on the wave only: every branch here is wave-uniform
  for (int step = 0; step + 1 < nsteps; ++step) compute(step, std::true_type());
  if (nsteps > 0) compute(nsteps - 1, std::false_type());
  st.m = m;
  st.l = l;
  st.lx = lx;
}

template <int DT, int G, class List>
__device__ __forceinline__ void attend_positions(const DecodeParams& p, const SplitCtx& c, const List& list, const int32_t* pages,
                                                 int pos_begin, int pos_end, const u32x4 (&qb)[4], AttnState<G>& st) {
  if (p.stream_rows)
    attend_rows<DT, G, true>(p, c, list, pages, pos_begin, pos_end, qb, st);
  else
    attend_rows<DT, G, false>(p, c, list, pages, pos_begin, pos_end, qb, st);
}

// An empty selection: the output rows are zero, the log-sum-exp -inf.
template <int G>
__device__ __forceinline__ void write_empty_rows(const DecodeParams& p, int b, int hs) {
  for (int i = threadIdx.x; i < G * ABSB_HEAD_DIM; i += DEC_THREADS) {
    const size_t row = (size_t)b * p.g.Hq + (size_t)hs * G + (i >> 7);
    static_cast<uint16_t*>(p.out)[row * ABSB_HEAD_DIM + (i & 127)] = 0;
    if (p.lse && (i & 127) == 0) p.lse[row] = -__builtin_inff();
  }
}

// A wait ran out: the segment's output cannot be completed (one split's ticket is missing for good, so nobody merges).  Its rows
// are set to NaN so that nobody takes stale values for results, by every work-group whose wait did: others of the segment may
// have come just in time, or have seen a count on its way past the one they wait for.
template <int DT, int G>
__device__ __forceinline__ void poison_rows(const DecodeParams& p, int b, int hs) {
  const uint16_t nan16 = DT == ABSB_F16 ? (uint16_t)0x7e00 : (uint16_t)0x7fc0;
  for (int i = threadIdx.x; i < G * ABSB_HEAD_DIM; i += DEC_THREADS) {
    const size_t row = (size_t)b * p.g.Hq + (size_t)hs * G + (i >> 7);
    static_cast<uint16_t*>(p.out)[row * ABSB_HEAD_DIM + (i & 127)] = nan16;
    if (p.lse && (i & 127) == 0) p.lse[row] = __builtin_nanf("");
  }
}

// The end of a work-group's attention: the four wave states are folded into the work-group's partial;
// with one split per segment it is normalised and written out; otherwise it goes to slot `split` of
// the segment's partials, the work-group draws a ticket, and the one that draws ticket nsplit - 1
// merges the segment's `nsplit` partials with the log-sum-exp rule and writes the output rows.
// `slots`: partial slots per segment (the stride of the partial arrays).  `on_last`: called by every thread
// of the segment's last work-group (the merging one, or the only one) ahead of the merge, for words of the segment
// that have to go back to zero: every other work-group of the segment has drawn its ticket by then.  Every
// thread of the work-group must call; returns (to all of them) whether this was the segment's last one.
template <int DT, int G, class OnLast>
__device__ __forceinline__ bool finish_split(const DecodeParams& p, int s, int b, int hs, int split, int nsplit, int slots,
                                             AttnState<G>& st, char* lds, OnLast&& on_last) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  char* s_stage = lds;
  float (*s_m)[DEC_WAVES] = reinterpret_cast<float (*)[DEC_WAVES]>(lds + DEC_LDS_STATE);
  float (*s_l)[DEC_WAVES] = s_m + ABSB_MAX_GROUP;
  float (*s_lx)[DEC_WAVES] = s_l + ABSB_MAX_GROUP;
  int* s_bcast = reinterpret_cast<int*>(lds + DEC_LDS_STATE + 3 * ABSB_MAX_GROUP * DEC_WAVES * 4);
  float m = st.m, l = st.l, lx = st.lx;

  // ---- the wave's state: m per head (lane = head), l summed over the four groups.  (The addresses that the hand-over below
  // needs are asked for here, to arrive with the barrier: behind it they would be two more round trips.)
  uint64_t at_o = addr(p.part_o), at_ml = addr(p.part_ml), at_tickets = addr(p.tickets);
  l = across_rows(l, FAdd());
  lx = across_rows(lx, FAdd());
  constexpr int HEADS = 4 * head_sets(G);
  if (lane < HEADS) s_m[lane][wave] = m;
  asm volatile("" : "+s"(at_o), "+s"(at_ml), "+s"(at_tickets));
  __syncthreads();
  // work-group maximum per head; own state rescaled to it, so that the four states simply add up.  (Every lane works out its
  // head's factor, and all read it from there.  A read of LDS per head, behind the writes of the one before, and addresses
  // fetched where they are used took longer: 1 x 4K 9.4 -> 9.1 us a step, 8 x 32K 20.5 -> 20.3, a step of a decode loop over 4
  // requests 15.3 -> 14.9; three copies of a layer in turn.)
  float* s_o = reinterpret_cast<float*>(s_stage);  // [DEC_WAVES][G][128]
  const float4_t ms = *reinterpret_cast<const float4_t*>(s_m[lane & (HEADS - 1)]);
  const float rescale = fast_exp2(m - fmaxf(fmaxf(ms[0], ms[1]), fmaxf(ms[2], ms[3])));
  if (lane < G) {
    s_l[lane][wave] = l * rescale;
    s_lx[lane][wave] = lx * rescale;
  }
#pragma unroll
  for (int hd = 0; hd < G; ++hd) {
    const float a = bitcast<float>(__builtin_amdgcn_readlane(bitcast<int>(rescale), hd));
    *reinterpret_cast<float2*>(s_o + ((size_t)wave * G + hd) * ABSB_HEAD_DIM + lane * 2) =
        make_float2(st.o[hd >> 2][0][hd & 3] * a, st.o[hd >> 2][1][hd & 3] * a);
  }
  __syncthreads();
  // ---- the work-group's partial: thread -> column (head g, channels 4*c4..4*c4+3), G*32 columns
  constexpr int NCOL = G * 32;
  constexpr int CP = NCOL <= 32 ? 32 : NCOL <= 64 ? 64 : NCOL <= 128 ? 128 : 256;  // columns, padded to 2^k
  constexpr int SL = DEC_THREADS / CP;                                             // split lanes per column
  const int col = tid & (CP - 1), sl = tid / CP;
  const int g = min(col, NCOL - 1) >> 5, c4 = col & 31;
  float4_t O = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int w = 0; w < DEC_WAVES; ++w)
    O += *reinterpret_cast<const float4_t*>(s_o + ((size_t)w * G + g) * ABSB_HEAD_DIM + c4 * 4);
  float M = fmaxf(fmaxf(s_m[g][0], s_m[g][1]), fmaxf(s_m[g][2], s_m[g][3]));
  float Lsum = (s_l[g][0] + s_l[g][1]) + (s_l[g][2] + s_l[g][3]);
  float Lx = (s_lx[g][0] + s_lx[g][1]) + (s_lx[g][2] + s_lx[g][3]);

  if (nsplit > 1) {
    // Publish the partial, take a ticket; the work-group that draws the segment's last ticket merges.
    // Visibility across the chip's L2 slices without a cache write-back: partials are written and
    // read with device-coherent accesses (the sc1 cache policy, which the non-coherent cache levels
    // do not serve), a writer waits for its stores to be acknowledged before it draws its ticket,
    // and the merging group issues its reads only after its ticket has come back.  Nobody waits
    // for anybody.
    constexpr int COHERENT = 16;  // cache-policy operand of the buffer instructions: sc1
    const size_t slot0 = (size_t)s * slots;
    const __amdgpu_buffer_rsrc_t part_o = __builtin_amdgcn_make_buffer_rsrc(
        from_addr<float>(at_o) + slot0 * G * ABSB_HEAD_DIM, 0, slots * G * ABSB_HEAD_DIM * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t part_ml =
        __builtin_amdgcn_make_buffer_rsrc(from_addr<float>(at_ml) + slot0 * G * 4, 0, slots * G * 16, 0x00020000);
    if (tid < NCOL) {
      __builtin_amdgcn_raw_buffer_store_b128(bitcast<u32x4>(O), part_o, ((split * G + g) * ABSB_HEAD_DIM + c4 * 4) * 4,
                                             0, COHERENT);
      if (c4 == 0)
        __builtin_amdgcn_raw_buffer_store_b128(bitcast<u32x4>(float4_t{M, Lsum, Lx, 0.0f}), part_ml,
                                               (split * G + g) * 16, 0, COHERENT);
    }
    int32_t* ticket = from_addr<int32_t>(at_tickets) + (size_t)s * ABSB_TICKET_STRIDE;
    int& s_last = s_bcast[0];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's stores have been acknowledged
    __syncthreads();                                   // ... and so have everybody's
    if (tid == 0)
      s_last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nsplit - 1;
    __syncthreads();
    if (!s_last) return false;
    // every counter a launch touches is back at zero when the launch ends
    if (tid == 0)
      __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    on_last();

    // log-sum-exp merge: split lane `sl` of a column takes splits sl, sl + SL, ..., U of them per memory round trip,
    // folded into a running (M, Lsum, O).  What bounds it is how fast one compute unit pulls lines that no cache holds: the
    // maxima and sums, which all columns of a head need, are fetched once, by a thread per split and head, and handed
    // round in LDS.  (Fetched by every thread, in half of the load instructions: 32 splits of four heads, 1 x 128K,
    // 16.5 -> 16.1 us a step; 16 x 8K-128K 42.7 -> 42.0.  With U = 16, one trip for 32 splits, 16.1 and 42.1.)
    M = M_INIT;
    Lsum = 0.0f;
    Lx = 0.0f;
    O = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float4_t* s_ml = reinterpret_cast<float4_t*>(s_stage + DEC_LDS_ML);  // [SL * U][G]
    auto merge = [&](auto unroll) __attribute__((always_inline)) {
      constexpr int U = decltype(unroll)::value;
      static_assert(SL * U * G <= DEC_THREADS, "a thread per split and head of a trip");
      for (int i0 = 0; i0 < nsplit; i0 += SL * U) {
        float4_t ml = {-__builtin_inff(), 0.0f, 0.0f, 0.0f};  // of no split: weight 0, beside M_INIT too
        if (tid < SL * U * G && i0 * G + tid < nsplit * G)
          ml = bitcast<float4_t>(__builtin_amdgcn_raw_buffer_load_b128(part_ml, (i0 * G + tid) * 16, 0, COHERENT));
        float4_t ov[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = min(i0 + sl + u * SL, nsplit - 1);
          ov[u] = bitcast<float4_t>(
              __builtin_amdgcn_raw_buffer_load_b128(part_o, ((i * G + g) * ABSB_HEAD_DIM + c4 * 4) * 4, 0, COHERENT));
        }
        if (i0) __syncthreads();  // the trip before has been read
        if (tid < SL * U * G) s_ml[tid] = ml;
        __syncthreads();
        float bm = M;
#pragma unroll
        for (int u = 0; u < U; ++u) bm = fmaxf(bm, s_ml[(sl + u * SL) * G + g].x);
        const float a = fast_exp2(M - bm);
        O *= a;
        Lsum *= a;
        Lx *= a;
        M = bm;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float4_t mlu = s_ml[(sl + u * SL) * G + g];
          const float w = fast_exp2(mlu.x - bm);
          O += ov[u] * w;
          Lsum = __builtin_fmaf(mlu.y, w, Lsum);
          Lx = __builtin_fmaf(mlu.z, w, Lx);
        }
      }
    };
    if (nsplit <= SL * (MRG_UNROLL / 2))
      merge(std::integral_constant<int, MRG_UNROLL / 2>());
    else
      merge(std::integral_constant<int, MRG_UNROLL>());
    if (SL > 1) {  // fold the split lanes of a column (the staging area is free again)
      float* s_red = reinterpret_cast<float*>(s_stage);  // [SL][CP][8] (at most 8 KB)
      __syncthreads();
      float* mine = s_red + ((size_t)sl * CP + col) * 8;
      *reinterpret_cast<float4_t*>(mine) = float4_t{M, Lsum, Lx, 0.0f};
      *reinterpret_cast<float4_t*>(mine + 4) = O;
      __syncthreads();
      if (sl == 0) {
        float bm = M;
#pragma unroll
        for (int k = 1; k < SL; ++k) bm = fmaxf(bm, s_red[((size_t)k * CP + col) * 8]);
        const float a = fast_exp2(M - bm);
        O *= a;
        Lsum *= a;
        Lx *= a;
        M = bm;
#pragma unroll
        for (int k = 1; k < SL; ++k) {
          const float* sr = s_red + ((size_t)k * CP + col) * 8;
          const float w = fast_exp2(sr[0] - bm);
          Lsum = __builtin_fmaf(sr[1], w, Lsum);
          Lx = __builtin_fmaf(sr[2], w, Lx);
#pragma unroll
          for (int j = 0; j < 4; ++j) O[j] = __builtin_fmaf(sr[4 + j], w, O[j]);
        }
      }
    }
  }

  if (nsplit <= 1) on_last();

  // ---- normalise and write the group's output rows
  if (tid < NCOL) {
    const size_t row = (size_t)b * p.g.Hq + (size_t)hs * G + g;
    const bool any = Lsum > 0.0f;
    const float inv = any ? 1.0f / Lsum : 0.0f;
    const uint32_t lo = (uint32_t)Elem<DT>::narrow(O[0] * inv) | ((uint32_t)Elem<DT>::narrow(O[1] * inv) << 16);
    const uint32_t hi = (uint32_t)Elem<DT>::narrow(O[2] * inv) | ((uint32_t)Elem<DT>::narrow(O[3] * inv) << 16);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + row * ABSB_HEAD_DIM + c4 * 4) = make_uint2(lo, hi);
    if (p.lse && c4 == 0) p.lse[row] = any ? (M + __builtin_log2f(Lx)) * 0.6931471805599453f : -__builtin_inff();
  }
  return true;
}

// Waits (thread 0, bounded in time) until the 32-bit word at `flag` is non-zero; every thread of the
// work-group returns the value seen (0: the wait ran into its limit; *status is then set).  Two
// barriers inside.  `s_word`: one word of LDS.
__device__ __forceinline__ int wait_for_flag(const int32_t* flag, int32_t* status, int* s_word) {
  if (threadIdx.x == 0) {
    int v = ld_i32<true>(flag);
    if (!v) {
      const uint64_t t0 = wall_clock64();
      do {
        __builtin_amdgcn_s_sleep(8);
        v = ld_i32<true>(flag);
      } while (!v && wall_clock64() - t0 < DEC_WAIT_LIMIT_TICKS);
    }
    if (!v) st_i32<true>(status, 1);
    *s_word = v;
  }
  __syncthreads();
  const int v = *s_word;
  __syncthreads();  // the word may be reused
  return v;
}

// Partial (and, for the last arriver, merged) attention of split `split` of segment s by one
// work-group of DEC_THREADS threads.  LISTED == false: the block list was complete before the
// launch.  LISTED == true (the pipelined one-launch step): the list is being produced by another work-group of
// this launch with a lower index; its length K_s is recomputed here from the budget, the
// work-group waits (bounded) for the segment's flag before it reads the list with device-coherent
// loads, and the segment's last work-group clears the flag again; a wait that ran out leaves NaN in
// the segment's rows.  `lds`: DEC_LDS_BYTES.
template <int DT, int G, bool LISTED>
__device__ __forceinline__ void decode_split(const DecodeParams& p, int s, int split, char* lds) {
  // s is a SELECTION segment: its G (= the template's) query heads start at head hs * G; hk is the
  // KV head whose rows they read
  const SegMap sm = seg_map(s, p.g.Hsel, p.g.Rk, p.g.Hkv);
  const int b = sm.b, hs = sm.hs, hk = sm.hk;
  const int lb = p.g.heads.log2_block(hk);
  constexpr int SRC = LISTED ? LIST_COHERENT : LIST_PLAIN;
  const int pos_begin = split * p.split_tokens;

  // never beyond what the launch covers (a list longer than promised is cut, not overrun)
  int nsel;
  bool listed = LISTED || p.sel_cnt;  // false: everything is selected, there is no list
  if (LISTED || !p.sel_cnt) {
    const int rows = p.cent_off[sm.s + 1] - p.cent_off[sm.s];
    nsel = blocks_in_use(p.g.tight, rows, p.seq_lens, b, lb);
    if (LISTED) {
      const int T = p.budget[b];
      if (p.some_dense && T >= p.seq_lens[b]) listed = false;
      nsel = budget_blocks(T, lb, nsel, p.sel_stride);
    }
  } else {
    nsel = p.sel_cnt[s];
  }
  const ListRef<SRC> list{listed ? p.sel_idx + (size_t)s * p.sel_stride : nullptr, (listed ? p.sel_stride : max(nsel, 1)) - 1};
  const int ntok = min(nsel << lb, p.max_splits * p.split_tokens);
  if (ntok == 0 && split == 0) write_empty_rows<G>(p, b, hs);
  if (pos_begin >= ntok) return;
  const int pos_end = min(ntok, pos_begin + p.split_tokens);

  SplitCtx c;
  c.b = b;
  c.hs = hs;
  c.hk = hk;
  c.lb = lb;
  c.L = p.seq_lens[b];
  c.lP = p.g.log2_page;
  const int32_t* pages = p.page_table + (size_t)b * p.g.pt_stride;
  int* s_bcast = reinterpret_cast<int*>(lds + DEC_LDS_STATE + 3 * ABSB_MAX_GROUP * DEC_WAVES * 4);
  const int nsplit = (ntok + p.split_tokens - 1) / p.split_tokens;

  u32x4 qb[4];
  load_q<G>(p.q + ((size_t)b * p.g.Hq + (size_t)hs * G) * ABSB_HEAD_DIM, qb);

  int32_t* flag = LISTED ? p.flags + (size_t)s * ABSB_TICKET_STRIDE : nullptr;
  if (LISTED && listed) {
    // The list comes from a work-group with a lower index, which never waits for anything and was
    // dispatched before this one: the wait ends.  The time limit only makes that unconditional.
    if (!wait_for_flag(flag, p.status, s_bcast + 1)) {
      poison_rows<DT, G>(p, b, hs);  // nobody will complete this segment's rows
      return;
    }
  }

  AttnState<G> st;
  st.reset();
  attend_positions<DT, G>(p, c, list, pages, pos_begin, pos_end, qb, st);
  finish_split<DT, G>(p, s, b, hs, split, nsplit, p.max_splits, st, lds, [&]() {
    if (LISTED && listed && threadIdx.x == 0) st_i32<true>(flag, 0);  // every reader of the list has drawn its ticket
  });
}

// Attention work-group `id`: a selection segment (nseg or beyond: none) and which of its splits it does.  Segment by
// segment; but the Rk segments that read one KV head's rows do a split one after the other on the same die (work-groups
// go to the eight dies in turn), whose L2 then has the rows that their lists have in common: a selection per query head,
// 8 x 32K: 43.5 -> 39.0 us a step, 8 x 4000 20.8 -> 17.0, 1 x 128K 21.9 -> 21.9.  (The estimation work-groups in that
// order, too: 38.9, 17.1, but 23.9.)
__device__ __forceinline__ int segment_split(int id, int splits, int Rk, int* split) {
  int u = id, r = 0;
  if (Rk > 1) {
    const int y = id >> 3;
    u = ((y / Rk) << 3) + (id & 7);
    r = y % Rk;
  }
  const int s = u / splits;
  *split = u - s * splits;
  return Rk > 1 ? s * Rk + r : s;
}
// How many work-groups that takes.
inline int64_t attention_grid(int nseg, int splits, int Rk) {
  const int64_t u = (int64_t)(nseg / Rk) * splits;
  return Rk > 1 ? (u + 7) / 8 * 8 * Rk : u;
}

}  // namespace absb

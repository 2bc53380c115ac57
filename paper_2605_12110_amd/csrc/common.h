// Internal declarations shared by the translation units of libabsb.so (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "absb.h"

#define ABSB_HEAD_DIM 128
#define ABSB_MAX_KV_HEADS 64
#define ABSB_MAX_GROUP 8
#define ABSB_MAX_SEL_BLOCKS (1 << 17)  // blocks per segment the selection holds (its LDS bitmap)
#define ABSB_HIDDEN __attribute__((visibility("hidden")))
// Split counters sit 256 bytes apart: counters that share a memory line serialise each other's
// atomic updates (measured: 8 segments x 32 arrivals on one line cost 2.7 us, apart 0.x us).
#define ABSB_TICKET_STRIDE 64
#define BUILD_RUNS_OF 512        // tokens a work-group of the store build pools at a time
#define BUILD_MAX_COPIES 8       // of the words that its work-groups raise together

namespace absb {

// Per-KV-head block sizes as log2, passed to kernels by value.  Four to a word: a byte of the kernel's arguments at an
// index known only at run time would be a vector load, half a microsecond in front of everything else.
struct HeadTable {
  uint32_t packed[ABSB_MAX_KV_HEADS / 4];
  __host__ __device__ int log2_block(int h) const { return (int)(packed[h >> 2] >> (8 * (h & 3)) & 255u); }
};

// Shape of the layer and of the paged cache, passed to kernels by value.
struct Geometry {
  int32_t Bt, Hq, Hkv, G;
  // Selection segments.  Group selection (default): one per (request, KV head), whose G query
  // heads share the list: Hsel = Hkv, Gd = G, Rk = 1.  Per-query-head selection: one per
  // (request, query head): Hsel = Hq, Gd = 1, Rk = G selection segments read each KV head's store.
  int32_t Hsel, Gd, Rk;
  int32_t agg_max;    // 1: a group's shared score is the maximum over its query heads (else their sum)
  int32_t log2_page;  // P = 1 << log2_page
  int32_t pt_stride;
  int32_t repr;       // absb_repr: vectors per block = repr + 1
  int32_t sink_tokens, recent_tokens;  // forced blocks of the selection (0 = none)
  int32_t tight;      // 1: the block layout is that of the current lengths (off[s+1] - off[s] = N_s)
  int64_t s_page, s_head, s_tok;  // element strides of the K/V caches
  HeadTable heads;
};

// Host-side sizes derived from (layer, batch).
struct Plan {
  int32_t nseg;             // selection segments: Bt * Hsel
  int32_t nstore;           // store segments: Bt * Hkv
  int64_t total;            // total centroids (rows of the store)
  int32_t max_blocks;       // max_s N_s
  int32_t sel_stride;       // max_s K_s (0 when no budget was given)
  int64_t max_tokens;       // max_s (upper bound of selected tokens of a segment)
  int64_t sum_tokens;       // sum_s of the same bound
  int32_t split_tokens;     // tokens per split-K work-group
  int32_t max_splits;       // grid.x of the decode kernels
  int32_t small;            // the pipelined step in the form of small.hip
  int32_t own;              // ... of own.hip
  int32_t some_dense, all_dense;  // requests whose budget covers their context (everything is selected): any, all
  int32_t stream_rows;      // attention: K and V rows are read past the caches
  int32_t one_launch;       // absb_decode_fused: the whole step as one launch (else one launch per stage)
  int32_t step_form;        // absb_step_form actually used (never ABSB_STEP_AUTO)
  int32_t shared;           // the one-launch step in the form of shared.hip
  int32_t score_chunk;      // centroids per work-group in score
  int32_t build_max_chunks; // max_b build_chunks(L_b)
  int32_t build_copies;     // of a segment's ranges while its chunks are pooled (a power of two)
  int32_t build_pitch;      // words between what two segments' chunks share
  // workspace carving (byte offsets, 256-aligned)
  size_t ws_part_o, ws_part_ml, ws_tickets;       // decode partials, per-segment split counters
  size_t ws_score_tickets, ws_flags, ws_status;   // more counters of the one-launch step
  size_t ws_finished, ws_listed, ws_counts, ws_hist;  // ... and of its form with a shared selection
  size_t ws_cand;
  size_t ws_head_bytes;                           // all counters: the part absb_workspace_init clears
  size_t ws_scores, ws_sel_idx, ws_sel_cnt;       // fused step intermediates
  size_t ws_cent, ws_meet;                        // build intermediates
  size_t ws_decode_bytes, ws_fused_bytes, ws_build_bytes, ws_bytes;
};

// Validates the host-visible arguments and fills geometry + plan.  `need_budget`: budget_host
// must be present (topk, fused); otherwise it is used when present.  `sel_stride_in` > 0 bounds
// the selected-token estimate for the stand-alone decode.  `lean`: a workspace without the shared
// selection's histogram rows and candidates, and so a step without it.
ABSB_HIDDEN int make_plan(const absb_layer* layer, const absb_batch* batch, bool need_budget,
                          int32_t sel_stride_in, Geometry* geo, Plan* plan, bool lean = false);

// The store build cuts a segment into chunks of a few runs of BUILD_RUNS_OF tokens, a work-group each: one run as long as
// that makes at most BUILD_CHUNKS of them (1280 work-groups fit the chip, 1024 that pool extrema; while one segment takes
// most of the places, the next one's cannot fill the gaps: 400000 tokens of 8 heads 207 us as 782 chunks of a run, 169 as 391 of two; with at
// most 256 chunks more rows than need to go through memory: 180000 tokens 83 us against 72), and never more than
// BUILD_MAX_RUNS.
constexpr int BUILD_CHUNKS = 512, BUILD_MAX_RUNS = 8;
__host__ __device__ constexpr int build_runs(int L) {
  const int runs = (int)(((int64_t)L + BUILD_RUNS_OF * BUILD_CHUNKS - 1) / (BUILD_RUNS_OF * BUILD_CHUNKS));
  return runs < BUILD_MAX_RUNS ? runs : BUILD_MAX_RUNS;
}
__host__ __device__ constexpr int build_chunks(int L) {
  const int tokens = build_runs(L) * BUILD_RUNS_OF;
  return (int)(((int64_t)L + tokens - 1) / tokens);
}
// The most chunks that a context of L tokens or any shorter one makes: longer chunks can make fewer of them (262144 tokens
// 512, 262145 257).
__host__ __device__ constexpr int build_most_chunks(int L) {
  const int one_run = (int)(((int64_t)L + BUILD_RUNS_OF - 1) / BUILD_RUNS_OF), now = build_chunks(L);
  return one_run < BUILD_CHUNKS ? one_run : now > BUILD_CHUNKS ? now : BUILD_CHUNKS;
}
static_assert(build_chunks(BUILD_RUNS_OF * BUILD_CHUNKS) == BUILD_CHUNKS && build_chunks(BUILD_RUNS_OF * BUILD_CHUNKS + 1) < BUILD_CHUNKS &&
              build_chunks(BUILD_RUNS_OF * BUILD_CHUNKS * BUILD_MAX_RUNS) == BUILD_CHUNKS, "at most BUILD_CHUNKS while chunks grow");

// What the build's chunks of a segment share, in words (zero when its kernel starts; W values per block): copies of the
// minima and maxima per value, a flag per copy, a 64-bit counter (each on memory lines of its own), a bit per chunk
// that left, and copies of those bits.
__host__ __device__ constexpr int meet_flags(int W, int copies) { return copies * 2 * W; }
__host__ __device__ constexpr int meet_state(int W, int copies) { return meet_flags(W, copies) + copies * 32; }
__host__ __device__ constexpr int meet_left(int W, int copies) { return meet_state(W, copies) + 32; }
__host__ __device__ constexpr int meet_used(int W, int copies, int chunks) {  // (the copies of the bits need not be zero)
  return meet_left(W, copies) + (chunks + 31) / 32;
}
__host__ __device__ constexpr int meet_words(int W, int copies, int chunks) {
  return meet_left(W, copies) + (copies + 1) * ((chunks + 31) / 32);
}

// Launchers (one per stage); all enqueue on `stream` and return an absb_status.
ABSB_HIDDEN int launch_build(const Geometry& g, const Plan& pl, int dtype, const void* k_cache,
                             const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off,
                             uint8_t* codes, float* qscale, float* qmin, char* ws, hipStream_t stream);
ABSB_HIDDEN int launch_score(const Geometry& g, const Plan& pl, int dtype, const void* q, const uint8_t* codes,
                             const float* qscale, const float* qmin, const int32_t* cent_off, const int32_t* seq_lens,
                             int32_t* scores, int32_t* score_exp, hipStream_t stream);
// append == false: only (re)compute the tail state from the cache
ABSB_HIDDEN int launch_append(const Geometry& g, const Plan& pl, int dtype, bool append, const void* k_cache,
                              const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off,
                              uint8_t* codes, const float* qscale, const float* qmin, float* tail,
                              int32_t* clamped, hipStream_t stream);
ABSB_HIDDEN int launch_topk(const Geometry& g, const Plan& pl, const int32_t* scores, const int32_t* cent_off,
                            const int32_t* budget, const int32_t* seq_lens, int32_t* sel_idx, int32_t* sel_cnt,
                            int32_t sel_stride,
                            int32_t* tickets, hipStream_t stream);
ABSB_HIDDEN int launch_decode(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q,
                              const void* k_cache, const void* v_cache, const int32_t* page_table,
                              const int32_t* seq_lens, const int32_t* sel_idx, const int32_t* sel_cnt,
                              int32_t sel_stride, void* out, float* lse, char* ws, bool tickets_cleared,
                              hipStream_t stream);
// ... over all blocks of every context: the list is the identity and is not read
ABSB_HIDDEN int launch_decode_dense(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q,
                                    const void* k_cache, const void* v_cache, const int32_t* page_table,
                                    const int32_t* seq_lens, const int32_t* cent_off, void* out, float* lse, char* ws,
                                    hipStream_t stream);

// The whole step in one launch (estimation, selection and attention work-groups in one grid).
ABSB_HIDDEN bool fused_one_launch_fits(const Plan& pl);
ABSB_HIDDEN int launch_fused(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q,
                             const uint8_t* codes, const float* qscale, const float* qmin, const void* k_cache,
                             const void* v_cache, const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off,
                             const int32_t* budget, int32_t* sel_idx_out, int32_t* sel_cnt, void* out, float* lse,
                             char* ws, hipStream_t stream);
// The whole step in one launch for short segments: every attention work-group scores and selects for itself.
constexpr int SMALL_MAX_BLOCKS = 512;
ABSB_HIDDEN int launch_small(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q,
                             const uint8_t* codes, const float* qscale, const float* qmin, const void* k_cache,
                             const void* v_cache, const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off,
                             const int32_t* budget, int32_t* sel_idx_out, int32_t* sel_cnt, void* out, float* lse,
                             char* ws, hipStream_t stream);
// The whole step in one launch for segments of medium length: every attention work-group selects for itself, from scores that
// the estimation work-groups hand over.
constexpr int OWN_MAX_BLOCKS = 4096;
ABSB_HIDDEN bool own_fits(const Plan& pl);
ABSB_HIDDEN int launch_own(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q,
                           const uint8_t* codes, const float* qscale, const float* qmin, const void* k_cache,
                           const void* v_cache, const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off,
                           const int32_t* budget, int32_t* sel_idx_out, int32_t* sel_cnt, void* out, float* lse,
                           char* ws, hipStream_t stream);
ABSB_HIDDEN int launch_workspace_init(const Plan& pl, char* ws, hipStream_t stream);
// The whole step in one launch for long segments: the work-groups that score a segment select for it together.
constexpr int SHARED_MAX_CHUNKS = 64;     // of a segment
constexpr int SHARED_MAX_CHUNK = 2048;    // blocks of a chunk: 2^17 blocks / 64 chunks
constexpr int SHARED_HIST_BINS = 1024;    // words of a segment's histogram row
constexpr int SHARED_MAX_SEGMENTS = 512;  // beyond, workspaces have no histogram rows
constexpr int SHARED_LIST = 2048;         // list entries an attention work-group holds
__host__ __device__ inline int shared_chunk_blocks(int max_blocks) {
  const int cb = ((max_blocks + SHARED_MAX_CHUNKS - 1) / SHARED_MAX_CHUNKS + 63) & ~63;
  return cb < 512 ? 512 : cb;
}
ABSB_HIDDEN bool shared_fits(const Plan& pl);
ABSB_HIDDEN int launch_shared(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q,
                              const uint8_t* codes, const float* qscale, const float* qmin, const void* k_cache,
                              const void* v_cache, const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off,
                              const int32_t* budget, int32_t* sel_idx_out, int32_t* sel_cnt, void* out, float* lse,
                              char* ws, hipStream_t stream);

ABSB_HIDDEN int launch_stream_read(const void* src, size_t bytes, uint32_t* sink, int num_cus, hipStream_t stream);

ABSB_HIDDEN int launch_head_recall(const float* lse_sel, const float* lse_all, float* recall, int nseg, int G,
                                   hipStream_t stream);

__host__ __device__ constexpr size_t max_sz(size_t a, size_t b) { return a > b ? a : b; }

inline int check_launch() { return hipGetLastError() == hipSuccess ? ABSB_OK : ABSB_ERR_HIP; }

// A kernel's leading arguments, which the build has in scalar registers when a wave starts (14 words), a few to a vector:
// every argument of a launch costs the host 0.02 us, whatever its size (a decode loop of short steps waits for the host).
typedef uint64_t addr2 __attribute__((ext_vector_type(2)));
typedef int32_t int2v __attribute__((ext_vector_type(2)));
typedef int32_t int4v __attribute__((ext_vector_type(4)));
__host__ __device__ inline uint64_t addr(const void* p) { return reinterpret_cast<uint64_t>(p); }

// ------------------------------------------------------------------ device helpers
#ifdef __HIPCC__
// Brings the kernel's arguments from byte FROM on into the scalar cache, all lines at once (together with whatever has been
// asked for before): a dozen cold lines, which the code would else ask for one after the other, wherever it first
// needs something from one, 0.3 us each.  (The attention work-groups of the one-launch forms do without: they have time
// until their lists come, and in a large batch the fetch costs more than it brings, 39.0 -> 39.6 us a step.)
template <int FROM, int BYTES>
__device__ __forceinline__ void fetch_arguments() {
  constexpr int FIRST = FROM / 64, LINES = (FROM + BYTES + 63) / 64 - FIRST;
  uint32_t got;
  __builtin_amdgcn_sched_barrier(0);
  asm volatile(
      ".set absb_at, %2\n\t"
      ".rept %3\n\t"
      "s_load_dword %0, %1, absb_at\n\t"
      ".set absb_at, absb_at + 64\n\t"
      ".endr\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&s"(got)
      : "s"(__builtin_amdgcn_kernarg_segment_ptr()), "n"(FIRST * 64), "n"(LINES));
  __builtin_amdgcn_sched_barrier(0);
}

// A pointer from a leading argument (to device memory, which the compiler would know of a pointer argument).
template <typename T>
__device__ __forceinline__ T* from_addr(uint64_t a) {
  return (T*)(__attribute__((address_space(1))) T*)a;
}

// Selection segment t -> request b, selection head hs (first query head = hs * Gd), KV head hk,
// store segment s = b * Hkv + hk, and where the segment's scores start in the score array:
// the Rk selection segments of a store segment lie side by side, Rk * off[s] + (hs % Rk) * rows.
struct SegMap {
  int b, hs, hk, s;
};
__device__ __forceinline__ SegMap seg_map(int t, int Hsel, int Rk, int Hkv) {
  SegMap m;
  m.b = t / Hsel;
  m.hs = t % Hsel;
  m.hk = m.hs / Rk;
  m.s = m.b * Hkv + m.hk;
  return m;
}
__device__ __forceinline__ int64_t score_base(const SegMap& m, int Rk, int off, int rows) {
  return (int64_t)Rk * off + (int64_t)(m.hs % Rk) * rows;
}
// Device-coherent 32-bit accesses for data handed from one work-group to another inside a launch
// (relaxed, agent scope: served past the caches that are not coherent across the chip).  The
// hand-off protocol around them: the writer waits until its stores are acknowledged
// (s_waitcnt vmcnt(0) + work-group barrier), then publishes a counter or flag with a relaxed
// agent-scope atomic; the reader issues its loads only after it has seen that counter or flag.
template <bool COH>
__device__ __forceinline__ int32_t ld_i32(const int32_t* p) {
  if (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool COH>
__device__ __forceinline__ void st_i32(int32_t* p, int32_t v) {
  if (COH)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}
__device__ __forceinline__ void wait_stores_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// K_s = min(N_s, ceil(T_b / B_h)) (Sec. 3.4, kernel 2), never more than the list has room for.
__device__ __forceinline__ int budget_blocks(int T, int log2_block, int blocks, int sel_stride) {
  const int K = (int)(((int64_t)T + (1 << log2_block) - 1) >> log2_block);
  return min(min(K, blocks), sel_stride);
}

// Blocks in use of a segment: all rows of a tight layout (no need to wait for the length then);
// otherwise N_s = ceil(L_b / B_h), never more than the layout has rows for.
__device__ __forceinline__ int blocks_in_use(bool tight, int rows, int L, int log2_block) {
  return tight ? rows : min(rows, (int)(((int64_t)L + (1 << log2_block) - 1) >> log2_block));
}
__device__ __forceinline__ int blocks_in_use(bool tight, int rows, const int32_t* seq_lens, int b, int log2_block) {
  return tight ? rows : blocks_in_use(tight, rows, seq_lens[b], log2_block);
}

template <typename To, typename From>
__device__ __forceinline__ To bitcast(From v) {
  return __builtin_bit_cast(To, v);
}

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// Element traits of the two storage formats.  A 32-bit word holds two consecutive channels
// (low half = even channel).
template <int DT>
struct Elem;

template <>
struct Elem<ABSB_F16> {
  static __device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2(bitcast<half2_t>(a), bitcast<half2_t>(b), c, false);
  }
  static __device__ __forceinline__ float lo(uint32_t v) { return (float)bitcast<half2_t>(v).x; }
  static __device__ __forceinline__ float hi(uint32_t v) { return (float)bitcast<half2_t>(v).y; }
  static __device__ __forceinline__ float widen(uint16_t v) { return (float)bitcast<_Float16>(v); }
  static __device__ __forceinline__ uint16_t narrow(float f) { return bitcast<uint16_t>((_Float16)f); }
};

template <>
struct Elem<ABSB_BF16> {
  static __device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(bitcast<bf16x2_t>(a), bitcast<bf16x2_t>(b), c, false);
  }
  static __device__ __forceinline__ float lo(uint32_t v) { return bitcast<float>(v << 16); }
  static __device__ __forceinline__ float hi(uint32_t v) { return bitcast<float>(v & 0xffff0000u); }
  static __device__ __forceinline__ float widen(uint16_t v) { return bitcast<float>((uint32_t)v << 16); }
  static __device__ __forceinline__ uint16_t narrow(float f) {  // round to nearest, ties to even
    uint32_t u = bitcast<uint32_t>(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
  }
};

// DPP controls (GFX9 encoding).
enum : int {
  DPP_QUAD_XOR1 = 0xB1,        // quad_perm:[1,0,3,2]
  DPP_QUAD_XOR2 = 0x4E,        // quad_perm:[2,3,0,1]
  DPP_ROW_MIRROR = 0x140,      // lane i <- lane 15-i within a row of 16
  DPP_ROW_HALF_MIRROR = 0x141  // lane i <- lane 7-i within a half row of 8
};

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return bitcast<float>(__builtin_amdgcn_update_dpp(0, bitcast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

// Sum over the 16 lanes of a DPP row; every lane of the row ends with the same bits.
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f<DPP_QUAD_XOR1>(v);
  v += dpp_f<DPP_QUAD_XOR2>(v);
  v += dpp_f<DPP_ROW_HALF_MIRROR>(v);
  v += dpp_f<DPP_ROW_MIRROR>(v);
  return v;
}
__device__ __forceinline__ int quad_sum(int v) {
  v += dpp_i<DPP_QUAD_XOR1>(v);
  v += dpp_i<DPP_QUAD_XOR2>(v);
  return v;
}

// Reductions and scans over a wave built from DPP row operations and four lane reads.  They
// replace ds_bpermute shuffle chains (each shuffle is an LDS-crossbar round trip of >100 cycles).
// All 64 lanes must be active.
template <typename Op>
__device__ __forceinline__ uint32_t row16_reduce_u32(uint32_t v, Op op) {  // every lane of a row gets the row's result
  v = op(v, (uint32_t)dpp_i<DPP_QUAD_XOR1>((int)v));
  v = op(v, (uint32_t)dpp_i<DPP_QUAD_XOR2>((int)v));
  v = op(v, (uint32_t)dpp_i<DPP_ROW_HALF_MIRROR>((int)v));
  v = op(v, (uint32_t)dpp_i<DPP_ROW_MIRROR>((int)v));
  return v;
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, Op op) {  // wave-uniform result
  v = row16_reduce_u32(v, op);
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16),
                 c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return op(op(a, b), op(c, d));
}
__device__ __forceinline__ float wave_max_f32(float v) {
  v = fmaxf(v, dpp_f<DPP_QUAD_XOR1>(v));
  v = fmaxf(v, dpp_f<DPP_QUAD_XOR2>(v));
  v = fmaxf(v, dpp_f<DPP_ROW_HALF_MIRROR>(v));
  v = fmaxf(v, dpp_f<DPP_ROW_MIRROR>(v));
  const float a = bitcast<float>(__builtin_amdgcn_readlane(bitcast<int>(v), 0)),
              b = bitcast<float>(__builtin_amdgcn_readlane(bitcast<int>(v), 16)),
              c = bitcast<float>(__builtin_amdgcn_readlane(bitcast<int>(v), 32)),
              d = bitcast<float>(__builtin_amdgcn_readlane(bitcast<int>(v), 48));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}
// Inclusive prefix sum over the wave in lane order; *total receives the wave's sum.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v, uint32_t* total) {
  v += (uint32_t)dpp_i<0x111>((int)v);  // row_shr:1 (lanes shifted in from outside the row read 0)
  v += (uint32_t)dpp_i<0x112>((int)v);  // row_shr:2
  v += (uint32_t)dpp_i<0x114>((int)v);  // row_shr:4
  v += (uint32_t)dpp_i<0x118>((int)v);  // row_shr:8
  const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15), t1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 31),
                 t2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 47), t3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
  const int row = (int)(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) >> 4);
  v += (row >= 1 ? t0 : 0u) + (row >= 2 ? t1 : 0u) + (row >= 3 ? t2 : 0u);
  *total = t0 + t1 + t2 + t3;
  return v;
}
#endif  // __HIPCC__

}  // namespace absb

// The whole decode step in one launch for short segments, where every attention work-group scores and selects
// for itself.
//
// At a few hundred blocks a segment the hand-overs of the pipelined form (fused.hip) cost more than the work they
// hand over: scores out, acknowledged, ticket, keys back in, list out, acknowledged, flag, list in, each a
// trip to memory.  Here every work-group (split, segment) reads all of its segment's codes (N * 64 bytes: the
// splits of a segment run on one die and share its L2), keeps the scores in LDS, selects, and attends over its
// own split of the list; only the split-K merge is left of the hand-overs.  Scores, selection and the order of
// the list are those of the pipelined form, so the output is the same bit for bit.  4K context, batch 1,
// 8 heads: 13.4 -> 11.3 us a step, and 9.3 with the selection by single waves and the arguments fetched at once (below).
//
// Compiled with -ffp-contract=off, as the estimation stage requires.
#include "decode_dev.h"
#include "score_dev.h"
#include "topk_dev.h"

namespace absb {

struct SmallParams {
  int32_t max_blocks;
  ScoreParams sc;
  TopkParams tk;
  DecodeParams dc;
};

constexpr int SMALL_THREADS = DEC_THREADS;
constexpr int SMALL_WAVES = SMALL_THREADS / 64;
constexpr size_t small_max(size_t a, size_t b) { return a > b ? a : b; }
// LDS: scratch of the stages (one after the other), then the scores, then the list
constexpr size_t SMALL_LDS_SCRATCH =
    small_max(small_max((size_t)DEC_LDS_BYTES, 2 * TOPK_RANK_MAX * 4 + SMALL_MAX_BLOCKS / 8), small_max(score_lds_bytes<0>(), score_lds_bytes<1>())) / 16 * 16 + 16;

// What is selected of a segment: K of its N blocks, of which [0, lo) and [hi, N) are forced and [lo, hi) compete.
struct SmallShape {
  int N, K, lo, hi;
};

// The selection of a segment whose scores are in LDS (at most 64 * R of its blocks compete, one at least): the same list
// in the same order as topk_segment's hand-over.  A selection by a work-group of four waves passes from barrier to barrier:
// 3.3 us for 512 blocks, most of it waiting.  Here every wave holds all keys and finds the threshold bin by itself, a bit
// of its number at a time (the keys beyond a candidate are counted with wave-wide comparisons, no LDS and no barrier), so
// that one barrier is left, in front of the ranking of the few keys inside the bin: 3.3 -> 2.3 us for 512 blocks (4K
// context, batch 1: 11.1 -> 10.6 us a step; the rest, to 9.3, is what the arguments took).
template <int R>
__device__ __forceinline__ void select_in_lds(const SmallShape& g, const int32_t* s_score, int32_t* s_list, uint32_t* s_cand, int32_t* out) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nforced = g.lo + (g.N - g.hi), Kc = g.K - nforced, Nc = g.hi - g.lo;
  // the keys that compete (block lo + i is the i-th) as their distance from the lowest, plus one; zero: none
  uint32_t key[R], kmin = ~0u, kmax = 0u;
#pragma unroll
  for (int i = 0; i < R; ++i) key[i] = ordered_key(s_score[g.lo + min(64 * i + lane, Nc - 1)]);
#pragma unroll
  for (int i = 0; i < R; ++i) {  // (copies of the last key change neither)
    kmin = min(kmin, key[i]);
    kmax = max(kmax, key[i]);
  }
  kmin = wave_reduce_u32(kmin, UMin());
  const uint32_t range = wave_reduce_u32(kmax, UMax()) - kmin;
#pragma unroll
  for (int i = 0; i < R; ++i) key[i] = 64 * i + lane < Nc ? key[i] - kmin + 1 : 0u;
  auto beyond = [&](uint32_t x) __attribute__((always_inline)) {  // how many competing keys are at least x above the lowest
    int n = 0;
#pragma unroll
    for (int i0 = 0; i0 < R; i0 += 8) {  // (comparisons in groups: a count waits for its comparison, the next one need not)
      uint64_t m[8];
#pragma unroll
      for (int i = 0; i < 8 && i0 + i < R; ++i) m[i] = __ballot(key[i0 + i] > x);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 8 && i0 + i < R; ++i) n += (int)__popcll(m[i]);
    }
    return n;
  };
  const int bits = 32 - __builtin_clz(range | 1u);
  const int shift = bits > TOPK_DIGIT_BITS ? bits - TOPK_DIGIT_BITS : 0;
  uint32_t floor_ = 0;  // the lowest key of the threshold bin
#pragma unroll 1
  for (uint32_t bit = 1u << (bits - 1); bit >> shift; bit >>= 1)
    if (beyond(floor_ | bit) >= Kc) floor_ |= bit;
  const uint32_t above = floor_ + (1u << shift);  // (no overflow: a range of scores stays below 2^32 - 2^21)
  // how many keys lie above the bin and inside it; how many of those belong to the waves before this one (wave w hands
  // over the blocks that threads [64 w, 64 w + 64) of a work-group would, 256 at a time)
  int n_above = 0, n_in = 0, at = 0, cand_at = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int a = (int)__popcll(__ballot(key[i] > above)), c = (int)__popcll(__ballot(key[i] > floor_)) - a;
    n_above += a;
    n_in += c;
    at += (i & (SMALL_WAVES - 1)) < wave ? a : 0;
    cand_at += (i & (SMALL_WAVES - 1)) < wave ? c : 0;
  }
  const int need = Kc - n_above;
  const bool direct = n_in <= TOPK_RANK_MAX;
  constexpr int OWN = (R + SMALL_WAVES - 1) / SMALL_WAVES;
  uint32_t own[OWN];
  int admitted = -1;  // the candidate that this thread ranks and that is admitted
  if (direct) {
    for (int i = tid; i < nforced; i += SMALL_THREADS) s_list[i] = i < g.lo ? i : g.hi + (i - g.lo);
    at += nforced;
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const int j = SMALL_THREADS * k + tid;
      own[k] = j < Nc ? ordered_key(s_score[g.lo + min(j, Nc - 1)]) - kmin + 1 : 0u;
      const uint64_t a = __ballot(own[k] > above), c = __ballot(own[k] > floor_) & ~a;
      at += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(a >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)a, 0u));
      if (c) {  // (few have any)
        if ((c >> lane) & 1u) {
          const int slot = cand_at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(c >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)c, 0u));
          s_cand[slot] = own[k];
          s_cand[TOPK_RANK_MAX + slot] = (uint32_t)j;
        }
        cand_at += (int)__popcll(c);
      }
    }
#pragma unroll
    for (int k = 0; k < OWN; ++k)
      if (own[k] > above) s_list[at++] = g.lo + SMALL_THREADS * k + tid;
    __syncthreads();
    if (tid < n_in) {  // exact rank of every candidate: key descending, index ascending
      const uint32_t mk = s_cand[tid], mi = s_cand[TOPK_RANK_MAX + tid];
      int rank = 0;
#pragma unroll 4
      for (int u = 0; u < n_in; ++u) {
        const uint32_t ok = s_cand[u], oi = s_cand[TOPK_RANK_MAX + u];
        rank += ok > mk || (ok == mk && oi < mi);
      }
      if (rank < need) s_list[nforced + n_above + rank] = g.lo + (admitted = (int)mi);
    }
  }
  if (direct && !out) return;
  if (direct) {
    // ---- the caller's list, in ascending order, from a bit per competing block.  (By the search and the passes below, over
    // all keys, it cost 3.0 us a step at 1024 blocks, which this form took then, this way 0.4.)
    uint64_t* s_taken = reinterpret_cast<uint64_t*>(s_cand + 2 * TOPK_RANK_MAX);
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const uint64_t a = __ballot(own[k] > above);
      if (lane == 0) s_taken[SMALL_WAVES * k + wave] = a;
    }
    __syncthreads();
    if (admitted >= 0) atomicOr(reinterpret_cast<uint32_t*>(s_taken) + (admitted >> 5), 1u << (admitted & 31));
    __syncthreads();
    const uint64_t mine = lane < SMALL_WAVES * OWN ? s_taken[lane] : 0;
    uint32_t all;
    const int before = (int)(wave_incl_scan_u32((uint32_t)__popcll(mine), &all) - (uint32_t)__popcll(mine));
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const int w = SMALL_WAVES * k + wave;
      const uint64_t sel = readlane_u64(mine, w);
      const int p = g.lo + __builtin_amdgcn_readlane(before, w) +
                    (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(sel >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)sel, 0u));
      if ((sel >> lane) & 1u) out[p] = g.lo + 64 * w + lane;
    }
    for (int i = tid; i < nforced; i += SMALL_THREADS)  // [0, lo) in front, [hi, N) behind
      out[i < g.lo ? i : i + Kc] = i < g.lo ? i : g.hi + (i - g.lo);
    return;
  }
  // ---- the bin is crowded: the threshold key itself, then the keys above it and the first ones that equal it, in order of
  // their index
#pragma unroll 1
  for (uint32_t bit = (1u << shift) >> 1; bit; bit >>= 1)
    if (beyond(floor_ | bit) >= Kc) floor_ |= bit;
  int left = Kc - beyond(floor_ + 1), pos = g.lo;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int j = g.lo + 64 * i + lane;
    const uint64_t eq = __ballot(key[i] == floor_ + 1);
    const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0u));
    const uint64_t sel = __ballot(key[i] > floor_ + 1 || (key[i] == floor_ + 1 && before < left));
    left = max(left - (int)__popcll(eq), 0);
    if (wave == (i & (SMALL_WAVES - 1)) && ((sel >> lane) & 1u)) {
      const int p = pos + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(sel >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)sel, 0u));
      s_list[p] = j;
      if (out) out[p] = j;
    }
    pos += (int)__popcll(sel);
  }
  for (int i = tid; i < nforced; i += SMALL_THREADS) {
    const int p = i < g.lo ? i : i + Kc, j = i < g.lo ? i : g.hi + (i - g.lo);
    s_list[p] = j;
    if (out) out[p] = j;
  }
}

// What a work-group needs before anything else, as arguments of their own in front: the build asks for them to be in
// scalar registers when a wave starts (the rest of the arguments are cold lines of memory, 0.5 us for the first and 0.3
// for every further one the code came upon: the codes were asked for 1.9 us after the wave had started).  The grid's
// three dimensions say which segment and split it is, without divisions.
constexpr int SMALL_LEADING = 6 * 8 + 2 * 4;  // bytes of them
template <int DT, int G, int REP>
__global__ __launch_bounds__(SMALL_THREADS, 4) void small_step_kernel(addr2 off_lens, addr2 budget_codes, addr2 q_qscale,
                                                                      int2v Hsel_tight, SmallParams p) {
  extern __shared__ __align__(16) char lds[];
  const auto cent_off = from_addr<const int32_t>(off_lens.x), seq_lens = from_addr<const int32_t>(off_lens.y);
  const auto budget = from_addr<const int32_t>(budget_codes.x);
  const auto codes = from_addr<const uint8_t>(budget_codes.y);
  const auto q = from_addr<const uint16_t>(q_qscale.x);
  const auto qscale = from_addr<const float>(q_qscale.y);
  const int Hsel = Hsel_tight.x, tight = Hsel_tight.y;
  // split-major: with a multiple of eight segments, the splits of a segment land on one die
  const int hs = blockIdx.x, b = blockIdx.y, split = blockIdx.z, t = b * Hsel + hs, tid = threadIdx.x;
  // cold lines, all asked for at once
  const int off = cent_off[t], end = cent_off[t + 1], T = budget[b];
  SplitCtx c;
  c.L = seq_lens[b];
  fetch_arguments<SMALL_LEADING, sizeof(SmallParams)>();
  int32_t* s_score = reinterpret_cast<int32_t*>(lds + SMALL_LDS_SCRATCH);
  int32_t* s_list = s_score + p.max_blocks;
  const int lb = p.dc.g.heads.log2_block(hs);
  const int N = blocks_in_use(tight, end - off, c.L, lb);
  const int pos_begin = split * p.dc.split_tokens;

  u32x4 qb[4];
  load_q<G>(q + ((size_t)t * G) * ABSB_HEAD_DIM, qb);
  c.b = b;
  c.hs = hs;
  c.hk = hs;
  c.lb = lb;
  c.lP = p.dc.g.log2_page;
  if (!p.dc.some_dense || T < c.L)  // (else the budget covers the context: no score decides anything)
    score_blocks<DT, REP, false, 4>(
        p.sc, score_source<REP>(q, qscale, codes, t, t, G, off, N), G, t, 0, p.max_blocks, lds,
        [&](int j, int32_t sc) __attribute__((always_inline)) { s_score[j] = sc; }, nullptr);

  const int nsel = budget_blocks(T, lb, N, p.dc.sel_stride);
  const int ntok = min(nsel << lb, p.dc.max_splits * p.dc.split_tokens);
  if (pos_begin >= ntok) return;
  const int pos_end = min(ntok, pos_begin + p.dc.split_tokens);
  const int nsplit = (ntok + p.dc.split_tokens - 1) / p.dc.split_tokens;
  __syncthreads();  // the scores are in LDS; the estimation's scratch is free

  SmallShape g{N, nsel, 0, N};
  if (p.tk.sink_tokens > 0) g.lo = min(N, (int)(((int64_t)p.tk.sink_tokens + (1 << lb) - 1) >> lb));
  if (p.tk.recent_tokens > 0) g.hi = max(g.lo, min(N, max(0, c.L - p.tk.recent_tokens) >> lb));
  // the caller's list and count come from the first split's work-group
  int32_t* out = split == 0 && p.tk.sel_idx ? p.tk.sel_idx + (size_t)t * p.tk.sel_stride : nullptr;
  if (split == 0 && tid == 0) p.tk.sel_cnt[t] = nsel;
  if (out)
    for (int i = nsel + tid; i < p.tk.sel_stride; i += SMALL_THREADS) out[i] = -1;
  uint32_t* s_cand = reinterpret_cast<uint32_t*>(lds);
  if (nsel >= N || g.lo + (N - g.hi) >= nsel) {  // no score decides anything
    for (int i = tid; i < nsel; i += SMALL_THREADS) {
      const int j = nsel >= N || i < g.lo ? i : g.hi + (i - g.lo);
      s_list[i] = j;
      if (out) out[i] = j;
    }
  } else if (g.hi - g.lo <= 256) {
    select_in_lds<4>(g, s_score, s_list, s_cand, out);
  } else {
    select_in_lds<SMALL_MAX_BLOCKS / 64>(g, s_score, s_list, s_cand, out);
  }
  __syncthreads();

  const ListRef<LIST_LOCAL> list{s_list, nsel - 1};
  const int32_t* pages = p.dc.page_table + (size_t)b * p.dc.g.pt_stride;
  AttnState<G> st;
  st.reset();
  attend_positions<DT, G>(p.dc, c, list, pages, pos_begin, pos_end, qb, st);
  finish_split<DT, G>(p.dc, t, b, hs, split, nsplit, p.dc.max_splits, st, lds, []() {});
}

template <int DT, int G>
static void launch_small_rep(const SmallParams& p, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(SMALL_THREADS), lds, stream,
                       addr2{addr(p.sc.cent_off), addr(p.sc.seq_lens)}, addr2{addr(p.tk.budget), addr(p.sc.codes)},
                       addr2{addr(p.sc.q), addr(p.sc.qscale)}, int2v{p.sc.Hsel, p.sc.tight}, p);
  };
  if (repr == ABSB_REPR_MEAN)
    launch(small_step_kernel<DT, G, 0>);
  else
    launch(small_step_kernel<DT, G, 1>);
}

template <int DT>
static void launch_small_group(const SmallParams& p, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  switch (p.dc.g.Gd) {
    case 1: launch_small_rep<DT, 1>(p, repr, grid, lds, stream); break;
    case 2: launch_small_rep<DT, 2>(p, repr, grid, lds, stream); break;
    case 3: launch_small_rep<DT, 3>(p, repr, grid, lds, stream); break;
    case 4: launch_small_rep<DT, 4>(p, repr, grid, lds, stream); break;
    case 5: launch_small_rep<DT, 5>(p, repr, grid, lds, stream); break;
    case 6: launch_small_rep<DT, 6>(p, repr, grid, lds, stream); break;
    case 7: launch_small_rep<DT, 7>(p, repr, grid, lds, stream); break;
    default: launch_small_rep<DT, 8>(p, repr, grid, lds, stream); break;
  }
}

int launch_small(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q, const uint8_t* codes,
                 const float* qscale, const float* qmin, const void* k_cache, const void* v_cache, const int32_t* page_table,
                 const int32_t* seq_lens, const int32_t* cent_off, const int32_t* budget, int32_t* sel_idx_out,
                 int32_t* sel_cnt, void* out, float* lse, char* ws, hipStream_t stream) {
  if (pl.max_blocks > SMALL_MAX_BLOCKS) return ABSB_ERR_UNSUPPORTED;
  SmallParams p;
  p.max_blocks = pl.max_blocks;
  p.sc = make_score_params(g, pl, q, codes, qscale, qmin, cent_off, seq_lens, nullptr, nullptr);
  p.tk = make_topk_params(g, nullptr, cent_off, budget, seq_lens, sel_idx_out, sel_cnt, pl.sel_stride, nullptr);
  p.dc = make_decode_params(g, pl, sm_scale, q, k_cache, v_cache, page_table, seq_lens, nullptr, nullptr, pl.sel_stride, out,
                            lse, ws);
  p.dc.some_dense = pl.some_dense;
  const dim3 grid((unsigned)g.Hsel, (unsigned)g.Bt, (unsigned)pl.max_splits);
  const size_t lds = SMALL_LDS_SCRATCH + (size_t)(pl.max_blocks + pl.sel_stride) * 4;
  if (dtype == ABSB_F16)
    launch_small_group<ABSB_F16>(p, g.repr, grid, lds, stream);
  else
    launch_small_group<ABSB_BF16>(p, g.repr, grid, lds, stream);
  return check_launch();
}

}  // namespace absb

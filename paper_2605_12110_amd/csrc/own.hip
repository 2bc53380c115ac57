// The whole decode step in one launch for segments of medium length, where every attention work-group selects for itself.
//
// In the pipelined form (fused.hip) the segment's last estimation work-group selects: it draws its number, reads the scores
// back, selects, writes the list, waits until it is acknowledged, raises a flag, and the attention work-groups, idle
// until then, read flag and list: 5.8 us from the scores to a list in every attention work-group (8 x 32K, 2048 blocks).
// A few thousand scores are little enough for every attention work-group to read them all, as soon as the chunks of
// its segment have counted themselves in, and to select from registers and LDS: the list never goes through
// memory, and two of the hand-overs are gone.  Pipelined / this, us a step: 8 x 32K 23.4 / 21.1, max-min 4 x 20K-64K 18.7 /
// 16.8, group maximum 4 x 64K (4096 blocks) 37.3 / 34.3, a selection per query head 8 x 32K 39.0 / 35.7, 1 x 1024
// blocks 13.2 / 11.4.
//
//   estimation work-group (chunk of a segment): scores its blocks (score_dev.h), stores the scores device-coherently, waits
//     for the acknowledgements and counts itself in.  If the caller wants the list, the last one to do so selects for
//     the caller, in ascending order (topk_dev.h); nobody waits for that.
//   attention work-group (split of a segment): waits until all chunks are counted in, selects, keeps the entries of its
//     split, and goes on as in decode_dev.h.  Blocks and their order are those of the pipelined form's list, so the output is
//     the same bit for bit.
//
// Progress: estimation work-groups never wait.  Attention work-groups wait only for work-groups with lower indices, which
// the hardware starts first; the wait is bounded in time besides (status word, NaN rows).  The segment's last attention
// work-group sets the chunks' counter back to zero.
//
// Compiled with -ffp-contract=off, as the estimation stage requires.
#include "decode_dev.h"
#include "score_dev.h"
#include "topk_dev.h"

namespace absb {

struct OwnParams {
  int32_t some_dense, want_list, nseg;
  ScoreParams sc;
  TopkParams tk;
  DecodeParams dc;
  int32_t* arrived;  // [nseg], ABSB_TICKET_STRIDE apart: chunks whose scores are out
};

constexpr int OWN_THREADS = DEC_THREADS;
constexpr int OWN_LIST = 2048;  // list entries an attention work-group holds
constexpr int OWN_LDS_LIST = (int)(max_sz(DEC_LDS_BYTES, sizeof(TopkShared)) + 15) / 16 * 16;  // behind epilogue and selection

// Entries [e0, e1) of the list of a segment whose blocks compete (at most 256 * R of them), into s_list: the list that
// topk_segment hands over, in its order.  A histogram over the top 11 bits of the keys' range, the bin that holds the K-th,
// exact ranks of the few keys inside it; a crowded bin is cut down by further digits to one key, whose members go by index.
// Barriers and LDS passes bound it, so a thread keeps its keys in registers: slot i is competing block 256 i + tid.
template <int R>
__device__ __forceinline__ void own_select(const SegShape& g, const int32_t* scores, int e0, int e1, TopkShared& sh, int32_t* s_list) {
  constexpr int NT = OWN_THREADS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int Nc = g.hi - g.lo;
  const uint32_t Kc = (uint32_t)(g.K - g.nforced);
  uint32_t key[R];
#pragma unroll
  for (int i = 0; i < R; ++i) key[i] = ordered_key(ld_i32<true>(scores + g.lo + min(i * NT + tid, Nc - 1)));
  for (int i = tid; i < (TOPK_BINS + 64) / 4; i += NT) reinterpret_cast<u32x4*>(sh.hist)[i] = u32x4{0u, 0u, 0u, 0u};

  // ---- range of the keys (copies of the last one change neither end)
  uint32_t kmin = ~0u, kmax = 0u;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    kmin = min(kmin, key[i]);
    kmax = max(kmax, key[i]);
  }
  kmin = wave_reduce_u32(kmin, UMin());
  kmax = wave_reduce_u32(kmax, UMax());
  if (lane == 0) {
    sh.red[wave] = kmin;
    sh.red[TOPK_SLOTS + wave] = kmax;
  }
  __syncthreads();
  kmin = min(min(sh.red[0], sh.red[1]), min(sh.red[2], sh.red[3]));
  kmax = max(max(sh.red[TOPK_SLOTS], sh.red[TOPK_SLOTS + 1]), max(sh.red[TOPK_SLOTS + 2], sh.red[TOPK_SLOTS + 3]));
  const int bits = 32 - __builtin_clz((kmax - kmin) | 1u);
  int shift = bits > TOPK_DIGIT_BITS ? bits - TOPK_DIGIT_BITS : 0;
#pragma unroll
  for (int i = 0; i < R; ++i) key[i] -= kmin;
  const uint32_t valid = (1u << max(0, min(R, (Nc - tid + NT - 1) / NT))) - 1u;  // slots that hold a block
  static_assert(R < 32, "a bit per slot");

  // ---- the bin of the Kc-th key.  (Other slots count into a dump word of their lane: no change of the execution mask.)
#pragma unroll
  for (int i = 0; i < R; ++i) atomicAdd(&sh.hist[valid >> i & 1u ? key[i] >> shift : (uint32_t)(TOPK_BINS + lane)], 1u);
  __syncthreads();
  pick_bin<NT>(sh, tid, lane, wave, Kc);
  uint32_t bin = sh.bcast[0], need = Kc - sh.bcast[1], total;
  const uint32_t inside = sh.bcast[2];
  if (inside <= (uint32_t)TOPK_RANK_MAX) {
    uint32_t above = 0, in = 0;
#pragma unroll
    for (int i = R - 1; i >= 0; --i) {
      above = above << 1 | (uint32_t)(key[i] >> shift > bin);
      in = in << 1 | (uint32_t)(key[i] >> shift == bin);
    }
    above &= valid;
    in &= valid;
    const uint32_t at = block_excl_scan<NT>((uint32_t)__popc(above) | (uint32_t)__popc(in) << 16, sh.wave_b, lane, wave, &total);
    const int cand0 = g.K - (int)need;  // the first admitted candidate's place
    const bool tail = e1 > cand0;
    for (int i = e0 + tid; i < min(e1, g.nforced); i += NT) s_list[i - e0] = g.given(i);
    int pos = g.nforced + (int)(at & 0xffffu) - e0;
    while (above) {
      const int i = __builtin_ctz(above);
      above &= above - 1;
      if (pos >= 0 && pos < e1 - e0) s_list[pos] = g.lo + i * NT + tid;
      ++pos;
    }
    if (tail) {  // exact ranks: key descending, index ascending
      uint32_t slot = at >> 16;
      while (in) {
        const int i = __builtin_ctz(in);
        in &= in - 1;
        sh.cand_key[slot] = pick_reg<R>(key, i);
        sh.cand_idx[slot] = (uint32_t)(g.lo + i * NT + tid);
        ++slot;
      }
      __syncthreads();
      if (tid < (int)inside) {
        const uint32_t mk = sh.cand_key[tid], mi = sh.cand_idx[tid];
        int rank = 0;
#pragma unroll 4
        for (uint32_t u = 0; u < inside; ++u) rank += sh.cand_key[u] > mk || (sh.cand_key[u] == mk && sh.cand_idx[u] < mi);
        const int p = cand0 + rank;
        if (rank < (int)need && p >= e0 && p < e1) s_list[p - e0] = (int)mi;
      }
    }
  } else {
#pragma unroll 1
    while (shift > 0) {  // the next digit, of the bin's keys alone
      const int next = shift > TOPK_DIGIT_BITS ? shift - TOPK_DIGIT_BITS : 0;
      __syncthreads();
      for (int i = tid; i < TOPK_BINS / 4; i += NT) reinterpret_cast<u32x4*>(sh.hist)[i] = u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
#pragma unroll
      for (int i = 0; i < R; ++i)
        if ((valid >> i & 1u) && key[i] >> shift == bin) atomicAdd(&sh.hist[(key[i] >> next) - (bin << (shift - next))], 1u);
      __syncthreads();
      pick_bin<NT>(sh, tid, lane, wave, need);
      bin = (bin << (shift - next)) + sh.bcast[0];
      need -= sh.bcast[1];
      shift = next;
    }
    // in order of the index: forced ones in front, the keys beyond the threshold and the first `need` that equal it, forced ones
    for (int i = e0 + tid; i < e1; i += NT)
      if (i < g.lo || i >= g.lo + (int)Kc) s_list[i - e0] = i < g.lo ? i : g.hi + (i - g.lo - (int)Kc);
    uint32_t gt = 0, eq = 0;  // of the slots before
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const bool real = valid >> i & 1u, beyond = real && key[i] > bin, equal = real && key[i] == bin;
      __syncthreads();
      const uint32_t at = block_excl_scan<NT>((uint32_t)beyond | (uint32_t)equal << 16, sh.wave_a, lane, wave, &total);
      const uint32_t e = eq + (at >> 16);
      const int p = g.lo + (int)(gt + (at & 0xffffu) + min(e, need));
      if ((beyond || (equal && e < need)) && p >= e0 && p < e1) s_list[p - e0] = g.lo + i * NT + tid;
      gt += total & 0xffffu;
      eq += total >> 16;
    }
  }
  __syncthreads();
}

// Waits (thread 0, bounded in time) until the word at `word` is `want`; every thread of the work-group returns whether it
// got there (else *status is set).  Two barriers inside.  `s_word`: one word of LDS.
__device__ __forceinline__ bool wait_for_count(const int32_t* word, int want, int32_t* status, int* s_word) {
  if (threadIdx.x == 0) {
    bool there = ld_i32<true>(word) == want;
    if (!there) {
      const uint64_t t0 = wall_clock64();
      do {
        __builtin_amdgcn_s_sleep(4);
        there = ld_i32<true>(word) == want;
      } while (!there && wall_clock64() - t0 < DEC_WAIT_LIMIT_TICKS);
    }
    if (!there) st_i32<true>(status, 1);
    *s_word = there;
  }
  __syncthreads();
  const bool there = *s_word != 0;
  __syncthreads();  // the word may be reused
  return there;
}

template <int DT, int G>
__device__ __forceinline__ void own_split(const OwnParams& p, int s, int split, char* lds) {
  const DecodeParams& d = p.dc;
  const SegMap sm = seg_map(s, d.g.Hsel, d.g.Rk, d.g.Hkv);
  const int b = sm.b, hs = sm.hs, lb = d.g.heads.log2_block(sm.hk);
  const int tid = threadIdx.x;
  const int pos_begin = split * d.split_tokens;
  const int off = d.cent_off[sm.s];
  const int rows = d.cent_off[sm.s + 1] - off;
  const int L = d.seq_lens[b], T = d.budget[b];
  const int N = blocks_in_use(d.g.tight, rows, L, lb);
  const SegShape g = seg_shape(p.tk, N, lb, L, T);
  const int ntok = min(g.K << lb, d.max_splits * d.split_tokens);
  if (pos_begin >= ntok) return;
  const int pos_end = min(ntok, pos_begin + d.split_tokens);
  const int nsplit = (ntok + d.split_tokens - 1) / d.split_tokens;
  SplitCtx c;
  c.b = b;
  c.hs = hs;
  c.hk = sm.hk;
  c.lb = lb;
  c.L = L;
  c.lP = d.g.log2_page;
  u32x4 qb[4];
  load_q<G>(d.q + ((size_t)b * d.g.Hq + (size_t)hs * G) * ABSB_HEAD_DIM, qb);

  const int e0 = pos_begin >> lb, e1 = ((pos_end - 1) >> lb) + 1;  // at most OWN_LIST entries (checked on the host)
  int32_t* s_list = reinterpret_cast<int32_t*>(lds + OWN_LDS_LIST);
  int* s_word = reinterpret_cast<int*>(lds + DEC_LDS_STATE + 3 * ABSB_MAX_GROUP * DEC_WAVES * 4);
  int32_t* arrived = p.arrived + (size_t)s * ABSB_TICKET_STRIDE;
  const bool scored = !p.some_dense || T < L;  // (else the budget covers the context: nobody scores for this request)
  if (scored && !wait_for_count(arrived, (N + p.sc.chunk - 1) / p.sc.chunk, d.status, s_word)) {
    poison_rows<DT, G>(d, b, hs);
    return;
  }
  if (!g.compete()) {  // no score decides anything
    for (int i = e0 + tid; i < e1; i += OWN_THREADS) s_list[i - e0] = g.given(i);
    __syncthreads();
  } else {
    TopkShared& sh = *reinterpret_cast<TopkShared*>(lds);
    const int32_t* scores = p.sc.scores + score_base(sm, d.g.Rk, off, rows);
    if (g.hi - g.lo <= 8 * OWN_THREADS)
      own_select<8>(g, scores, e0, e1, sh, s_list);
    else
      own_select<OWN_MAX_BLOCKS / OWN_THREADS>(g, scores, e0, e1, sh, s_list);
  }

  const int32_t* pages = d.page_table + (size_t)b * d.g.pt_stride;
  AttnState<G> st;
  st.reset();
  attend_positions<DT, G>(d, c, StretchRef{s_list, e0, e1 - 1}, pages, pos_begin, pos_end, qb, st);
  finish_split<DT, G>(d, s, b, hs, split, nsplit, d.max_splits, st, lds, [&]() __attribute__((always_inline)) {
    if (scored && tid == 0) st_i32<true>(arrived, 0);  // every other split has seen it and drawn its ticket
  });
}

// (What an estimation work-group needs first comes as arguments of their own: see small.hip.)
constexpr int OWN_LEADING = 5 * 8 + 4 * 4;  // bytes of them
template <int DT, int G, int REP>
__global__ __launch_bounds__(OWN_THREADS, 4) void own_step_kernel(addr2 off_lens, addr2 codes_q, int4v shape, uint64_t qscale_, OwnParams p) {
  const auto cent_off = from_addr<const int32_t>(off_lens.x), seq_lens = from_addr<const int32_t>(off_lens.y);
  const auto codes = from_addr<const uint8_t>(codes_q.x);
  const auto q = from_addr<const uint16_t>(codes_q.y);
  const auto qscale = from_addr<const float>(qscale_);
  const int n_score = shape.x, chunks_per_seg = shape.y, Rk_ = shape.z, tight = shape.w;
  extern __shared__ __align__(16) char lds[];
  const int Rk = G == 1 ? Rk_ : 1;  // (groups of one are the only ones that may select per query head)
  const int bid = blockIdx.x, tid = threadIdx.x;
  if (bid >= n_score) {
    int split;
    const int s = segment_split(bid - n_score, p.dc.max_splits, Rk, &split);
    if (Rk == 1 || s < p.nseg) own_split<DT, G>(p, s, split, lds);
    return;
  }
  const int s = bid / chunks_per_seg, chunk = bid - s * chunks_per_seg, store = Rk == 1 ? s : s / Rk;
  const int off = cent_off[store], end = cent_off[store + 1];
  fetch_arguments<OWN_LEADING, sizeof(OwnParams)>();
  const int rows = end - off;
  const SegMap sm = seg_map(s, p.sc.Hsel, Rk, p.sc.Hkv);
  const int lb = p.sc.heads.log2_block(sm.hk);
  if (p.some_dense) {
    // requests whose budget covers their context: no score decides anything, the attention knows its list
    if (p.tk.budget[sm.b] >= seq_lens[sm.b]) {
      if (chunk) return;
      const int N = blocks_in_use(tight, rows, seq_lens, sm.b, lb);
      if (tid == 0) p.tk.sel_cnt[s] = N;
      if (p.want_list)
        for (int i = tid; i < p.tk.sel_stride; i += OWN_THREADS) p.tk.sel_idx[(size_t)s * p.tk.sel_stride + i] = i < N ? i : -1;
      return;
    }
  }
  const int N = blocks_in_use(tight, rows, seq_lens, sm.b, lb);
  if (!score_chunk<DT, REP, true, 8>(p.sc, score_source<REP>(q, qscale, codes, s, store, G, off, N), G, s, chunk,
                                     p.sc.scores + score_base(sm, Rk, off, rows), lds))
    return;
  wait_stores_acknowledged();
  __syncthreads();  // every thread's scores are visible device-wide; the estimation's LDS is free
  int32_t* arrived = p.arrived + (size_t)s * ABSB_TICKET_STRIDE;
  if (!p.want_list) {
    if (tid == 0) {
      __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (chunk == 0) p.tk.sel_cnt[s] = budget_blocks(p.tk.budget[sm.b], lb, N, p.tk.sel_stride);
    }
    return;
  }
  int* s_last = reinterpret_cast<int*>(lds);
  if (tid == 0)
    *s_last = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (N + p.sc.chunk - 1) / p.sc.chunk - 1;
  __syncthreads();
  if (!*s_last) return;
  __syncthreads();  // everybody has read the word before the selection reuses the memory
  TopkShared& sh = *reinterpret_cast<TopkShared*>(lds);
  uint32_t* bitmap = reinterpret_cast<uint32_t*>(lds + ((sizeof(TopkShared) + 15) & ~size_t(15)));
  topk_segment<OWN_THREADS, OWN_MAX_BLOCKS / OWN_THREADS, true>(p.tk, s, sh, bitmap);
}

template <int DT, int G>
static void launch_own_rep(const OwnParams& p, int n_score, int chunks_per_seg, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(OWN_THREADS), lds, stream, addr2{addr(p.sc.cent_off), addr(p.sc.seq_lens)},
                       addr2{addr(p.sc.codes), addr(p.sc.q)}, int4v{n_score, chunks_per_seg, p.sc.Rk, p.sc.tight}, addr(p.sc.qscale), p);
  };
  if (repr == ABSB_REPR_MEAN)
    launch(own_step_kernel<DT, G, 0>);
  else
    launch(own_step_kernel<DT, G, 1>);
}

template <int DT>
static void launch_own_group(const OwnParams& p, int n_score, int chunks_per_seg, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  switch (p.dc.g.Gd) {
    case 1: launch_own_rep<DT, 1>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 2: launch_own_rep<DT, 2>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 3: launch_own_rep<DT, 3>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 4: launch_own_rep<DT, 4>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 5: launch_own_rep<DT, 5>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 6: launch_own_rep<DT, 6>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 7: launch_own_rep<DT, 7>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    default: launch_own_rep<DT, 8>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
  }
}

bool own_fits(const Plan& pl) {
  return pl.max_blocks <= OWN_MAX_BLOCKS && pl.split_tokens <= 8 * OWN_LIST && fused_one_launch_fits(pl);
}

int launch_own(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q, const uint8_t* codes, const float* qscale,
               const float* qmin, const void* k_cache, const void* v_cache, const int32_t* page_table, const int32_t* seq_lens,
               const int32_t* cent_off, const int32_t* budget, int32_t* sel_idx_out, int32_t* sel_cnt, void* out, float* lse,
               char* ws, hipStream_t stream) {
  if (!own_fits(pl)) return ABSB_ERR_UNSUPPORTED;
  OwnParams p;
  int32_t* scores = reinterpret_cast<int32_t*>(ws + pl.ws_scores);
  p.some_dense = pl.some_dense;
  p.want_list = sel_idx_out ? 1 : 0;
  p.nseg = pl.nseg;
  p.sc = make_score_params(g, pl, q, codes, qscale, qmin, cent_off, seq_lens, scores, nullptr);
  p.tk = make_topk_params(g, scores, cent_off, budget, seq_lens, sel_idx_out, sel_cnt, pl.sel_stride, nullptr);
  p.dc = make_decode_params(g, pl, sm_scale, q, k_cache, v_cache, page_table, seq_lens, nullptr, nullptr, pl.sel_stride, out,
                            lse, ws);
  p.dc.budget = budget;
  p.dc.cent_off = cent_off;
  p.dc.status = reinterpret_cast<int32_t*>(ws + pl.ws_status);
  p.arrived = reinterpret_cast<int32_t*>(ws + pl.ws_score_tickets);
  // (one work-group a segment writes the lists when every context is covered)
  const int chunks_per_seg = pl.all_dense ? 1 : (pl.max_blocks + pl.score_chunk - 1) / pl.score_chunk;
  const int n_score = chunks_per_seg * pl.nseg;
  const dim3 grid((unsigned)(n_score + attention_grid(pl.nseg, pl.max_splits, g.Rk)));
  const size_t lds = max_sz(max_sz((size_t)OWN_LDS_LIST + OWN_LIST * 4, topk_lds_bytes(pl.max_blocks)), score_lds_bytes<1>());
  if (dtype == ABSB_F16)
    launch_own_group<ABSB_F16>(p, n_score, chunks_per_seg, g.repr, grid, lds, stream);
  else
    launch_own_group<ABSB_BF16>(p, n_score, chunks_per_seg, g.repr, grid, lds, stream);
  return check_launch();
}

}  // namespace absb

// The whole decode step in one launch for short segments, where every attention work-group scores and selects
// for itself.
//
// At a few hundred blocks a segment the hand-overs of the pipelined form (fused.hip) cost more than the work they
// hand over: scores out, acknowledged, ticket, keys back in, list out, acknowledged, flag, list in, each a
// trip to memory.  Here every work-group (split, segment) reads all of its segment's codes (N * 64 bytes: the
// splits of a segment run on one die and share its L2), keeps the scores in LDS, selects, and attends over its
// own split of the list; only the split-K merge is left of the hand-overs.  Scores, selection and the order of
// the list are those of the pipelined form, so the output is the same bit for bit.  4K context, batch 1,
// 8 heads: 13.4 -> 11.3 us a step.
//
// Compiled with -ffp-contract=off, as the estimation stage requires.
#include "decode_dev.h"
#include "score_dev.h"
#include "topk_dev.h"

namespace absb {

struct SmallParams {
  int32_t nseg, max_blocks;
  ScoreParams sc;
  TopkParams tk;
  DecodeParams dc;
};

constexpr int SMALL_THREADS = DEC_THREADS;
__host__ __device__ constexpr size_t small_max(size_t a, size_t b) { return a > b ? a : b; }
// LDS: scratch of the stages (one after the other), then the scores, then the list
constexpr size_t SMALL_LDS_SCRATCH =
    small_max(small_max((size_t)DEC_LDS_BYTES, topk_lds_bytes(SMALL_MAX_BLOCKS)), small_max(score_lds_bytes<0>(), score_lds_bytes<1>()) + 16) / 16 * 16 + 16;

template <int DT, int G, int REP>
__global__ __launch_bounds__(SMALL_THREADS, 4) void small_step_kernel(SmallParams p) {
  extern __shared__ __align__(16) char lds[];
  // split-major: with a multiple of eight segments, the splits of a segment land on one die
  const int t = blockIdx.x % p.nseg, split = blockIdx.x / p.nseg;
  int32_t* s_score = reinterpret_cast<int32_t*>(lds + SMALL_LDS_SCRATCH);
  int32_t* s_list = s_score + p.max_blocks;
  const SegMap sm = seg_map(t, p.dc.g.Hsel, p.dc.g.Rk, p.dc.g.Hkv);
  const int b = sm.b, hs = sm.hs;
  const int lb = p.dc.g.heads.log2_block[sm.hk];
  const int pos_begin = split * p.dc.split_tokens;

  u32x4 qb[4];
  load_q<G>(p.dc, b, hs, qb);
  SplitCtx c;
  c.b = b;
  c.hs = hs;
  c.hk = sm.hk;
  c.lb = lb;
  c.L = p.dc.seq_lens[b];
  c.lP = p.dc.g.log2_page;
  const int T = p.tk.budget[b];
  const bool everything = p.dc.some_dense && T >= c.L;  // the budget covers the context: no score decides anything
  int N = 0;
  if (!everything)
    N = score_blocks<DT, REP, false, 4>(
        p.sc, t, 0, p.max_blocks, lds, [&](int j, int32_t sc) __attribute__((always_inline)) { s_score[j] = sc; }, nullptr);
  else
    N = blocks_in_use(p.tk.tight, p.tk.cent_off[sm.s + 1] - p.tk.cent_off[sm.s], p.tk.seq_lens, b, lb);

  const int nsel = budget_blocks(T, lb, N, p.dc.sel_stride);
  const int ntok = min(nsel << lb, p.dc.max_splits * p.dc.split_tokens);
  if (pos_begin >= ntok) return;
  const int pos_end = min(ntok, pos_begin + p.dc.split_tokens);
  const int nsplit = (ntok + p.dc.split_tokens - 1) / p.dc.split_tokens;
  __syncthreads();  // the scores are in LDS; the estimation's scratch is free

  TopkShared& sh = *reinterpret_cast<TopkShared*>(lds);
  uint32_t* bitmap = reinterpret_cast<uint32_t*>(lds + ((sizeof(TopkShared) + 15) & ~size_t(15)));
  const LocalSelection loc{s_score, s_list, split == 0};
  topk_segment<SMALL_THREADS, SMALL_MAX_BLOCKS / SMALL_THREADS, false, true, true>(p.tk, t, sh, bitmap, loc);
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
  if (repr == ABSB_REPR_MEAN)
    hipLaunchKernelGGL((small_step_kernel<DT, G, 0>), grid, dim3(SMALL_THREADS), lds, stream, p);
  else
    hipLaunchKernelGGL((small_step_kernel<DT, G, 1>), grid, dim3(SMALL_THREADS), lds, stream, p);
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
  p.nseg = pl.nseg;
  p.max_blocks = pl.max_blocks;
  p.sc = make_score_params(g, pl, q, codes, qscale, qmin, cent_off, seq_lens, nullptr, nullptr);
  p.tk = make_topk_params(g, nullptr, cent_off, budget, seq_lens, sel_idx_out, sel_cnt, pl.sel_stride, nullptr);
  p.dc = make_decode_params(g, pl, sm_scale, q, k_cache, v_cache, page_table, seq_lens, nullptr, nullptr, pl.sel_stride, out,
                            lse, ws);
  p.dc.some_dense = pl.some_dense;
  const dim3 grid((unsigned)(pl.nseg * pl.max_splits));
  const size_t lds = SMALL_LDS_SCRATCH + (size_t)(pl.max_blocks + pl.sel_stride) * 4;
  if (dtype == ABSB_F16)
    launch_small_group<ABSB_F16>(p, g.repr, grid, lds, stream);
  else
    launch_small_group<ABSB_BF16>(p, g.repr, grid, lds, stream);
  return check_launch();
}

}  // namespace absb

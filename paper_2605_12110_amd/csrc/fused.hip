// The whole decode step (score -> select -> attention over the selection, Sec. 3.4 kernels 1-3)
// in ONE launch.
//
// At batch 1 the step moves ~20 MB, i.e. a few microseconds of HBM time, so three dependent
// launches cost more in launch floors and drained pipelines than in work; and at large batches
// the selection of one segment (one CU, instruction-bound) can run under the attention of others.
// Work-groups take one of two roles by their index:
//
//   [0, n_score)        estimation of one chunk of one segment's blocks (score_dev.h).  Scores are
//                       stored device-coherently; the work-group then draws a ticket from the
//                       segment's counter, and the one that draws the last ticket runs the
//                       segment's selection (topk_dev.h): it stores the selected blocks
//                       device-coherently in the order it finds them, raises the segment's flag,
//                       and only then writes the ascending list if the caller asked for one.
//   [n_score, grid)     attention over one split of one segment's selection (decode_dev.h): the
//                       work-group loads its queries, waits for the segment's flag, reads the
//                       blocks with device-coherent loads (attention does not depend on their
//                       order beyond rounding) and proceeds as in the stand-alone kernel
//                       (partials, ticket, the last arriver merges).
//
// This is the form for segments beyond 4096 blocks whose chunks should not wait for each other (shared.hip): grids of
// estimation work-groups that outgrow the chip or are nearly all empty, the group's maximum beyond 8192 blocks.  Shorter
// segments are selected by every attention work-group (own.hip, small.hip), unless the caller asks for splits longer than
// own.hip holds.
//
// Progress: estimation/selection work-groups never wait for anything.  Attention work-groups wait
// only for work-groups with lower indices; the hardware starts work-groups in index order, so
// every work-group waited for is already running or done.  The wait is also bounded in time, so
// the launch ends whatever happens (a wait that ran out sets the status word; its segment's
// output rows are then set to NaN).
//
// Counters (estimation tickets, flags, attention tickets; 256 bytes apart) must be zero when the
// launch starts and are zero again when it ends: absb_workspace_init clears them once.
//
// Compiled with -ffp-contract=off, as the estimation stage requires.
#include "decode_dev.h"
#include "score_dev.h"
#include "topk_dev.h"

namespace absb {

struct FusedParams {
  int32_t some_dense, nseg;
  ScoreParams sc;
  TopkParams tk;
  DecodeParams dc;
  int32_t* score_tickets;  // [nseg], ABSB_TICKET_STRIDE apart
};

constexpr int FUSED_THREADS = DEC_THREADS;

// (What an estimation work-group needs first comes as arguments of their own: see small.hip.)
constexpr int FUSED_LEADING = 5 * 8 + 4 * 4;  // bytes of them
template <int DT, int G, int REP>
__global__ __launch_bounds__(FUSED_THREADS, 4) void fused_step_kernel(addr2 off_lens, addr2 codes_q, int4v shape, uint64_t qscale_, FusedParams p) {
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
    if (Rk == 1 || s < p.nseg) decode_split<DT, G, true>(p.dc, s, split, lds);
    return;
  }
  const int s = bid / chunks_per_seg, chunk = bid - s * chunks_per_seg, store = Rk == 1 ? s : s / Rk;
  const int off = cent_off[store], end = cent_off[store + 1];
  fetch_arguments<FUSED_LEADING, sizeof(FusedParams)>();
  const int rows = end - off;
  const SegMap sm = seg_map(s, p.sc.Hsel, Rk, p.sc.Hkv);
  if (p.some_dense) {
    // requests whose budget covers their context: no score decides anything, the attention knows its list
    if (p.tk.budget[sm.b] >= seq_lens[sm.b]) {
      if (chunk) return;
      const int N = blocks_in_use(tight, rows, seq_lens, sm.b, p.tk.heads.log2_block(sm.hk));
      if (tid == 0) p.tk.sel_cnt[s] = N;
      if (p.tk.sel_idx)
        for (int i = tid; i < p.tk.sel_stride; i += FUSED_THREADS) p.tk.sel_idx[(size_t)s * p.tk.sel_stride + i] = i < N ? i : -1;
      return;
    }
  }
  const int N = blocks_in_use(tight, rows, seq_lens, sm.b, p.sc.heads.log2_block(sm.hk));
  if (!score_chunk<DT, REP, true>(p.sc, score_source<REP>(q, qscale, codes, s, store, G, off, N), G, s, chunk,
                                  p.sc.scores + score_base(sm, Rk, off, rows), lds))
    return;

  // ---- hand the chunk's scores over; the segment's last chunk goes on to select
  wait_stores_acknowledged();
  __syncthreads();  // every thread's scores are visible device-wide; the estimation's LDS is free
  int* s_last = reinterpret_cast<int*>(lds);
  if (tid == 0) {
    int32_t* ticket = p.score_tickets + (size_t)s * ABSB_TICKET_STRIDE;
    const int nchunks = (N + p.sc.chunk - 1) / p.sc.chunk;
    const int last =
        __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nchunks - 1;
    if (last) st_i32<true>(ticket, 0);
    *s_last = last;
  }
  __syncthreads();
  if (!*s_last) return;
  __syncthreads();  // everybody has read the word before the selection reuses the memory

  TopkShared& sh = *reinterpret_cast<TopkShared*>(lds);
  uint32_t* bitmap = reinterpret_cast<uint32_t*>(lds + ((sizeof(TopkShared) + 15) & ~size_t(15)));
  const int tiles = (N + FUSED_THREADS - 1) / FUSED_THREADS;
  if (tiles <= 8)
    topk_segment<FUSED_THREADS, 8, true, true>(p.tk, s, sh, bitmap);
  else if (tiles <= 16)
    topk_segment<FUSED_THREADS, 16, true, true>(p.tk, s, sh, bitmap);
  else if (tiles <= 32)
    topk_segment<FUSED_THREADS, 32, true, true>(p.tk, s, sh, bitmap);
  else if (tiles <= 64)
    topk_segment<FUSED_THREADS, 64, true, true>(p.tk, s, sh, bitmap);
  else
    topk_segment<FUSED_THREADS, 0, true, true>(p.tk, s, sh, bitmap);
  // (the selection raises the segment's flag itself, as soon as its members are known)
}

// Clears the counters at the start of a workspace (all three kinds, and the status word).
__global__ void clear_counters_kernel(int32_t* head, int nwords) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nwords) head[i] = 0;
}

int launch_workspace_init(const Plan& pl, char* ws, hipStream_t stream) {
  const int nwords = (int)(pl.ws_head_bytes / 4);
  hipLaunchKernelGGL(clear_counters_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, stream,
                     reinterpret_cast<int32_t*>(ws), nwords);
  return check_launch();
}

template <int DT, int G>
static void launch_fused_rep(const FusedParams& p, int n_score, int chunks_per_seg, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(FUSED_THREADS), lds, stream,
                       addr2{addr(p.sc.cent_off), addr(p.sc.seq_lens)}, addr2{addr(p.sc.codes), addr(p.sc.q)},
                       int4v{n_score, chunks_per_seg, p.sc.Rk, p.sc.tight}, addr(p.sc.qscale), p);
  };
  if (repr == ABSB_REPR_MEAN)
    launch(fused_step_kernel<DT, G, 0>);
  else
    launch(fused_step_kernel<DT, G, 1>);
}

template <int DT>
static void launch_fused_group(const FusedParams& p, int n_score, int chunks_per_seg, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  switch (p.dc.g.Gd) {
    case 1: launch_fused_rep<DT, 1>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 2: launch_fused_rep<DT, 2>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 3: launch_fused_rep<DT, 3>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 4: launch_fused_rep<DT, 4>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 5: launch_fused_rep<DT, 5>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 6: launch_fused_rep<DT, 6>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 7: launch_fused_rep<DT, 7>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    default: launch_fused_rep<DT, 8>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
  }
}

bool fused_one_launch_fits(const Plan& pl) {
  if (pl.max_blocks > TOPK_MAX_BLOCKS) return false;
  const int64_t cps = (pl.max_blocks + pl.score_chunk - 1) / pl.score_chunk;
  const int64_t grid = cps * pl.nseg + pl.max_splits * ((int64_t)pl.nseg + 8 * ABSB_MAX_GROUP);  // (or a little less)
  return grid < (int64_t(1) << 31) - 1;
}

int launch_fused(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q, const uint8_t* codes,
                 const float* qscale, const float* qmin, const void* k_cache, const void* v_cache, const int32_t* page_table,
                 const int32_t* seq_lens, const int32_t* cent_off, const int32_t* budget, int32_t* sel_idx_out,
                 int32_t* sel_cnt, void* out, float* lse, char* ws, hipStream_t stream) {
  if (!fused_one_launch_fits(pl)) return ABSB_ERR_UNSUPPORTED;
  FusedParams p;
  int32_t* scores = reinterpret_cast<int32_t*>(ws + pl.ws_scores);
  p.sc = make_score_params(g, pl, q, codes, qscale, qmin, cent_off, seq_lens, scores, nullptr);
  // the attention reads the workspace's list (any order); the caller's, if wanted, is ascending
  int32_t* work_list = reinterpret_cast<int32_t*>(ws + pl.ws_sel_idx);
  p.tk = make_topk_params(g, scores, cent_off, budget, seq_lens, sel_idx_out, sel_cnt, pl.sel_stride, nullptr);
  p.tk.work_list = work_list;
  p.tk.flags = reinterpret_cast<int32_t*>(ws + pl.ws_flags);
  p.dc = make_decode_params(g, pl, sm_scale, q, k_cache, v_cache, page_table, seq_lens, work_list, sel_cnt,
                            pl.sel_stride, out, lse, ws);
  p.dc.budget = budget;
  p.some_dense = p.dc.some_dense = pl.some_dense;
  p.dc.cent_off = cent_off;
  p.dc.flags = reinterpret_cast<int32_t*>(ws + pl.ws_flags);
  p.dc.status = reinterpret_cast<int32_t*>(ws + pl.ws_status);
  p.score_tickets = reinterpret_cast<int32_t*>(ws + pl.ws_score_tickets);
  // (one work-group a segment writes the lists when every context is covered)
  const int chunks_per_seg = pl.all_dense ? 1 : (pl.max_blocks + pl.score_chunk - 1) / pl.score_chunk;
  p.nseg = pl.nseg;
  const int n_score = chunks_per_seg * pl.nseg;
  const dim3 grid((unsigned)(n_score + attention_grid(pl.nseg, pl.max_splits, g.Rk)));
  const size_t lds = max_sz(max_sz((size_t)DEC_LDS_BYTES, topk_lds_bytes(pl.max_blocks)), score_lds_bytes<1>());
  if (dtype == ABSB_F16)
    launch_fused_group<ABSB_F16>(p, n_score, chunks_per_seg, g.repr, grid, lds, stream);
  else
    launch_fused_group<ABSB_BF16>(p, n_score, chunks_per_seg, g.repr, grid, lds, stream);
  return check_launch();
}

}  // namespace absb

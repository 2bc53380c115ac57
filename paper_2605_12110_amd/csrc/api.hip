// Host side of libabsb.so: argument validation, size planning, workspace carving and the
// extern "C" entry points.  Nothing here touches the device except through the launchers.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "common.h"

namespace absb {

static inline bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }
static inline int ilog2(int64_t v) {
  int r = 0;
  while ((int64_t(1) << (r + 1)) <= v) ++r;
  return r;
}
static inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }
static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The split-K partials of a step with that many splits a segment: outputs, and (max, rounded sum, exact sum, -) a head.
static size_t partial_bytes(const Geometry& g, const Plan& p, int64_t splits) {
  const size_t rows = (size_t)p.nseg * (size_t)splits * g.Gd;
  return align256(rows * ABSB_HEAD_DIM * 4) + align256(rows * 4 * 4);
}
// Blocks per estimation work-group: 256, or 512 where that would make more than two work-groups a compute unit in the
// one-launch step, which pay their prologue and keep attention work-groups from their places.  256 / 512, us a step: group
// maximum 4 x 64K 32.1 / 33.0 (512 work-groups of 256), 8 x 32K 21.0 / 21.1 (512); a selection per query head, 8 x 32K 38.3 /
// 35.7 (2048).
static int default_score_chunk(const Plan& p) { return p.nseg * ceil_div(p.max_blocks, 256) > 512 ? 512 : 256; }
constexpr int MAX_SPLITS_CHOSEN = 64;  // of a segment, unless the caller says what a split is

int make_plan(const absb_layer* layer, const absb_batch* batch, bool need_budget, int32_t sel_stride_in,
              Geometry* geo, Plan* pl, bool lean) {
  if (!layer || !batch) return ABSB_ERR_NULL;
  if (!layer->block_size || !batch->seq_lens_host) return ABSB_ERR_NULL;
  if (need_budget && !batch->budget_host) return ABSB_ERR_NULL;
  if (layer->head_dim != ABSB_HEAD_DIM) return ABSB_ERR_UNSUPPORTED;
  if (layer->dtype != ABSB_F16 && layer->dtype != ABSB_BF16) return ABSB_ERR_UNSUPPORTED;
  const int Hq = layer->num_q_heads, Hkv = layer->num_kv_heads;
  if (Hq < 1 || Hkv < 1 || Hq % Hkv != 0) return ABSB_ERR_BAD_SHAPE;
  if (Hq / Hkv > ABSB_MAX_GROUP || Hkv > ABSB_MAX_KV_HEADS) return ABSB_ERR_UNSUPPORTED;
  if (layer->block_repr != ABSB_REPR_MEAN && layer->block_repr != ABSB_REPR_MINMAX) return ABSB_ERR_UNSUPPORTED;
  const int P = layer->page_size;
  if (!is_pow2(P) || P < 8 || P > 65536) return ABSB_ERR_BAD_SHAPE;
  const int64_t sp = layer->kv_stride_page, sh = layer->kv_stride_head, st = layer->kv_stride_tok;
  if (sp <= 0 || sh <= 0 || st < ABSB_HEAD_DIM || (sp % 8) || (sh % 8) || (st % 8)) return ABSB_ERR_BAD_SHAPE;
  if (!(layer->sm_scale >= 0.0f) || std::isinf(layer->sm_scale)) return ABSB_ERR_BAD_SHAPE;
  if (layer->sink_tokens < 0 || layer->recent_tokens < 0) return ABSB_ERR_BAD_SHAPE;
  if (layer->selection != ABSB_SELECT_GROUP && layer->selection != ABSB_SELECT_PER_QUERY_HEAD &&
      layer->selection != ABSB_SELECT_GROUP_MAX)
    return ABSB_ERR_UNSUPPORTED;
  if (layer->selection == ABSB_SELECT_GROUP_MAX && layer->block_repr != ABSB_REPR_MEAN) return ABSB_ERR_UNSUPPORTED;
  const bool per_q = layer->selection == ABSB_SELECT_PER_QUERY_HEAD;
  const int Hsel = per_q ? Hq : Hkv;
  const int Bt = batch->batch;
  if (Bt < 1 || (int64_t)Bt * Hsel > 65535) return ABSB_ERR_BAD_SHAPE;  // segments index grid.y

  Geometry g = {};
  g.Bt = Bt;
  g.Hq = Hq;
  g.Hkv = Hkv;
  g.G = Hq / Hkv;
  g.Hsel = Hsel;
  g.Gd = per_q ? 1 : g.G;
  g.Rk = per_q ? g.G : 1;
  g.agg_max = layer->selection == ABSB_SELECT_GROUP_MAX;
  g.log2_page = ilog2(P);
  g.pt_stride = batch->pt_stride;
  g.repr = layer->block_repr;
  g.tight = batch->cap_lens_host ? 0 : 1;
  g.sink_tokens = layer->sink_tokens;
  g.recent_tokens = layer->recent_tokens;
  g.s_page = sp;
  g.s_head = sh;
  g.s_tok = st;
  for (int h = 0; h < Hkv; ++h) {
    const int B = layer->block_size[h];
    if (!is_pow2(B) || B < 8 || B > 128) return ABSB_ERR_BAD_BLOCK_SIZE;
    // both are powers of two, so B | P or P | B holds: blocks never straddle a page partially
    g.heads.packed[h >> 2] |= (uint32_t)ilog2(B) << (8 * (h & 3));
  }

  Plan p = {};
  const absb_launch_opts& opts = batch->opts;
  if (opts.step_form < ABSB_STEP_AUTO || opts.step_form > ABSB_STEP_PER_STAGE) return ABSB_ERR_BAD_SHAPE;
  if (opts.split_tokens < 0 || opts.split_tokens % 64 || opts.score_chunk < 0 || opts.score_chunk % 64 ||
      opts.unit_tokens < 0 || opts.unit_tokens % 64 || opts.counters_zero < 0 || opts.counters_zero > 1)
    return ABSB_ERR_BAD_SHAPE;
  p.nseg = Bt * Hsel;
  p.nstore = Bt * Hkv;
  int64_t max_len = 0, in_use = 0;  // in_use: blocks of the current lengths (p.total: of the layout's)
  for (int b = 0; b < Bt; ++b) {
    const int64_t L = batch->seq_lens_host[b];
    if (L < 1) return ABSB_ERR_BAD_SHAPE;
    const int64_t cap = batch->cap_lens_host ? batch->cap_lens_host[b] : L;  // the layout's length
    if (cap < L) return ABSB_ERR_BAD_SHAPE;
    if (L > max_len) max_len = L;
    p.build_max_chunks = std::max(p.build_max_chunks, build_chunks((int)L));
    if (batch->budget_host) {
      if (batch->budget_host[b] < 1) return ABSB_ERR_BAD_SHAPE;
      (batch->budget_host[b] >= L ? p.some_dense : p.all_dense) = 1;  // (all_dense holds "some are not" until the end)
    }
    for (int h = 0; h < Hkv; ++h) {
      const int lb = g.heads.log2_block(h);  // (shifts: a 64-bit division a segment and quantity is most of a plan's time)
      const int64_t B = int64_t(1) << lb, N = (L + B - 1) >> lb;
      int64_t K = N;
      if (batch->budget_host) {
        const int64_t kb = (batch->budget_host[b] + B - 1) >> lb;
        if (kb < K) K = kb;
        if (K > p.sel_stride) p.sel_stride = (int32_t)K;
      }
      if (sel_stride_in > 0 && sel_stride_in < K) K = sel_stride_in;
      p.total += (cap + B - 1) >> lb;
      in_use += N;
      if (N > p.max_blocks) p.max_blocks = (int32_t)N;
      const int64_t tok = K * B;
      if (tok > p.max_tokens) p.max_tokens = tok;
      p.sum_tokens += tok * g.Rk;  // every selection segment of the KV head reads its own tokens
    }
  }
  p.all_dense = p.some_dense && !p.all_dense;
  if (!batch->budget_host) p.sel_stride = p.max_blocks;
  // entry points that select (they are the ones that need the budgets) refuse on the host what the
  // selection cannot hold, before anything is enqueued
  if (need_budget && p.max_blocks > ABSB_MAX_SEL_BLOCKS) return ABSB_ERR_UNSUPPORTED;
  if (p.total >= (int64_t(1) << 31) - 1) return ABSB_ERR_BAD_SHAPE;
  if ((int64_t)batch->pt_stride < ceil_div(max_len, P)) return ABSB_ERR_BAD_SHAPE;

  // How absb_decode_fused is enqueued.  Measured on MI355X (three copies of a layer in
  // turn, here and below): one launch against one per stage, 1 request of 4K 9.3 / 15.1 us, 8 of 32K 20.2 / 26.2, 1 of
  // 128K 16.0 / 20.5, 16 of 8K-128K 40.6 / 47.6.  A selection by one work-group holds 16384 blocks in its registers;
  // beyond (keys re-read) it takes several times longer (1 request of 256K 63.5 us a step against 19.4 shared, below).  Very long lists (budgets near the context) go to the per-stage
  // path: its attention kernel reads the lists through the L2.
  const bool by_shape = p.max_blocks <= 16384 && p.sel_stride <= 4096;
  // Segments beyond 4096 blocks: the work-groups that score a segment share its selection, unless the grid of them is
  // large.  They wait for each other, twice as long as the scores alone take, and those that are waiting hold back the
  // others beyond four a compute unit.  So: at most two a compute unit, or four if hardly any of the grid is empty, or (empty
  // ones leave at once) as long as the ones with blocks are three a compute unit, four beyond 16384 blocks, where the
  // alternative is a launch per stage.  How many have blocks is taken as how many the blocks in use fill; a layout's room to
  // grow counts for nothing.  One work-group's selection / shared, us a step (those, of the grid): 16 x 10K-73K in blocks of 16, max-min 34.4 / 31.8 and 8 % 59.3 / 57.0 (660 of 1152), 8 x 20K-128K, 4096 36.6 / 35.8
  // (470 of 2048), 16 x 8K-128K 42.0 / 40.8 (575 of 2048); 16 x 5K-128K in blocks of 8 to 128 40.4 / 41.1 (830 of 4096), 16 x
  // 96K 41.3 / 41.5 (900 of 1536), 16 x 128K in blocks of 16 48.8 / 49.4 (all of 2048); and a grid that is nearly all empty
  // keeps the few that wait from their places: one request of 131000 beside 16 of 7 to 1000 tokens 21.9 / 27.1 (150 of 2176), two
  // beside 14 of 2000 31.4 / 31.0 (283 of 2048).  Per stage / shared: 4 x 256K, 2048 30.8 / 29.7 (794 of 2048).  Query heads that select for themselves leave the order in which they find each other's rows in
  // a die's L2: 2 x 128K 26.5 / 24.3 (906 of 1024), but 16 x 10K-73K 87 / 109 (2600 of 4608).
  // (This is a limit on time, not what makes the waits end: beyond 96128 blocks a segment three fit a compute unit, not
  // four, and 1024 of them still take 52 us against 90 at 16 segments of 131072 blocks.  See "Progress" in shared.hip.)
  const int shared_chunk = shared_chunk_blocks(p.max_blocks);
  const int64_t shared_grid = (int64_t)p.nseg * ceil_div(p.max_blocks, shared_chunk), shared_real = ceil_div(in_use * g.Rk, shared_chunk);
  const bool shared_pays = shared_grid <= 512 || (shared_grid <= 1024 && 2 * shared_real >= shared_grid) ||
                           (g.Rk == 1 && shared_real <= (p.max_blocks > 16384 ? 1024 : 768) && 8 * shared_real >= shared_grid);
  const bool by_units = !by_shape && p.max_blocks > 16384 && shared_pays;
  p.step_form = opts.step_form != ABSB_STEP_AUTO ? opts.step_form
                : by_shape ? ABSB_STEP_PIPELINED : by_units ? ABSB_STEP_UNITS : ABSB_STEP_PER_STAGE;
  p.one_launch = p.step_form != ABSB_STEP_PER_STAGE;
  // Short segments: every attention work-group scores and selects for itself (small.hip) as long as reading all
  // of a segment's codes takes less than the hand-over it saves.  This / scored once (own.hip), 8 heads, blocks of 16: 1 request,
  // budget 512, 256 blocks 8.7 / 10.5 us, 512 9.7 / 10.9, 768 11.5 / 11.0, 1024 12.0 / 11.0; 4 requests, budget 2048, 512
  // 14.3 / 14.8, 768 16.0 / 15.0; 16 requests, budget 2048, 512 28.9 / 30.0, 768 31.2 / 30.9.  Max-min rows, 4 requests, 512 12.7 / 13.3,
  // 768 14.8 / 13.5.  Group maximum, 512 blocks, four heads 10.2 / 10.9.  With a selection per query head the scores are G
  // times as many.
  p.small = opts.step_form == ABSB_STEP_AUTO && by_shape && g.Rk == 1 && p.max_blocks <= SMALL_MAX_BLOCKS;
  // split-K shape, in 64-token granules (one work-group step).  Swept on MI355X (256 CUs) when three
  // work-groups fitted a compute unit; four do now, and the sweep has not been repeated: the kernel was
  // fastest with about two work-groups per CU, all resident at once and each streaming as long as
  // possible; a work-group needs at least two steps to amortise its set-up; and since one work-group
  // merges a segment's partials, a segment should not be cut into more than 64.
  // (the shape follows the batch, not the enqueue knob: every form of the step then cuts the
  // segments alike)
  int st_tok = opts.split_tokens;
  const int64_t cap_tok = ceil_div(ceil_div(p.max_tokens, MAX_SPLITS_CHOSEN), 64) * 64;
  if (st_tok <= 0 && p.step_form == ABSB_STEP_UNITS && !lean && opts.unit_tokens > 0)
    st_tok = (int)std::max<int64_t>(opts.unit_tokens, cap_tok);
  if (st_tok <= 0) {
    const int64_t target_wgs = 640;
    int64_t t = ceil_div(ceil_div(p.sum_tokens, target_wgs), 64) * 64;
    if (t < 128) t = p.sum_tokens / 128 >= 128 ? 128 : 64;  // one step only when two would leave the chip idle
    // In the one-launch step the attention work-groups of a large batch start segment by segment as
    // the lists come out, not all at once: sweeps there favour ~1100 work-groups of at least four
    // steps (config 4 43.5 -> 42.0 us, config 5 at budget 8192 41.4 -> 39.2).
    if (by_shape && batch->budget_host && p.sum_tokens >= 65536)
      t = std::max<int64_t>(256, ceil_div(ceil_div(p.sum_tokens, 1100), 64) * 64);
    // Segments of (nearly) equal lists: all splits the same size, if that makes two or four work-groups a compute unit (of
    // 256) or hardly fewer, of at least 512 tokens each while two are left: a split's set-up and its part of the
    // merge are paid less often, and no compute unit has one more than the others.  Two only where the estimation
    // work-groups leave two of the four places of every compute unit free: where they take more, the attention's go to
    // where places are left or come free first, and two are no longer two everywhere.  Without / with, us a step: 4 x 64K
    // group maximum, lists of 8192 tokens 39.5 / 37.1, 8 x 64K, lists of 3000 33.5 / 30.3 (512 estimation work-groups), a
    // selection per query head, 8 x 32K, 4096 72.3 / 65.5 (1024 and 1024); with more than 512 beside two a compute unit it
    // would be 37.9 / 44.1 (8 x 96K, 4096: 768) and 27.3 / 33.3 (per query head, 4 x 64K, 2048: 1024).  Other numbers
    // lose: 920 work-groups 61.7 / 62.1 (5 x 40K, 14519), 576 35.3 / 37.6 (9 x 60K, 4096), 768 45.7 / 47.6 (8 x 40K, 16
    // heads, 3200); so do splits of which the last is hardly filled, and segments beyond 8192 blocks, whose estimation
    // work-groups are many: 36.8 / 43.3 (5 x 72K-150K, 6506).
    if (by_shape && batch->budget_host && p.max_blocks <= 8192 && p.sum_tokens >= 131072 &&
        20 * p.sum_tokens >= 19 * p.nseg * p.max_tokens) {
      int64_t even = std::max<int64_t>({256, std::min<int64_t>(512, ceil_div(p.sum_tokens, 512)), ceil_div(p.sum_tokens, 1024)});
      even = ceil_div(ceil_div(p.max_tokens, std::max<int64_t>(1, p.max_tokens / even)), 64) * 64;
      const int64_t splits = ceil_div(p.max_tokens, even), wgs = p.nseg * splits;
      const bool two = wgs >= 448 && wgs <= 512 && p.nseg * ceil_div(p.max_blocks, default_score_chunk(p)) <= 512;
      if (25 * splits * even <= 26 * p.max_tokens && (two || (wgs >= 960 && wgs <= 1024))) t = even;
    }
    if (t < cap_tok) t = cap_tok;
    st_tok = (int)t;
  }
  // Rows that a step reads once and that the 256 MB last-level cache could not keep for the next step anyway
  // are read nontemporally: they neither wait for a place in the caches nor push the codes and lists
  // out (dense read of 537 MB: 111 -> 99 us, 142 MB of a batch: 51.1 -> 47.2 us a step; 67 MB, which a cache
  // may still hold, 27.0 -> 27.5).  Query heads with lists of their own share rows: those stay cached.
  p.stream_rows = g.Rk == 1 && p.sum_tokens * 512 >= int64_t(96) << 20;
  p.split_tokens = st_tok;
  p.max_splits = (int32_t)ceil_div(p.max_tokens, st_tok);
  if (p.max_splits < 1) p.max_splits = 1;
  if (p.max_splits > 65535) return ABSB_ERR_BAD_SHAPE;
  if ((int64_t)p.max_splits * st_tok >= (int64_t(1) << 31)) return ABSB_ERR_BAD_SHAPE;  // positions are 32-bit

  // The pipelined form shares the selection, too, from where a segment's scores are too many for every attention
  // work-group to read (own.hip).  Own selection / shared at 4096 blocks: 1 request, 4096 15.7 / 16.5 us, 8 requests, 2048 23.3 / 23.9.
  // One work-group's selection / shared beyond: 6144 blocks, 1 request, 512 14.5 / 13.8, 4 requests, 2048 21.1 / 19.1, group
  // maximum, 8192, 1 request 17.8 / 16.8, 8 requests 31.5 / 30.1.  Level with max-min rows and a list for the caller: 8 x 9K-75K (4700
  // blocks), 1024 20.5 / 20.6, 2048 27.7 / 26.9, 4096 34.8 / 34.9; without it 20.7 / 20.6, 28.0 / 26.9, 34.5 / 33.6; mean rows with it
  // 19.1 / 18.3, 27.3 / 24.9, 34.0 / 32.5.  Beyond 8192 blocks the group's maximum keeps to one work-group's
  // selection, and that costs: group maximum, blocks of 8, lists of 2048, 12288 blocks, 1 request 19.5 / 17.0, 8 requests 38.4 / 38.4, 16384
  // blocks, 1 request 20.0 / 17.3, 4 requests 28.7 / 25.8.  That line dates from when one work-group's selection was the faster there and has yet
  // to be moved.  (Forced beyond 16384 blocks, the pipelined form keeps to one work-group a segment and to the ascending order.)
  p.shared = p.step_form == ABSB_STEP_UNITS || (p.step_form == ABSB_STEP_PIPELINED && !p.small && (!g.agg_max || p.max_blocks <= 8192) &&
                                                p.max_blocks > OWN_MAX_BLOCKS && p.max_blocks <= 16384 && shared_pays);
  const bool rows = !lean && p.nseg <= SHARED_MAX_SEGMENTS;  // the workspace has histogram rows and room for candidates
  p.shared = p.shared && rows && shared_fits(p);

  p.score_chunk = opts.score_chunk > 0 ? opts.score_chunk : p.one_launch ? default_score_chunk(p) : 256;
  p.own = p.step_form == ABSB_STEP_PIPELINED && !p.small && !p.shared && own_fits(p);

  // workspace: the split counters of the attention kernel come first, at the same place in every
  // carving (nothing else ever writes there); behind them the three users overlap, since they
  // never run concurrently on one workspace
  p.ws_tickets = 0;
  const size_t ctr = align256((size_t)p.nseg * ABSB_TICKET_STRIDE * 4);
  p.ws_score_tickets = ctr;
  p.ws_flags = 2 * ctr;
  p.ws_status = 3 * ctr;
  p.ws_finished = 3 * ctr + 256;
  p.ws_listed = 4 * ctr + 256;
  p.ws_counts = 5 * ctr + 256;  // SHARED_MAX_CHUNKS words a segment: as far apart as the counters
  static_assert(SHARED_MAX_CHUNKS <= ABSB_TICKET_STRIDE, "a segment's counts words take the place of one counter");
  p.ws_hist = 6 * ctr + 256;
  const size_t head = p.ws_hist + (rows ? (size_t)p.nseg * SHARED_HIST_BINS * 4 : 0);
  p.ws_head_bytes = head;
  size_t o = head;
  p.ws_scores = o;
  o += align256((size_t)p.total * g.Rk * 4);
  p.ws_sel_idx = o;
  o += align256((size_t)p.nseg * (size_t)(p.sel_stride > 0 ? p.sel_stride : 1) * 4);
  p.ws_sel_cnt = o;
  o += align256((size_t)p.nseg * 4);
  p.ws_part_o = o;
  p.ws_part_ml = o + align256((size_t)p.nseg * p.max_splits * g.Gd * ABSB_HEAD_DIM * 4);
  o += partial_bytes(g, p, p.max_splits);
  p.ws_decode_bytes = o;  // the stand-alone decode uses the same offsets (the head is left unused)
  p.ws_cand = o;  // the shared selection's candidates
  if (rows) o += align256((size_t)p.total * g.Rk * 8);
  p.ws_fused_bytes = o;
  size_t bo = head;
  p.ws_cent = bo;
  const size_t width = (size_t)ABSB_HEAD_DIM * (g.repr + 1);  // values per block
  bo += align256((size_t)p.total * width * 4);
  p.ws_meet = bo;
  // the chunks of a segment share its words in groups of at most 16 (~10 ns an update of a line), or in the most groups
  const auto copies_for = [](int chunks) {
    int copies = 1;
    while (copies < BUILD_MAX_COPIES && copies * 16 < chunks) copies *= 2;
    return copies;
  };
  p.build_copies = copies_for(p.build_max_chunks);
  // ... in a place that never shrinks as contexts grow, as every other part: a workspace for a capacity has room for every
  // length on the way
  const int most = build_most_chunks((int)max_len);
  p.build_pitch = (int32_t)(align256((size_t)meet_words((int)width, copies_for(most), most) * 4) / 4);
  bo += (size_t)p.nstore * p.build_pitch * 4;
  p.ws_build_bytes = bo;
  p.ws_bytes = p.ws_fused_bytes > p.ws_build_bytes ? p.ws_fused_bytes : p.ws_build_bytes;

  if (geo) *geo = g;
  if (pl) *pl = p;
  return ABSB_OK;
}

// A workspace for every length on the way to the capacity.  All parts grow with the lengths (the build's shared words
// because they are placed for the most chunks of any shorter context) except the partials: longer lists get longer splits,
// and so at times fewer of them.
static size_t growing_workspace_bytes(const absb_layer* layer, const absb_batch* batch, const Plan& now) {
  absb_batch longest = *batch;
  longest.seq_lens_host = batch->cap_lens_host;
  longest.pt_stride = INT32_MAX;  // (the page table may grow with the contexts)
  Geometry g;
  Plan p;
  if (make_plan(layer, &longest, false, 0, &g, &p) != ABSB_OK) return now.ws_bytes;
  const int64_t most = batch->opts.split_tokens > 0 ? p.max_splits : std::min<int64_t>(MAX_SPLITS_CHOSEN, ceil_div(p.max_tokens, 64));
  const size_t step = p.ws_fused_bytes - partial_bytes(g, p, p.max_splits) + partial_bytes(g, p, std::max<int64_t>(most, p.max_splits));
  return std::max({now.ws_bytes, p.ws_build_bytes, step});
}

static int check_ws(const void* ws, size_t have, size_t need) {
  if (need == 0) return ABSB_OK;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) || have < need) return ABSB_ERR_WORKSPACE;
  return ABSB_OK;
}

static float resolve_scale(const absb_layer* layer) {
  return layer->sm_scale > 0.0f ? layer->sm_scale : 1.0f / std::sqrt((float)layer->head_dim);
}

}  // namespace absb

using namespace absb;

extern "C" {

int absb_plan(const absb_layer* layer, const absb_batch* batch, int32_t* cent_off_host,
              int64_t* total_centroids, int32_t* sel_stride, size_t* workspace_bytes) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (cent_off_host) {
    int32_t acc = 0;
    cent_off_host[0] = 0;
    for (int b = 0; b < g.Bt; ++b)
      for (int h = 0; h < g.Hkv; ++h) {
        const int64_t B = layer->block_size[h];
        const int64_t cap = batch->cap_lens_host ? batch->cap_lens_host[b] : batch->seq_lens_host[b];
        acc += (int32_t)((cap + B - 1) / B);
        cent_off_host[b * g.Hkv + h + 1] = acc;
      }
  }
  if (total_centroids) *total_centroids = p.total;
  if (sel_stride) *sel_stride = p.sel_stride;
  if (workspace_bytes) *workspace_bytes = batch->cap_lens_host ? growing_workspace_bytes(layer, batch, p) : p.ws_bytes;
  return ABSB_OK;
}

int absb_build_centroids(const absb_layer* layer, const absb_batch* batch, const void* k_cache, uint8_t* codes,
                         float* qscale, float* qmin, void* workspace, size_t workspace_bytes, void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!k_cache || !codes || !qscale || !qmin || !batch->seq_lens || !batch->page_table || !batch->cent_off)
    return ABSB_ERR_NULL;
  rc = check_ws(workspace, workspace_bytes, p.ws_build_bytes);
  if (rc != ABSB_OK) return rc;
  return launch_build(g, p, layer->dtype, k_cache, batch->page_table, batch->seq_lens, batch->cent_off, codes,
                      qscale, qmin, static_cast<char*>(workspace), static_cast<hipStream_t>(stream));
}

int absb_score(const absb_layer* layer, const absb_batch* batch, const void* q, const uint8_t* codes,
               const float* qscale, int32_t* scores, int32_t* score_exp, void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!q || !codes || !qscale || !scores || !batch->cent_off || !batch->seq_lens) return ABSB_ERR_NULL;
  if (g.agg_max && !batch->qmin) return ABSB_ERR_NULL;
  return launch_score(g, p, layer->dtype, q, codes, qscale, batch->qmin, batch->cent_off, batch->seq_lens, scores, score_exp,
                      static_cast<hipStream_t>(stream));
}

int absb_topk(const absb_layer* layer, const absb_batch* batch, const int32_t* scores, int32_t* sel_idx,
              int32_t* sel_cnt, int32_t sel_stride, void* workspace, size_t workspace_bytes, void* stream) {
  (void)workspace;
  (void)workspace_bytes;  // the selection needs no scratch memory
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, true, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!scores || !sel_idx || !sel_cnt || !batch->cent_off || !batch->budget) return ABSB_ERR_NULL;
  if (!batch->seq_lens) return ABSB_ERR_NULL;
  if (sel_stride < p.sel_stride) return ABSB_ERR_BAD_SHAPE;
  return launch_topk(g, p, scores, batch->cent_off, batch->budget, batch->seq_lens, sel_idx, sel_cnt, sel_stride, nullptr,
                     static_cast<hipStream_t>(stream));
}

int absb_sparse_decode(const absb_layer* layer, const absb_batch* batch, const void* q, const void* k_cache,
                       const void* v_cache, const int32_t* sel_idx, const int32_t* sel_cnt, int32_t sel_stride,
                       void* out, float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  if (sel_stride < 1) return layer && batch ? ABSB_ERR_BAD_SHAPE : ABSB_ERR_NULL;
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, sel_stride, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!q || !k_cache || !v_cache || !sel_idx || !sel_cnt || !out || !batch->seq_lens || !batch->page_table)
    return ABSB_ERR_NULL;
  rc = check_ws(workspace, workspace_bytes, p.ws_decode_bytes);
  if (rc != ABSB_OK) return rc;
  return launch_decode(g, p, layer->dtype, resolve_scale(layer), q, k_cache, v_cache, batch->page_table,
                       batch->seq_lens, sel_idx, sel_cnt, sel_stride, out, lse, static_cast<char*>(workspace),
                       batch->opts.counters_zero == 1, static_cast<hipStream_t>(stream));
}

static int decode_fused(const absb_layer* layer, const absb_batch* batch, bool lean, const void* q, const uint8_t* codes,
                        const float* qscale, const void* k_cache, const void* v_cache, void* out, float* lse,
                        int32_t* sel_idx_out, int32_t* sel_cnt_out, void* workspace, size_t workspace_bytes,
                        void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, true, 0, &g, &p, lean);
  if (rc != ABSB_OK) return rc;
  if (!q || !codes || !qscale || !k_cache || !v_cache || !out || !batch->seq_lens || !batch->page_table ||
      !batch->cent_off || !batch->budget)
    return ABSB_ERR_NULL;
  if (g.agg_max && !batch->qmin) return ABSB_ERR_NULL;
  rc = check_ws(workspace, workspace_bytes, p.ws_fused_bytes);
  if (rc != ABSB_OK) return rc;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  int32_t* scores = reinterpret_cast<int32_t*>(ws + p.ws_scores);
  int32_t* sel_idx = sel_idx_out ? sel_idx_out : reinterpret_cast<int32_t*>(ws + p.ws_sel_idx);
  int32_t* sel_cnt = sel_cnt_out ? sel_cnt_out : reinterpret_cast<int32_t*>(ws + p.ws_sel_cnt);
  if (p.shared)
    return launch_shared(g, p, layer->dtype, resolve_scale(layer), q, codes, qscale, batch->qmin, k_cache, v_cache, batch->page_table,
                         batch->seq_lens, batch->cent_off, batch->budget, sel_idx_out, sel_cnt, out, lse, ws, st);
  if (p.small)
    return launch_small(g, p, layer->dtype, resolve_scale(layer), q, codes, qscale, batch->qmin, k_cache, v_cache, batch->page_table,
                        batch->seq_lens, batch->cent_off, batch->budget, sel_idx_out, sel_cnt, out, lse, ws, st);
  if (p.own)
    return launch_own(g, p, layer->dtype, resolve_scale(layer), q, codes, qscale, batch->qmin, k_cache, v_cache, batch->page_table,
                      batch->seq_lens, batch->cent_off, batch->budget, sel_idx_out, sel_cnt, out, lse, ws, st);
  if (p.step_form == ABSB_STEP_PIPELINED && fused_one_launch_fits(p))
    return launch_fused(g, p, layer->dtype, resolve_scale(layer), q, codes, qscale, batch->qmin, k_cache, v_cache, batch->page_table,
                        batch->seq_lens, batch->cent_off, batch->budget, sel_idx_out, sel_cnt, out, lse, ws, st);
  if (p.all_dense) {
    // no score decides anything; the lists (0, 1, 2, ...) are only written if the caller wants them
    if (sel_idx_out || sel_cnt_out) {
      rc = launch_topk(g, p, scores, batch->cent_off, batch->budget, batch->seq_lens, sel_idx, sel_cnt, p.sel_stride, nullptr, st);
      if (rc != ABSB_OK) return rc;
    }
    return launch_decode_dense(g, p, layer->dtype, resolve_scale(layer), q, k_cache, v_cache, batch->page_table,
                               batch->seq_lens, batch->cent_off, out, lse, ws, st);
  }
  rc = launch_score(g, p, layer->dtype, q, codes, qscale, batch->qmin, batch->cent_off, batch->seq_lens, scores, nullptr, st);
  if (rc != ABSB_OK) return rc;
  // the selection kernel also clears the split counters of the attention kernel behind it
  rc = launch_topk(g, p, scores, batch->cent_off, batch->budget, batch->seq_lens, sel_idx, sel_cnt, p.sel_stride,
                   reinterpret_cast<int32_t*>(ws + p.ws_tickets), st);
  if (rc != ABSB_OK) return rc;
  return launch_decode(g, p, layer->dtype, resolve_scale(layer), q, k_cache, v_cache, batch->page_table,
                       batch->seq_lens, sel_idx, sel_cnt, p.sel_stride, out, lse, ws, true, st);
}

int absb_decode_fused(const absb_layer* layer, const absb_batch* batch, const void* q, const uint8_t* codes,
                      const float* qscale, const void* k_cache, const void* v_cache, void* out, float* lse,
                      int32_t* sel_idx_out, int32_t* sel_cnt_out, void* workspace, size_t workspace_bytes,
                      void* stream) {
  return decode_fused(layer, batch, false, q, codes, qscale, k_cache, v_cache, out, lse, sel_idx_out, sel_cnt_out, workspace,
                      workspace_bytes, stream);
}

int absb_step_form_used(const absb_layer* layer, const absb_batch* batch) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, true, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (p.step_form == ABSB_STEP_UNITS && p.shared) return ABSB_STEP_UNITS;
  if (p.step_form == ABSB_STEP_PIPELINED && fused_one_launch_fits(p)) return ABSB_STEP_PIPELINED;
  return ABSB_STEP_PER_STAGE;
}

int absb_status_offset(const absb_layer* layer, const absb_batch* batch, size_t* offset) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!offset) return ABSB_ERR_NULL;
  *offset = p.ws_status;
  return ABSB_OK;
}

int absb_workspace_init(const absb_layer* layer, const absb_batch* batch, void* workspace, size_t workspace_bytes,
                        void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  rc = check_ws(workspace, workspace_bytes, p.ws_head_bytes);
  if (rc != ABSB_OK) return rc;
  return launch_workspace_init(p, static_cast<char*>(workspace), static_cast<hipStream_t>(stream));
}

int absb_tail_init(const absb_layer* layer, const absb_batch* batch, const void* k_cache, float* tail, void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!k_cache || !tail || !batch->seq_lens || !batch->page_table) return ABSB_ERR_NULL;
  return launch_append(g, p, layer->dtype, false, k_cache, batch->page_table, batch->seq_lens, nullptr, nullptr,
                       nullptr, nullptr, tail, nullptr, static_cast<hipStream_t>(stream));
}

int absb_append_token(const absb_layer* layer, const absb_batch* batch, const void* k_cache, uint8_t* codes,
                      const float* qscale, const float* qmin, float* tail, int32_t* clamped, void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!k_cache || !codes || !qscale || !qmin || !tail || !batch->seq_lens || !batch->page_table || !batch->cent_off)
    return ABSB_ERR_NULL;
  return launch_append(g, p, layer->dtype, true, k_cache, batch->page_table, batch->seq_lens, batch->cent_off, codes,
                       qscale, qmin, tail, clamped, static_cast<hipStream_t>(stream));
}

int absb_head_recall(const absb_layer* layer, const absb_batch* batch, const float* lse_selected,
                     const float* lse_dense, float* recall, void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, false, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  if (!lse_selected || !lse_dense || !recall) return ABSB_ERR_NULL;
  return launch_head_recall(lse_selected, lse_dense, recall, p.nstore, g.G, static_cast<hipStream_t>(stream));
}

int absb_assign_block_sizes(int32_t n_samples, int32_t n_heads, int32_t n_cand, const float* recall_host,
                            const int32_t* cand, double tau, int32_t* block_size_out, double* mean_out) {
  if (!recall_host || !cand || !block_size_out) return ABSB_ERR_NULL;
  if (n_samples < 1 || n_heads < 1 || n_cand < 1 || n_cand > 64 || !(tau >= 0.0)) return ABSB_ERR_BAD_SHAPE;
  if (!is_pow2(cand[0]) || cand[0] < 8 || cand[0] > 128) return ABSB_ERR_BAD_BLOCK_SIZE;
  for (int k = 1; k < n_cand; ++k) {
    if (!is_pow2(cand[k]) || cand[k] > 128) return ABSB_ERR_BAD_BLOCK_SIZE;
    if (cand[k] <= cand[k - 1]) return ABSB_ERR_BAD_SHAPE;
  }
  // Eq. (2), head by head.  First Recall(h, B) for every candidate: the mean over the samples (which
  // are whatever the caller measured recall on: one row per request of every calibration input),
  // accumulated in binary64 in sample order.  Then the candidates are tried from the largest down:
  // the set {B : Recall(h, B) >= tau * Recall(h, B_min)} is read as written, so the first one that
  // passes is its maximum, whatever the candidates below it do; B_min is in the set for tau <= 1 and
  // is the answer when nothing passes.
  const size_t row = (size_t)n_heads * n_cand;
  for (int h = 0; h < n_heads; ++h) {
    double recall_of[64];
    for (int k = 0; k < n_cand; ++k) recall_of[k] = 0.0;
    const float* sample = recall_host + (size_t)h * n_cand;
    for (int i = 0; i < n_samples; ++i, sample += row)
      for (int k = 0; k < n_cand; ++k) recall_of[k] += (double)sample[k];
    for (int k = 0; k < n_cand; ++k) {
      recall_of[k] /= (double)n_samples;
      if (mean_out) mean_out[(size_t)h * n_cand + k] = recall_of[k];
    }
    const double floor_of_head = tau * recall_of[0];
    int chosen = n_cand - 1;
    while (chosen > 0 && !(recall_of[chosen] >= floor_of_head)) --chosen;
    block_size_out[h] = cand[chosen];
  }
  return ABSB_OK;
}

int absb_stream_read(const void* src, size_t bytes, void* sink, void* stream) {
  if (!src || !sink) return ABSB_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(src) & 15) return ABSB_ERR_BAD_SHAPE;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return ABSB_ERR_HIP;
  return launch_stream_read(src, bytes, static_cast<uint32_t*>(sink), cus, static_cast<hipStream_t>(stream));
}

const char* absb_strerror(int status) {
  switch (status) {
    case ABSB_OK: return "ok";
    case ABSB_ERR_NULL: return "a required pointer is NULL";
    case ABSB_ERR_BAD_SHAPE: return "invalid shape, length, stride, budget or list width";
    case ABSB_ERR_BAD_BLOCK_SIZE: return "block size must be a power of two in [8,128]";
    case ABSB_ERR_UNSUPPORTED: return "unsupported configuration (head_dim, group size, head count or dtype)";
    case ABSB_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case ABSB_ERR_HIP: return "HIP launch failed";
    case ABSB_ERR_STATIC_WORKSPACE:
      return "the batch needs more scratch memory than the library's built-in array holds (ABSB_STATIC_WORKSPACE_BYTES); "
             "use absb_decode_fused with a workspace of the caller's";
    default: return "unknown status";
  }
}

}  // extern "C"

// ------------------------------------------------------------------ the step for callers that cannot allocate
//
// absb_decode_fused with the workspace taken from device memory that the library's code object
// holds: a file-scope array, one copy per GPU, there from the moment the library is loaded on that
// GPU until the process ends.  Nothing is allocated or freed by the call, by the library or by any
// runtime routine it uses.
namespace absb {

static __device__ __align__(256) unsigned char scratch[ABSB_STATIC_WORKSPACE_BYTES];

constexpr int kMaxDevices = 64;
struct StaticWorkspace {
  char* ptr = nullptr;        // this device's copy of `scratch` (a device address; the array's name is not one)
  size_t head_bytes = 0;      // counters cleared for a batch shape whose counters take this many bytes
};
static StaticWorkspace g_static_ws[kMaxDevices];
static std::mutex g_static_ws_lock;

// Device address of the current device's scratch array, resolved once per device.
static int static_workspace(int* dev_out, StaticWorkspace** slot) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ABSB_ERR_HIP;
  StaticWorkspace& w = g_static_ws[dev];
  if (!w.ptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ABSB_ERR_HIP;
    w.ptr = static_cast<char*>(p);
    w.head_bytes = 0;
  }
  *dev_out = dev;
  *slot = &w;
  return ABSB_OK;
}

}  // namespace absb

extern "C" {

int absb_decode_fused_static(const absb_layer* layer, const absb_batch* batch, const void* q, const uint8_t* codes,
                             const float* qscale, const void* k_cache, const void* v_cache, void* out, float* lse,
                             int32_t* sel_idx_out, int32_t* sel_cnt_out, void* stream) {
  Geometry g;
  Plan p;
  int rc = make_plan(layer, batch, true, 0, &g, &p);
  if (rc != ABSB_OK) return rc;
  // Near the array's size the shared selection's memory (4 KB a segment, 8 bytes a block) is given up before the call is.
  const bool lean = p.ws_fused_bytes > (size_t)ABSB_STATIC_WORKSPACE_BYTES;
  if (lean) {
    rc = make_plan(layer, batch, true, 0, &g, &p, true);
    if (rc != ABSB_OK) return rc;
    if (p.ws_fused_bytes > (size_t)ABSB_STATIC_WORKSPACE_BYTES) return ABSB_ERR_STATIC_WORKSPACE;
  }
  std::lock_guard<std::mutex> hold(g_static_ws_lock);
  int dev = 0;
  StaticWorkspace* w = nullptr;
  rc = static_workspace(&dev, &w);
  if (rc != ABSB_OK) return rc;
  // The array keeps what the last call left.  The counters at its start are zero after every
  // completed step, but where they sit follows the batch shape: a first call on this device, or a
  // call whose counters take a different number of bytes than the last one's, clears them first
  // (a small fill kernel on the caller's stream, ordered before the step).
  if (w->head_bytes != p.ws_head_bytes) {
    rc = launch_workspace_init(p, w->ptr, static_cast<hipStream_t>(stream));
    if (rc != ABSB_OK) return rc;
    w->head_bytes = p.ws_head_bytes;
  }
  return decode_fused(layer, batch, lean, q, codes, qscale, k_cache, v_cache, out, lse, sel_idx_out, sel_cnt_out, w->ptr,
                      (size_t)ABSB_STATIC_WORKSPACE_BYTES, stream);
}

}  // extern "C"

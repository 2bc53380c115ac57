// The whole decode step in one launch for long segments, with the selection shared by the work-groups that score.
//
// A selection by one work-group passes over all keys of a segment on one compute unit: 9 us for 16384 blocks,
// twice that for 32768, while the attention waits.  Here the scores never leave the work-groups that computed
// them: what they exchange is a histogram, a few kilobytes a segment whatever its length.
//
//   estimation work-group (chunk c of segment t):
//     1. scores its blocks into LDS (score_dev.h) and counts them in bins that follow from the query's fixed-point
//        weights alone, so that every chunk of the segment uses the same ones; adds its counts to the segment's row
//        in memory (device atomics);
//     2. waits until the segment's chunks have counted themselves in, then reads the row until it holds all blocks that
//        compete: every chunk finds the bin that holds the K_s-th largest score;
//     3. writes its blocks above the bin to its own stretch of the segment's list area, the few inside it
//        (candidates) as (score, index) pairs, and how many of each it has to its counts word;
//     4. the chunk that gets here last clears what chunks share, writes the caller's list and count if asked, and takes over where the
//        bin is too crowded to rank its members (ties): the exact selection of topk_dev.h over the segment's
//        scores, which the chunks then store instead of lists.
//   attention work-group (split of segment t): waits for the chunks' counts words, places its stretch of the
//     selection (blocks above the bin in ascending order, then the admitted candidates by rank, which only
//     the splits that reach that far work out, exactly: score descending, index ascending), and goes on as in
//     decode_dev.h.  The order is a function of the scores alone.
//
// The bins: 1024 of equal width over the range that the scores can take at all (every code lies in [0, 15]).  With
// 128 independent channels that is about 45 standard deviations, so a bin holds 0.2 % of the blocks in the
// tail where the threshold lies.
//
// Progress rests on work-groups starting in the grid's order, not on the whole grid being resident (a caller may
// ask for this form at any size, a large segment's LDS lets three work-groups into a compute unit, and other
// streams may hold places).  Estimation work-groups come first, a segment's chunks side by side, and wait only
// for the other chunks of their segment.  So of those that have started, only the segment that is being
// dispatched can be waiting for one that has not, with at most SHARED_MAX_CHUNKS - 1 work-groups: every
// segment before it finishes and gives its places back.  Attention work-groups wait only for work-groups
// with lower indices.  Several launches at once hold back at most that many places each.  Every wait is
// bounded in time; one that runs out sets the status word and leaves NaN in the segment's rows.
//
// Counters, histogram rows and counts words must be zero when the launch starts and are zero again when it ends:
// the chunk that finishes last clears what only chunks use, while the attention runs, the work-group that merges a
// segment's partials the words that the attention reads, ahead of the merge.  (With all of it left to that work-group, behind
// its merge, a step ended later: 1 x 128K 17.3 us against 16.5, 1 x 256K 20.6 / 19.7.)  A counter that did not start at zero
// shows: a chunk that takes itself for the last one and goes by what the others have found sees whether all their counts words
// are out, and the work-group that merges sees whether a last chunk has been there and nobody has counted after it.
//
// Compiled with -ffp-contract=off, as the estimation stage requires.
#include "decode_dev.h"
#include "score_dev.h"
#include "topk_dev.h"

namespace absb {

constexpr int SHARED_THREADS = DEC_THREADS;
constexpr int SHARED_BINS = SHARED_HIST_BINS;
constexpr int SHARED_BPT = SHARED_BINS / SHARED_THREADS;              // bins a thread owns
static_assert(SHARED_BINS == 4 * SHARED_THREADS, "a thread clears four words of a row");
constexpr int SHARED_PER = SHARED_MAX_CHUNK / SHARED_THREADS;         // blocks of a chunk a thread owns at most
constexpr int SHARED_MAX_CAND = 512;                                  // longest list of candidates that is ranked
constexpr uint32_t SHARED_CROWDED = 0x40000000u;                      // counts word: the list comes from the last chunk
constexpr uint32_t SHARED_THERE = 0x80000000u;                        // counts word: always set (zero = not yet)
constexpr int SHARED_GAVE_UP = 1 << 20;                               // arrived: beyond any number of chunks

struct SharedParams {
  int32_t want_list;
  ScoreParams sc;
  TopkParams tk;
  DecodeParams dc;
  int32_t* arrived;    // [nseg], ABSB_TICKET_STRIDE apart: chunks that have sent their counts; more: one has waited too long
  int32_t* finished;   // [nseg] likewise: chunks whose counts word is out
  uint32_t* listed;    // [nseg][SHARED_MAX_CHUNKS]: the counts words once more, for the last chunk
  int32_t* crowd_flag; // [nseg] likewise: 1 = the crowded segment's work list is complete
  uint32_t* hist;      // [nseg][SHARED_BINS]
  uint32_t* counts;    // [nseg][SHARED_MAX_CHUNKS]
  int32_t* area;       // [total]: a chunk's blocks above the bin, at its first block's place (crowded: its scores)
  uint64_t* cand;      // [total]: its candidates, (index << 32 | score - lowest possible score)
};

// LDS of an estimation work-group behind the estimation's own
constexpr int SHARED_LDS_SCORE = 4096;                                            // int32 [SHARED_MAX_CHUNK]
constexpr int SHARED_LDS_HIST = SHARED_LDS_SCORE + SHARED_MAX_CHUNK * 4;          // uint32 [SHARED_BINS]
constexpr int SHARED_LDS_WORDS = SHARED_LDS_HIST + SHARED_BINS * 4;               // 64 words of scan / broadcast scratch
constexpr int SHARED_LDS_SCORING = SHARED_LDS_WORDS + 64 * 4;
static_assert(score_lds_bytes<0>() <= SHARED_LDS_SCORE && score_lds_bytes<1>() <= SHARED_LDS_SCORE, "estimation LDS");
// LDS of an attention work-group: candidates share the epilogue's bytes, the list does not
constexpr int SHARED_LDS_CAND_KEY = 0;                                            // uint32 [SHARED_MAX_CAND]
constexpr int SHARED_LDS_CAND_IDX = SHARED_LDS_CAND_KEY + SHARED_MAX_CAND * 4;    // uint32 [SHARED_MAX_CAND]
static_assert(SHARED_LDS_CAND_IDX + SHARED_MAX_CAND * 4 <= DEC_LDS_STATE, "attention LDS");
constexpr int SHARED_LDS_LIST = (DEC_LDS_BYTES + 15) / 16 * 16;                   // int32 [SHARED_LIST]
constexpr int SHARED_LDS_ATTENTION = SHARED_LDS_LIST + SHARED_LIST * 4;

__host__ __device__ constexpr size_t shared_max(size_t a, size_t b) { return a > b ? a : b; }

// The bins of a segment's scores.
struct ScoreBins {
  uint32_t lo, mul;  // mul: bins per unit of score, in 2^-32; 0: a bin is one score
  __device__ __forceinline__ explicit ScoreBins(const ScoreRange& r) {
    lo = (uint32_t)r.lo;
    const uint32_t span = (uint32_t)r.hi - (uint32_t)r.lo;
    mul = span < (uint32_t)SHARED_BINS ? 0u : (uint32_t)((float)SHARED_BINS * 0x1p32f / ((float)span + 1.0f));
  }
  __device__ __forceinline__ int of(int32_t score) const {
    const uint32_t rel = (uint32_t)score - lo;
    return (int)min(mul ? __umulhi(rel, mul) : rel, (uint32_t)SHARED_BINS - 1u);
  }
};

// The chunk that holds entry i, `before` counting the entries of the chunks before: the last u < C with before[u] <= i.
__device__ __forceinline__ int chunk_of(const int32_t* before, int C, int i) {
  int u = 0;
#pragma unroll
  for (int sb = SHARED_MAX_CHUNKS / 2; sb > 0; sb >>= 1)
    if (u + sb < C && before[u + sb] <= i) u += sb;
  return u;
}

// ------------------------------------------------------------------ estimation
template <int DT, int G, int REP>
__device__ __forceinline__ void shared_chunk(const SharedParams& p, const ScoreSource& src, int t, int c, int off, int rows, char* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t* s_score = reinterpret_cast<int32_t*>(lds + SHARED_LDS_SCORE);
  uint32_t* s_hist = reinterpret_cast<uint32_t*>(lds + SHARED_LDS_HIST);
  uint32_t* s_words = reinterpret_cast<uint32_t*>(lds + SHARED_LDS_WORDS);  // [0,16), [16,32) scan slots, 32.. broadcast
#pragma unroll
  for (int k = 0; k < SHARED_BPT; ++k) s_hist[k * SHARED_THREADS + tid] = 0;
  const int chunk = p.sc.chunk, j0 = c * chunk;
  ScoreRange range;
  // Lengths and budgets are wanted behind the scores.  Their lines are cold: asked for first, or through scalar
  // loads (which return in any order, so that a wait for one is a wait for all), they would delay the scores; vector
  // loads behind those of the codes do not.
  const SegMap sm = seg_map(t, p.tk.Hsel, p.tk.Rk, p.tk.Hkv);
  int T = 0, L = 0;
  const int lb = p.tk.heads.log2_block(sm.hk), N = src.N;
  const bool any = score_blocks<DT, REP, true, 8>(
      p.sc, src, G, t, j0, chunk, lds, [&](int j, int32_t sc) __attribute__((always_inline)) { s_score[j - j0] = sc; }, &range,
      [&]() __attribute__((always_inline)) {
        const int same = sm.b + (tid >> 10);  // (a lane's own index as far as the compiler can tell)
        T = p.tk.budget[same];
        L = p.tk.seq_lens[same];
      });
  if (!any) return;
  const int n = min(N - j0, chunk), C = (N + chunk - 1) / chunk;
  __syncthreads();

  const SegShape g = seg_shape(p.tk, N, lb, __builtin_amdgcn_readfirstlane(L), __builtin_amdgcn_readfirstlane(T));
  int32_t* out = p.want_list ? p.tk.sel_idx + (size_t)t * p.tk.sel_stride : nullptr;
  if (!g.compete()) {  // nobody waits for this segment's chunks
    if (c != 0) return;
    if (tid == 0) p.tk.sel_cnt[t] = g.K;
    if (out)
      for (int i = tid; i < p.tk.sel_stride; i += SHARED_THREADS) out[i] = i < g.K ? g.given(i) : -1;
    return;
  }

  // ---- 1. the chunk's counts into the segment's row.  A thread owns `per` consecutive blocks (at most SHARED_PER);
  // bin of a forced block: beyond all, of none: before all
  const ScoreBins bins(range);
  const int per = (n + SHARED_THREADS - 1) / SHARED_THREADS, ia = tid * per;
  int bin[SHARED_PER];
#pragma unroll
  for (int k = 0; k < SHARED_PER; ++k) {
    bin[k] = -1;
    if (k < per && ia + k < n) {
      const int j = j0 + ia + k;
      bin[k] = bins.of(s_score[ia + k]);
      if (j >= g.lo && j < g.hi)
        atomicAdd(&s_hist[bin[k]], 1u);
      else
        bin[k] = SHARED_BINS;
    }
  }
  __syncthreads();
  uint32_t* row = p.hist + (size_t)t * SHARED_BINS;
#pragma unroll
  for (int k = 0; k < SHARED_BPT; ++k) {
    const uint32_t v = s_hist[k * SHARED_THREADS + tid];
    if (v) __hip_atomic_fetch_add(row + k * SHARED_THREADS + tid, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // ---- 2. the threshold bin: thread tid owns SHARED_BPT bins, thread 0 the highest.  The row is complete when it holds
  // every block that competes; that alone says so, and whoever reads it then has it.  The counter of the chunks only says
  // when looking is worth while, so nobody waits for his additions to be acknowledged before he raises it; it is one word.
  // (Looking at the row itself, 4 KB a chunk and turn, keeps a large grid from its scores: 2 x 504807 tokens in blocks of
  // 16, 1024 estimation work-groups, 33.4 us a step against 29.0; 3 x 325527 51.2 / 47.6; 1 x 131072 17.7 / 17.4.  With
  // the additions acknowledged first: 30.5, 48.0 and 17.7.)
  const int first = SHARED_BINS - SHARED_BPT * (tid + 1);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(row, 0, SHARED_BINS * 4, 0x00020000);
  int32_t* arrived = p.arrived + (size_t)t * ABSB_TICKET_STRIDE;
  const uint64_t since = wall_clock64();
  if (tid == 0) {
    int v = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    while (v < C && wall_clock64() - since < DEC_WAIT_LIMIT_TICKS) {
      __builtin_amdgcn_s_sleep(2);
      v = ld_i32<true>(arrived);
    }
  }
  __syncthreads();
  uint32_t cnt[SHARED_BPT], total, above;
  for (int turn = 0;; turn ^= 1) {  // (scratch words in turns: a wave is at most one barrier ahead)
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < SHARED_BPT; k += 4) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (first + k) * 4, 0, 16 /* sc1 */);
      cnt[k] = v.x, cnt[k + 1] = v.y, cnt[k + 2] = v.z, cnt[k + 3] = v.w;
    }
    if (tid == 0) s_words[40 + turn] = ld_i32<true>(arrived) > C || wall_clock64() - since >= DEC_WAIT_LIMIT_TICKS;
#pragma unroll
    for (int k = 0; k < SHARED_BPT; ++k) sum += cnt[k];
    above = block_excl_scan<SHARED_THREADS>(sum, s_words + 16 * turn, lane, wave, &total);
    if (s_words[40 + turn]) {  // one chunk that gives up speaks for all; the segment's attention runs into its limit, too
      if (tid == 0) {
        st_i32<true>(arrived, SHARED_GAVE_UP);
        st_i32<true>(p.dc.status, 1);
      }
      return;
    }
    if (total == (uint32_t)(g.hi - g.lo)) break;
    __builtin_amdgcn_s_sleep(2);
  }
  const uint32_t Kc = (uint32_t)(g.K - g.nforced);
#pragma unroll
  for (int k = SHARED_BPT - 1; k >= 0; --k) {
    if (above < Kc && Kc <= above + cnt[k]) {
      s_words[33] = (uint32_t)(first + k);
      s_words[34] = above;
      s_words[35] = cnt[k];
    }
    above += cnt[k];
  }
  __syncthreads();
  const int d1 = (int)s_words[33];
  const int need = (int)(Kc - s_words[34]), n_in = (int)s_words[35];
  const bool whole = need == n_in;
  const bool crowded = n_in > SHARED_MAX_CAND && !whole;

  // ---- 3. classify
  const int64_t place = score_base(sm, p.tk.Rk, off, rows) + j0;
  uint32_t word = SHARED_THERE | SHARED_CROWDED;
  if (crowded) {
#pragma unroll 1
    for (int i = tid; i < n; i += SHARED_THREADS) st_i32<true>(p.area + place + i, s_score[i]);
  } else {
    // blocks above the bin (all of it, if it is admitted whole): sure; inside it: candidates
    const int bar = whole ? d1 - 1 : d1;
    uint32_t mine = 0;  // sure ones, candidates << 16
#pragma unroll
    for (int k = 0; k < SHARED_PER; ++k) mine += bin[k] > bar ? 1u : bin[k] == d1 ? 0x10000u : 0u;
    uint32_t at = block_excl_scan<SHARED_THREADS>(mine, s_words + 16, lane, wave, &total);
#pragma unroll
    for (int k = 0; k < SHARED_PER; ++k) {
      const int j = j0 + ia + k;
      if (bin[k] > bar) {
        st_i32<true>(p.area + place + (at & 0xffffu), j);
        ++at;
      } else if (bin[k] == d1) {
        const uint32_t rel = (uint32_t)s_score[ia + k] - (uint32_t)range.lo;
        __hip_atomic_store(p.cand + place + (at >> 16), ((uint64_t)(uint32_t)j << 32) | rel, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        at += 0x10000u;
      }
    }
    word = SHARED_THERE | total;  // at most 2048 of either kind
  }
  wait_stores_acknowledged();
  __syncthreads();
  const bool relied = out || crowded;  // the last chunk reads what the others have found
  if (tid == 0) {
    uint32_t* counts = p.counts + (size_t)t * SHARED_MAX_CHUNKS + c;
    st_i32<true>(reinterpret_cast<int32_t*>(counts), (int32_t)word);
    if (relied) st_i32<true>(reinterpret_cast<int32_t*>(p.listed + (size_t)t * SHARED_MAX_CHUNKS + c), (int32_t)word);
    wait_stores_acknowledged();
    s_words[36] = __hip_atomic_fetch_add(p.finished + (size_t)t * ABSB_TICKET_STRIDE, 1, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) == C - 1;
  }
  __syncthreads();
  if (!s_words[36]) return;

  // ---- 4. the segment's last chunk: every other one has read the row and drawn its number.  Before it goes by what the others
  // have found, its first wave looks whether all counts words are out: with one missing, `finished` did not start at zero, and
  // nothing is cleared, which the merging work-group sees.
  uint32_t* s_key = reinterpret_cast<uint32_t*>(lds);                       // [SHARED_MAX_CAND]
  uint32_t* s_idx = s_key + SHARED_MAX_CAND;                                // [SHARED_MAX_CAND]
  uint32_t* s_bm = reinterpret_cast<uint32_t*>(lds + SHARED_LDS_SCORING);   // a bit per block
  int32_t* s_sure = reinterpret_cast<int32_t*>(s_idx + SHARED_MAX_CAND);    // [SHARED_MAX_CHUNKS]
  int32_t* s_cand = s_sure + SHARED_MAX_CHUNKS;                             // [SHARED_MAX_CHUNKS]
  const int nwords = out && !crowded ? (N + 31) >> 5 : 0;
  int32_t* listed = reinterpret_cast<int32_t*>(p.listed + (size_t)t * SHARED_MAX_CHUNKS);
  u32x4 sums = {0u, 0u, 0u, 0u};  // blocks above the bin, candidates, whether a word is missing
  if (relied) {
    const uint32_t cw = wave == 0 && lane < C ? (uint32_t)ld_i32<true>(listed + lane) : 0u;  // lane = chunk
#pragma unroll 1
    for (int w = tid; w < nwords; w += SHARED_THREADS) s_bm[w] = 0;
    if (wave == 0) {
      const uint32_t ns = cw & 0xffffu, ncd = (cw >> 16) & 0xfffu;
      uint32_t sure, ncand;
      const uint32_t sure_to = wave_incl_scan_u32(ns, &sure), cand_to = wave_incl_scan_u32(ncd, &ncand);
      const uint32_t missing = __any(lane < C && cw == 0u);
      s_sure[lane] = (int)(sure_to - ns);
      s_cand[lane] = (int)(cand_to - ncd);
      if (lane == 0) *reinterpret_cast<u32x4*>(s_words + 44) = u32x4{sure, ncand, missing, 0u};
    }
    __syncthreads();
    sums = *reinterpret_cast<const u32x4*>(s_words + 44);
    if (sums.z) return;
  }
  const auto clear = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, rsrc, tid * 16, 0, 16 /* sc1 */);
    if (relied && tid < SHARED_MAX_CHUNKS) st_i32<true>(listed + tid, 0);
    if (tid == 0) {
      st_i32<true>(arrived, 0);
      st_i32<true>(p.finished + (size_t)t * ABSB_TICKET_STRIDE, 0);
    }
  };
  if (crowded) {
    clear();
    __syncthreads();  // the words are read; the selection's LDS overlaps them
    TopkShared& sh = *reinterpret_cast<TopkShared*>(lds);
    uint32_t* bitmap = reinterpret_cast<uint32_t*>(lds + ((sizeof(TopkShared) + 15) & ~size_t(15)));
    topk_segment<SHARED_THREADS, 0, true, true>(p.tk, t, sh, bitmap);  // raises the segment's flag itself
    return;
  }
  if (tid == 0) p.tk.sel_cnt[t] = g.K;
  if (!out) {
    clear();
    return;
  }
  // the caller's ascending list, from the chunks' lists: a bitmap, then one scan
  const int64_t seg_place = place - j0;
  const uint32_t sure = sums.x, ncand = sums.y;
  for (int i = tid; i < (int)sure; i += SHARED_THREADS) {
    const int u = chunk_of(s_sure, C, i);
    const int j = ld_i32<true>(p.area + seg_place + (int64_t)u * chunk + (i - s_sure[u]));
    atomicOr(&s_bm[j >> 5], 1u << (j & 31));
  }
  const int nc = min((int)ncand, SHARED_MAX_CAND);
  for (int i = tid; i < nc; i += SHARED_THREADS) {
    const int u = chunk_of(s_cand, C, i);
    const uint64_t pr = __hip_atomic_load(p.cand + seg_place + (int64_t)u * chunk + (i - s_cand[u]), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
    s_key[i] = (uint32_t)pr;
    s_idx[i] = (uint32_t)(pr >> 32);
  }
  __syncthreads();
  clear();  // (ahead of the loads above these would wait for its acknowledgement: 1 x 256K with the list, 0.1 us a step)
#pragma unroll 1
  for (int k = tid; k < nc; k += SHARED_THREADS) {
    const uint32_t mk = s_key[k], mi = s_idx[k];
    int rank = 0;
    for (int u = 0; u < nc; ++u) rank += s_key[u] > mk || (s_key[u] == mk && s_idx[u] < mi);
    if (rank < need) atomicOr(&s_bm[mi >> 5], 1u << (mi & 31));
  }
  for (int i = g.K + tid; i < p.tk.sel_stride; i += SHARED_THREADS) out[i] = -1;
  __syncthreads();
  const int wpt = (nwords + SHARED_THREADS - 1) / SHARED_THREADS;
  const int wa = min(tid * wpt, nwords), wb = min(wa + wpt, nwords);
  uint32_t bits = 0;
  for (int w = wa; w < wb; ++w) bits += (uint32_t)__popc(s_bm[w]);
  uint32_t at = block_excl_scan<SHARED_THREADS>(bits, s_words, lane, wave, &total);
  for (int w = wa; w < wb; ++w) {
    uint32_t left = s_bm[w];
    while (left) {
      const int bpos = __builtin_ctz(left);
      left &= left - 1;
      if (at < (uint32_t)g.K) out[at] = (w << 5) + bpos;  // always true for consistent counts; keeps stores in bounds
      ++at;
    }
  }
}

// ------------------------------------------------------------------ attention
template <int DT, int G>
__device__ __forceinline__ void shared_split(const SharedParams& p, int t, int split, char* lds) {
  const DecodeParams& d = p.dc;
  const SegMap sm = seg_map(t, d.g.Hsel, d.g.Rk, d.g.Hkv);
  const int b = sm.b, hs = sm.hs, lb = d.g.heads.log2_block(sm.hk);
  const int tid = threadIdx.x, lane = tid & 63;
  const int pos_begin = split * d.split_tokens;
  const int off = d.cent_off[sm.s];
  const int rows = d.cent_off[sm.s + 1] - off;
  const int L = d.seq_lens[b];
  const int N = blocks_in_use(d.g.tight, rows, d.seq_lens, b, lb);
  const SegShape g = seg_shape(p.tk, N, lb, L, d.budget[b]);
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

  const int e0 = pos_begin >> lb, e1 = ((pos_end - 1) >> lb) + 1;  // at most SHARED_LIST entries (checked on the host)
  int32_t* s_list = reinterpret_cast<int32_t*>(lds + SHARED_LDS_LIST);
  int* s_word = reinterpret_cast<int*>(lds + DEC_LDS_STATE + 3 * ABSB_MAX_GROUP * DEC_WAVES * 4);
  const int chunk = p.sc.chunk, C = (N + chunk - 1) / chunk;
  const bool compete = g.compete();
  bool crowded = false;
  if (!compete) {
    for (int i = e0 + tid; i < e1; i += SHARED_THREADS) s_list[i - e0] = g.given(i);
    __syncthreads();
  } else {
    // ---- the chunks' counts words: lane i waits for chunk i's
    const int32_t* counts = reinterpret_cast<const int32_t*>(p.counts + (size_t)t * SHARED_MAX_CHUNKS);
    uint32_t word = SHARED_THERE;
    if (lane < C) word = (uint32_t)ld_i32<true>(counts + lane);
    bool there = !__any(word == 0u);
    if (!there) {
      const uint64_t t0 = wall_clock64();
      do {
        __builtin_amdgcn_s_sleep(8);
        if (lane < C) word = (uint32_t)ld_i32<true>(counts + lane);
        there = !__any(word == 0u);
      } while (!there && wall_clock64() - t0 < DEC_WAIT_LIMIT_TICKS);
    }
    // (every wave waits for itself; the waves agree unless one of them ran into its limit)
    const int gone = __syncthreads_or(!there);
    if (gone) {
      if (tid == 0) st_i32<true>(d.status, 1);
      poison_rows<DT, G>(d, b, hs);
      return;
    }
    crowded = __builtin_amdgcn_readfirstlane((int)word) & (int)SHARED_CROWDED;
    if (crowded) {
      if (!wait_for_flag(p.crowd_flag + (size_t)t * ABSB_TICKET_STRIDE, d.status, s_word)) {
        poison_rows<DT, G>(d, b, hs);
        return;
      }
      const int32_t* list = p.tk.work_list + (size_t)t * p.tk.sel_stride;
      for (int i = e0 + tid; i < e1; i += SHARED_THREADS) s_list[i - e0] = ld_i32<true>(list + i);
      __syncthreads();
    } else {
      const uint32_t ns = word & 0xffffu, nc = lane < C ? (word >> 16) & 0xfffu : 0u;  // lane = chunk
      uint32_t sure_, n_in;
      const int to = (int)wave_incl_scan_u32(ns, &sure_);                 // blocks up to and with this chunk's
      const int cand_from = (int)(wave_incl_scan_u32(nc, &n_in) - nc);    // candidates before this chunk's
      const int sure = (int)sure_;
      const int64_t place = score_base(sm, p.tk.Rk, off, rows);
      // entry i of the blocks above the bin lies in chunk u, the first one with to(u) > i: the stretch's entries lie in
      // few chunks, whose bounds are scalars
      const int stop = min(e1, sure);
      const int u0 = min(__popcll(__ballot(to <= e0)), C - 1), u1 = min(__popcll(__ballot(to < stop)), C - 1);
      const int from0 = u0 ? __builtin_amdgcn_readlane(to, u0 - 1) : 0;
      // (requested before the list: a candidate of the lane's chunk, the waves take turns; few chunks have more)
      const int wave = tid >> 6;
      const bool tail = e1 > sure;  // the stretch reaches the admitted candidates
      uint64_t pr = 0;
      if (tail && wave < (int)nc)
        pr = __hip_atomic_load(p.cand + place + (int64_t)lane * chunk + wave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int i = e0 + tid; i < stop; i += SHARED_THREADS) {
        int u = u0, from = from0;
        for (int v = u0; v < u1; ++v) {
          const int bound = __builtin_amdgcn_readlane(to, v);
          if (i >= bound) u = v + 1, from = bound;
        }
        s_list[i - e0] = ld_i32<true>(p.area + place + (int64_t)u * chunk + (i - from));
      }
      if (tail) {  // rank all candidates
        uint32_t* s_key = reinterpret_cast<uint32_t*>(lds + SHARED_LDS_CAND_KEY);
        uint32_t* s_idx = reinterpret_cast<uint32_t*>(lds + SHARED_LDS_CAND_IDX);
        const int nin = min((int)n_in, SHARED_MAX_CAND);
        for (int q = wave; __any(q < (int)nc); q += DEC_WAVES) {
          if (q < (int)nc && cand_from + q < SHARED_MAX_CAND) {
            if (q != wave) pr = __hip_atomic_load(p.cand + place + (int64_t)lane * chunk + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_key[cand_from + q] = (uint32_t)pr;
            s_idx[cand_from + q] = (uint32_t)(pr >> 32);
          }
        }
        __syncthreads();
        // candidate k's rank, counted by 2^x threads: every one takes a part of the list
        int x = 0;
        while (x < 5 && (nin << (x + 1)) <= SHARED_THREADS) ++x;
        const int part = tid & ((1 << x) - 1);
        for (int k = tid >> x; k < nin; k += SHARED_THREADS >> x) {
          const uint32_t mk = s_key[k], mi = s_idx[k];
          int at = 0;
#pragma unroll 8
          for (int u = part; u < nin; u += 1 << x) at += s_key[u] > mk || (s_key[u] == mk && s_idx[u] < mi);
          for (int y = 1; y < 1 << x; y <<= 1) at += __shfl_xor(at, y);
          at += sure;
          if (part == 0 && at >= e0 && at < e1) s_list[at - e0] = (int)mi;
        }
      }
      __syncthreads();
    }
  }

  const int32_t* pages = d.page_table + (size_t)b * d.g.pt_stride;
  AttnState<G> st;
  st.reset();
  attend_positions<DT, G>(d, c, StretchRef{s_list, e0, e1 - 1}, pages, pos_begin, pos_end, qb, st);
  // The segment's last split: every other one has drawn its ticket, so the words that splits read go back to zero, ahead of
  // the merge.  The chunks' own counters are back at zero, or about to be, if a last chunk has been there (all counts
  // words were out long before) and nobody has counted after it; otherwise they did not start there, the caller's list may be
  // missing, and the row may not be clear.
  const int32_t* finished = p.finished + (size_t)t * ABSB_TICKET_STRIDE;
  const int32_t* arrived = p.arrived + (size_t)t * ABSB_TICKET_STRIDE;
  int fin = 0, arr = 0;  // (put together behind the merge only: any use ahead of it waits for them and the stores in front)
  const bool last = finish_split<DT, G>(d, t, b, hs, split, nsplit, d.max_splits, st, lds, [&]() __attribute__((always_inline)) {
    if (!compete) return;
    if (tid < SHARED_MAX_CHUNKS) st_i32<true>(reinterpret_cast<int32_t*>(p.counts + (size_t)t * SHARED_MAX_CHUNKS) + tid, 0);
    if (tid == 0) {
      fin = ld_i32<true>(finished);
      arr = ld_i32<true>(arrived);
      if (crowded) st_i32<true>(p.crowd_flag + (size_t)t * ABSB_TICKET_STRIDE, 0);
    }
  });
  if (!last || !compete) return;
  if (tid == 0) {  // (finish_split uses the word in front)
    s_word[1] = fin;
    s_word[2] = arr;
  }
  __syncthreads();
  if (!(s_word[1] | s_word[2])) return;
  __syncthreads();
  if (tid == 0) {
    const uint64_t t0 = wall_clock64();
    int left;
    do {
      __builtin_amdgcn_s_sleep(2);
      left = ld_i32<true>(finished) | ld_i32<true>(arrived);
    } while (left && wall_clock64() - t0 < DEC_WAIT_LIMIT_TICKS);
    if (left) st_i32<true>(d.status, 1);
    s_word[1] = left;
  }
  __syncthreads();
  if (s_word[1]) poison_rows<DT, G>(d, b, hs);
}

// (What an estimation work-group needs first comes as arguments of their own: see small.hip.)
constexpr int SHARED_LEADING = 5 * 8 + 4 * 4;  // bytes of them
template <int DT, int G, int REP>
__global__ __launch_bounds__(SHARED_THREADS, 4) void shared_step_kernel(addr2 off_lens, addr2 codes_q, int4v shape, uint64_t qscale_, SharedParams p) {
  const auto cent_off = from_addr<const int32_t>(off_lens.x), seq_lens = from_addr<const int32_t>(off_lens.y);
  const auto codes = from_addr<const uint8_t>(codes_q.x);
  const auto q = from_addr<const uint16_t>(codes_q.y);
  const auto qscale = from_addr<const float>(qscale_);
  const int n_score = shape.x, chunks_per_seg = shape.y, Rk = shape.z, tight = shape.w;
  extern __shared__ __align__(16) char lds[];
  const int bid = blockIdx.x;
  if (bid >= n_score) {
    shared_split<DT, G>(p, (bid - n_score) / p.dc.max_splits, (bid - n_score) % p.dc.max_splits, lds);
    return;
  }
  const int t = bid / chunks_per_seg, store = Rk == 1 ? t : t / Rk;
  const int off = cent_off[store], end = cent_off[store + 1];
  fetch_arguments<SHARED_LEADING, sizeof(SharedParams)>();
  int N = end - off;
  if (!tight) {
    const SegMap sm = seg_map(t, p.tk.Hsel, Rk, p.tk.Hkv);
    N = blocks_in_use(false, end - off, seq_lens[sm.b], p.tk.heads.log2_block(sm.hk));
  }
  shared_chunk<DT, G, REP>(p, score_source<REP>(q, qscale, codes, t, store, G, off, N), t, bid % chunks_per_seg, off, end - off, lds);
}

template <int DT, int G>
static void launch_shared_rep(const SharedParams& p, int n_score, int chunks_per_seg, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(SHARED_THREADS), lds, stream,
                       addr2{addr(p.sc.cent_off), addr(p.sc.seq_lens)}, addr2{addr(p.sc.codes), addr(p.sc.q)},
                       int4v{n_score, chunks_per_seg, p.sc.Rk, p.sc.tight}, addr(p.sc.qscale), p);
  };
  if (repr == ABSB_REPR_MEAN)
    launch(shared_step_kernel<DT, G, 0>);
  else
    launch(shared_step_kernel<DT, G, 1>);
}

template <int DT>
static void launch_shared_group(const SharedParams& p, int n_score, int chunks_per_seg, int repr, dim3 grid, size_t lds, hipStream_t stream) {
  switch (p.dc.g.Gd) {
    case 1: launch_shared_rep<DT, 1>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 2: launch_shared_rep<DT, 2>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 3: launch_shared_rep<DT, 3>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 4: launch_shared_rep<DT, 4>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 5: launch_shared_rep<DT, 5>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 6: launch_shared_rep<DT, 6>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    case 7: launch_shared_rep<DT, 7>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
    default: launch_shared_rep<DT, 8>(p, n_score, chunks_per_seg, repr, grid, lds, stream); break;
  }
}

bool shared_fits(const Plan& pl) {
  return pl.max_blocks <= TOPK_MAX_BLOCKS && pl.nseg <= SHARED_MAX_SEGMENTS && pl.split_tokens <= 8 * SHARED_LIST;
}

int launch_shared(const Geometry& g, const Plan& pl, int dtype, float sm_scale, const void* q, const uint8_t* codes,
                  const float* qscale, const float* qmin, const void* k_cache, const void* v_cache, const int32_t* page_table,
                  const int32_t* seq_lens, const int32_t* cent_off, const int32_t* budget, int32_t* sel_idx_out,
                  int32_t* sel_cnt, void* out, float* lse, char* ws, hipStream_t stream) {
  if (!shared_fits(pl)) return ABSB_ERR_UNSUPPORTED;
  SharedParams p;
  int32_t* scores = reinterpret_cast<int32_t*>(ws + pl.ws_scores);
  p.sc = make_score_params(g, pl, q, codes, qscale, qmin, cent_off, seq_lens, scores, nullptr);
  p.sc.chunk = shared_chunk_blocks(pl.max_blocks);
  p.tk = make_topk_params(g, scores, cent_off, budget, seq_lens, sel_idx_out, sel_cnt, pl.sel_stride, nullptr);
  p.tk.work_list = reinterpret_cast<int32_t*>(ws + pl.ws_sel_idx);
  p.tk.flags = reinterpret_cast<int32_t*>(ws + pl.ws_flags);
  p.dc = make_decode_params(g, pl, sm_scale, q, k_cache, v_cache, page_table, seq_lens, nullptr, nullptr, pl.sel_stride, out,
                            lse, ws);
  p.dc.budget = budget;
  p.dc.cent_off = cent_off;
  p.dc.status = reinterpret_cast<int32_t*>(ws + pl.ws_status);
  p.arrived = reinterpret_cast<int32_t*>(ws + pl.ws_score_tickets);
  p.finished = reinterpret_cast<int32_t*>(ws + pl.ws_finished);
  p.listed = reinterpret_cast<uint32_t*>(ws + pl.ws_listed);
  p.crowd_flag = reinterpret_cast<int32_t*>(ws + pl.ws_flags);
  p.hist = reinterpret_cast<uint32_t*>(ws + pl.ws_hist);
  p.counts = reinterpret_cast<uint32_t*>(ws + pl.ws_counts);
  p.area = scores;
  p.cand = reinterpret_cast<uint64_t*>(ws + pl.ws_cand);
  p.want_list = sel_idx_out ? 1 : 0;
  const int chunks_per_seg = (pl.max_blocks + p.sc.chunk - 1) / p.sc.chunk, n_score = chunks_per_seg * pl.nseg;
  const dim3 grid((unsigned)(n_score + pl.nseg * pl.max_splits));
  size_t lds = shared_max(shared_max((size_t)SHARED_LDS_SCORING, (size_t)SHARED_LDS_ATTENTION), topk_lds_bytes(pl.max_blocks));
  const size_t lds_list = SHARED_LDS_SCORING + (size_t)((pl.max_blocks + 31) / 32) * 4;
  if (lds < lds_list) lds = lds_list;
  if (dtype == ABSB_F16)
    launch_shared_group<ABSB_F16>(p, n_score, chunks_per_seg, g.repr, grid, lds, stream);
  else
    launch_shared_group<ABSB_BF16>(p, n_score, chunks_per_seg, g.repr, grid, lds, stream);
  return check_launch();
}

}  // namespace absb

// Centroid store build: block pooling (mean pooling, or channel-wise maxima and minima: Sec. 2.2 and
// its footnote), per-channel asymmetric INT4 quantization (Sec. 3.3) and the flattened,
// prefix-sum-delimited code array (Sec. 3.4, kernel 1).  Runs once per context (prefill side), reads
// every key once.
//
// A block is a row of W = 128 * R values: R = 1 the mean, R = 2 the maxima followed by the minima.
//
// Arithmetic is fixed so that the 4-bit codes are reproducible bit for bit: binary32 running sum
// of a block's keys in token order, one IEEE division by the number of valid tokens (extrema need
// comparisons only), exact min/max per (segment, value), scale = (max-min)/15 and 15/(max-min) as two
// IEEE divisions, code = clamp(round-half-even((c - min) * (15/(max-min)))).  Compiled with
// -ffp-contract=off.
//
// Three launches:
//   1. pool: a work-group owns BUILD_CHUNK consecutive tokens of a segment, a wave a quarter of them; a block
//      is closed whenever the running token index reaches its boundary: its binary32 row goes to the
//      workspace and into the work-group's minima / maxima per value;
//   2. params: reduces the partial extrema per segment and writes qscale, qmin (and 15/range);
//   3. codes: quantizes the rows, eight values per lane packed into one 32-bit store.
#include "common.h"

namespace absb {

struct BuildParams {
  const uint16_t* k;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const int32_t* cent_off;
  float* cent;     // [total][W]
  float* minmax;   // [nseg][max_chunks][2][W]
  float* qinv;     // [nseg][W]
  float* qscale;   // [nseg][W]
  float* qmin;     // [nseg][W]
  uint8_t* codes;  // [total][W/2]
  int32_t max_chunks;
  Geometry g;
};

constexpr int BUILD_THREADS = 256;
constexpr int BUILD_GROUPS = BUILD_THREADS / 16;
constexpr int BUILD_WAVES = BUILD_THREADS / 64;
constexpr int BUILD_RUN = BUILD_CHUNK / BUILD_WAVES;  // tokens a wave pools: whole blocks of every size
constexpr int BUILD_BATCH = 32;                       // rows it requests at once
constexpr int CODES_BLOCKS = 64;                      // blocks per work-group of the codes kernel
static_assert(BUILD_RUN % 128 == 0, "a wave's tokens are whole blocks");

// Read-only arrays at wave-uniform addresses: scalar loads, which do not queue behind the rows in flight.
typedef __attribute__((address_space(4))) const int32_t scalar_i32;
__device__ __forceinline__ scalar_i32* as_scalar(const int32_t* p) { return (scalar_i32*)(uintptr_t)p; }

// Bound by the stream of keys, 256 bytes a token and KV head.  A wave reads one row per load instruction, a lane
// two channels: a block's sum stays in one lane in token order, and the row's address is a scalar.  32 rows
// are in flight while 32 are pooled.  The keys are read once and nothing else wants them, so they pass the
// caches by (nontemporal loads).  Against 16-lane row-groups of 128-bit loads, whose page lookups sat behind
// the rows in flight (loads return in order), on a 128K context of 8 heads (268 MB of keys): 72 -> 55 us, of
// which the rows written out are 10 us (44 us = 6.0 TB/s without them).
template <int DT, int REP>
__global__ __launch_bounds__(BUILD_THREADS, 4) void build_pool_kernel(BuildParams p) {
  constexpr int W = ABSB_HEAD_DIM * (REP + 1);
  __shared__ float2 s_ext[BUILD_WAVES][2][W / 2];
  const int s = blockIdx.y, chunk = blockIdx.x;
  const int b = s / p.g.Hkv, h = s % p.g.Hkv;
  const int L = as_scalar(p.seq_lens)[b];
  const int t0 = chunk * BUILD_CHUNK;
  if (t0 >= L) return;
  const int off = as_scalar(p.cent_off)[s];
  const int lb = p.g.heads.log2_block[h], lP = p.g.log2_page;
  const int B = 1 << lb;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tA = t0 + wave * BUILD_RUN, tB = min(tA + BUILD_RUN, L);

  // extrema over this wave's blocks, per vector of the row (v = 0: mean or maxima, 1: minima)
  float mn[REP + 1][2], mx[REP + 1][2];
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    mn[v][0] = mn[v][1] = __builtin_inff();
    mx[v][0] = mx[v][1] = -__builtin_inff();
  }
  if (tA < tB) {
    scalar_i32* pt = as_scalar(p.page_table + (size_t)b * p.g.pt_stride);
    const char* kh = reinterpret_cast<const char*>(p.k + (size_t)h * p.g.s_head) + lane * 4;
    const int tok_mask = (1 << lP) - 1;
    const size_t pitch = (size_t)p.g.s_tok * 2;
    // rows [t, t + BUILD_BATCH); rows past the end repeat earlier ones (legal addresses), skipped below
    auto load = [&](int t, uint32_t (&r)[BUILD_BATCH]) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < BUILD_BATCH / 8; ++q) {
        const int tq = min(t + 8 * q, (tB - 1) & ~7);  // eight rows from a multiple of eight lie in one page
        const char* base = kh + ((size_t)pt[tq >> lP] * p.g.s_page + (size_t)(tq & tok_mask) * p.g.s_tok) * 2;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          r[8 * q + i] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(base + (size_t)min(i, tB - 1 - tq) * pitch));
      }
    };
    // the open block: its running sum (mean pooling) or its maxima / minima so far
    float acc[REP + 1][2];
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        acc[0][c] = REP ? -__builtin_inff() : 0.0f;
        if (REP) acc[REP][c] = __builtin_inff();
      }
    };
    auto fold = [&](uint32_t w) __attribute__((always_inline)) {
      const float lo = Elem<DT>::lo(w), hi = Elem<DT>::hi(w);
      if (REP) {
        acc[0][0] = fmaxf(acc[0][0], lo);
        acc[0][1] = fmaxf(acc[0][1], hi);
        acc[REP][0] = fminf(acc[REP][0], lo);
        acc[REP][1] = fminf(acc[REP][1], hi);
      } else {
        acc[0][0] = acc[0][0] + lo;
        acc[0][1] = acc[0][1] + hi;
      }
    };
    auto pool = [&](int t, const uint32_t (&r)[BUILD_BATCH]) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < BUILD_BATCH / 8; ++q) {
        const int tq = t + 8 * q;
        if (tq >= tB) continue;
        if (tq + 8 <= tB) {
#pragma unroll
          for (int i = 0; i < 8; ++i) fold(r[8 * q + i]);
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (tq + i < tB) fold(r[8 * q + i]);
        }
        if (((tq + 8) & (B - 1)) == 0 || tq + 8 >= tB) {  // the block that holds token tq is complete
          const int j = tq >> lb;
          const float fn = (float)min(B, L - (j << lb));
#pragma unroll
          for (int v = 0; v <= REP; ++v) {
            const float x = REP ? acc[v][0] : acc[v][0] / fn, y = REP ? acc[v][1] : acc[v][1] / fn;
            mn[v][0] = fminf(mn[v][0], x);
            mn[v][1] = fminf(mn[v][1], y);
            mx[v][0] = fmaxf(mx[v][0], x);
            mx[v][1] = fmaxf(mx[v][1], y);
            *reinterpret_cast<float2*>(p.cent + ((size_t)off + j) * W + v * ABSB_HEAD_DIM + lane * 2) = make_float2(x, y);
          }
          reset();
        }
      }
    };
    reset();
    uint32_t even[BUILD_BATCH], odd[BUILD_BATCH];
    load(tA, even);
    for (int t = tA;;) {
      const int t1 = t + BUILD_BATCH, t2 = t1 + BUILD_BATCH;
      if (t1 < tB) load(t1, odd);
      pool(t, even);
      if (t1 >= tB) break;
      if (t2 < tB) load(t2, even);
      pool(t1, odd);
      if (t2 >= tB) break;
      t = t2;
    }
  }

  // ---- fold the waves: thread -> (kind, two values)
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    s_ext[wave][0][v * 64 + lane] = make_float2(mn[v][0], mn[v][1]);
    s_ext[wave][1][v * 64 + lane] = make_float2(mx[v][0], mx[v][1]);
  }
  __syncthreads();
  if (tid < W) {
    const int kind = tid / (W / 2), c = tid % (W / 2);
    float2 x = s_ext[0][kind][c];
#pragma unroll
    for (int w = 1; w < BUILD_WAVES; ++w) {
      const float2 y = s_ext[w][kind][c];
      x.x = kind ? fmaxf(x.x, y.x) : fminf(x.x, y.x);
      x.y = kind ? fmaxf(x.y, y.y) : fminf(x.y, y.y);
    }
    float* dst = p.minmax + ((size_t)s * p.max_chunks + chunk) * 2 * W;
    *reinterpret_cast<float2*>(dst + kind * W + 2 * c) = x;
  }
}

// grid (segment, 32 values of the row): 32 values x 32 chunk lanes; min/max are exact in any order.
constexpr int PARAMS_THREADS = 1024;
constexpr int PARAMS_VALUES = 32;
constexpr int PARAMS_LANES = PARAMS_THREADS / PARAMS_VALUES;

__global__ __launch_bounds__(PARAMS_THREADS) void build_params_kernel(BuildParams p) {
  const int W = ABSB_HEAD_DIM * (p.g.repr + 1);
  const int s = blockIdx.x, cl = threadIdx.x / PARAMS_VALUES, c = threadIdx.x % PARAMS_VALUES;
  const int ch = blockIdx.y * PARAMS_VALUES + c;  // value index in the row
  const int nchunks = (p.seq_lens[s / p.g.Hkv] + BUILD_CHUNK - 1) / BUILD_CHUNK;
  float mn = __builtin_inff(), mx = -__builtin_inff();
  for (int i0 = cl; i0 < nchunks; i0 += 8 * PARAMS_LANES) {
    float a[8], z[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = min(i0 + u * PARAMS_LANES, nchunks - 1);  // the tail repeats a chunk: harmless for min/max
      const float* src = p.minmax + ((size_t)s * p.max_chunks + i) * 2 * W;
      a[u] = src[ch];
      z[u] = src[W + ch];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      mn = fminf(mn, a[u]);
      mx = fmaxf(mx, z[u]);
    }
  }
  __shared__ float s_mn[PARAMS_LANES][PARAMS_VALUES], s_mx[PARAMS_LANES][PARAMS_VALUES];
  s_mn[cl][c] = mn;
  s_mx[cl][c] = mx;
  __syncthreads();
  if (cl != 0) return;
#pragma unroll
  for (int k = 1; k < PARAMS_LANES; ++k) {
    mn = fminf(mn, s_mn[k][c]);
    mx = fmaxf(mx, s_mx[k][c]);
  }
  const float rng = mx - mn;
  float sc = 0.0f, inv = 0.0f;
  if (rng > 0.0f) {
    sc = rng / 15.0f;
    inv = 15.0f / rng;
  }
  p.qscale[(size_t)s * W + ch] = sc;
  p.qmin[(size_t)s * W + ch] = mn;
  p.qinv[(size_t)s * W + ch] = inv;
}

// grid (64 blocks, segment, vector of the row)
__global__ __launch_bounds__(BUILD_THREADS) void build_codes_kernel(BuildParams p) {
  const int W = ABSB_HEAD_DIM * (p.g.repr + 1);
  const int s = blockIdx.y, v = blockIdx.z;
  const int off = p.cent_off[s];
  const int lb = p.g.heads.log2_block[s % p.g.Hkv];
  const int N = blocks_in_use(p.g.tight, p.cent_off[s + 1] - off, p.seq_lens, s / p.g.Hkv, lb);
  const int j0 = blockIdx.x * CODES_BLOCKS;
  if (j0 >= N) return;
  const int jend = min(N, j0 + CODES_BLOCKS);
  const int tid = threadIdx.x, grp = tid >> 4, li = tid & 15;
  const int col = v * ABSB_HEAD_DIM + li * 8;  // first of this lane's eight values in the row
  float mn[8], inv[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    mn[c] = p.qmin[(size_t)s * W + col + c];
    inv[c] = p.qinv[(size_t)s * W + col + c];
  }
  for (int j = j0 + grp; j < jend; j += BUILD_GROUPS) {
    const float4* src = reinterpret_cast<const float4*>(p.cent + ((size_t)off + j) * W + col);
    const float4 a = src[0], z = src[1];
    const float cen[8] = {a.x, a.y, a.z, a.w, z.x, z.y, z.z, z.w};
    uint32_t packed = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float x = cen[c] - mn[c];
      const float y = x * inv[c];
      float r = __builtin_rintf(y);
      r = fminf(fmaxf(r, 0.0f), 15.0f);
      packed |= (uint32_t)r << (4 * c);
    }
    // byte i of a row holds value 2i (low nibble) and 2i+1 (high nibble): little-endian nibble n
    // of this word is value col + n
    *reinterpret_cast<uint32_t*>(p.codes + ((size_t)off + j) * (W / 2) + col / 2) = packed;
  }
}

// Decode-time maintenance.  A 16-lane row-group per segment, each lane 8 channels.
struct AppendParams {
  const uint16_t* k;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const int32_t* cent_off;
  uint8_t* codes;
  const float* qscale;
  const float* qmin;
  float* tail;  // [nseg][W]
  int32_t* clamped;  // [nseg] or null
  int32_t nseg;
  Geometry g;
};

// One key folded into the pooled state of a block (first: it is the block's first key and starts the state).
template <int DT, int REP>
__device__ __forceinline__ void fold_key(float (&st)[REP + 1][8], const uint4& row, bool first) {
  const uint32_t w[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float lo = Elem<DT>::lo(w[c]), hi = Elem<DT>::hi(w[c]);
    if (REP) {
      st[0][2 * c] = first ? lo : fmaxf(st[0][2 * c], lo);
      st[0][2 * c + 1] = first ? hi : fmaxf(st[0][2 * c + 1], hi);
      st[REP][2 * c] = first ? lo : fminf(st[REP][2 * c], lo);
      st[REP][2 * c + 1] = first ? hi : fminf(st[REP][2 * c + 1], hi);
    } else {
      st[0][2 * c] = first ? lo : st[0][2 * c] + lo;
      st[0][2 * c + 1] = first ? hi : st[0][2 * c + 1] + hi;
    }
  }
}

template <int REP>
__device__ __forceinline__ void store_tail(float* tail, const float (&st)[REP + 1][8]) {
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    *reinterpret_cast<float4*>(tail + v * ABSB_HEAD_DIM) = make_float4(st[v][0], st[v][1], st[v][2], st[v][3]);
    *reinterpret_cast<float4*>(tail + v * ABSB_HEAD_DIM + 4) = make_float4(st[v][4], st[v][5], st[v][6], st[v][7]);
  }
}

// Recomputes the pooled state of every segment's last block from the cache (its tokens, in order).  The
// keys enter the state one after the other, so the kernel is a chain of memory round trips unless they are
// requested together: one lane per eight tokens looks up their page (a block of 128 tokens has 16 such
// runs), then 32 rows are in flight at a time.  One key per round trip cost 33 us for blocks of 64 tokens.
constexpr int TAIL_ROWS = 32;

template <int DT, int REP>
__global__ __launch_bounds__(BUILD_THREADS) void tail_kernel(AppendParams p) {
  constexpr int W = ABSB_HEAD_DIM * (REP + 1);
  const int tid = threadIdx.x, grp = tid >> 4, li = tid & 15;
  const int s = blockIdx.x * BUILD_GROUPS + grp;
  if (s >= p.nseg) return;
  const int b = s / p.g.Hkv, h = s % p.g.Hkv;
  const int lb = p.g.heads.log2_block[h], lP = p.g.log2_page;
  const int t_new = p.seq_lens[b] - 1, t0 = (t_new >> lb) << lb;
  const int32_t* pt = p.page_table + (size_t)b * p.g.pt_stride;
  const uint16_t* k = p.k + (size_t)h * p.g.s_head + (size_t)li * 8;
  // the page of tokens [t0 + 8*li, +8): they lie in one page (t0 is a multiple of eight, P >= 8)
  const int my_page = pt[min(t0 + 8 * li, t_new) >> lP];

  float st[REP + 1][8];
  for (int base = t0; base <= t_new; base += TAIL_ROWS) {
    uint4 row[TAIL_ROWS];
#pragma unroll
    for (int r = 0; r < TAIL_ROWS; ++r) {  // rows past the newest token repeat it (a legal address), skipped below
      const int t = min(base + r, t_new);
      const int page = __shfl(my_page, (t - t0) >> 3, 16);
      row[r] = *reinterpret_cast<const uint4*>(k + (size_t)page * p.g.s_page + (size_t)(t & ((1 << lP) - 1)) * p.g.s_tok);
    }
#pragma unroll
    for (int r = 0; r < TAIL_ROWS; ++r)
      if (base + r <= t_new) fold_key<DT, REP>(st, row[r], base + r == t0);
  }
  store_tail<REP>(p.tail + (size_t)s * W + li * 8, st);
}

// Folds the key of the newest token (position L - 1) into the pooled state of the segment's last block and
// re-emits that block's 4-bit row under the store's frozen ranges.  When the new token completes its block
// the row is final: the number of its values that the frozen range does not hold is then added to the
// segment's counter (the signal for a re-ranging policy).
//
// Bound by latency: length -> page-table entry -> key is the only chain, so everything else (state, ranges,
// the row's place) is requested before it.
template <int DT, int REP>
__global__ __launch_bounds__(BUILD_THREADS) void append_kernel(AppendParams p) {
  constexpr int W = ABSB_HEAD_DIM * (REP + 1);
  const int tid = threadIdx.x, grp = tid >> 4, li = tid & 15;
  const int s = blockIdx.x * BUILD_GROUPS + grp;
  if (s >= p.nseg) return;
  const int b = s / p.g.Hkv, h = s % p.g.Hkv;
  const int t_new = p.seq_lens[b] - 1;
  float* tail = p.tail + (size_t)s * W + li * 8;
  float st[REP + 1][8], scale[REP + 1][8], mn[REP + 1][8];
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    const size_t at = (size_t)s * W + v * ABSB_HEAD_DIM + li * 8;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<float4*>(&st[v][4 * q]) = *reinterpret_cast<const float4*>(tail + v * ABSB_HEAD_DIM + 4 * q);
      *reinterpret_cast<float4*>(&scale[v][4 * q]) = *reinterpret_cast<const float4*>(p.qscale + at + 4 * q);
      *reinterpret_cast<float4*>(&mn[v][4 * q]) = *reinterpret_cast<const float4*>(p.qmin + at + 4 * q);
    }
  }
  const int off = p.cent_off[s];
  const int lb = p.g.heads.log2_block[h], lP = p.g.log2_page;
  const int j = t_new >> lb, t0 = j << lb;
  const int page = p.page_table[(size_t)b * p.g.pt_stride + (t_new >> lP)];
  const uint4 row = *reinterpret_cast<const uint4*>(p.k + (size_t)page * p.g.s_page + (size_t)h * p.g.s_head +
                                                    (size_t)(t_new & ((1 << lP) - 1)) * p.g.s_tok + (size_t)li * 8);
  fold_key<DT, REP>(st, row, t_new == t0);
  store_tail<REP>(tail, st);

  const float fn = (float)(t_new - t0 + 1);
  const size_t row_at = ((size_t)off + j) * (W / 2);
  int outside = 0;
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    const int col = v * ABSB_HEAD_DIM + li * 8;
    uint32_t packed = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float value = REP ? st[v][c] : st[v][c] / fn;
      const float sc = scale[v][c];
      float r = 0.0f;
      if (sc > 0.0f) {
        const float inv = 1.0f / sc;
        const float x = value - mn[v][c];
        r = __builtin_rintf(x * inv);
        outside += !(r >= 0.0f && r <= 15.0f);
        r = fminf(fmaxf(r, 0.0f), 15.0f);  // a NaN ends up at 0
      } else {
        outside += value != mn[v][c];  // a channel that was constant at build time
      }
      packed |= (uint32_t)r << (4 * c);
    }
    *reinterpret_cast<uint32_t*>(p.codes + row_at + col / 2) = packed;
  }
  if (p.clamped && ((t_new + 1) & ((1 << lb) - 1)) == 0) {  // the block is complete (wave-uniform per row-group)
    outside += __shfl_xor(outside, 1);
    outside += __shfl_xor(outside, 2);
    outside += __shfl_xor(outside, 4);
    outside += __shfl_xor(outside, 8);
    // this row-group is the segment's only writer; an add without return value, so that nothing waits for it
    if (li == 0 && outside)
      __hip_atomic_fetch_add(p.clamped + s, outside, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int DT, int REP>
static void launch_append_kernel(bool append, const AppendParams& p, hipStream_t stream) {
  const dim3 grid((unsigned)((p.nseg + BUILD_GROUPS - 1) / BUILD_GROUPS)), block(BUILD_THREADS);
  if (append)
    hipLaunchKernelGGL((append_kernel<DT, REP>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((tail_kernel<DT, REP>), grid, block, 0, stream, p);
}

int launch_append(const Geometry& g, const Plan& pl, int dtype, bool append, const void* k_cache,
                  const int32_t* page_table, const int32_t* seq_lens, const int32_t* cent_off, uint8_t* codes,
                  const float* qscale, const float* qmin, float* tail, int32_t* clamped, hipStream_t stream) {
  AppendParams p;
  p.k = static_cast<const uint16_t*>(k_cache);
  p.page_table = page_table;
  p.seq_lens = seq_lens;
  p.cent_off = cent_off;
  p.codes = codes;
  p.qscale = qscale;
  p.qmin = qmin;
  p.tail = tail;
  p.clamped = clamped;
  p.nseg = pl.nstore;
  p.g = g;
  if (dtype == ABSB_F16 && g.repr == ABSB_REPR_MEAN)
    launch_append_kernel<ABSB_F16, 0>(append, p, stream);
  else if (dtype == ABSB_F16)
    launch_append_kernel<ABSB_F16, 1>(append, p, stream);
  else if (g.repr == ABSB_REPR_MEAN)
    launch_append_kernel<ABSB_BF16, 0>(append, p, stream);
  else
    launch_append_kernel<ABSB_BF16, 1>(append, p, stream);
  return check_launch();
}

int launch_build(const Geometry& g, const Plan& pl, int dtype, const void* k_cache, const int32_t* page_table,
                 const int32_t* seq_lens, const int32_t* cent_off, uint8_t* codes, float* qscale, float* qmin,
                 char* ws, hipStream_t stream) {
  BuildParams p;
  p.k = static_cast<const uint16_t*>(k_cache);
  p.page_table = page_table;
  p.seq_lens = seq_lens;
  p.cent_off = cent_off;
  p.cent = reinterpret_cast<float*>(ws + pl.ws_cent);
  p.minmax = reinterpret_cast<float*>(ws + pl.ws_minmax);
  p.qinv = reinterpret_cast<float*>(ws + pl.ws_qinv);
  p.qscale = qscale;
  p.qmin = qmin;
  p.codes = codes;
  p.max_chunks = pl.build_max_chunks;
  p.g = g;
  const unsigned R = (unsigned)g.repr + 1;
  const dim3 grid((unsigned)pl.build_max_chunks, (unsigned)pl.nstore), block(BUILD_THREADS);
  if (dtype == ABSB_F16 && g.repr == ABSB_REPR_MEAN)
    hipLaunchKernelGGL((build_pool_kernel<ABSB_F16, 0>), grid, block, 0, stream, p);
  else if (dtype == ABSB_F16)
    hipLaunchKernelGGL((build_pool_kernel<ABSB_F16, 1>), grid, block, 0, stream, p);
  else if (g.repr == ABSB_REPR_MEAN)
    hipLaunchKernelGGL((build_pool_kernel<ABSB_BF16, 0>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((build_pool_kernel<ABSB_BF16, 1>), grid, block, 0, stream, p);
  int rc = check_launch();
  if (rc != ABSB_OK) return rc;
  hipLaunchKernelGGL(build_params_kernel, dim3((unsigned)pl.nstore, R * ABSB_HEAD_DIM / PARAMS_VALUES), dim3(PARAMS_THREADS), 0, stream, p);
  rc = check_launch();
  if (rc != ABSB_OK) return rc;
  hipLaunchKernelGGL(build_codes_kernel, dim3((unsigned)((pl.max_blocks + CODES_BLOCKS - 1) / CODES_BLOCKS), grid.y, R), block, 0, stream, p);
  return check_launch();
}

}  // namespace absb

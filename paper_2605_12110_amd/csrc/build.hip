// Centroid store build (prefill side) and its maintenance while decoding.
//
// Build: block pooling (mean pooling, or channel-wise maxima and minima: Sec. 2.2 and its footnote), per-channel
// asymmetric INT4 quantization (Sec. 3.3) and the flattened, prefix-sum-delimited code array (Sec. 3.4, kernel 1).
// Runs once per context, reads every key once.
//
// A block is a row of W = 128 * R values: R = 1 the mean, R = 2 the maxima followed by the minima.
//
// Arithmetic is fixed so that the 4-bit codes are reproducible bit for bit: binary32 running sum
// of a block's keys in token order, one IEEE division by the number of valid tokens (extrema need
// comparisons only), exact min/max per (segment, value), scale = (max-min)/15 and 15/(max-min) as two
// IEEE divisions, code = clamp(round-half-even((c - min) * (15/(max-min)))).  Compiled with
// -ffp-contract=off.
//
// One kernel (behind one that clears a few words a segment): a work-group owns a chunk of consecutive
// tokens of a segment, a wave a quarter of them, and a row stays in the registers of the wave that pooled it until the
// segment's ranges are known:
//   1. pool: a block is closed whenever the running token index reaches its boundary;
//   2. ranges: the chunk's minima and maxima per value go into the segment's words in memory (device atomics on
//      integers that order like the floats), then the chunk signs in on the segment's counter;
//   3. when all of the segment's chunks have signed in, every chunk reads the ranges and quantizes its own rows.
// A chunk does not wait for ever, nor where too many others are missing: it then writes its binary32 rows to the
// workspace, marks itself, and leaves.  The chunks that are there when the segment is complete (the last to sign in
// always is) quantize the rows of those that left.  So nothing rests on which work-groups run at the same time:
// every work-group ends, and every row is quantized, whatever the order.
#include <climits>
#include <type_traits>

#include "common.h"

namespace absb {

struct BuildParams {
  const uint16_t* k;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const int32_t* cent_off;
  float* cent;     // [total][W]: rows of the chunks that left
  uint32_t* meet;  // [nseg][pitch]: what a segment's chunks share
  float* qscale;   // [nseg][W]
  float* qmin;     // [nseg][W]
  uint8_t* codes;  // [total][W/2]
  int32_t pitch, copies;
  Geometry g;
};

constexpr int BUILD_THREADS = 256;
constexpr int BUILD_GROUPS = BUILD_THREADS / 16;
constexpr int BUILD_WAVES = BUILD_THREADS / 64;
constexpr int BUILD_RUN = BUILD_RUNS_OF / BUILD_WAVES;  // tokens a wave pools at a time: whole blocks of every size
constexpr int BUILD_BATCH = 32;                       // rows it requests at once
constexpr int BUILD_EIGHTS = BUILD_RUN / 8;           // rows it may end up with (blocks of eight tokens)
static_assert(BUILD_RUN == 128, "a wave's tokens are whole blocks of every size, in four batches");
// A chunk waits while at most so many of its segment's chunks are missing (it would keep their places from them
// otherwise: 1280 fit the chip with mean pooling, 1024 with extrema, and another launch may want some), and at most so
// long (100 MHz ticks; the tests' second library is built with 1: whoever is not there at the first look leaves).
#ifndef ABSB_BUILD_WAIT_TICKS
#define ABSB_BUILD_WAIT_TICKS 20000
#endif
constexpr uint32_t BUILD_MISSING = 512;
constexpr uint64_t BUILD_WAIT_TICKS = ABSB_BUILD_WAIT_TICKS;

// What the chunks of a segment share (meet_...: common.h).  Chunk c raises copy c % copies of the minima and maxima (as
// keys, below); the chunk that signs in last makes all copies equal to their common maximum and raises the flags.  One
// copy for everybody is what everybody would queue for: updates and reads of one memory line take ~10 ns each,
// whoever makes them (a 128K context of 8 heads, 256 chunks a segment: 104 us with one copy and one flag, 51 with
// eight, 46 if every chunk kept its extrema to itself).
// The counter holds the chunks that signed in [0, 32) and those that left [32, 64); a chunk's bit says that its rows
// are in the workspace.  The last chunk copies the bits for everybody before it raises the flags, so that all who are
// there go by the same ones when they share out the rows of those that left.
constexpr uint32_t MEET_COMPLETE = 1, MEET_SOME_LEFT = 2;  // of a flag

// Unsigned integers that order like the floats; zero lies below all of them.  Minima are kept as the
// complement, so that both are raised by a maximum.
__device__ __forceinline__ uint32_t float_key(float x) {
  const uint32_t u = bitcast<uint32_t>(x);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) { return bitcast<float>(k ^ ((k >> 31) ? 0x80000000u : 0xffffffffu)); }

// Read-only arrays at wave-uniform addresses: scalar loads, which do not queue behind the rows in flight.
typedef __attribute__((address_space(4))) const int32_t scalar_i32;
typedef __attribute__((address_space(1))) uint32_t global_u32;
__device__ __forceinline__ scalar_i32* as_scalar(const int32_t* p) { return (scalar_i32*)(uintptr_t)p; }

__global__ void build_clear_kernel(BuildParams p, int words) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) p.meet[(size_t)blockIdx.y * p.pitch + i] = 0;
}

// The two 4-bit codes of a lane's two values, low nibble first.
__device__ __forceinline__ uint32_t code_pair(float x, float y, const float (&mn)[2], const float (&inv)[2]) {
  const float a = fminf(fmaxf(__builtin_rintf((x - mn[0]) * inv[0]), 0.0f), 15.0f);
  const float b = fminf(fmaxf(__builtin_rintf((y - mn[1]) * inv[1]), 0.0f), 15.0f);
  return (uint32_t)a | ((uint32_t)b << 4);
}

// A row in the registers of its wave: two values per vector and lane.  Means take a register each; extrema are
// values of the K/V type, so two fit one.
template <int DT, int REP>
struct KeptRow;
template <int DT>
struct KeptRow<DT, 0> {
  float x, y;
  __device__ __forceinline__ void set(const float (&r)[1][2]) { x = r[0][0], y = r[0][1]; }
  __device__ __forceinline__ void get(float (&r)[1][2]) const { r[0][0] = x, r[0][1] = y; }
};
template <int DT>
struct KeptRow<DT, 1> {
  uint32_t v[2];
  __device__ __forceinline__ void set(const float (&r)[2][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = (uint32_t)Elem<DT>::narrow(r[i][0]) | ((uint32_t)Elem<DT>::narrow(r[i][1]) << 16);
  }
  __device__ __forceinline__ void get(float (&r)[2][2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) r[i][0] = Elem<DT>::lo(v[i]), r[i][1] = Elem<DT>::hi(v[i]);
  }
};

// Bound by the stream of keys, 256 bytes a token and KV head.  A wave reads one row per load instruction, a lane
// two channels: a block's sum stays in one lane in token order, and the row's address is a scalar.  64 rows
// are in flight, 32 of them while 32 are pooled.  The keys are read once and nothing else wants them, so they pass the
// caches by (nontemporal loads).  Rows kept in registers (16 of eight tokens at most: 32 registers of 96) instead of
// written out, read back and quantized by a kernel of their own, on 128K of 8 heads (268 MB of keys): 67 -> 51 us,
// 16 requests of 8K-128K (2.35 GB): 535 -> 419 us; the keys alone take 46 and 397.  Contexts so long that their rows
// do not all stay (a chunk of several runs): 262144 tokens 123 -> 105 us, 524288 233 -> 222.
template <int DT, int REP>
__global__ __launch_bounds__(BUILD_THREADS, REP ? 4 : 5) void build_kernel(BuildParams p) {
  constexpr int W = ABSB_HEAD_DIM * (REP + 1);
  __shared__ float2 s_ext[BUILD_WAVES][2][W / 2];
  __shared__ uint32_t s_word[4];
  const int s = blockIdx.y, chunk = blockIdx.x;
  const int b = s / p.g.Hkv, h = s % p.g.Hkv;
  const int L = as_scalar(p.seq_lens)[b];
  const int runs = build_runs(L);
  const int t0 = chunk * runs * BUILD_RUNS_OF;
  if (t0 >= L) return;
  const int last_run = min(runs, (L - t0 + BUILD_RUNS_OF - 1) / BUILD_RUNS_OF) - 1;
  const int off = as_scalar(p.cent_off)[s];
  const int lb = p.g.heads.log2_block(h), lP = p.g.log2_page;
  const int B = 1 << lb;
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tA, tB;  // the wave's tokens of the run
  // whether the eighth of tokens [t, t + 8) completes a block
  auto closes = [&](int t) __attribute__((always_inline)) { return t < tB && (((t + 8) & (B - 1)) == 0 || t + 8 >= tB); };

  // ---- 1. pool
  // extrema over this wave's blocks, per vector of the row (v = 0: mean or maxima, 1: minima)
  float mn[REP + 1][2], mx[REP + 1][2];
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    mn[v][0] = mn[v][1] = __builtin_inff();
    mx[v][0] = mx[v][1] = -__builtin_inff();
  }
  KeptRow<DT, REP> kept[BUILD_EIGHTS];  // of the block that ends with the wave's i-th eighth
  // a row to the workspace, where other work-groups may have to read it
  auto row_out = [&](int t, const float (&r)[REP + 1][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v <= REP; ++v)
      __hip_atomic_store(reinterpret_cast<uint64_t*>(p.cent + ((size_t)off + (t >> lb)) * W + v * ABSB_HEAD_DIM + lane * 2),
                         bitcast<uint64_t>(make_float2(r[v][0], r[v][1])), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // FULL: no row is missing, so no load, address or fold depends on where the context ends.  KEEP: the run's rows stay
  // in registers, else they go to the workspace.
  auto pool_run = [&](auto full_, auto keep_) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_)::value, KEEP = decltype(keep_)::value;
    scalar_i32* pt = as_scalar(p.page_table + (size_t)b * p.g.pt_stride);
    const uint64_t kh = reinterpret_cast<uint64_t>(p.k + (size_t)h * p.g.s_head);
    const int tok_mask = (1 << lP) - 1;
    const uint64_t pitch = (uint64_t)p.g.s_tok * 2;
    int32_t page[BUILD_EIGHTS];  // eight rows from a multiple of eight lie in one page
#pragma unroll
    for (int q = 0; q < BUILD_EIGHTS; ++q) page[q] = pt[(FULL ? tA + 8 * q : min(tA + 8 * q, (tB - 1) & ~7)) >> lP];
    // rows of batch n; rows past the end repeat rows of the last eighth (legal addresses)
    auto load = [&](auto batch, uint32_t (&r)[BUILD_BATCH]) __attribute__((always_inline)) {
      constexpr int Q0 = decltype(batch)::value * (BUILD_BATCH / 8);
#pragma unroll
      for (int q = 0; q < BUILD_BATCH / 8; ++q) {
        const int tq = FULL ? tA + 8 * (Q0 + q) : min(tA + 8 * (Q0 + q), (tB - 1) & ~7);
        uint64_t row = kh + ((uint64_t)page[Q0 + q] * (uint64_t)p.g.s_page + (uint64_t)(tq & tok_mask) * (uint64_t)p.g.s_tok) * 2;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          asm("" : "+s"(row));  // stays a scalar, the lane's part being the load's offset
          r[8 * q + i] = __builtin_nontemporal_load((const global_u32*)row + lane);
          if (FULL || tq + i + 1 < tB) row += pitch;
        }
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
    const float whole = bitcast<float>((uint32_t)(127 - lb) << 23);  // 1/B: a product with it is the quotient by B, bit for bit
    auto close = [&](float (&r)[REP + 1][2]) __attribute__((always_inline)) {  // a finished row into the extrema
#pragma unroll
      for (int v = 0; v <= REP; ++v)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          mn[v][c] = fminf(mn[v][c], r[v][c]);
          mx[v][c] = fmaxf(mx[v][c], r[v][c]);
        }
    };
    auto pool = [&](auto batch, const uint32_t (&r)[BUILD_BATCH]) __attribute__((always_inline)) {
      constexpr int Q0 = decltype(batch)::value * (BUILD_BATCH / 8);
#pragma unroll
      for (int q = 0; q < BUILD_BATCH / 8; ++q) {
        const int tq = tA + 8 * (Q0 + q);
        // (rows past the end: nothing to a sum; copies of rows of the last block change none of its extrema)
#pragma unroll
        for (int i = 0; i < 8; ++i) fold(FULL || REP || tq + i < tB ? r[8 * q + i] : 0u);
        if (((tq + 8) & (B - 1)) == 0 && (FULL || tq + 8 <= tB)) {
#pragma unroll
          for (int c = 0; c < 2; ++c)
            if (!REP) acc[0][c] *= whole;
          close(acc);
          if (KEEP)
            kept[Q0 + q].set(acc);
          else
            row_out(tq, acc);
          reset();
        }
      }
    };
    typedef std::integral_constant<int, 0> B0;
    typedef std::integral_constant<int, 1> B1;
    typedef std::integral_constant<int, 2> B2;
    typedef std::integral_constant<int, 3> B3;
    reset();
    uint32_t even[BUILD_BATCH], odd[BUILD_BATCH];
    load(B0(), even);
    load(B1(), odd);
    pool(B0(), even);
    load(B2(), even);
    pool(B1(), odd);
    load(B3(), odd);
    pool(B2(), even);
    pool(B3(), odd);
    if (!FULL && (tB & (B - 1))) {  // the context ends inside a block
      const float fn = (float)(tB & (B - 1));
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (!REP) acc[0][c] = acc[0][c] / fn;
      close(acc);
#pragma unroll
      for (int q = 0; q < BUILD_EIGHTS; ++q) {
        int ends = (tB - 1 - tA) >> 3;
        asm("" : "+s"(ends));  // (a comparison per eighth: a store at a computed place would put the rows into memory)
        if (q == ends) kept[q].set(acc);
      }
    }
  };
  tA = t0 + wave * BUILD_RUN;
#pragma unroll 1
  for (int run = 0; run < last_run; ++run, tA += BUILD_RUNS_OF) {
    tB = tA + BUILD_RUN;
    pool_run(std::true_type(), std::false_type());
  }
  tB = min(tA + BUILD_RUN, L);
  if (tA + BUILD_RUN <= L)  // all of the tokens exist, and so all blocks are whole
    pool_run(std::true_type(), std::true_type());
  else if (tA < tB)
    pool_run(std::false_type(), std::true_type());

  // ---- 2. ranges: the waves' extrema folded (word i: minima, then maxima; R words a thread), and into the segment's
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    s_ext[wave][0][v * 64 + lane] = make_float2(mn[v][0], mn[v][1]);
    s_ext[wave][1][v * 64 + lane] = make_float2(mx[v][0], mx[v][1]);
  }
  __syncthreads();
  uint32_t word[REP + 1];
#pragma unroll
  for (int u = 0; u <= REP; ++u) {
    const int i = u * BUILD_THREADS + tid, kind = i / W, c = i % W;
    float x = reinterpret_cast<const float*>(s_ext[0][kind])[c];
#pragma unroll
    for (int w = 1; w < BUILD_WAVES; ++w) {
      const float y = reinterpret_cast<const float*>(s_ext[w][kind])[c];
      x = kind ? fmaxf(x, y) : fminf(x, y);
    }
    word[u] = kind ? float_key(x) : ~float_key(x);
  }
  const uint32_t C = (uint32_t)build_chunks(L);
  uint32_t* meet = p.meet + (size_t)s * p.pitch;
  uint32_t* left = meet + meet_left(W, p.copies);
  const int words = (int)(C + 31) / 32;  // of bits
  bool last = true;         // to sign in
  uint32_t some_left = 0;   // rows in the workspace that somebody has to take on
  if (C > 1) {              // (a segment of one chunk shares nothing)
    const int group = chunk & (p.copies - 1);
    uint32_t* copy = meet + group * 2 * W + tid;
    uint32_t* flag = meet + meet_flags(W, p.copies) + group * 32;
    uint64_t* state = reinterpret_cast<uint64_t*>(meet + meet_state(W, p.copies));
#pragma unroll
    for (int u = 0; u <= REP; ++u)
      __hip_atomic_fetch_max(copy + u * BUILD_THREADS, word[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_stores_acknowledged();
    __syncthreads();
    if (tid == 0) {
      const uint64_t now = __hip_atomic_fetch_add(state, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
      uint32_t seen = 0;
      if ((uint32_t)now != C && C - (uint32_t)now <= BUILD_MISSING) {
        const uint64_t since = wall_clock64();
        do {
          __builtin_amdgcn_s_sleep(24);
          seen = (uint32_t)ld_i32<true>(reinterpret_cast<const int32_t*>(flag));
        } while (!seen && wall_clock64() - since < BUILD_WAIT_TICKS);
      }
      s_word[0] = seen;
      s_word[1] = (uint32_t)now == C;
      s_word[2] = now >> 32 ? MEET_SOME_LEFT : 0u;  // (of the last: nobody who finds the segment incomplete leaves any more)
    }
    __syncthreads();
    uint32_t seen = s_word[0];
    last = s_word[1];
    if (!seen && !last) {
      // ---- leave: rows out, a bit for whoever is there at the end; unless the segment became complete meanwhile
#pragma unroll
      for (int q = 0; q < BUILD_EIGHTS; ++q) {
        const int t = tA + 8 * q;
        if (!closes(t)) continue;
        float r[REP + 1][2];
        kept[q].get(r);
        row_out(t, r);
      }
      wait_stores_acknowledged();
      __syncthreads();
      if (tid == 0) {
        __hip_atomic_fetch_or(left + (chunk >> 5), 1u << (chunk & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_stores_acknowledged();
        const uint64_t was = __hip_atomic_fetch_add(state, (uint64_t)1 << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_word[0] = 0;
        if ((uint32_t)was == C) {  // it did: stay.  (The last chunk has signed in and waits for nobody before it raises the flag)
          do {
            __builtin_amdgcn_s_sleep(8);
            s_word[0] = (uint32_t)ld_i32<true>(reinterpret_cast<const int32_t*>(flag));
          } while (!s_word[0]);
        }
      }
      __syncthreads();
      seen = s_word[0];
      if (!seen) return;
    }
    // the segment's words: once the flag is up in any copy, before as the maximum of all
#pragma unroll
    for (int u = 0; u <= REP; ++u) {
      if (!last) {
        word[u] = (uint32_t)ld_i32<true>(reinterpret_cast<const int32_t*>(copy + u * BUILD_THREADS));
      } else {
        uint32_t x[BUILD_MAX_COPIES];
#pragma unroll
        for (int k = 0; k < BUILD_MAX_COPIES; ++k)
          x[k] = (uint32_t)ld_i32<true>(reinterpret_cast<const int32_t*>(meet + (k & (p.copies - 1)) * 2 * W + u * BUILD_THREADS + tid));
#pragma unroll
        for (int k = 0; k < BUILD_MAX_COPIES; ++k) word[u] = max(word[u], x[k]);
      }
    }
    some_left = (last ? s_word[2] : seen) & MEET_SOME_LEFT;
    if (last) {
#pragma unroll
      for (int u = 0; u <= REP; ++u)
        for (int k = 0; k < p.copies; ++k) st_i32<true>(reinterpret_cast<int32_t*>(meet + k * 2 * W + u * BUILD_THREADS + tid), (int32_t)word[u]);
      if (some_left)
        for (int w = tid; w < words; w += BUILD_THREADS) {
          const int32_t bits = ld_i32<true>(reinterpret_cast<const int32_t*>(left + w));
          for (int k = 0; k < p.copies; ++k) st_i32<true>(reinterpret_cast<int32_t*>(left + (k + 1) * words + w), bits);
        }
      wait_stores_acknowledged();
      __syncthreads();
      if ((int)tid < p.copies)
        st_i32<true>(reinterpret_cast<int32_t*>(meet + meet_flags(W, p.copies) + tid * 32), (int32_t)(MEET_COMPLETE | some_left));
    }
  }
  uint32_t* s_meet = reinterpret_cast<uint32_t*>(s_ext);
  __syncthreads();
#pragma unroll
  for (int u = 0; u <= REP; ++u) s_meet[u * BUILD_THREADS + tid] = word[u];
  __syncthreads();

  // ---- 3. the ranges of this lane's values, and its rows' codes
  float lo[REP + 1][2], inv[REP + 1][2];
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    const int c = v * ABSB_HEAD_DIM + lane * 2;
    const uint64_t kn = reinterpret_cast<const uint64_t*>(s_meet)[c / 2], kx = reinterpret_cast<const uint64_t*>(s_meet)[(W + c) / 2];
    float scale[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      lo[v][i] = key_float(~(uint32_t)(kn >> (32 * i)));
      const float rng = key_float((uint32_t)(kx >> (32 * i))) - lo[v][i];
      scale[i] = inv[v][i] = 0.0f;
      if (rng > 0.0f) {
        scale[i] = rng / 15.0f;
        inv[v][i] = 15.0f / rng;
      }
    }
    if (last && wave == 0) {
      *reinterpret_cast<float2*>(p.qscale + (size_t)s * W + c) = make_float2(scale[0], scale[1]);
      *reinterpret_cast<float2*>(p.qmin + (size_t)s * W + c) = make_float2(lo[v][0], lo[v][1]);
    }
  }
  // byte i of a vector's 64 holds its value 2i (low nibble) and 2i+1 (high nibble): a lane's two
  uint8_t* codes = p.codes + (size_t)off * (W / 2) + lane;
#pragma unroll
  for (int q = 0; q < BUILD_EIGHTS; ++q) {
    const int t = tA + 8 * q;
    if (!closes(t)) continue;
    float r[REP + 1][2];
    kept[q].get(r);
#pragma unroll
    for (int v = 0; v <= REP; ++v) codes[(size_t)(t >> lb) * (W / 2) + v * 64] = (uint8_t)code_pair(r[v][0], r[v][1], lo[v], inv[v]);
  }
  // the codes of the rows of a run that went through the workspace
  auto rows_back = [&](int t) __attribute__((always_inline)) {
    constexpr int U = BUILD_EIGHTS / (REP + 1);  // rows at once
    const int end = (min(t + BUILD_RUNS_OF, L) + B - 1) >> lb;
    for (int j0 = (t >> lb) + wave; j0 < end; j0 += U * BUILD_WAVES) {
      uint64_t r[REP + 1][U];
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int v = 0; v <= REP; ++v) {
          const float* row = p.cent + ((size_t)off + min(j0 + i * BUILD_WAVES, end - 1)) * W;  // past the end: the last again
          r[v][i] = __hip_atomic_load(reinterpret_cast<const uint64_t*>(row + v * ABSB_HEAD_DIM + lane * 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int j = j0 + i * BUILD_WAVES;
        if (j >= end) break;
#pragma unroll
        for (int v = 0; v <= REP; ++v) {
          const float2 x = bitcast<float2>(r[v][i]);
          codes[(size_t)j * (W / 2) + v * 64] = (uint8_t)code_pair(x.x, x.y, lo[v], inv[v]);
        }
      }
    }
  };
#pragma unroll 1
  for (int run = 0; run < last_run; ++run) rows_back(t0 + run * BUILD_RUNS_OF);
  if (!some_left) return;

  // ---- 4. the chunks that left, shared out among those that are here: this one is the mine-th of `here`, and takes on
  // the mine-th of those that left, the (mine + here)-th, ...
  const uint32_t* bits = left + ((chunk & (p.copies - 1)) + 1) * words;
  int gone = 0, mine = chunk;
  for (int w0 = 0; w0 < words; w0 += 64) {
    const int w = w0 + (int)lane;
    const uint32_t x = w < words ? (uint32_t)ld_i32<true>(reinterpret_cast<const int32_t*>(bits + w)) : 0u;
    const uint32_t below = w < (chunk >> 5) ? ~0u : w == (chunk >> 5) ? (1u << (chunk & 31)) - 1u : 0u;
    uint32_t n, n_below;
    wave_incl_scan_u32((uint32_t)__popc(x), &n);
    wave_incl_scan_u32((uint32_t)__popc(x & below), &n_below);
    gone += (int)n;
    mine -= (int)n_below;
    if (w == (chunk >> 5) && (x >> (chunk & 31) & 1u)) mine = INT_MAX;  // its bit came in time: nobody counts on this one
  }
  mine = (int)wave_reduce_u32((uint32_t)mine, [](uint32_t a, uint32_t b) { return max(a, b); });
  const int here = (int)C - gone;
  for (int w0 = 0, base = 0; w0 < words && mine < gone; w0 += 64) {
    const int w = w0 + (int)lane;
    const uint32_t x = w < words ? (uint32_t)ld_i32<true>(reinterpret_cast<const int32_t*>(bits + w)) : 0u;
    uint32_t n;
    const int to = base + (int)wave_incl_scan_u32((uint32_t)__popc(x), &n);
    base += (int)n;
    for (; mine < base; mine += here) {
      const int at = __popcll(__ballot(to <= mine));  // lane whose word holds it
      uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, at);
      for (int skip = mine - (__builtin_amdgcn_readlane(to, at) - __popc(y)); skip > 0; --skip) y &= y - 1;
      const int t = ((w0 + at) * 32 + __builtin_ctz(y)) * runs * BUILD_RUNS_OF, end = min(t + runs * BUILD_RUNS_OF, L);
#pragma unroll 1
      for (int u = t; u < end; u += BUILD_RUNS_OF) rows_back(u);
    }
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
  const int lb = p.g.heads.log2_block(h), lP = p.g.log2_page;
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
// (What the chain starts with comes as arguments of their own, in scalar registers when a wave
// starts: a decode loop of 8 tokens and 4 layers 748 -> 735 us, 0.4 an append.)
template <int DT, int REP>
__global__ __launch_bounds__(BUILD_THREADS) void append_kernel(addr2 lens_pages, addr2 keys_tails, addr2 qscale_qmin, int2v nseg_Hkv, AppendParams p) {
  constexpr int W = ABSB_HEAD_DIM * (REP + 1);
  const auto seq_lens = from_addr<const int32_t>(lens_pages.x), page_table = from_addr<const int32_t>(lens_pages.y);
  const auto keys = from_addr<const uint16_t>(keys_tails.x);
  const auto tails = from_addr<float>(keys_tails.y);
  const auto qscale = from_addr<const float>(qscale_qmin.x), qmin = from_addr<const float>(qscale_qmin.y);
  const int nseg = nseg_Hkv.x, Hkv = nseg_Hkv.y;
  const int tid = threadIdx.x, grp = tid >> 4, li = tid & 15;
  const int s = blockIdx.x * BUILD_GROUPS + grp;
  if (s >= nseg) return;
  const int b = s / Hkv, h = s % Hkv;
  const int t_new = seq_lens[b] - 1;
  float* tail = tails + (size_t)s * W + li * 8;
  float st[REP + 1][8], scale[REP + 1][8], mn[REP + 1][8];
#pragma unroll
  for (int v = 0; v <= REP; ++v) {
    const size_t at = (size_t)s * W + v * ABSB_HEAD_DIM + li * 8;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<float4*>(&st[v][4 * q]) = *reinterpret_cast<const float4*>(tail + v * ABSB_HEAD_DIM + 4 * q);
      *reinterpret_cast<float4*>(&scale[v][4 * q]) = *reinterpret_cast<const float4*>(qscale + at + 4 * q);
      *reinterpret_cast<float4*>(&mn[v][4 * q]) = *reinterpret_cast<const float4*>(qmin + at + 4 * q);
    }
  }
  const int off = p.cent_off[s];
  const int lb = p.g.heads.log2_block(h), lP = p.g.log2_page;
  const int j = t_new >> lb, t0 = j << lb;
  const int page = page_table[(size_t)b * p.g.pt_stride + (t_new >> lP)];
  const uint4 row = *reinterpret_cast<const uint4*>(keys + (size_t)page * p.g.s_page + (size_t)h * p.g.s_head +
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
    hipLaunchKernelGGL((append_kernel<DT, REP>), grid, block, 0, stream, addr2{addr(p.seq_lens), addr(p.page_table)}, addr2{addr(p.k), addr(p.tail)},
                       addr2{addr(p.qscale), addr(p.qmin)}, int2v{p.nseg, p.g.Hkv}, p);
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
  p.meet = reinterpret_cast<uint32_t*>(ws + pl.ws_meet);
  p.qscale = qscale;
  p.qmin = qmin;
  p.codes = codes;
  p.pitch = pl.build_pitch;
  p.copies = pl.build_copies;
  p.g = g;
  const dim3 grid((unsigned)pl.build_max_chunks, (unsigned)pl.nstore), block(BUILD_THREADS);
  if (pl.build_max_chunks > 1) {  // (segments of one chunk share nothing)
    const int words = meet_used(ABSB_HEAD_DIM * (g.repr + 1), pl.build_copies, pl.build_max_chunks);
    hipLaunchKernelGGL(build_clear_kernel, dim3((unsigned)((words + 255) / 256), grid.y), dim3(256), 0, stream, p, words);
    const int rc = check_launch();
    if (rc != ABSB_OK) return rc;
  }
  if (dtype == ABSB_F16 && g.repr == ABSB_REPR_MEAN)
    hipLaunchKernelGGL((build_kernel<ABSB_F16, 0>), grid, block, 0, stream, p);
  else if (dtype == ABSB_F16)
    hipLaunchKernelGGL((build_kernel<ABSB_F16, 1>), grid, block, 0, stream, p);
  else if (g.repr == ABSB_REPR_MEAN)
    hipLaunchKernelGGL((build_kernel<ABSB_BF16, 0>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((build_kernel<ABSB_BF16, 1>), grid, block, 0, stream, p);
  return check_launch();
}

}  // namespace absb

// What the persistent decode kernels (step_kernel.h, step_batch.h) and the streaming output layers (head_one.h,
// head_batch.h) share: the exchange between workgroups, requests, staging, the geometry and the streaming loop of a
// matrix-vector product, attention over the cache pages.  Compiled for workgroups of MDI_STEP_WAVES wavefronts, in a
// namespace of its own for each.
#pragma once
#include <type_traits>

#include "bounded_wait.h"
#include "device_utils.h"

#ifndef MDI_STEP_WAVES
#error "MDI_STEP_WAVES: wavefronts per workgroup"
#endif
#define MDI_STEP_CAT2(a, b) a##b
#define MDI_STEP_CAT(a, b) MDI_STEP_CAT2(a, b)

namespace mdi {
namespace MDI_STEP_CAT(step_w, MDI_STEP_WAVES) {

#define MDI_GLOBAL __attribute__((address_space(1)))

constexpr int kStepWaves = MDI_STEP_WAVES;       // wavefronts per workgroup
constexpr int kStepThreads = 64 * kStepWaves;


constexpr int kTile = 4;                 // items per register tile (two 16-byte loads each)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
struct Tile { u32x4 r[2 * kTile]; };

// Tagged exchange.  A store is acknowledged before every compute die can read it back, so a flag raised after it
// proves nothing to a reader; the data validates itself: value and the writing phase's counter travel in one 8-byte
// store, and a reader that finds another counter simply loads again.  No ordering between stores is needed.
__device__ __forceinline__ void st_tag(tagged_t* p, float v, unsigned tag) {
  __hip_atomic_store((MDI_GLOBAL tagged_t*)p, ((tagged_t)tag << 32) | (tagged_t)__float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ tagged_t ld_raw(const tagged_t* p) { return __hip_atomic_load((const MDI_GLOBAL tagged_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float tag_value(tagged_t u) { return __uint_as_float((uint32_t)u); }
// A wait that expires raises the partition's error word and its workgroup's failure flag (an index in lds_flag()); the
// other waits of the workgroup then end at their next look at the flag.
constexpr int kFailed = 2;
__device__ __forceinline__ int* lds_flag() { extern __shared__ float smem[]; return (int*)(smem + 16); }
// (The same for all lanes of the wavefront that are active: its loops have no lanes to keep apart.)
__device__ __forceinline__ bool poll_again(int& polls, int spin_limit, int* err) {
  return may_poll_again(
      polls, spin_limit, [&]() { return __builtin_amdgcn_readfirstlane(__hip_atomic_load(lds_flag() + kFailed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0; },
      [&]() {
        __hip_atomic_store(lds_flag() + kFailed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store((MDI_GLOBAL int*)err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      });
}
// Asks again while any lane of the wavefront misses something: bad() says whether this one does.  A loop that lanes leave
// one by one keeps a copy of every word asked for, and moves all of them in every round.
template <typename BAD, typename ASK>
__device__ __forceinline__ void poll_while(const BAD& bad, const ASK& ask, int spin_limit, int* err) {
  int it = 0;
  while (__ballot(bad()) != 0) {
    if (!poll_again(it, spin_limit, err)) break;
    __builtin_amdgcn_s_sleep(1);
    ask();
  }
}
// Returns the value once its tag is `tag`, or whatever is there when the wait ends otherwise.
__device__ __forceinline__ float settle(const tagged_t* p, tagged_t u, unsigned tag, int spin_limit, int* err) {
  poll_while([&]() { return (uint32_t)(u >> 32) != tag; }, [&]() { u = ld_raw(p); }, spin_limit, err);
  return tag_value(u);
}

template <typename T> struct Unpack;
template <> struct Unpack<float> {
  __device__ static __forceinline__ void go(const u32x4& t, float (&v)[4]) {
    v[0] = __uint_as_float(t.x); v[1] = __uint_as_float(t.y); v[2] = __uint_as_float(t.z); v[3] = __uint_as_float(t.w);
  }
};
template <> struct Unpack<bf16_t> {
  __device__ static __forceinline__ void go(const u32x4& t, float (&v)[8]) {
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xFFFF0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xFFFF0000u);
    v[4] = __uint_as_float(t.z << 16); v[5] = __uint_as_float(t.z & 0xFFFF0000u);
    v[6] = __uint_as_float(t.w << 16); v[7] = __uint_as_float(t.w & 0xFFFF0000u);
  }
};

// Loads through buffer descriptors.  An offset of kNowhere, or a descriptor of nothing, reads as zero and touches no
// memory, so a lane without a word, or an absent bias, needs no branch around its load (which would merge the loaded
// register with another value, and where the compiler copies to do so it waits for the load there and then), and an
// address costs one register and an immediate instead of two additions.
typedef __amdgpu_buffer_rsrc_t Buffer;
constexpr uint32_t kNowhere = 0x80000000u;
__device__ __forceinline__ Buffer buffer_at(const void* p) { return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, p ? 0x7FFFFFFF : 0, 0x00020000); }
__device__ __forceinline__ float ld_f32(Buffer b, uint32_t off) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, 0)); }
constexpr int kAgentScope = 0x10;        // the sc1 bit: the load is answered by what all dies see
__device__ __forceinline__ tagged_t ld_word(Buffer b, uint32_t off) {
  return __builtin_bit_cast(tagged_t, __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, 0, kAgentScope));
}

// The kernel's arguments, as if read for the first time: a phase loads what it needs of them when it starts, instead of
// keeping everything that some phase needs in scalar registers (of which there are not nearly enough) all the time.
template <typename AR>
__device__ __forceinline__ const AR& args_again() {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const AR*)(const __attribute__((address_space(4))) AR*)p;
}
// Two exchanged words as one 16-byte piece.  Each of them carries its own counter, so only 8 bytes need to be seen whole.
__device__ __forceinline__ u32x4 ld_two(Buffer b, uint32_t off, uint32_t uniform) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, (int)uniform, kAgentScope));
}
__device__ __forceinline__ void st_two(Buffer b, uint32_t off, uint32_t uniform, float v0, float v1, unsigned tag) {
  __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(v0), tag, __float_as_uint(v1), tag}, b, (int)off, (int)uniform, kAgentScope);
}
// An offset that the compiler takes for a new one, so that a poll's loads are not taken for those of the one before.
__device__ __forceinline__ uint32_t fresh(uint32_t off) { asm volatile("" : "+v"(off)); return off; }

enum StepPhase { PH_QKV = 0, PH_ATTN = 1, PH_OPROJ = 2, PH_UP = 3, PH_DOWN = 4 };

// optional timeline for profiling: thread 0 of every workgroup records a 100 MHz timestamp
__device__ __forceinline__ void stamp(const StepArgs& a, const StepSlot& S, int layer, int ph, int k) {
  if (S.trace && threadIdx.x == 0)
    S.trace[(((long)(blockIdx.x % a.nwg) * a.n_layer + layer) * 5 + ph) * 8 + k] = wall_clock64();
}


// LDS map (floats): [0,16) reduction scratch, [16,20) flags,
// [128, 128+part_floats) pair partials, then the vector.
constexpr int kLdsPart = 128;
__device__ __forceinline__ float* lds_red() { extern __shared__ float smem[]; return smem; }
__device__ __forceinline__ float* lds_part() { extern __shared__ float smem[]; return smem + kLdsPart; }
__device__ __forceinline__ float* lds_vec(int part_floats) { extern __shared__ float smem[]; return smem + kLdsPart + part_floats; }

// Waits for every load of this wavefront, those of no interest any more (a stream's tiles past its end) too: placed before a
// phase's results are stored.  A register that such a load may still write is waited for when it is next used, at the start
// of the next phase, and by then that means waiting for the stores as well: they share the counter with the loads.
__device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// N words at once, asked for again until all of a thread's carry the counter `tag`: one round trip however many were
// early (word by word, eight early words cost eight).  Asked for before a phase's weights, awaited after: loads return
// in order, and the workgroup that everybody waits for finds its words there.
// at(i, z): byte offset of word i; z is zero, and unknown to the compiler, so that the loads of one poll are not taken for
// those of the one before.  live(i): whether this thread wants word i at all; the others count as seen (asking for some
// word again in their place would have every workgroup hammer one line of memory).
struct AllLive { __device__ __forceinline__ bool operator()(int) const { return true; } };
template <int N, typename AT, typename LT = AllLive>
__device__ __forceinline__ void ask_words(tagged_t (&raw)[N], Buffer b, const AT& at, const LT& live = LT()) {
  uint32_t z = 0u;
  asm volatile("" : "+v"(z));
#pragma unroll
  for (int i = 0; i < N; ++i) raw[i] = ld_word(b, live(i) ? at(i, z) : kNowhere);
}
template <int N, typename AT, typename LT = AllLive>
__device__ __forceinline__ void await_words(tagged_t (&raw)[N], Buffer b, const AT& at, unsigned tag, int spin_limit, int* err, const LT& live = LT()) {
  poll_while([&]() {
    uint32_t bad = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) bad |= live(i) ? (uint32_t)(raw[i] >> 32) ^ tag : 0u;
    return bad != 0;
  }, [&]() { ask_words(raw, b, at, live); }, spin_limit, err);
}

// ---------------------------------------------------------------------------
// vector staging: n floats written earlier in this launch by other workgroups -> LDS
// With gain != nullptr (RMSNorm) the staged values are x[i] * gain[i] and the return value is this thread's share of
// sum(x^2); the common factor 1/rms is applied to the finished dot products.  Otherwise the values are staged as they
// are and the return value is this thread's share of their sum.
// A thread takes pairs tid, tid + threads, ...; its first four (and their gains) have been requested before.
struct VecAsk { u32x4 raw[4]; u32x2 gain[4]; };
__device__ __forceinline__ void vec_words(VecAsk& v, const tagged_t* src, int n, int q0) {
  const Buffer b = buffer_at(src);
  const uint32_t o = fresh((uint32_t)q0 * 16u);
#pragma unroll
  for (int j = 0; j < 4; ++j) v.raw[j] = ld_two(b, 2 * (q0 + j * kStepThreads) < n ? o + (uint32_t)(j * kStepThreads) * 16u : kNowhere, 0);
}
__device__ __forceinline__ void vec_ask(VecAsk& v, const tagged_t* src, int n, const float* gain, int q0) {
  vec_words(v, src, n, q0);
  const Buffer gb = buffer_at(gain);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    v.gain[j] = __builtin_amdgcn_raw_buffer_load_b64(gb, 2 * (q0 + j * kStepThreads) < n ? (q0 + j * kStepThreads) * 8 : (int)kNowhere, 0, 0);
}
template <bool kRms>
__device__ __forceinline__ float stage_coherent(VecAsk& v, const tagged_t* src, int n, float* xs, const float* gain, unsigned tag, int spin_limit, int* err, int tid) {
  float ss = 0.f;
  for (int q0 = tid; 2 * q0 < n; q0 += 4 * kStepThreads) {
    if (q0 != tid) vec_ask(v, src, n, kRms ? gain : nullptr, q0);
    poll_while([&]() {
      uint32_t bad = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) bad |= 2 * (q0 + j * kStepThreads) < n ? (v.raw[j].y ^ tag) | (v.raw[j].w ^ tag) : 0u;
      return bad != 0;
    }, [&]() { vec_words(v, src, n, q0); }, spin_limit, err);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = q0 + j * kStepThreads;
      const float x0 = __uint_as_float(v.raw[j].x), x1 = __uint_as_float(v.raw[j].z);   // (zeros past the end)
      ss += kRms ? x0 * x0 : x0; ss += kRms ? x1 * x1 : x1;
      if (2 * q < n) *reinterpret_cast<float2*>(xs + 2 * q) = kRms ? float2{x0 * __uint_as_float(v.gain[j].x), x1 * __uint_as_float(v.gain[j].y)} : float2{x0, x1};
    }
  }
  return ss;
}

// Sum over the workgroup, every thread gets it.  One barrier; `red` is a strip of kStepWaves floats that the previous
// call did not use.
__device__ __forceinline__ float step_sum(float v, float* red, int tid) {
  const float w = wave_sum_to_lane63(v);
  if ((tid & 63) == 63) red[tid >> 6] = w;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int k = 0; k < kStepWaves; ++k) t += red[k];
  return t;
}

// LayerNorm of the staged vector, each thread on the pairs it staged itself; s = its share of their sum.
__device__ __forceinline__ void layer_norm(float* xs, int n, float s, float eps, Buffer g, Buffer b, float* red, int tid) {
  auto two = [&](Buffer p, int q) __attribute__((always_inline)) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(p, 2 * q < n ? q * 8 : (int)kNowhere, 0, 0);
    return float2{__uint_as_float(v.x), __uint_as_float(v.y)};
  };
  auto apply = [&](int q, const float2& gv, const float2& bv, float mean, float rstd) __attribute__((always_inline)) {
    if (2 * q >= n) return;
    float2* p = reinterpret_cast<float2*>(xs) + q;
    const float2 x = *p;
    *p = float2{(x.x - mean) * rstd * gv.x + bv.x, (x.y - mean) * rstd * gv.y + bv.y};
  };
  const float2 g0 = two(g, tid), b0 = two(b, tid);      // the first gains and biases are on their way during the sums
  const float mean = step_sum(s, red, tid) / (float)n;
  float s2 = 0.f;
  for (int q = tid; 2 * q < n; q += kStepThreads) {
    const float2 x = reinterpret_cast<const float2*>(xs)[q];
    s2 += (x.x - mean) * (x.x - mean); s2 += (x.y - mean) * (x.y - mean);
  }
  const float rstd = 1.f / sqrtf(step_sum(s2, red + kStepWaves, tid) / (float)n + eps);
  apply(tid, g0, b0, mean, rstd);
  for (int q = tid + kStepThreads; 2 * q < n; q += kStepThreads) apply(q, two(g, q), two(b, q), mean, rstd);
}

__device__ __forceinline__ void normalise(float* xs, int n, int norm_kind, float eps, const float* g, const float* b, float* red) {
  if (norm_kind == MDI_NORM_LAYERNORM) {
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += kStepThreads) s += xs[i];
    const float mean = block_sum(s, red) / (float)n;
    float s2 = 0.f;
    for (int i = threadIdx.x; i < n; i += kStepThreads) { const float c = xs[i] - mean; s2 += c * c; }
    const float rstd = 1.f / sqrtf(block_sum(s2, red) / (float)n + eps);
    for (int i = threadIdx.x; i < n; i += kStepThreads) xs[i] = (xs[i] - mean) * rstd * g[i] + (b ? b[i] : 0.f);
  } else {
    float s2 = 0.f;
    for (int i = threadIdx.x; i < n; i += kStepThreads) s2 += xs[i] * xs[i];
    const float rstd = 1.f / sqrtf(block_sum(s2, red) / (float)n + eps);
    for (int i = threadIdx.x; i < n; i += kStepThreads) xs[i] = xs[i] * rstd * g[i];
  }
}

// ---------------------------------------------------------------------------
// GEMV phase geometry (all values uniform across the wavefront)
struct Geo {
  const char* W;
  int N, units, cpp;     // rows, 16-byte units per row, 64-lane chunks per row
  int row_bytes;
  int p_lo, n_pl;        // this workgroup owns n_pl pairs: blocks of 2^bshift consecutive pairs, block b of the
  int bshift, nwg;       // matrix going to workgroup b % nwg (p_lo = workgroup index).  At any moment the grid
                         // reads one contiguous window of the matrix, and a workgroup stays >= 64 KiB in place.
  int n_k;               // this wavefront's items: item k is flat index wave + k * wavefronts, flat = pair * cpp + chunk
  int dq, dr;            // wavefronts div and mod cpp: how (pair, chunk) moves from one item to the next
  int pl0, c0;           // the wavefront's first item
  // first row of pair p = (p >> rsh) * rmul + (p & rmask), its partner rstep rows on: rows (2p, 2p + 1), or RoPE partners
  // (i, i + h/2) inside heads of h rows (head sizes are powers of two)
  int rsh, rmask, rmul, rstep;
};
template <typename WT, bool kRope>
__device__ __forceinline__ Geo make_geo(const GemvGeo& P, long w_off, int wg, int nwg, int wave, int h) {
  Geo g;
  g.W = (const char*)P.W + w_off;
  g.N = P.N; g.units = P.units; g.cpp = P.cpp; g.row_bytes = P.units * 16;
  g.p_lo = wg; g.nwg = nwg; g.bshift = P.bshift;
  const int own = P.own_q + (wg < P.own_r ? 1 : 0);
  g.n_pl = (own << P.bshift) - (wg == P.last_wg ? P.last_short : 0);
  const int flat = g.n_pl * g.cpp;
  g.n_k = flat > wave ? (flat - wave + kStepWaves - 1) / kStepWaves : 0;
  g.dq = P.dq; g.dr = P.dr;
  g.pl0 = (int)((unsigned)(wave * P.cpp_magic) >> 16); g.c0 = wave - g.pl0 * g.cpp;
  if (kRope) {
    const int half = h >> 1;
    g.rsh = 31 - __builtin_clz(half); g.rmask = half - 1; g.rmul = h; g.rstep = half;
  } else {
    g.rsh = 0; g.rmask = 0; g.rmul = 2; g.rstep = 1;
  }
  return g;
}
__device__ __forceinline__ void geo_next(const Geo& g, int& pl, int& c) {
  c += g.dr; pl += g.dq;
  if (c >= g.cpp) { c -= g.cpp; ++pl; }
}
__device__ __forceinline__ int geo_pair(const Geo& g, int pl) {     // local pair index -> pair index in the matrix
  return ((((pl >> g.bshift) * g.nwg) + g.p_lo) << g.bshift) + (pl & ((1 << g.bshift) - 1));
}
__device__ __forceinline__ int geo_row(const Geo& g, int p, int j) {
  return (p >> g.rsh) * g.rmul + (p & g.rmask) + j * g.rstep;
}

// the step's own input (token embedding + learned position, or the previous stage's activation), staged as stage_coherent
// does it - same arithmetic, element order and thread mapping, so that a layer gives the same bits whether it is the first
// of its partition or not (where the model is cut changes nothing); gres: the residual phases' rows
template <typename WT, bool kLn>
__device__ __forceinline__ float stage_input(const StepArgs& a, const StepSlot& S, float* xs, const float* gain, const Geo& gres, unsigned tag, int tid) {
  const int n = a.d;
  if (S.in_kind == IN_TOKEN) {
    const long tok = checked_token(S.in, 0, a.vocab, a.err);
    for (int i = tid; i < n; i += kStepThreads) {
      float v = Storage<WT>::get((const WT*)a.wte + tok * n + i);
      if (a.wpe) v += Storage<WT>::get((const WT*)a.wpe + (long)S.pos * n + i);
      xs[i] = v;
    }
  } else {
    for (int i = tid; i < n; i += kStepThreads) xs[i] = load_kind(S.in, S.in_kind, i);
  }
  __syncthreads();
  // rows this workgroup owns in the residual phases get their starting value
  for (int pl = tid; pl < gres.n_pl; pl += kStepThreads) {
    const int r = 2 * geo_pair(gres, pl);
    st_tag(S.xres + r, xs[r], tag);
    if (r + 1 < n) st_tag(S.xres + r + 1, xs[r + 1], tag);
  }
  __syncthreads();                                   // those rows have been read
  float ss = 0.f;
  for (int q = tid; 2 * q < n; q += kStepThreads) {
    float2* p = reinterpret_cast<float2*>(xs) + q;
    const float2 x = *p;
    ss += kLn ? x.x : x.x * x.x; ss += kLn ? x.y : x.y * x.y;
    if (!kLn) { const MDI_GLOBAL float* g = (const MDI_GLOBAL float*)gain; *p = float2{x.x * g[2 * q], x.y * g[2 * q + 1]}; }
  }
  return ss;
}

// Where a wavefront stands in its items (local pair, chunk of the row): tiles are issued, and multiplied, in order, so
// each side keeps a cursor and moves it item by item instead of dividing the item index again for every tile.
struct Cursor {
  int pl, c;
  int row_pl;                          // the local pair whose rows b0, b1 are (-1: none yet)
  Buffer b0, b1;                       // (issue side only) a pair's rows, each as long as a row; they stay the same over its chunks
};
__device__ __forceinline__ Cursor cursor_start(const Geo& g) {
  Cursor cur;
  cur.pl = g.pl0; cur.c = g.c0; cur.row_pl = -1; cur.b0 = cur.b1 = buffer_at(nullptr);
  return cur;
}

// Every call issues exactly 2 * kTile loads, whatever the geometry: a fixed number of loads per tile is what lets
// the compiler wait for one tile while the next stays in flight (its counters cannot follow conditional loads).
// Items past the end of the wavefront's share, and lanes past the end of a row, read nothing; gemv_compute skips the former
// and masks the latter or multiplies them by zeros.  All of this is scalar arithmetic, which the wavefronts of a
// compute unit share one unit for, on the critical path of a phase's start: it is kept short.
__device__ __forceinline__ void gemv_issue(Tile& t, const Geo& g, Cursor& cur, int lane) {
  int pl = cur.pl, c = cur.c;
#pragma unroll
  for (int s = 0; s < kTile; ++s) {
    const bool own = pl < g.n_pl;
    if (pl != cur.row_pl) {                                     // uniform; long rows keep a pair for several items
      const int r0 = own ? geo_row(g, geo_pair(g, pl), 0) : 0, r1 = min(r0 + g.rstep, g.N - 1);
      cur.b0 = __builtin_amdgcn_make_buffer_rsrc((void*)(g.W + (long)r0 * g.row_bytes), 0, g.row_bytes, 0x00020000);
      cur.b1 = __builtin_amdgcn_make_buffer_rsrc((void*)(g.W + (long)r1 * g.row_bytes), 0, g.row_bytes, 0x00020000);
      cur.row_pl = pl;
    }
    const int off = own ? lane * 16 : (int)kNowhere, at = own ? c * 1024 : 0;
    t.r[2 * s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(cur.b0, off, at, 0));
    t.r[2 * s + 1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(cur.b1, off, at, 0));
    geo_next(g, pl, c);
  }
  cur.pl = pl; cur.c = c;
}

// kPadded: the caller has zeros in xs behind the vector, up to a whole number of 64-lane chunks, so the lanes past the
// end of a row (which hold zeros, see gemv_issue) find finite numbers there and need no case of their own.
template <typename WT, bool kPadded>
__device__ __forceinline__ void gemv_compute(const Tile& t, const Geo& g, int ti, Cursor& cur, int wave, int lane, const float* xs,
                                             float* part, float& acc0, float& acc1) {
  constexpr int V = Storage<WT>::kVec;
  int pl = cur.pl, c = cur.c;
#pragma unroll
  for (int s = 0; s < kTile; ++s) {
    int npl = pl, nc = c;
    geo_next(g, npl, nc);
    const int k = ti * kTile + s;
    if (k < g.n_k) {                                         // uniform
      const int unit = c * 64 + lane;
      if (kPadded || unit < g.units) {
        float w0[V], w1[V], xv[V];
        Unpack<WT>::go(t.r[2 * s], w0);
        Unpack<WT>::go(t.r[2 * s + 1], w1);
#pragma unroll
        for (int e = 0; e < V; e += 4) {
          const float4 q4 = *reinterpret_cast<const float4*>(xs + unit * V + e);
          xv[e] = q4.x; xv[e + 1] = q4.y; xv[e + 2] = q4.z; xv[e + 3] = q4.w;
        }
#pragma unroll
        for (int e = 0; e < V; ++e) { acc0 = fmaf(w0[e], xv[e], acc0); acc1 = fmaf(w1[e], xv[e], acc1); }
      }
      if (npl != pl || k == g.n_k - 1) {                     // this wavefront's share of the pair is complete
        const float r0 = wave_sum_to_lane63(acc0), r1 = wave_sum_to_lane63(acc1);
        if (lane == 63) { part[(pl * 2) * kStepWaves + wave] = r0; part[(pl * 2 + 1) * kStepWaves + wave] = r1; }
        acc0 = 0.f; acc1 = 0.f;
      }
    }
    pl = npl; c = nc;
  }
  cur.pl = pl; cur.c = c;
}

// What a phase's epilogue needs beside the sums, for pair pl: QKV: (cos, sin); all: the biases.  A thread's first pair's
// are fetched before the stream.
template <typename T> __device__ __forceinline__ float rounded(float v);   // as the storage type holds it
template <> __device__ __forceinline__ float rounded<float>(float v) { return v; }
template <> __device__ __forceinline__ float rounded<bf16_t>(float v) { return bf16_to_f32(f32_to_bf16(v)); }
template <typename T> __device__ __forceinline__ T stored(float v);
template <> __device__ __forceinline__ float stored<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t stored<bf16_t>(float v) { return f32_to_bf16(v); }
struct FinOps { float c, s, b0, b1; int p, r0, r1; };
template <int ph, bool kSwiglu>
__device__ __forceinline__ FinOps fin_ops(const Geo& g, const StepArgs& a, const StepSlot& S, long w_off, int pl) {
  FinOps o{};
  const bool own = pl < g.n_pl;
  o.p = geo_pair(g, own ? pl : 0); o.r0 = geo_row(g, o.p, 0); o.r1 = geo_row(g, o.p, 1);
  if constexpr (!(ph == PH_UP && kSwiglu)) {
    const float* bias = a.pr[ph == PH_QKV ? 0 : ph - 1].bias;
    const Buffer b = buffer_at(bias ? (const char*)bias + w_off : nullptr);
    o.b0 = ld_f32(b, own ? (uint32_t)o.r0 * 4u : kNowhere);
    o.b1 = ld_f32(b, own && o.r1 < g.N ? (uint32_t)o.r1 * 4u : kNowhere);
  }
  if constexpr (ph == PH_QKV) {
    const bool turned = own && (o.r0 >> (31 - __builtin_clz(a.h))) < a.H + a.K;   // (head sizes are powers of two)
    const u32x2 cs = __builtin_amdgcn_raw_buffer_load_b64(buffer_at(S.rope), turned ? (o.r0 & (a.h - 1)) * 8 : (int)kNowhere, 0, 0);
    o.c = __uint_as_float(cs.x); o.s = __uint_as_float(cs.y);
  }
  return o;
}

// Sums the wavefront slots of every pair and applies the phase's epilogue; kv: this layer's pages.
template <typename WT, int ph, bool kSwiglu>
__device__ __forceinline__ void gemv_finish(const Geo& g, int layer, const StepArgs& a, const StepSlot& S, char* kv, const float* part,
                                            float row_scale, tagged_t x0_pre, tagged_t x1_pre, FinOps ops, long w_off, unsigned epoch, int tid) {
  const unsigned wtag = epoch + 1;                            // what this phase writes carries the next counter
  for (int pl = tid; pl < g.n_pl; pl += kStepThreads) {
    float v0 = 0.f, v1 = 0.f;
#pragma unroll
    for (int w = 0; w < kStepWaves; ++w) { v0 += part[(pl * 2) * kStepWaves + w]; v1 += part[(pl * 2 + 1) * kStepWaves + w]; }
    v0 *= row_scale; v1 *= row_scale;
    if (pl != tid) ops = fin_ops<ph, kSwiglu>(g, a, S, w_off, pl);
    const int p = ops.p, r0 = ops.r0, r1 = ops.r1;
    if constexpr (ph == PH_QKV) {
      v0 += ops.b0; v1 += ops.b1;
      const int head = r0 >> (31 - __builtin_clz(a.h)), i = r0 & (a.h - 1);
      if (S.rope && head < a.H + a.K) {
        const float t0 = v0 * ops.c - v1 * ops.s, t1 = v0 * ops.s + v1 * ops.c;
        v0 = t0; v1 = t1;
      }
      if (head < a.H) {
        st_tag(S.q + r0, v0, wtag); st_tag(S.q + r1, v1, wtag);
      } else {
        // the cache row is for later launches (plain stores); this launch's attention takes the same
        // rounded values from the tagged copy
        const bool is_v = head >= a.H + a.K;
        const int kvh = head - a.H - (is_v ? a.K : 0);
        MDI_GLOBAL WT* dst = (MDI_GLOBAL WT*)kv + S.kv_tok_off + (long)(kvh * 2 + (is_v ? 1 : 0)) * a.pt_h + i;
        dst[0] = stored<WT>(v0); dst[a.h >> 1] = stored<WT>(v1);
        tagged_t* kn = S.knew + (is_v ? a.K * a.h : 0) + kvh * a.h + i;
        st_tag(kn, rounded<WT>(v0), wtag); st_tag(kn + (a.h >> 1), rounded<WT>(v1), wtag);
      }
    } else if constexpr (ph == PH_UP) {
      if constexpr (kSwiglu) {
        st_tag(S.u + p, silu_f(v0) * v1, wtag);              // rows (2f, 2f+1) = (gate_f, up_f)
      } else {
        v0 += ops.b0; v1 += ops.b1;
        const bool tanh_form = a.mlp_kind == MDI_MLP_GELU_TANH;
        st_tag(S.u + r0, tanh_form ? gelu_tanh_f(v0) : gelu_erf_f(v0), wtag);
        if (r1 < g.N) st_tag(S.u + r1, tanh_form ? gelu_tanh_f(v1) : gelu_erf_f(v1), wtag);
      }
    } else {                                                  // residual phases
      const bool last = ph == PH_DOWN && layer == a.n_layer - 1;
      const bool two = r1 < g.N;
      // rows of the first kStepThreads pairs were fetched before the stream
      const bool pre = pl == tid;
      // this workgroup wrote these rows itself: two phases ago (output projection) or one (down projection)
      const unsigned rtag = ph == PH_OPROJ ? epoch - 2 : epoch - 1;
      const float x0 = settle(S.xres + r0, pre ? x0_pre : ld_raw(S.xres + r0), rtag, a.spin_limit, a.err);
      const float x1 = two ? settle(S.xres + r1, pre ? x1_pre : ld_raw(S.xres + r1), rtag, a.spin_limit, a.err) : 0.f;
      v0 += x0 + ops.b0;
      st_tag(S.xres + r0, v0, wtag);
      if (last) store_kind(S.act_out, a.act_kind, r0, v0);
      if (two) {
        v1 += x1 + ops.b1;
        st_tag(S.xres + r1, v1, wtag);
        if (last) store_kind(S.act_out, a.act_kind, r1, v1);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// attention phase geometry
struct AttnGeo {
  bool active;
  int hg, split, kvh, s0, s1, s1p;
  int L, tpw, sub, hoff;
  int n_k;                // this wavefront's steps: step k covers tokens s0 + (k * wavefronts + wave) * tpw ..
  float f2, f4, f8, f16;  // 1 when a position's values are spread over at least that many lanes, else 0
  int pt_sh;              // log2(tokens per page) when that is a power of two, else -1 ...
  unsigned pt_magic;      // ... and then position / page size = high word of position * pt_magic (exact while
                          // position * page size < 2^32, which creating the partition checks)
};
// Sum over the g.L lanes that share a position, in every one of them.  Inside a row of 16 lanes every step is taken,
// multiplied by the step's flag: no branch on the (run-time) lane count in the streaming loop.  Same order of
// additions as group_sum.
template <int CTRL>
__device__ __forceinline__ float dpp_add_if(float v, float flag) {
  const int moved = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false);
  return fmaf(__int_as_float(moved), flag, v);
}
__device__ __forceinline__ float group_sum_lanes(float v, const AttnGeo& g) {
  v = dpp_add_if<kDppXor1>(v, g.f2);
  v = dpp_add_if<kDppXor2>(v, g.f4);
  v = dpp_add_if<kDppHalfMirror>(v, g.f8);
  v = dpp_add_if<kDppMirror>(v, g.f16);
  if (g.L >= 32) v += __shfl_xor(v, 16, 64);
  if (g.L >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}
__device__ __forceinline__ int page_of(const AttnGeo& g, int tok) {
  return g.pt_sh >= 0 ? tok >> g.pt_sh : (int)__umulhi((unsigned)tok, g.pt_magic);
}

template <typename WT, int G, typename AR, typename SL>
__device__ __forceinline__ AttnGeo make_attn_geo(const AR& a, const SL& S, int wg, int wave, int lane) {
  constexpr int V = Storage<WT>::kVec;
  AttnGeo g;
  g.L = a.h / V; g.tpw = 64 / g.L; g.sub = lane / g.L; g.hoff = (lane % g.L) * V;
  g.active = wg < a.n_hg * S.n_splits;
  g.hg = g.active ? wg % a.n_hg : 0;
  g.split = g.active ? wg / a.n_hg : 0;
  g.kvh = (g.hg * G) / (a.H / a.K);
  g.s0 = g.split * S.chunk;
  g.s1 = min(S.ctx, g.s0 + S.chunk);
  g.s1p = min(g.s1, S.ctx - 1);                               // the newest row is written in this launch
  const int steps = g.active && g.s1p > g.s0 ? (g.s1p - g.s0 + g.tpw - 1) / g.tpw : 0;
  g.n_k = steps > wave ? (steps - wave + kStepWaves - 1) / kStepWaves : 0;
  g.f2 = g.L >= 2 ? 1.f : 0.f; g.f4 = g.L >= 4 ? 1.f : 0.f; g.f8 = g.L >= 8 ? 1.f : 0.f; g.f16 = g.L >= 16 ? 1.f : 0.f;
  g.pt_sh = (a.pt & (a.pt - 1)) == 0 ? __builtin_ctz(a.pt) : -1;
  g.pt_magic = g.pt_sh >= 0 ? 0u : 0xFFFFFFFFu / (unsigned)a.pt + 1u;
  return g;
}

// Page numbers of the tokens of tile ti (slots without a token take token 0's).  The table entries of every position
// before the newest were written by earlier launches, so they are fetched a tile pair ahead of the rows they locate:
// a row's address then never waits for a table look-up.
template <typename AR, typename SL>
__device__ __forceinline__ void attn_pages(int (&pg)[kTile], const AttnGeo& g, const AR& a, const SL& S, int ti, int wave) {
  const MDI_GLOBAL int32_t* table = (const MDI_GLOBAL int32_t*)S.table;
#pragma unroll
  for (int s = 0; s < kTile; ++s) {
    const int k = ti * kTile + s;
    int tok = g.s0 + (k * kStepWaves + wave) * g.tpw + g.sub;
    if (!(k < g.n_k && tok < g.s1p)) tok = 0;
    pg[s] = __hip_atomic_load(table + page_of(g, tok), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Issues exactly 2 * kTile row loads (see gemv_issue) for tile ti, whose page numbers are in pg, then asks for the
// page numbers of the tile that goes into the same registers next; slots without a token re-read token 0.
template <typename WT, typename AR, typename SL>
__device__ __forceinline__ void attn_issue(Tile& t, int (&pg)[kTile], const AttnGeo& g, const AR& a, const SL& S, const void* pool_,
                                           int ti, int wave) {
  const MDI_GLOBAL WT* pool = (const MDI_GLOBAL WT*)pool_;
#pragma unroll
  for (int s = 0; s < kTile; ++s) {
    const int k = ti * kTile + s;
    int tok = g.s0 + (k * kStepWaves + wave) * g.tpw + g.sub;
    if (!(k < g.n_k && tok < g.s1p)) tok = 0;
    const int in_page = tok - page_of(g, tok) * a.pt;
    const MDI_GLOBAL WT* kp = pool + ((long)pg[s] * a.K + g.kvh) * 2 * a.pt_h + (long)in_page * a.h + g.hoff;
    t.r[2 * s] = *reinterpret_cast<const MDI_GLOBAL u32x4*>(kp);
    t.r[2 * s + 1] = *reinterpret_cast<const MDI_GLOBAL u32x4*>(kp + a.pt_h);
  }
  attn_pages(pg, g, a, S, ti + 2, wave);
}

template <typename WT, int G>
struct AttnState {
  float m[G], l[G], o[G][Storage<WT>::kVec];
};

template <typename WT, int G>
__device__ __forceinline__ void attn_update_f(AttnState<WT, G>& st, const AttnGeo& g, int h, const float (&kf)[Storage<WT>::kVec],
                                              const float (&vf)[Storage<WT>::kVec], bool valid, const float* qs) {
  constexpr int V = Storage<WT>::kVec;
#pragma unroll
  for (int gi = 0; gi < G; ++gi) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < V; e += 4) {
      const float4 q4 = *reinterpret_cast<const float4*>(qs + gi * h + g.hoff + e);
      s = fmaf(q4.x, kf[e], s); s = fmaf(q4.y, kf[e + 1], s); s = fmaf(q4.z, kf[e + 2], s); s = fmaf(q4.w, kf[e + 3], s);
    }
    s = group_sum_lanes(s, g);
    if (valid) {
      const float mn = fmaxf(st.m[gi], s);
      const float alpha = __expf(st.m[gi] - mn), p = __expf(s - mn);
      st.m[gi] = mn;
      st.l[gi] = st.l[gi] * alpha + p;
#pragma unroll
      for (int e = 0; e < V; ++e) st.o[gi][e] = st.o[gi][e] * alpha + p * vf[e];
    }
  }
}

// One tile = kTile cached positions per lane group.  The scores of all of them first, then ONE rescaling of the running
// sums to the new maximum, then the weighted values: a rescaling per position (as attn_update_f does for the single
// newest row) costs as many multiplications as the values themselves.
template <typename WT, int G>
__device__ __forceinline__ void attn_compute(AttnState<WT, G>& st, const Tile& t, const AttnGeo& g, int h, int ti, int wave,
                                             const float* qs) {
  constexpr int V = Storage<WT>::kVec;
  float sc[kTile][G];
  bool ok[kTile];
#pragma unroll
  for (int s = 0; s < kTile; ++s) {
    const int k = ti * kTile + s;
    const int tok = g.s0 + (k * kStepWaves + wave) * g.tpw + g.sub;
    ok[s] = k < g.n_k && tok < g.s1p;
    if (k < g.n_k) {                                     // uniform
      float kf[V];
      Unpack<WT>::go(t.r[2 * s], kf);
#pragma unroll
      for (int gi = 0; gi < G; ++gi) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < V; e += 4) {
          const float4 q4 = *reinterpret_cast<const float4*>(qs + gi * h + g.hoff + e);
          d = fmaf(q4.x, kf[e], d); d = fmaf(q4.y, kf[e + 1], d); d = fmaf(q4.z, kf[e + 2], d); d = fmaf(q4.w, kf[e + 3], d);
        }
        sc[s][gi] = group_sum_lanes(d, g);
      }
    } else {
#pragma unroll
      for (int gi = 0; gi < G; ++gi) sc[s][gi] = -1e30f;
    }
  }
#pragma unroll
  for (int gi = 0; gi < G; ++gi) {
    float mn = st.m[gi];
#pragma unroll
    for (int s = 0; s < kTile; ++s) mn = ok[s] ? fmaxf(mn, sc[s][gi]) : mn;
    const float alpha = __expf(st.m[gi] - mn);
    st.m[gi] = mn;
    st.l[gi] *= alpha;
#pragma unroll
    for (int e = 0; e < V; ++e) st.o[gi][e] *= alpha;
  }
#pragma unroll
  for (int s = 0; s < kTile; ++s) {
    if (ti * kTile + s < g.n_k) {                        // uniform
      float vf[V];
      Unpack<WT>::go(t.r[2 * s + 1], vf);
#pragma unroll
      for (int gi = 0; gi < G; ++gi) {
        const float p = ok[s] ? __expf(sc[s][gi] - st.m[gi]) : 0.f;
        st.l[gi] += p;
#pragma unroll
        for (int e = 0; e < V; ++e) st.o[gi][e] = fmaf(p, vf[e], st.o[gi][e]);
      }
    }
  }
}

// The streaming loop of the attention phase: two tiles in flight, each multiplied while the other's rows arrive.
template <typename WT, int G, typename AR, typename SL>
__device__ __forceinline__ void attn_stream(AttnState<WT, G>& st, Tile& A, Tile& B, int (&pgA)[kTile], int (&pgB)[kTile], const AttnGeo& ga,
                                            const AR& a, const SL& S, const void* kv, int nte, int wave, const float* xs) {
#pragma nounroll
  for (int t = 2; t < nte; t += 2) {
    attn_compute<WT, G>(st, A, ga, a.h, t - 2, wave, xs);
    attn_issue<WT>(A, pgA, ga, a, S, kv, t, wave);
    attn_compute<WT, G>(st, B, ga, a.h, t - 1, wave, xs);
    attn_issue<WT>(B, pgB, ga, a, S, kv, t + 1, wave);
  }
  if (nte) {                               // (the last two tiles: nothing more to ask for)
    attn_compute<WT, G>(st, A, ga, a.h, nte - 2, wave, xs);
    attn_compute<WT, G>(st, B, ga, a.h, nte - 1, wave, xs);
  }
}

// What attention reads of this launch's QKV product: this thread's word of the queries, and in the last wavefront (the
// one with the fewest query words) the newest position's K/V row, already rounded to the storage type.
template <typename WT> struct AttnAsk { tagged_t q[1], kv[2 * Storage<WT>::kVec]; };
template <int G, typename AR>
__device__ __forceinline__ uint32_t attn_q_at(const AttnGeo& g, const AR& a, int i, uint32_t z) {
  return (uint32_t)(g.hg * G * a.h + i) * 8u + z;
}
template <typename WT, typename AR>
__device__ __forceinline__ uint32_t attn_kv_at(const AttnGeo& g, const AR& a, int e, uint32_t z) {
  constexpr int V = Storage<WT>::kVec;
  return (uint32_t)(g.kvh * a.h + (e < V ? e : a.K * a.h + e - V) + g.hoff) * 8u + z;
}
template <typename WT, int G, typename AR, typename SL>
__device__ __forceinline__ void attn_ask(AttnAsk<WT>& k, const AttnGeo& g, const AR& a, const SL& S, int wave, int tid) {
  const bool newest = g.active && g.s1 == S.ctx && wave == kStepWaves - 1;
  ask_words(k.q, buffer_at(S.q), [&](int, uint32_t z) { return attn_q_at<G>(g, a, tid, z); }, [&](int) { return g.active && tid < G * a.h; });
  ask_words(k.kv, buffer_at(S.knew), [&](int e, uint32_t z) { return attn_kv_at<WT>(g, a, e, z); }, [&](int) { return newest; });
}
// queries into LDS (pre-scaled), the newest position into the last wavefront's running sums
template <typename WT, int G, typename AR, typename SL>
__device__ __forceinline__ void attn_begin(AttnState<WT, G>& st, AttnAsk<WT>& k, const AttnGeo& g, const AR& a, const SL& S, float* qs, int wave, unsigned epoch, int tid) {
  constexpr int V = Storage<WT>::kVec;
#pragma unroll
  for (int gi = 0; gi < G; ++gi) {
    st.m[gi] = -1e30f; st.l[gi] = 0.f;
#pragma unroll
    for (int e = 0; e < V; ++e) st.o[gi][e] = 0.f;
  }
  const bool newest = g.active && g.s1 == S.ctx && wave == kStepWaves - 1;
  if (g.active) {
    for (int i = tid; i < G * a.h; i += kStepThreads) {
      auto at = [&](int, uint32_t z) { return attn_q_at<G>(g, a, i, z); };
      if (i != tid) ask_words(k.q, buffer_at(S.q), at);
      await_words(k.q, buffer_at(S.q), at, epoch, a.spin_limit, a.err);
      qs[i] = tag_value(k.q[0]) * a.scale;
    }
    if (newest) await_words(k.kv, buffer_at(S.knew), [&](int e, uint32_t z) { return attn_kv_at<WT>(g, a, e, z); }, epoch, a.spin_limit, a.err);
  }
  __syncthreads();
  if (newest) {
    float kf[V], vf[V];
#pragma unroll
    for (int e = 0; e < V; ++e) { kf[e] = g.sub == 0 ? tag_value(k.kv[e]) : 0.f; vf[e] = g.sub == 0 ? tag_value(k.kv[V + e]) : 0.f; }
    attn_update_f<WT, G>(st, g, a.h, kf, vf, g.sub == 0, qs);
  }
}

// Folds the wavefront's token sub-groups, leaves one record per (wavefront, head) in LDS.
template <typename WT, int G>
__device__ __forceinline__ void attn_to_lds(AttnState<WT, G>& st, const AttnGeo& g, int h, float* sm, int wave) {
  constexpr int V = Storage<WT>::kVec;
  const int rec = h + 2;
  for (int off = g.L; off < 64; off <<= 1) {
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
      const float mo = __shfl_xor(st.m[gi], off, 64), lo = __shfl_xor(st.l[gi], off, 64);
      const float mn = fmaxf(st.m[gi], mo);
      const float sa = __expf(st.m[gi] - mn), sb = __expf(mo - mn);
      st.l[gi] = st.l[gi] * sa + lo * sb;
#pragma unroll
      for (int e = 0; e < V; ++e) st.o[gi][e] = st.o[gi][e] * sa + __shfl_xor(st.o[gi][e], off, 64) * sb;
      st.m[gi] = mn;
    }
  }
  __syncthreads();                                             // queries in LDS are no longer needed
  if (g.sub == 0) {                                            // [wave][g][h + 2]
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
      float* r = sm + (wave * G + gi) * rec;
#pragma unroll
      for (int e = 0; e < V; ++e) r[g.hoff + e] = st.o[gi][e];
      if (g.hoff == 0) { r[h] = st.m[gi]; r[h + 1] = st.l[gi]; }
    }
  }
  __syncthreads();
}

// Counts an arrival; whether it was the last of n.  The count wraps to zero with that one, in the same operation: a store
// of zero after it would have to be seen everywhere before the next layer's first arrival, and nothing waits for it - a
// phase waits for data, of which the other wavefronts' may be out first.
__device__ __forceinline__ bool last_of(unsigned* arrivals, unsigned n) { return atomicInc(arrivals, n - 1u) == n - 1u; }

// Wavefront records -> split partial (or the final output when there is one split);
// the last workgroup of a head group to arrive folds the splits in split order.
template <int G, typename AR, typename SL>
__device__ __forceinline__ void attn_finish(const AttnGeo& g, const AR& a, const SL& S, const float* sm, int* s_flag, unsigned epoch, int tid) {
  const unsigned wtag = epoch + 1;
  const int h = a.h, rec = h + 2;
  if (!g.active) return;
  const bool single = S.n_splits == 1;
  for (int idx = tid; idx < G * h; idx += kStepThreads) {
    const int gi = idx / h, e = idx - gi * h;
    float m = -1e30f;
    for (int w = 0; w < kStepWaves; ++w) m = fmaxf(m, sm[(w * G + gi) * rec + h]);
    float l = 0.f, o = 0.f;
    for (int w = 0; w < kStepWaves; ++w) {
      const float* r = sm + (w * G + gi) * rec;
      const float sc = __expf(r[h] - m);
      l += r[h + 1] * sc; o += r[e] * sc;
    }
    const int head = g.hg * G + gi;
    if (single) {
      st_tag(S.o + (long)head * h + e, o / l, wtag);
    } else {
      tagged_t* pr = S.part + ((long)head * kMaxSplits + g.split) * rec;
      st_tag(pr + e, o, wtag);
      if (e == 0) { st_tag(pr + h, m, wtag); st_tag(pr + h + 1, l, wtag); }
    }
  }
  if (single) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  if (tid == 0) s_flag[1] = last_of(S.tickets + g.hg, (unsigned)S.n_splits);
  __syncthreads();
  if (!s_flag[1]) return;
  for (int idx = tid; idx < G * h; idx += kStepThreads) {
    const int gi = idx / h, e = idx - gi * h;
    const int head = g.hg * G + gi;
    const tagged_t* pr = S.part + (long)head * kMaxSplits * rec;
    // splits are folded in split order, eight at a time so that their loads are in flight together
    float m = -1e30f, l = 0.f, o = 0.f;
    for (int sp0 = 0; sp0 < S.n_splits; sp0 += 8) {
      tagged_t rm[8], rl[8], ro[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool ok = sp0 + k < S.n_splits;
        const tagged_t* r = pr + (sp0 + k) * rec;
        rm[k] = ok ? ld_raw(r + h) : 0ull; rl[k] = ok ? ld_raw(r + h + 1) : 0ull; ro[k] = ok ? ld_raw(r + e) : 0ull;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (sp0 + k < S.n_splits) {
          const tagged_t* r = pr + (sp0 + k) * rec;
          const float mk = settle(r + h, rm[k], wtag, a.spin_limit, a.err);
          const float lk = settle(r + h + 1, rl[k], wtag, a.spin_limit, a.err);
          const float ok_ = settle(r + e, ro[k], wtag, a.spin_limit, a.err);
          const float mn = fmaxf(m, mk);
          const float sa = __expf(m - mn), sb = __expf(mk - mn);
          l = l * sa + lk * sb;
          o = o * sa + ok_ * sb;
          m = mn;
        }
      }
    }
    st_tag(S.o + (long)head * h + e, o / l, wtag);
  }
}

// ---------------------------------------------------------------------------

}  // namespace step_w<waves>
}  // namespace mdi

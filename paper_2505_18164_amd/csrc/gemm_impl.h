// The matrix products of a first visit (Alg. 1 round 0, Alg. 2 "first iteration"): C[T, N] = A[T, Kd] W[N, Kd]^T with
// fp32 accumulation, A the activations of T prompt positions, W a weight matrix.  bf16 storage runs on
// v_mfma_f32_16x16x32_bf16, fp32 storage on v_mfma_f32_16x16x4_f32 (exact fp32 products).
//
// One workgroup computes BN weight rows x BT positions, transposed (C^T = W A^T: a lane then owns one position and
// eight consecutive outputs, so residual, activation and gate/up pairs need no other lane).  A step of the inner
// dimension is 128 bytes of every row; both operands travel global -> LDS without passing registers
// (buffer_load_dwordx4 ... lds), a ring of NBW / NBA steps deep, so that a step has one to three steps of arithmetic
// to arrive; one barrier per step.  Fragments of the next half step are read from LDS between the matrix
// instructions of the current one.  The steps that still ask for others are a loop of their own without a condition in
// it.  The 16-byte pieces of a row are permuted by the row number (the permutation is applied to the global address, LDS
// then holds it for free), which spreads the reads over the banks.
//
// What bounds it depends on the tile.  Timed with one of the three parts of a step left out at a time (1024 positions, cold
// weights): 128 x 128 tiles take 0.60 us a step to load (53 bytes per ns and compute unit, at a depth of three steps as at
// five: what a compute unit keeps on its way over the latency of memory; 75 with the weights in the memory-side cache, 86
// from L2), 0.41 to multiply, 0.35 to read LDS, 0.68 together.  256 x 256: 1.25 to load, 1.37 to multiply, 0.66 to read
// LDS, 1.8 together; there the clock gives way as well, 1.6 - 1.9 GHz (2.1 with small tiles; a loop of nothing but matrix
// instructions on random operands runs at 1.9 - 2.1).  So few positions want tiles with few bytes per product, many
// positions tiles that divide their number well.  16x16x32 instructions against 32x32x16 ones, half the accumulator traffic
// per product: 283 against 310 us at 4096 x 4096 x 11008, and a clock 10 % higher.
// The loop without conditions is 1 to 6 % faster than one with a test before every load (192 x 256: 2.5 %, 64 x 64: 6 %).
// Spreading a step's loads over both halves, or over the first quarter, reading the fragments earlier, wavefront priority
// around the products: between nothing and 5 % slower.

// Included by gemm_bf16.hip and gemm_f32.hip, which hold the tile shapes of their storage type.
#pragma once

#include <type_traits>
#include <utility>

#include "device_utils.h"
#include "visit_internal.h"

namespace mdi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// 64 x 16 bytes global -> LDS: lane l's piece lands at lds + 16 l.  An offset at or past the descriptor's 2^31 - 1
// bytes reads as zero.
__device__ __forceinline__ void dma_piece(uint32_t lds, u32x4 rsrc, int voff, int soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "m0", "memory");
}
__device__ __forceinline__ u32x4 buffer_of(const void* p) {
  const uint64_t a = (uint64_t)p;
  return u32x4{(uint32_t)a, (uint32_t)(a >> 32) & 0xFFFFu, 0x7FFFFFFFu, 0x00020000u};
}
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// One 16-byte fragment of each operand: 32 values of the inner dimension over the four lane groups in bf16, 16 in fp32.
template <typename T> struct Mac;
template <> struct Mac<bf16_t> {
  typedef bf16x8 frag;
  __device__ static __forceinline__ f32x4 go(const frag& w, const frag& a, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, c, 0, 0, 0); }
};
template <> struct Mac<float> {
  typedef f32x4 frag;
  __device__ static __forceinline__ f32x4 go(const frag& w, const frag& a, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], a[e], c, 0, 0, 0);
    return c;
  }
};

template <typename T> __device__ __forceinline__ void put8(void* base, long o, const float (&v)[8]);
template <> __device__ __forceinline__ void put8<float>(void* base, long o, const float (&v)[8]) {
  f32x4* p = reinterpret_cast<f32x4*>((float*)base + o);
  p[0] = f32x4{v[0], v[1], v[2], v[3]}; p[1] = f32x4{v[4], v[5], v[6], v[7]};
}
__device__ __forceinline__ uint32_t pack2(float lo, float hi) { return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16); }
template <> __device__ __forceinline__ void put8<bf16_t>(void* base, long o, const float (&v)[8]) {
  *reinterpret_cast<u32x4*>((bf16_t*)base + o) = u32x4{pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
}
template <typename T> __device__ __forceinline__ void put4(void* base, long o, float a, float b, float c, float d);
template <> __device__ __forceinline__ void put4<float>(void* base, long o, float a, float b, float c, float d) {
  *reinterpret_cast<f32x4*>((float*)base + o) = f32x4{a, b, c, d};
}
template <> __device__ __forceinline__ void put4<bf16_t>(void* base, long o, float a, float b, float c, float d) {
  *reinterpret_cast<u32x2*>((bf16_t*)base + o) = u32x2{pack2(a, b), pack2(c, d)};
}

// f(0), ..., f(N - 1) with the numbers as constants.  (A loop for the compiler to unroll is left as a loop when a tile has many
// products, and the fragments then end up in scratch memory.)
template <typename F, int... I> __device__ __forceinline__ void each_of(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F> __device__ __forceinline__ void each(F&& f) { each_of(static_cast<F&&>(f), std::make_integer_sequence<int, N>{}); }
// n things spread evenly over `over` places: the first that is due at place q or later.
constexpr int due(int q, int n, int over) { const int v = (q * n + over - 1) / over; return v < n ? v : n; }

// A workgroup is WN x WT wavefronts, each (BN / WN) weight rows x (BT / WT) positions.  bf16 tiles of four wavefronts are held to
// 256 registers: given all 512 the compiler keeps sums in the accumulation half and moves them to and fro in every step (96 x
// 128, of which a compute unit's LDS holds one anyway, 256 x 12288 x 4096: 42.9 -> 38.6 us; 64 x 96, 333 x 2560 x 2048: 16.0 ->
// 14.1).  In fp32 the same costs 1 %.
template <typename ST, int EPI, int BN, int BT, int WN, int WT, int NBW, int NBA>
__global__ __launch_bounds__(WN * WT * 64, sizeof(ST) == 2 ? 2 : WN * WT * 64 / 256) void k_gemm(GemmArgs a) {
  typedef Mac<ST> M;
  constexpr int NW = WN * WT, ES = (int)sizeof(ST);
  constexpr int TN = BN / WN / 16, TT = BT / WT / 16;   // 16 x 16 tiles per wavefront
  constexpr int LW = BN / 8 / NW, LA = BT / 8 / NW;     // 1-KiB pieces (8 rows) per wavefront and step
  constexpr int WB = BN * 128, AB = BT * 128;           // bytes of a step
  static_assert(TN % 2 == 0 && TT >= 1 && BN % (8 * NW) == 0 && BT % (8 * NW) == 0, "tile shape");
  static_assert(NBW >= NBA && (NBW == NBA || NBW == NBA + 1) && NBA >= 2, "ring depths");
  extern __shared__ __attribute__((aligned(1024))) unsigned char gemm_smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)gemm_smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave / WT, wt = wave % WT;
  // all arguments in one round trip (left alone they are asked for where they are first used, in three)
  if constexpr (EPI == GEPI_QKV)
    asm volatile("" ::"s"(a.A), "s"(a.W), "s"(a.bias), "s"(a.T), "s"(a.N), "s"(a.Kd), "s"(a.S), "s"(a.qkv.H), "s"(a.qkv.K), "s"(a.qkv.h), "s"(a.qkv.pt),
                 "s"(a.qkv.pt_sh), "s"(a.qkv.pt_magic), "s"(a.qkv.pos0), "s"(a.qkv.scale), "s"(a.qkv.rope), "s"(a.qkv.q_out), "s"(a.qkv.q_bf),
                 "s"(a.qkv.pool), "s"(a.qkv.table));
  else
    asm volatile("" ::"s"(a.A), "s"(a.W), "s"(a.bias), "s"(a.T), "s"(a.N), "s"(a.Kd), "s"(a.S), "s"(a.out_f32), "s"(a.out_act));

  // Workgroup -> tile.  Workgroups are handed to the eight compute dies in turn, and each die has an L2 of its own:
  // a die takes a contiguous range of tiles, ordered in groups of up to eight position tiles that share a weight
  // tile while it is in that L2.
  const int t_tiles = (a.T + BT - 1) / BT, n_tiles = (a.N + BN - 1) / BN, tiles = t_tiles * n_tiles;
  const int die = blockIdx.x & 7, seq = blockIdx.x >> 3, per_die = (tiles + 7) >> 3;
  const int idx = die * per_die + seq;
  if (seq >= per_die || idx >= tiles) return;
  const int grp = idx / (8 * n_tiles), rem = idx - grp * 8 * n_tiles, in_grp = min(8, t_tiles - grp * 8);
  const int tile_n = rem / in_grp, tile_t = grp * 8 + rem - tile_n * in_grp;
  const int n0 = tile_n * BN, t0 = tile_t * BT;

  // This split's steps.  Dies walk them from different starting points: in step they would all ask the same columns
  // of the activations, and rows a power of two apart of the weights, from memory at once (3 to 9 % on every shape).
  const int row_bytes = a.Kd * ES, nk_all = (row_bytes + 127) >> 7, per_split = (nk_all + a.S - 1) / a.S;
  const int k_lo = blockIdx.y * per_split, nk = min(per_split, nk_all - k_lo);
  const int rot = (die * nk) >> 3;
  const int tail = row_bytes & 127;                     // bytes of a partial last step: pieces past them are zero

  // Row r of a weight tile is output n0 + r.  The QKV product's outputs are dealt out in eights: four of the first half of a
  // head and the four they are rotated with, so that a pair is in one lane whatever the tile and wherever it starts.
  const int base = EPI == GEPI_QKV ? n0 & -a.qkv.h : n0;
  auto w_row = [&](int r) __attribute__((always_inline)) {          // counted from `base`; rows past the matrix re-read its last row
    const int n = min(n0 + r, a.N - 1);
    if constexpr (EPI != GEPI_QKV) return n - base;
    const int in = n & (a.qkv.h - 1);
    return n - in - base + 4 * (in >> 3) + (in & 3) + (in & 4 ? a.qkv.h >> 1 : 0);
  };
  const u32x4 rw = buffer_of((const char*)a.W + (long)base * row_bytes), ra = buffer_of((const char*)a.A + (long)t0 * row_bytes);
  // Row r of a weight tile keeps its 16-byte piece c at slot c ^ (r bit 1, r bits 3 - 4), of a position tile at
  // c ^ (r bits 1 - 3): the sixteen rows a fragment read touches then differ in (row parity, slot).
  auto w_slot = [](int r) { return ((r >> 1) & 1) | (((r >> 3) & 3) << 1); };
  auto a_slot = [](int r) { return (r >> 1) & 7; };
  int vw[LW], va[LA];
  bool zw[LW], za[LA];                                  // this lane's piece lies past a partial last step
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ w_slot(r);
    vw[i] = w_row(r) * row_bytes + (c << 4); zw[i] = tail && (c << 4) >= tail;
  }
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ a_slot(r);
    va[i] = min(r, a.T - 1 - t0) * row_bytes + (c << 4); za[i] = tail && (c << 4) >= tail;
  }
  const uint32_t lw0 = lds0 + wave * 1024, la0 = lds0 + NBW * WB + wave * 1024;
  auto k_of = [&](int kt) { const int k = kt + rot; return k_lo + (k >= nk ? k - nk : k); };
  auto load_w = [&](int i, int k, int buf) __attribute__((always_inline)) {
    dma_piece(lw0 + buf * WB + i * NW * 1024, rw, k == nk_all - 1 && zw[i] ? (int)0x80000000 : vw[i], k * 128);
  };
  auto load_a = [&](int i, int k, int buf) __attribute__((always_inline)) {
    dma_piece(la0 + buf * AB + i * NW * 1024, ra, k == nk_all - 1 && za[i] ? (int)0x80000000 : va[i], k * 128);
  };

  f32x4 acc[TN][TT];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Fragment addresses.  Position tiles: lane (m = l mod 16, g = l div 16) reads row m.  Weight tiles in pairs: rows
  // 8 (m / 4) + m mod 4 (+ 4 in the second), so that the pair leaves eight consecutive outputs 8 g .. 8 g + 7 in a lane.
  const int m = lane & 15, g = lane >> 4;
  int fa[2], fw[2][2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    fa[s] = m * 128 + (((4 * s + g) ^ a_slot(m)) << 4);
#pragma unroll
    for (int b = 0; b < 2; ++b) { const int r = 8 * (m >> 2) + 4 * b + (m & 3); fw[s][b] = r * 128 + (((4 * s + g) ^ w_slot(r)) << 4); }
  }
  const unsigned char* w_wave = gemm_smem + wn * (BN / WN) * 128;
  const unsigned char* a_wave = gemm_smem + NBW * WB + wt * (BT / WT) * 128;

  // The QKV product's epilogue rotates queries and keys and puts keys and values into the pages.  (A kernel of its own read the
  // rows back in fp32: 13.8 us at 1024 positions of the 7B shape, 8.2 at 256, 4.9 at 333 of TinyLlama.  The product itself, fp32
  // rows and a test before every load / this epilogue and the loop without, on the same tiles: 7168 outputs of rows of 5120, 64
  // positions 30.3 / 30.3 us, 192 44.1 / 42.8, 256 45.1 / 44.7.)  What it needs besides the sums, angles and page numbers, small tiles ask for
  // before the first step - asked for in the epilogue they cost 1.5 to 2 us more - and tiles that need the registers one position ahead.
  constexpr bool ASK_EARLY = TN * TT <= 12;
  const int h_sh = EPI == GEPI_QKV ? 31 - __builtin_clz(a.qkv.h) : 0;
  f32x4 cs[TT][TN / 2][2];                                         // (cos, sin) of four pairs
  int page[TT];
  auto head_of = [&](int p) __attribute__((always_inline)) { return (n0 + wn * (BN / WN) + 8 * g + 32 * p) >> h_sh; };
  auto pair_of = [&](int p) __attribute__((always_inline)) { return ((n0 + wn * (BN / WN) + 8 * g + 32 * p) & (a.qkv.h - 1)) >> 1; };
  auto page_no = [&](int pos) __attribute__((always_inline)) { return a.qkv.pt_sh >= 0 ? pos >> a.qkv.pt_sh : (int)__umulhi((unsigned)pos, a.qkv.pt_magic); };
  auto ask_pairs = [&](int j) __attribute__((always_inline)) {
    const QkvOut& o = a.qkv;
    const int pos = o.pos0 + min(t0 + wt * (BT / WT) + j * 16 + m, a.T - 1);
    if (n0 + BN > o.H << h_sh) page[j] = o.table[page_no(pos)];    // a tile of queries alone needs none
    if (!o.rope) return;
#pragma unroll
    for (int p = 0; p < TN / 2; ++p) {                             // (values and rows past the last have no use for theirs)
      const f32x4* r = reinterpret_cast<const f32x4*>(o.rope + (long)pos * (o.h >> 1) + pair_of(p));
      cs[j][p][0] = r[0]; cs[j][p][1] = r[1];
    }
  };
  if constexpr (EPI == GEPI_QKV && ASK_EARLY) {
#pragma unroll
    for (int j = 0; j < TT; ++j) ask_pairs(j);
  }

  // fill the rings; the first step waits only for its own pieces
#pragma unroll
  for (int p = 0; p < NBW; ++p) {
    if (p < nk) {
      const int k = k_of(p);
      if (p < NBA) {
#pragma unroll
        for (int i = 0; i < LA; ++i) load_a(i, k, p);
      }
#pragma unroll
      for (int i = 0; i < LW; ++i) load_w(i, k, p);
    }
  }
  if (nk >= NBW) wait_loads<(NBA - 1) * LA + (NBW - 1) * LW>(); else wait_loads<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  typename M::frag xw[2][TN], xa[2][TT];
#pragma unroll
  for (int j = 0; j < TT; ++j) xa[0][j] = *reinterpret_cast<const typename M::frag*>(a_wave + fa[0] + j * 2048);
#pragma unroll
  for (int i = 0; i < TN; ++i) xw[0][i] = *reinterpret_cast<const typename M::frag*>(w_wave + fw[0][i & 1] + (i >> 1) * 4096);

  constexpr int NF = TN + TT, NM = TN * TT, NL = LW + LA;
  int bw = 0, ba = 0;
  auto step = [&](auto steady, int kt) __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady)::value;               // both buffers that this step frees are filled again
    const int nbw = bw + 1 == NBW ? 0 : bw + 1, nba = ba + 1 == NBA ? 0 : ba + 1;
    const bool more_a = STEADY || kt + NBA < nk;
    const int kw = k_of(kt + NBW), ka = k_of(kt + NBA);
    each<2>([&](auto half) __attribute__((always_inline)) {
      constexpr int s = half, cur = s, nxt = s ^ 1;
      const unsigned char* wp = w_wave + (s ? nbw : bw) * WB;      // where the next half step's fragments are
      const unsigned char* ap = a_wave + (s ? nba : ba) * AB;
      if constexpr (s == 1) {
        // this wavefront has read all of step kt; the next step must have landed, for every wavefront.  Loads return
        // in order: what may still be on its way are the pieces issued after the next step's.
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (STEADY || kt + NBW <= nk) wait_loads<(NBW > NBA ? LW + (NBA - 2) * (LW + LA) : (NBW - 2) * (LW + LA))>(); else wait_loads<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      __builtin_amdgcn_sched_barrier(0);
      each<NM>([&](auto place) __attribute__((always_inline)) {
        constexpr int q = place, i = q / TT, j = q % TT;
        acc[i][j] = M::go(xw[cur][i], xa[cur][j], acc[i][j]);
        constexpr int f0 = due(q, NF, NM), f1 = due(q + 1, NF, NM);
        each<f1 - f0>([&](auto n) __attribute__((always_inline)) {
          constexpr int f = f0 + n;
          if constexpr (f < TT) xa[nxt][f] = *reinterpret_cast<const typename M::frag*>(ap + fa[nxt] + f * 2048);
          else { constexpr int i2 = f - TT; xw[nxt][i2] = *reinterpret_cast<const typename M::frag*>(wp + fw[nxt][i2 & 1] + (i2 >> 1) * 4096); }
        });
        if constexpr (s == 1) {                                    // refill the buffers this step has just freed
          constexpr int l0 = due(q, NL, NM), l1 = due(q + 1, NL, NM);
          each<l1 - l0>([&](auto n) __attribute__((always_inline)) {
            constexpr int l = l0 + n;
            if constexpr (l < LA) { if (more_a) load_a(l, ka, ba); }
            else if constexpr (STEADY) load_w(l - LA, kw, bw);
          });
        }
        __builtin_amdgcn_sched_barrier(0);                         // keep this order: reads and loads between the products
      });
    });
    bw = nbw; ba = nba;
  };
  int kt = 0;
  for (; kt + NBW < nk; ++kt) step(std::true_type{}, kt);
  for (; kt < nk; ++kt) step(std::false_type{}, kt);

  // ---- epilogue of the QKV product: lane = position t, four pairs (i, i + h / 2) of a head: rotated where the head is one of
  // the queries' or keys', then stored where it is wanted
  if constexpr (EPI == GEPI_QKV) {
    const QkvOut& o = a.qkv;
    const int half = o.h >> 1;
    if constexpr (!ASK_EARLY) ask_pairs(0);
#pragma unroll
    for (int j = 0; j < TT; ++j) {
      if (!ASK_EARLY && j + 1 < TT) ask_pairs(j + 1);
      const int t = t0 + wt * (BT / WT) + j * 16 + m;
      if (t >= a.T) continue;
#pragma unroll
      for (int p = 0; p < TN / 2; ++p) {
        const int hd = head_of(p), in = pair_of(p);
        if (hd >= o.H + 2 * o.K) continue;
        f32x4 x = acc[2 * p][j], y = acc[2 * p + 1][j];
        if (a.bias) {
          const float* b = a.bias + hd * o.h + in;
          x += *reinterpret_cast<const f32x4*>(b);
          y += *reinterpret_cast<const f32x4*>(b + half);
        }
        if (o.rope && hd < o.H + o.K) {
          const f32x4 c = {cs[j][p][0][0], cs[j][p][0][2], cs[j][p][1][0], cs[j][p][1][2]}, s = {cs[j][p][0][1], cs[j][p][0][3], cs[j][p][1][1], cs[j][p][1][3]};
          const f32x4 x0 = x;
          x = x0 * c - y * s;
          y = x0 * s + y * c;
        }
        if (hd < o.H) {
          const long to = ((long)t * o.H + hd) * o.h + in;
          if (o.q_bf) {
            x *= o.scale; y *= o.scale;
            put4<bf16_t>(o.q_bf, to, x[0], x[1], x[2], x[3]);
            put4<bf16_t>(o.q_bf, to + half, y[0], y[1], y[2], y[3]);
          } else {
            put4<float>(o.q_out, to, x[0], x[1], x[2], x[3]);
            put4<float>(o.q_out, to + half, y[0], y[1], y[2], y[3]);
          }
        } else {
          const int is_v = hd >= o.H + o.K, kv = hd - o.H - (is_v ? o.K : 0), pos = o.pos0 + t;
          const long to = ((((long)page[j] * o.K + kv) * 2 + is_v) * o.pt + (pos - page_no(pos) * o.pt)) * o.h + in;
          put4<ST>(o.pool, to, x[0], x[1], x[2], x[3]);
          put4<ST>(o.pool, to + half, y[0], y[1], y[2], y[3]);
        }
      }
    }
    return;
  }

  // ---- epilogue: lane = position t, outputs n .. n + 7 (N is a multiple of 8)
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    const int t = t0 + wt * (BT / WT) + j * 16 + m;
    const int nb = n0 + wn * (BN / WN) + 8 * g;
    if (t >= a.T) continue;
    f32x4 res[TN];
    if (EPI == GEPI_RESID) {
#pragma unroll
      for (int p = 0; p < TN / 2; ++p) {
        const int n = nb + 32 * p;
        if (n < a.N) { const f32x4* r = reinterpret_cast<const f32x4*>(a.out_f32 + (long)t * a.N + n); res[2 * p] = r[0]; res[2 * p + 1] = r[1]; }
      }
    }
#pragma unroll
    for (int p = 0; p < TN / 2; ++p) {
      const int n = nb + 32 * p;
      if (n >= a.N) continue;
      float v[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[e] = acc[2 * p][j][e]; v[4 + e] = acc[2 * p + 1][j][e]; }
      if (EPI == GEPI_PART) {
        put8<float>(a.out_f32, ((long)blockIdx.y * a.T + t) * a.N + n, v);
      } else if (EPI == GEPI_SWIGLU) {                             // rows (2f, 2f + 1) = (gate_f, up_f)
        put4<ST>(a.out_act, (long)t * (a.N >> 1) + (n >> 1), silu_f(v[0]) * v[1], silu_f(v[2]) * v[3], silu_f(v[4]) * v[5], silu_f(v[6]) * v[7]);
      } else {
        if (a.bias) {
          const f32x4* b = reinterpret_cast<const f32x4*>(a.bias + n);
          const f32x4 b0 = b[0], b1 = b[1];
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[e] += b0[e]; v[4 + e] += b1[e]; }
        }
        const long o = (long)t * a.N + n;
        if (EPI == GEPI_RESID) {
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[e] += res[2 * p][e]; v[4 + e] += res[2 * p + 1][e]; }
          put8<float>(a.out_f32, o, v);
          if (a.out_act) {
            if (a.act_aligned) put8<ST>(a.out_act, o, v);
            else
              for (int e = 0; e < 8; ++e) Storage<ST>::put((ST*)a.out_act + o + e, v[e]);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = a.gelu_tanh ? gelu_tanh_f(v[e]) : gelu_erf_f(v[e]);
          put8<ST>(a.out_act, o, v);
        }
      }
    }
  }
}

// Lets the current device's copy of the kernel have its LDS: a kernel gets 64 KiB by default.
template <typename ST, int EPI, int BN, int BT, int WN, int WT, int NBW, int NBA>
bool allow_shape() {
  constexpr size_t lds = (size_t)128 * (NBW * BN + NBA * BT);
  static_assert(lds <= 160 * 1024, "LDS of a compute unit");
  return lds <= 64 * 1024 || hipFuncSetAttribute((const void*)k_gemm<ST, EPI, BN, BT, WN, WT, NBW, NBA>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
}

template <typename ST, int EPI, int BN, int BT, int WN, int WT, int NBW, int NBA>
void launch_shape(hipStream_t s, const GemmArgs& a) {
  constexpr size_t lds = (size_t)128 * (NBW * BN + NBA * BT);
  const int tiles = ((a.T + BT - 1) / BT) * ((a.N + BN - 1) / BN);
  hipLaunchKernelGGL((k_gemm<ST, EPI, BN, BT, WN, WT, NBW, NBA>), dim3(8 * ((tiles + 7) / 8), a.S), dim3(WN * WT * 64), lds, s, a);
}

}  // namespace
}  // namespace mdi

// Decode step of SEVERAL queued messages with ONE pass over the partition's weights.
//
// The paper's node takes the messages of its input queue one at a time (Sec. III-A), so every later visit of a
// sample (Sec. III-D) streams all local weights again.  With several samples in flight (Sec. III-C) their messages
// wait in the queue together; here up to 16 of them go through every layer together: a 16-byte piece of a weight
// row is fetched once and multiplied with all the messages' vectors by one matrix instruction
// (v_mfma_f32_16x16x32_bf16: 16 weight rows x 32 columns times 32 x 16 messages), attention stays per sample over
// each sample's own cache.  The kernel is still bound by HBM: the matrix cores only take over the multiply-adds
// that the vector ALUs could not do for 16 messages at the rate the weights arrive.
//
// Same skeleton as k_step (one persistent launch, five phases per layer, self-validating tagged exchange), with these
// differences:
//   * One set of 8-wavefront workgroups, all messages in lockstep.
//   * No barrier: a phase waits for the words it reads, by reloading those whose counter is not the writing phase's
//     yet.  Phase counters, watched by every workgroup before it fetched the data, cost 3.2 us a round; 256
//     workgroups that watch 2048 words of data themselves take 1.65 us from store to store.  What binds a phase of the
//     small shapes is this chain of round trips (a store is seen elsewhere after about 1.2 us), so each is started as
//     early as it can be: words of the phase before are asked for ahead of this phase's weights, operands of the
//     epilogue before the products, and no stream asks for tiles past its end.  Together, per launch: 4 layers of GPT-2
//     with 3 messages 304 -> 183 us, 11 of TinyLlama with 4 846 -> 589 us, 8 of the 7B shape with 8 1178 -> 958 us.
//     What the counters also gave, that nobody overwrites what somebody still reads, follows from
//     the sums of squares: every workgroup publishes its share at the end of the output projection and of the down
//     projection, after all it read up to there, and every workgroup has seen the shares of all before it stores
//     anything in the QKV and the up product.  So whoever stores in QKV, attention or the output projection knows that
//     all have finished the layer before; whoever stores in the up or down product knows that all have finished this
//     layer's output projection.  Hence the residual vectors, the sums of squares and the sums exist twice, once from
//     the output projection to the up product and once from the down projection to QKV; every other vector is
//     written at least two such points after it was last read.
//   * Work unit of a product = a block of R (16 or 8) weight rows; blocks are dealt round-robin to workgroups; the
//     eight wavefronts of a workgroup split the block's columns among them and their partial 16 x 16 results are
//     added in LDS in wavefront order (deterministic, no float atomics).  RoPE partners (i, i + h/2) and SwiGLU
//     partners (gate_f, up_f) sit in the same block, so the epilogue of a row pair needs no other workgroup.
//   * Vectors that feed a product cross workgroups as bf16 PAIRS with the writing phase's counter in one 8-byte
//     word, already multiplied by the gain of the RMSNorm that follows (1/rms is applied to the finished products;
//     the sum of squares travels as one partial per workgroup and message).  Bytes exchanged per message are half
//     those of k_step's (float, counter) words, which matters now that 16 messages share a pass.  A vector kind is
//     ONE array [pair of columns][messages] for the whole launch: the lanes that hold the same columns of the messages
//     read consecutive words, and no line carries room for messages the launch does not have.
//   * The residual stream never leaves the workgroup that owns its rows: it stays in LDS for the whole launch.
//   * Products whose input is the d-sized normalised vector (QKV, MLP up) keep each wavefront's column slice of all
//     messages in registers for all the blocks of the phase; the others (output projection, MLP down: one block per
//     workgroup at the benchmark shapes, a long inner dimension) split the inner dimension among workgroups, so
//     that a workgroup reads a fraction of the vectors, and exchange 16 x 16 partial results (see KsGeo).
// Needs bf16 storage and widths that are multiples of 32; other shapes keep one pass per message.  With LayerNorm the vectors still travel as x * gain: the mean and the norm's bias enter the finished
// products through two precomputed vectors per matrix (W g and W b), see BatchArgs.
//
// Included by step_w8.hip after step_impl.h (shares its exchange, wait and attention helpers).
namespace mdi {
namespace step_w8 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ void st_pair(tagged_t* p, uint32_t bits, unsigned tag) {
  __hip_atomic_store(p, ((tagged_t)tag << 32) | (tagged_t)bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The low word of *p once its counter is `tag` (see settle in step_impl.h).
__device__ __forceinline__ uint32_t settle_bits(const tagged_t* p, tagged_t u, unsigned tag, int spin_limit, int* err) {
  int it = 0;
  while ((uint32_t)(u >> 32) != tag) {
    if (++it > spin_limit) { __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); break; }
    __builtin_amdgcn_s_sleep(1);
    u = ld_raw(p);
  }
  return (uint32_t)u;
}

// What the attention helpers of step_impl.h read of a message.
struct BatchView {
  const tagged_t *q, *knew;
  tagged_t *part, *ob;             // ob: the launch's [pair][messages] array of attention outputs
  unsigned* tickets;
  const int32_t* table;
  int ctx, n_splits, chunk, msg, n_msg;
};
__device__ __forceinline__ BatchView view_of(const BatchArgs& a, int j, tagged_t* ob) {
  char* base = a.slot0 + (long)j * a.slot_stride;
  BatchView v;
  v.q = (const tagged_t*)(base + a.off_q); v.knew = (const tagged_t*)(base + a.off_knew);
  v.part = (tagged_t*)(base + a.off_part); v.ob = ob; v.msg = j; v.n_msg = a.m;
  v.tickets = (unsigned*)(base + a.off_tickets);
  v.table = a.s[j].table; v.ctx = a.s[j].ctx; v.n_splits = a.s[j].n_splits; v.chunk = a.s[j].chunk;
  return v;
}


// ---------------------------------------------------------------------------
// geometry of a product (all values uniform across the wavefront)
struct BGeo {
  const char* W;        // matrix [N, Kd] bf16, row-major
  long row_bytes;
  int N, R;             // rows; rows per block (16 or 8)
  int rope_sh;          // >= 0: rows pair as RoPE partners (i, i + h/2), h = 2 << rope_sh; -1: rows (2p, 2p + 1)
  int nb_local;         // this workgroup's blocks: its block lb is block lb * nwg + wg of the matrix
  int ks0, nks;         // this wavefront's column steps [ks0, ks0 + nks), 32 columns each (products with a resident operand)
};
__device__ __forceinline__ BGeo make_bgeo(const void* W, int N, int Kd, int R, int rope_h, int wg, int nwg, int wave) {
  BGeo g;
  g.W = (const char*)W; g.row_bytes = 2L * Kd; g.N = N; g.R = R;
  g.rope_sh = rope_h ? 31 - __builtin_clz(rope_h >> 1) : -1;
  const int nblk = (N + R - 1) >> (R == 16 ? 4 : 3);
  g.nb_local = nblk > wg ? (nblk - wg + nwg - 1) / nwg : 0;
  // The columns are cut into one slice per wavefront; which wavefront takes which slice rotates with the workgroup,
  // so that at any moment the workgroups read different parts of the messages' vectors (every workgroup walks the
  // same vectors: in step they would all queue up at the same few memory channels).
  const int total = Kd >> 5, c = (total + kStepWaves - 1) / kStepWaves;
  g.ks0 = ((wave + wg) & (kStepWaves - 1)) * c;
  g.nks = max(0, min(c, total - g.ks0));
  if (g.nks == 0) g.ks0 = 0;          // a wavefront without columns still issues its (unused) loads inside the matrix
  return g;
}
// Row of the matrix that row i (< R) of block `block` stands for.  With RoPE pairing a block is R/2 consecutive
// rows of a head's first half followed by their partners in the second half.
__device__ __forceinline__ int block_row(const BGeo& g, int block, int i) {
  if (g.rope_sh < 0) return block * g.R + i;
  const int hsh = 31 - __builtin_clz(g.R >> 1);            // log2 of the rows a block takes of a half head
  const int bsh = g.rope_sh - hsh;                           // log2 of the blocks per head
  const int head = block >> bsh, off = (block & ((1 << bsh) - 1)) << hsh;
  return (head << (g.rope_sh + 1)) + off + (i & ((g.R >> 1) - 1)) + ((i >> hsh) << g.rope_sh);
}
// ---------------------------------------------------------------------------
// products whose second operand stays in registers (QKV, MLP up): Bv[ks] = this wavefront's column step ks of all
// messages.  A tile is 8 column steps of a block; with more than 8 steps per wavefront a block is two tiles.
constexpr int kWatchWords = 2048;
constexpr int kResSteps = 16;          // column steps a wavefront can keep: widths up to 8 * 16 * 32 = 4096
template <int HALF>
__device__ __forceinline__ void res_issue(Tile& t, const BGeo& g, int lb, int wg, int nwg, int lane) {
  const int i = lane & (g.R - 1) & 15, kg = lane >> 4;
  const int row = min(block_row(g, min(lb, max(g.nb_local - 1, 0)) * nwg + wg, i), g.N - 1);
  const uint32_t woff = (uint32_t)row * (uint32_t)g.row_bytes + (uint32_t)(kg << 4);
  const MDI_GLOBAL char* base = (const MDI_GLOBAL char*)g.W + ((long)g.ks0 << 6);
  const int last = max(g.nks - 1 - HALF * 8, 0);
#pragma unroll
  for (int s = 0; s < 8; ++s)
    t.r[s] = *reinterpret_cast<const MDI_GLOBAL u32x4*>(base + ((long)(HALF * 8 + min(s, last)) << 6) + woff);
}
template <int HALF, bool LAST_HALF>
__device__ __forceinline__ void res_compute(const Tile& t, const BGeo& g, int lb, const bf16x8 (&Bv)[kResSteps], f32x4& acc,
                                            float* part, int wave, int lane) {
  if (lb < 0 || lb >= g.nb_local) return;                        // uniform
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int ks = HALF * 8 + s;
    if (ks < g.nks)                                              // uniform
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, t.r[s]), Bv[ks], acc, 0, 0, 0);
  }
  if (LAST_HALF) {
    *reinterpret_cast<f32x4*>(part + (((lb * kStepWaves + wave) << 6) + lane) * 4) = acc;
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// ---------------------------------------------------------------------------
// Streamed products with the inner dimension split among workgroups.  Every workgroup used to read the whole
// vector of all messages for its one block of rows: 256 copies of it through the dies' L2s, twice the bytes of
// the matrix itself in the MLP down projection.  Here workgroup (q, s) takes column slice s of the eight row
// blocks 8 q .. 8 q + 7, one block per wavefront: it reads 1 / S of the vector - once, validated, into LDS, from
// where its eight wavefronts take the matrix instruction's second operand - and hands the 16 x 16 partial result
// of every block, as tagged words, to the workgroup that owns the block's residual rows, which adds the S partials
// in slice order.
struct KsGeo {
  int S, q, s;          // slices per block; this workgroup's block octet and slice (q >= octets: no work)
  int k0, nk;           // the slice: column steps [k0, k0 + nk)
  int blk, nblk;        // this wavefront's block; blocks of the product
  bool live;            // this wavefront has columns and a block
};
// c = column steps of a slice; q, s = workgroup divided by S, the same for the whole launch
__device__ __forceinline__ KsGeo make_ksgeo(int N, int Kd, int S, int c, int octets, int q, int s, int wave) {
  KsGeo g;
  g.S = S; g.q = q; g.s = s;
  const int ktot = Kd >> 5;
  g.k0 = min(g.s * c, ktot);
  g.nk = g.q < octets ? max(0, min(c, ktot - g.s * c)) : 0;
  g.nblk = (N + 15) >> 4;
  g.blk = g.q * kStepWaves + wave;
  g.live = g.nk > 0 && g.blk < g.nblk;
  return g;
}
// column steps 8 t .. 8 t + 7 of the slice (steps past its end repeat its last one)
__device__ __forceinline__ void ks_issue(Tile& t, const KsGeo& g, const char* W, uint32_t woff, int ti) {
  const MDI_GLOBAL char* base = (const MDI_GLOBAL char*)W + ((long)g.k0 << 6);
  const int last = max(g.nk - 1, 0);
#pragma unroll
  for (int s = 0; s < 8; ++s)
    t.r[s] = *reinterpret_cast<const MDI_GLOBAL u32x4*>(base + ((long)min(ti * 8 + s, last) << 6) + woff);
}
__device__ __forceinline__ void ks_compute(const Tile& t, const KsGeo& g, const u32x4* Bs, int ti, int lane, f32x4& acc) {
  const int n = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int ks = ti * 8 + s;
    if (ks < g.nk) {                                             // uniform
      const int gi = ks * 4 + kg;
      const u32x4 b = Bs[gi * 16 + (n ^ (gi & 15))];
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, t.r[s]), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
  }
}
// Sum over the wavefronts of element (row i, message j) of local block lb.
__device__ __forceinline__ float part_sum(const float* part, int lb, int i, int j) {
  const float* p = part + ((lb * kStepWaves) << 8) + ((((i >> 2) << 4) + j) << 2) + (i & 3);
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < kStepWaves; ++w) v += p[w << 8];
  return v;
}

// Wavefront records -> split partial, or the finished output when there is one split; the last workgroup of a head
// group to arrive folds the splits in split order (as attn_finish in step_impl.h).  The output leaves as bf16 pairs.
template <int G>
__device__ __forceinline__ void attn_finish_pairs(const AttnGeo& g, const BatchArgs& a, const BatchView& S, const float* sm, int* s_flag, unsigned epoch, int tid) {
  const unsigned wtag = epoch + 1;
  const int h = a.h, rec = h + 2, hp = h >> 1;
  const bool single = S.n_splits == 1;
  for (int idx = tid; idx < G * hp; idx += kStepThreads) {
    const int gi = idx / hp, e = (idx - gi * hp) * 2;
    float m = -1e30f;
    for (int w = 0; w < kStepWaves; ++w) m = fmaxf(m, sm[(w * G + gi) * rec + h]);
    float l = 0.f, o0 = 0.f, o1 = 0.f;
    for (int w = 0; w < kStepWaves; ++w) {
      const float* r = sm + (w * G + gi) * rec;
      const float sc = __expf(r[h] - m);
      l += r[h + 1] * sc; o0 += r[e] * sc; o1 += r[e + 1] * sc;
    }
    const int head = g.hg * G + gi;
    if (single) {
      st_pair(S.ob + (((long)head * h + e) >> 1) * S.n_msg + S.msg, pack_bf16x2(o0 / l, o1 / l), wtag);
    } else {
      tagged_t* pr = S.part + ((long)head * kMaxSplits + g.split) * rec;
      st_tag(pr + e, o0, wtag); st_tag(pr + e + 1, o1, wtag);
      if (e == 0) { st_tag(pr + h, m, wtag); st_tag(pr + h + 1, l, wtag); }
    }
  }
  if (single) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  if (tid == 0) s_flag[1] = last_of(S.tickets + g.hg, (unsigned)S.n_splits);
  __syncthreads();
  if (!s_flag[1]) return;
  for (int idx = tid; idx < G * hp; idx += kStepThreads) {
    const int gi = idx / hp, e = (idx - gi * hp) * 2;
    const int head = g.hg * G + gi;
    const tagged_t* pr = S.part + (long)head * kMaxSplits * rec;
    float m = -1e30f, l = 0.f, o0 = 0.f, o1 = 0.f;
    for (int sp0 = 0; sp0 < S.n_splits; sp0 += 4) {                // four splits' loads in flight together
      tagged_t rm[4], rl[4], ra[4], rb[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool ok = sp0 + k < S.n_splits;
        const tagged_t* r = pr + (sp0 + k) * rec;
        rm[k] = ok ? ld_raw(r + h) : 0ull; rl[k] = ok ? ld_raw(r + h + 1) : 0ull;
        ra[k] = ok ? ld_raw(r + e) : 0ull; rb[k] = ok ? ld_raw(r + e + 1) : 0ull;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (sp0 + k < S.n_splits) {
          const tagged_t* r = pr + (sp0 + k) * rec;
          const float mk = settle(r + h, rm[k], wtag, a.spin_limit, a.err);
          const float lk = settle(r + h + 1, rl[k], wtag, a.spin_limit, a.err);
          const float ak = settle(r + e, ra[k], wtag, a.spin_limit, a.err);
          const float bk = settle(r + e + 1, rb[k], wtag, a.spin_limit, a.err);
          const float mn = fmaxf(m, mk);
          const float sa = __expf(m - mn), sb = __expf(mk - mn);
          l = l * sa + lk * sb;
          o0 = o0 * sa + ak * sb; o1 = o1 * sa + bk * sb;
          m = mn;
        }
      }
    }
    st_pair(S.ob + (((long)head * h + e) >> 1) * S.n_msg + S.msg, pack_bf16x2(o0 / l, o1 / l), wtag);
  }
}

// ---------------------------------------------------------------------------
// Attention of four query heads that share a kv head, heads of 128, with the scores on the matrix cores.  On the vector
// ALUs a position costs four heads x (8 multiply-adds, 4 cross-lane adds, two 16-byte reads of q from LDS) per lane
// before its values are touched, and the phase ran at that pace: 115 us a layer for 16 messages with 6144 positions,
// where HBM needs 64 us; like this it takes 81 us (the whole 8-layer launch 1835 -> 1475 us).
//   * A tile is 16 positions of one page (pages and context splits are multiples of 16, so one page number serves it).
//     Keys in operand order: lane (i = l mod 16, kg = l div 16) holds columns 32 c + 8 kg .. + 7 of position i.
//   * The queries stay exact: column n of the second operand is head n mod 4, and its columns n div 4 = 0, 1, 2 are three
//     bf16 parts that add up to the 24 bits of q (the fourth is zero).  Adding the four columns of a head inside a row
//     of 16 lanes (two rotations) leaves the score of position 4 kg + r in register r of every lane of row kg.
//   * So a row of 16 lanes works on positions 4 kg .. 4 kg + 3 with running maximum, sum and output of its own, values
//     as 16-byte pieces (lane = 8 columns); a lane keeps maximum and sum of head n mod 4, and reads another head's weight
//     out of its quad (DPP).
template <int QUAD> __device__ __forceinline__ float quad_lane(float v) {       // lane QUAD of every four, to all four
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), QUAD * 0x55, 0xF, 0xF, false));
}
template <int K> __device__ __forceinline__ float row_rotate(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + K, 0xF, 0xF, false));
}
struct Attn4 {
  bf16x8 q[4];
  float m, l, o[4][8];
  int n_t;                       // tiles of the item's cached positions
};
// tile ti of this wavefront; tiles past the item's last re-read the sequence's first
__device__ __forceinline__ int attn4_tile(const AttnGeo& g, const Attn4& s, int ti, int wave) {
  const int t = ti * kStepWaves + wave;
  return t < s.n_t ? g.s0 + 16 * t : -1;
}
__device__ __forceinline__ int attn4_page(const AttnGeo& g, const Attn4& s, const BatchView& S, int ti, int wave) {
  const int base = max(attn4_tile(g, s, ti, wave), 0);
  return __hip_atomic_load((const MDI_GLOBAL int32_t*)S.table + page_of(g, base), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void attn4_issue(Tile& t, int& pg, const AttnGeo& g, const Attn4& s, const BatchArgs& a, const BatchView& S,
                                            const void* pool, int ti, int wave, int lane) {
  const int base0 = attn4_tile(g, s, ti, wave), base = max(base0, 0);
  const int page = __builtin_amdgcn_readfirstlane(pg);
  const MDI_GLOBAL char* kb = (const MDI_GLOBAL char*)pool + 2 * (((long)page * a.K + g.kvh) * 2 * a.pt_h + (long)(base - page_of(g, base) * a.pt) * 128);
  const uint32_t ko = (uint32_t)((lane & 15) * 256 + (lane >> 4) * 16);
  // a position past the last one has weight zero, and its values must be finite: the last one's
  const int end = base0 < 0 ? 15 : min(g.s1p - base - 1, 15), row = (lane >> 4) * 4;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    t.r[k] = *reinterpret_cast<const MDI_GLOBAL u32x4*>(kb + ko + 64 * k);
    t.r[4 + k] = *reinterpret_cast<const MDI_GLOBAL u32x4*>(kb + 2 * a.pt_h + (uint32_t)(min(row + k, end) * 256 + (lane & 15) * 16));
  }
  pg = attn4_page(g, s, S, ti + 2, wave);
}
__device__ __forceinline__ void attn4_compute(Attn4& s, const Tile& t, const AttnGeo& g, int ti, int wave, int lane) {
  const int base = attn4_tile(g, s, ti, wave);
  if (base < 0) return;                                          // uniform
  f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 4; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, t.r[k]), s.q[k], c, 0, 0, 0);
  float sc[4], p[4];
  bool ok[4];
  float mn = s.m;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float v = c[r] + row_rotate<4>(c[r]);
    sc[r] = v + row_rotate<8>(v);
    ok[r] = base + 4 * (lane >> 4) + r < g.s1p;
    mn = ok[r] ? fmaxf(mn, sc[r]) : mn;
  }
  if (__any(mn != s.m)) {                                        // rare after the first tiles
    const float alpha = __expf(s.m - mn);
    s.m = mn; s.l *= alpha;
    const float al[4] = {quad_lane<0>(alpha), quad_lane<1>(alpha), quad_lane<2>(alpha), quad_lane<3>(alpha)};
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
#pragma unroll
      for (int e = 0; e < 8; ++e) s.o[gi][e] *= al[gi];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) { p[r] = ok[r] ? __expf(sc[r] - mn) : 0.f; s.l += p[r]; }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float vf[8];
    Unpack<bf16_t>::go(t.r[4 + r], vf);
    const float w[4] = {quad_lane<0>(p[r]), quad_lane<1>(p[r]), quad_lane<2>(p[r]), quad_lane<3>(p[r])};
#pragma unroll
    for (int gi = 0; gi < 4; ++gi)
#pragma unroll
      for (int e = 0; e < 8; ++e) s.o[gi][e] = fmaf(w[gi], vf[e], s.o[gi][e]);
  }
}
// The whole stream of an item, between attn_begin (queries in qs, the newest position in `st`) and attn_to_lds.
__device__ __forceinline__ void attn4_stream(Attn4& s, AttnState<bf16_t, 4>& st, Tile& A, Tile& B, int& pgA, int& pgB, const AttnGeo& g,
                                             const BatchArgs& a, const BatchView& S, const void* kv, int wave, int lane, const float* qs) {
  const int n = lane & 15, part = n >> 2;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float4* qp = reinterpret_cast<const float4*>(qs + (n & 3) * 128 + 32 * k + 8 * (lane >> 4));
    const float4 lo = qp[0], hi = qp[1];
    const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t b0 = f32_to_bf16(v[e]);
      const float r1 = v[e] - bf16_bits_to_f32(b0);
      const uint32_t b1 = f32_to_bf16(r1);
      const uint32_t b2 = f32_to_bf16(r1 - bf16_bits_to_f32(b1));
      const uint32_t b = part == 0 ? b0 : part == 1 ? b1 : part == 2 ? b2 : 0u;
      if (e & 1) w[e >> 1] |= b << 16; else w[e >> 1] = b;
    }
    s.q[k] = __builtin_bit_cast(bf16x8, w);
  }
  const float m0 = st.m[0], m1 = st.m[1], m2 = st.m[2], m3 = st.m[3], l0 = st.l[0], l1 = st.l[1], l2 = st.l[2], l3 = st.l[3];
  s.m = (n & 2) ? ((n & 1) ? m3 : m2) : ((n & 1) ? m1 : m0);
  s.l = (n & 2) ? ((n & 1) ? l3 : l2) : ((n & 1) ? l1 : l0);
#pragma unroll
  for (int gi = 0; gi < 4; ++gi)
#pragma unroll
    for (int e = 0; e < 8; ++e) s.o[gi][e] = st.o[gi][e];
  const int n_w = (s.n_t - wave + kStepWaves - 1) / kStepWaves, nte = (max(n_w, 0) + 1) & ~1;
#pragma nounroll
  for (int t = 2; t < nte; t += 2) {
    attn4_compute(s, A, g, t - 2, wave, lane);
    attn4_issue(A, pgA, g, s, a, S, kv, t, wave, lane);
    attn4_compute(s, B, g, t - 1, wave, lane);
    attn4_issue(B, pgB, g, s, a, S, kv, t + 1, wave, lane);
  }
  if (nte) { attn4_compute(s, A, g, nte - 2, wave, lane); attn4_compute(s, B, g, nte - 1, wave, lane); }
  st.m[0] = quad_lane<0>(s.m); st.m[1] = quad_lane<1>(s.m); st.m[2] = quad_lane<2>(s.m); st.m[3] = quad_lane<3>(s.m);
  st.l[0] = quad_lane<0>(s.l); st.l[1] = quad_lane<1>(s.l); st.l[2] = quad_lane<2>(s.l); st.l[3] = quad_lane<3>(s.l);
#pragma unroll
  for (int gi = 0; gi < 4; ++gi)
#pragma unroll
    for (int e = 0; e < 8; ++e) st.o[gi][e] = s.o[gi][e];
}

__device__ __forceinline__ void bstamp(const BatchArgs& a, int layer, int ph, int k) {
  if (a.trace && threadIdx.x == 0)
    a.trace[(((long)blockIdx.x * a.n_layer + layer) * 5 + ph) * 8 + k] = wall_clock64();
}

// Per-message values that a thread needs for a message index of its own (a kernel argument cannot be indexed per lane).
struct BatchLds {
  const float2* rope[kMaxBatch];
  const void* in[kMaxBatch];
  void* out[kMaxBatch];
  long kv_off[kMaxBatch];
  long tok[kMaxBatch];
  int pos[kMaxBatch];
};

// Element `row` of message j's input vector (the token's embedding plus learned position, or the previous stage's activation).
__device__ __forceinline__ float batch_input(const BatchArgs& a, const BatchLds& sl, int j, int row) {
  if (a.in_kind == IN_TOKEN) {
    float v = bf16_to_f32(((const bf16_t*)a.wte)[sl.tok[j] * a.d + row]);
    if (a.wpe) v += bf16_to_f32(((const bf16_t*)a.wpe)[(long)sl.pos[j] * a.d + row]);
    return v;
  }
  return bf16_to_f32(((const bf16_t*)sl.in[j])[row]);
}

// What the epilogue of a phase needs beside the products, for item e: QKV: (cos, sin) of the row pair; residual
// products: the following norm's gains of the row pair; all: the biases, and the LayerNorm corrections [W g | W b].
struct EpiItem { int j, p, lb; };      // message, row pair (SwiGLU: quad) of the block, local block
__device__ __forceinline__ EpiItem epi_item(int e, int m, unsigned m_magic, int n_sh) {
  const int x = (int)__umulhi((unsigned)e, m_magic);            // e / m, see BatchArgs
  return EpiItem{e - x * m, x & ((1 << n_sh) - 1), x >> n_sh};
}
// Sums over the eight lanes of a message's row pairs, published by the first of them.
__device__ __forceinline__ void publish_sums(float s2, float s1, int p, tagged_t* ssq, tagged_t* ssum, unsigned tag) {
  s2 = dpp_add<kDppXor1, 0xF>(s2); s2 = dpp_add<kDppXor2, 0xF>(s2); s2 = dpp_add<kDppHalfMirror, 0xF>(s2);
  if (p == 0) st_tag(ssq, s2, tag);
  if (ssum) {
    s1 = dpp_add<kDppXor1, 0xF>(s1); s1 = dpp_add<kDppXor2, 0xF>(s1); s1 = dpp_add<kDppHalfMirror, 0xF>(s1);
    if (p == 0) st_tag(ssum, s1, tag);
  }
}
struct EpiOps { float g0, g1, b0, b1, n[4]; };
__device__ __forceinline__ EpiOps epi_ops(const BatchArgs& a, const StepLayer& L, const BGeo& g, const BatchLds& sl, const float* nc, int ph,
                                          bool last, int e, int n_items, int n_sh, int wg, int nwg) {
  EpiOps o{};
  if (e >= n_items) return o;
  const bool resid = ph == PH_OPROJ || ph == PH_DOWN;
  const EpiItem it = resid ? EpiItem{e >> 3, e & 7, 0} : epi_item(e, a.m, a.m_magic, n_sh);
  const int j = it.j, p = it.p, lb = it.lb;
  if (ph == PH_QKV) {
    const int r0 = block_row(g, lb * nwg + wg, p), r1 = r0 + (a.h >> 1);
    const int head = r0 >> (31 - __builtin_clz(a.h));             // (head sizes are powers of two)
    const float2* rope = sl.rope[j];
    if (rope && head < a.H + a.K) { const float2 cs = rope[r0 & (a.h - 1)]; o.g0 = cs.x; o.g1 = cs.y; }
    if (L.bqkv) { o.b0 = L.bqkv[r0]; o.b1 = L.bqkv[r1]; }
    if (nc) { o.n[0] = nc[r0]; o.n[1] = nc[r1]; o.n[2] = nc[g.N + r0]; o.n[3] = nc[g.N + r1]; }
    return o;
  }
  if (ph == PH_UP && a.mlp_kind == MDI_MLP_SWIGLU) return o;
  const int r0 = (lb * nwg + wg) * g.R + 2 * p;
  if (r0 >= g.N) return o;
  const float *bu = L.bup, *bo = L.bo, *bd = L.bdown, *g1 = L.ln1_g, *g2 = L.ln2_g;
  const float* bias = ph == PH_UP ? bu : ph == PH_OPROJ ? bo : bd;
  if (bias) { o.b0 = bias[r0]; o.b1 = bias[r0 + 1]; }
  if (ph == PH_UP) {
    if (nc) { o.n[0] = nc[r0]; o.n[1] = nc[r0 + 1]; o.n[2] = nc[g.N + r0]; o.n[3] = nc[g.N + r0 + 1]; }
  } else if (!last) {
    const float* gain = ph == PH_OPROJ ? g2 : advance(g1, a.w_stride);
    o.g0 = gain[r0]; o.g1 = gain[r0 + 1];
  }
  return o;
}

// G query heads per attention work item; kScoresOnMfma: see Attn4 (G = 4)
template <int G, bool kScoresOnMfma>
__global__ __launch_bounds__(kStepThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_step_batch(BatchArgs a) {
  typedef bf16_t WT;
  extern __shared__ float smem[];
  __shared__ BatchLds sl;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = blockIdx.x, nwg = a.nwg, m = a.m;
  int* s_flag = lds_flag();
  float* rscale = smem + 32;                     // [16] 1/rms (LayerNorm: 1/std) of every message's vector in the normed products
  float* rshift = smem + 64;                     // [16] LayerNorm: (mean - centre) / std of every message's vector
  float* rcen = smem + 80;                       // [16] LayerNorm: the centre the vectors are published around (see below)
  const bool ln = a.norm_kind == MDI_NORM_LAYERNORM;
  float* xres = smem + a.lds_xres;               // residual rows this workgroup owns: [16 rows][16 messages]
  float* part = smem + a.lds_part;               // the wavefronts' partial products [block][wavefront][lane][4]; attention scratch

  if (threadIdx.x == 0) {
    s_flag[kFailed] = 0;
    for (int j = 0; j < m; ++j) {
      const BatchSlot& S = a.s[j];
      sl.rope[j] = S.rope; sl.in[j] = S.in; sl.out[j] = S.act_out; sl.kv_off[j] = S.kv_tok_off; sl.pos[j] = S.pos;
      sl.tok[j] = a.in_kind == IN_TOKEN ? checked_token(S.in, 0, a.vocab, a.err) : 0;
      if (wg == 0 && S.table_entry) *S.table_entry = S.new_page;    // for later launches: no position before the newest lies on a page that starts now
    }
  }
  __syncthreads();

  // Residual rows of this workgroup (the output projection's and the down projection's rows: same geometry) start
  // as the launch's inputs.  They are also published exactly as a down projection publishes its result - pairs of
  // x times the first layer's gain, this workgroup's share of the sums of squares, both with the counter the
  // first phase expects - so that the first layer's QKV product is like any other.
  // LayerNorm: a vector travels as (x - c) g in bf16, c a number per message that every workgroup knows: rounding
  // x g itself would cost accuracy whenever |mean| >> std.  c is the mean of the message's vector at the previous
  // norm of the launch (every workgroup computes it, from the same sums in the same order), for the first norm the
  // mean of the input vector, which every workgroup forms here for itself.
  if (!ln) {
    if (threadIdx.x < kMaxBatch) rcen[threadIdx.x] = 0.f;
  } else {
    for (int j = wave; j < m; j += kStepWaves) {
      float u = 0.f;
      for (int r0 = lane; r0 < a.d; r0 += 512) {     // eight loads in flight
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = batch_input(a, sl, j, min(r0 + 64 * k, a.d - 1));
#pragma unroll
        for (int k = 0; k < 8; ++k) u += r0 + 64 * k < a.d ? v[k] : 0.f;
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) u += __shfl_xor(u, off, 64);
      if (lane == 0) rcen[j] = u / (float)a.d;
    }
  }
  __syncthreads();
  {
    // item (message j, row pair p) of the block of 16 rows this workgroup owns: eight neighbouring lanes share a message
    const int e = threadIdx.x, j = e >> 3, p = e & 7, r0 = wg * 16 + 2 * p;
    if (e < 8 * m) {
      float s2 = 0.f, s1 = 0.f;
      if (r0 < a.d) {
        const float x0 = batch_input(a, sl, j, r0), x1 = batch_input(a, sl, j, r0 + 1);
        float* xr = xres + 2 * p * 16 + j;
        xr[0] = x0; xr[16] = x1;
        st_pair(a.xn[0] + (r0 >> 1) * m + j, pack_bf16x2((x0 - rcen[j]) * a.l0.ln1_g[r0], (x1 - rcen[j]) * a.l0.ln1_g[r0 + 1]), a.epoch0);
        s2 = x0 * x0 + x1 * x1; s1 = x0 + x1;
      }
      publish_sums(s2, s1, p, a.ssq[0] + j * nwg + wg, ln ? a.ssum[0] + j * nwg + wg : nullptr, a.epoch0);
    }
  }
  __syncthreads();

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int ks_q = wg / a.str_S, ks_s = wg - ks_q * a.str_S;

#pragma nounroll
  for (int layer = 0; layer < a.n_layer; ++layer) {
    const StepLayer Lv = layer_at(a, layer);
#pragma nounroll
    for (int ph = 0; ph < 5; ++ph) {
      const unsigned epoch = a.epoch0 + (unsigned)(layer * 5 + ph);
      const unsigned wtag = epoch + 1;
      const int jm = gemv_index(ph);
      const int N = jm == 0 ? (a.H + 2 * a.K) * a.h : jm == 2 ? (a.mlp_kind == MDI_MLP_SWIGLU ? 2 * a.F : a.F) : a.d;
      const int Kd = jm == 1 ? a.H * a.h : jm == 3 ? a.F : a.d;
      const BGeo g = make_bgeo(layer_matrix(Lv, jm), N, Kd, jm == 0 ? a.R[0] : jm == 2 ? a.R[2] : a.R[1], jm == 0 ? a.h : 0, wg, nwg, wave);
      // LayerNorm corrections of this phase's product: [W g | W b], N floats each (QKV's first, then the up product's)
      const float* nc = ln ? a.nc0 + (long)layer * a.nc_stride + (jm == 2 ? 2L * (a.H + 2 * a.K) * a.h : 0L) : nullptr;
      // Per-lane addresses and epilogue indexes do not change from phase to phase; computed once outside the loops they
      // would occupy dozens of registers for the whole launch, so they are derived from values the compiler cannot see
      // through and are recomputed where they are used.
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, kg = lane >> 4, lane_msg = min(lane & 15, m - 1);   // lane_msg: the message this lane's column stands for (columns past m repeat the last)
      tagged_t* ob_l = a.ob;
      tagged_t* ub_l = a.ub;
      bstamp(a, layer, ph, 0);

      // Every kind of phase keeps its registers to itself (tiles in flight, the second operand, attention state are
      // declared inside its branch and given a value on every path), so that the compiler sees them dead elsewhere.
      // Each branch first issues the requests that depend on nothing another workgroup writes; they are on their way
      // while the words of the phase before arrive.  The epilogue's own operands (gains, biases, angles) are among
      // them: a thread keeps those of its first item, fetched again they would cost a round trip at the phase's end.
      if (ph == PH_ATTN) {
        // ---- attention: one work item = (message, head group, context split); items dealt round-robin
        for (int item = wg, slot = 0; item < a.n_items; item += nwg) {
          if (item != wg) __syncthreads();                           // the records in LDS have been read
          while (slot + 1 < m && item >= a.s[slot + 1].item_lo) ++slot;
          const BatchView V = view_of(a, slot, ob_l);
          const AttnGeo ga = make_attn_geo<WT, G>(a, V, item - a.s[slot].item_lo, wave, lane);
          AttnState<WT, G> st;
          AttnAsk<WT> ask{};
          Tile A, B;
          attn_ask<WT, G>(ask, ga, a, V, wave, epoch, tid);
          if constexpr (kScoresOnMfma) {
            Attn4 s4;
            s4.n_t = max(ga.s1p - ga.s0 + 15, 0) >> 4;
            int pgA = attn4_page(ga, s4, V, 0, wave), pgB = attn4_page(ga, s4, V, 1, wave);
            attn4_issue(A, pgA, ga, s4, a, V, Lv.kv, 0, wave, lane); attn4_issue(B, pgB, ga, s4, a, V, Lv.kv, 1, wave, lane);
            if (item == wg) bstamp(a, layer, ph, 1);
            attn_begin<WT, G>(st, ask, ga, a, V, part, wave, epoch, tid);
            if (item == wg) bstamp(a, layer, ph, 2);
            attn4_stream(s4, st, A, B, pgA, pgB, ga, a, V, Lv.kv, wave, lane, part);
          } else {
            int pgA[kTile], pgB[kTile];
            attn_pages(pgA, ga, a, V, 0, wave); attn_pages(pgB, ga, a, V, 1, wave);
            attn_issue<WT>(A, pgA, ga, a, V, Lv.kv, 0, wave); attn_issue<WT>(B, pgB, ga, a, V, Lv.kv, 1, wave);
            if (item == wg) bstamp(a, layer, ph, 1);
            attn_begin<WT, G>(st, ask, ga, a, V, part, wave, epoch, tid);
            if (item == wg) bstamp(a, layer, ph, 2);
            const int nte = ((ga.n_k + kTile - 1) / kTile + 1) & ~1;
            attn_stream<WT, G>(st, A, B, pgA, pgB, ga, a, V, Lv.kv, nte, wave, part);
          }
          if (item == wg) bstamp(a, layer, ph, 3);
          attn_to_lds<WT, G>(st, ga, a.h, part, wave);
          attn_finish_pairs<G>(ga, a, V, part, s_flag, epoch, tid);
        }
      } else {
        const int R = g.R, half = R >> 1;
        // epilogue items per block and message: row pairs, or quads of rows for SwiGLU; a power of two
        const int n_sh = (R == 16 ? 3 : 2) - (ph == PH_UP && a.mlp_kind == MDI_MLP_SWIGLU ? 1 : 0);
        const int n_items = (g.nb_local << n_sh) * m;
        const bool last = ph == PH_DOWN && layer == a.n_layer - 1;   // (both residual products only)
        EpiOps ops = epi_ops(a, Lv, g, sl, nc, ph, last, tid, n_items, n_sh, wg, nwg);
        if (ph == PH_QKV || ph == PH_UP) {
          // ---- a product whose second operand stays in registers: this wavefront's column slice of every message, as
          // published, bf16 pairs of x * gain.  Asked for first, before the weights: the sums of squares of all
          // messages.  Vectors of more than kWatchWords words are looked at only after every workgroup's first sum of
          // squares (which it stores last) is there: 256 workgroups that watch 32 KB each crowd out the stores they wait
          // for (TinyLlama, 4 messages: 629 us, ungated 644; the 7B shape with 8: 979 and 975).
          Tile A, B;
          bf16x8 Bv[kResSteps];
          const tagged_t* xn_in = ph == PH_QKV ? a.xn[0] : a.xn[1];  // (selected, not indexed: an index into the arguments costs a copy of them)
          const tagged_t* ssq_in = ph == PH_QKV ? a.ssq[0] : a.ssq[1];
          const tagged_t* ssum_in = ph == PH_QKV ? a.ssum[0] : a.ssum[1];
          const tagged_t* bbase = xn_in + (long)g.ks0 * (16 * m);
          const uint32_t boff = (uint32_t)(4 * kg * m + lane_msg) << 3;
          const int last_ks = max(g.nks - 1, 0);
          auto step_at = [&](int ks, int e, uint32_t z) __attribute__((always_inline)) { return word_at(bbase + min(ks, last_ks) * (16 * m) + e * m, boff + z); };
          const int sj = tid >> 5, sc = tid & 31;                    // sums: 32 threads per message, eight words each
          auto sum_at = [&](const tagged_t* v, int k, uint32_t z) __attribute__((always_inline)) {
            return word_at(v, (uint32_t)(min(sj, m - 1) * nwg + min(sc + 32 * k, nwg - 1)) * 8u + z);
          };
          tagged_t sqr[8] = {};
          const bool long_vec = (a.d >> 1) * m > kWatchWords;
          auto gate_at = [&](int, uint32_t z) __attribute__((always_inline)) { return word_at(ssq_in, (uint32_t)tid * 8u + z); };
          auto gated = [&](int) __attribute__((always_inline)) { return long_vec && tid < nwg; };
          tagged_t gate[1];
          ask_words(gate, gate_at, epoch, gated);
          if (sj < m) ask_words(sqr, [&](int k, uint32_t z) { return sum_at(ssq_in, k, z); }, epoch);
          if (g.nks > 8) { res_issue<0>(A, g, 0, wg, nwg, lane); res_issue<1>(B, g, 0, wg, nwg, lane); }
          else { res_issue<0>(A, g, 0, wg, nwg, lane); res_issue<0>(B, g, 1, wg, nwg, lane); }
          bstamp(a, layer, ph, 1);
          if (long_vec) {
            await_words(gate, gate_at, epoch, a.spin_limit, a.err, gated);
            for (int i = tid + kStepThreads; i < nwg; i += kStepThreads)
              poll_words(gate, [&](int, uint32_t z) { return word_at(ssq_in, (uint32_t)i * 8u + z); }, epoch, a.spin_limit, a.err);
            __syncthreads();
          }
          float sum2 = 0.f, sum1 = 0.f;                              // this thread's share of its message's sums
          if (sj < m) {
            await_words(sqr, [&](int k, uint32_t z) { return sum_at(ssq_in, k, z); }, epoch, a.spin_limit, a.err);
#pragma unroll
            for (int k = 0; k < 8; ++k) sum2 += sc + 32 * k < nwg ? tag_value(sqr[k]) : 0.f;
            if (ln) {
              poll_words(sqr, [&](int k, uint32_t z) { return sum_at(ssum_in, k, z); }, epoch, a.spin_limit, a.err);
#pragma unroll
              for (int k = 0; k < 8; ++k) sum1 += sc + 32 * k < nwg ? tag_value(sqr[k]) : 0.f;
            }
            for (int w = sc + 256; w < nwg; w += 32) {               // (more than 256 workgroups)
              auto at = [&](const tagged_t* v, uint32_t z) { return word_at(v, (uint32_t)(sj * nwg + w) * 8u + z); };
              tagged_t one[1];
              poll_words(one, [&](int, uint32_t z) { return at(ssq_in, z); }, epoch, a.spin_limit, a.err);
              sum2 += tag_value(one[0]);
              if (ln) { poll_words(one, [&](int, uint32_t z) { return at(ssum_in, z); }, epoch, a.spin_limit, a.err); sum1 += tag_value(one[0]); }
            }
          }
          auto fetch4 = [&](int h0, bf16x8& v0, bf16x8& v1, bf16x8& v2, bf16x8& v3) __attribute__((always_inline)) {
            if (h0 == 0 || h0 < g.nks) {             // uniform: a batch of steps that lies past the slice costs no round trip
              tagged_t xr[16];                         // steps past the slice repeat its last one: every register gets a value
              poll_words(xr, [&](int s, uint32_t z) { return step_at(h0 + (s >> 2), s & 3, z); }, epoch, a.spin_limit, a.err);
              auto low4 = [&](int s) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8, u32x4{(uint32_t)xr[s], (uint32_t)xr[s + 1], (uint32_t)xr[s + 2], (uint32_t)xr[s + 3]}); };
              v0 = low4(0); v1 = low4(4); v2 = low4(8); v3 = low4(12);
            } else {
              v0 = Bv[0]; v1 = Bv[0]; v2 = Bv[0]; v3 = Bv[0];
            }
          };
          fetch4(0, Bv[0], Bv[1], Bv[2], Bv[3]); fetch4(4, Bv[4], Bv[5], Bv[6], Bv[7]);
          fetch4(8, Bv[8], Bv[9], Bv[10], Bv[11]); fetch4(12, Bv[12], Bv[13], Bv[14], Bv[15]);
          bstamp(a, layer, ph, 2);
          // the stream: two tiles in flight, each multiplied while the other's rows arrive
          if (g.nks > 8) {
#pragma nounroll
            for (int lb = 1; lb < g.nb_local; ++lb) {
              res_compute<0, false>(A, g, lb - 1, Bv, acc, part, wave, lane);
              res_issue<0>(A, g, lb, wg, nwg, lane);
              res_compute<1, true>(B, g, lb - 1, Bv, acc, part, wave, lane);
              res_issue<1>(B, g, lb, wg, nwg, lane);
            }
            res_compute<0, false>(A, g, g.nb_local - 1, Bv, acc, part, wave, lane);
            res_compute<1, true>(B, g, g.nb_local - 1, Bv, acc, part, wave, lane);
          } else {
            int lb = 0;
#pragma nounroll
            for (; lb + 2 < g.nb_local; lb += 2) {
              res_compute<0, true>(A, g, lb, Bv, acc, part, wave, lane);
              res_issue<0>(A, g, lb + 2, wg, nwg, lane);
              res_compute<0, true>(B, g, lb + 1, Bv, acc, part, wave, lane);
              res_issue<0>(B, g, lb + 3, wg, nwg, lane);
            }
            res_compute<0, true>(A, g, lb, Bv, acc, part, wave, lane);
            res_compute<0, true>(B, g, lb + 1, Bv, acc, part, wave, lane);
          }
          bstamp(a, layer, ph, 3);
          // 1/rms of every message.  The shares of all workgroups have been seen before anything of this phase is stored
          // (see the top of the file).
#pragma unroll
          for (int off = 16; off >= 1; off >>= 1) { sum2 += __shfl_xor(sum2, off, 64); if (ln) sum1 += __shfl_xor(sum1, off, 64); }
          if (sj < m && sc == 0) {
            if (!ln) {
              rscale[sj] = 1.f / sqrtf(sum2 / (float)a.d + a.eps);
            } else {
              const float mean = sum1 / (float)a.d;
              const float rstd = 1.f / sqrtf(fmaxf(sum2 / (float)a.d - mean * mean, 0.f) + a.eps);
              rscale[sj] = rstd; rshift[sj] = rstd * (mean - rcen[sj]);
              rcen[sj] = mean;                                       // what the next norm's vector is published around
            }
          }
        } else {
          // ---- a product whose inner dimension is split among workgroups (see KsGeo)
          const KsGeo kq = make_ksgeo(N, Kd, a.str_S, ph == PH_OPROJ ? a.str_c[0] : a.str_c[1], a.str_oct, ks_q, ks_s, wave);
          Tile A, B;
          const uint32_t woff = (uint32_t)min(kq.blk * 16 + (lane & 15), N - 1) * (uint32_t)g.row_bytes + (uint32_t)(kg << 4);
          // the slice of every message's vector to LDS as [group of 8 columns][message]
          u32x4* Bs = reinterpret_cast<u32x4*>(part);
          const tagged_t* bvec = ph == PH_OPROJ ? ob_l : ub_l;
          const int n_units = kq.nk * 4 * m;                         // unit: eight columns of one message
          tagged_t raw[8] = {};
          int gi[2], n[2];
          int u_at = tid;
          auto unit_of = [&](int u0) __attribute__((always_inline)) {
            u_at = u0;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              const int u = u0 + r * kStepThreads;
              gi[r] = (int)__umulhi((unsigned)u, a.m_magic); n[r] = u - gi[r] * m;
            }
          };
          auto at = [&](int r, uint32_t z) __attribute__((always_inline)) {   // pairs 4 (4 k0 + gi) .. + 3
            return word_at(bvec + (long)kq.k0 * (16 * m) + (r & 3) * m, (uint32_t)(4 * gi[r >> 2] * m + n[r >> 2]) * 8u + z);
          };
          auto live = [&](int r) __attribute__((always_inline)) { return u_at + (r >> 2) * kStepThreads < n_units; };
          unit_of(tid);
          ask_words(raw, at, epoch, live);
          ks_issue(A, kq, g.W, woff, 0);
          ks_issue(B, kq, g.W, woff, 1);
          bstamp(a, layer, ph, 1);
          for (int u0 = tid; u0 < n_units; u0 += 2 * kStepThreads) {
            if (u0 != tid) { unit_of(u0); ask_words(raw, at, epoch, live); }
            await_words(raw, at, epoch, a.spin_limit, a.err, live);
#pragma unroll
            for (int r = 0; r < 2; ++r)
              if (u0 + r * kStepThreads < n_units)
                Bs[gi[r] * 16 + (n[r] ^ (gi[r] & 15))] = u32x4{(uint32_t)raw[4 * r], (uint32_t)raw[4 * r + 1], (uint32_t)raw[4 * r + 2], (uint32_t)raw[4 * r + 3]};
          }
          __syncthreads();
          bstamp(a, layer, ph, 2);
          acc = f32x4{0.f, 0.f, 0.f, 0.f};
          if (kq.live) {                                             // uniform per wavefront
            const int nt = ((kq.nk + 7) >> 3) + 1 & ~1;
#pragma nounroll
            for (int t = 2; t < nt; t += 2) {
              ks_compute(A, kq, Bs, t - 2, lane, acc);
              ks_issue(A, kq, g.W, woff, t);
              ks_compute(B, kq, Bs, t - 1, lane, acc);
              ks_issue(B, kq, g.W, woff, t + 1);
            }
            ks_compute(A, kq, Bs, nt - 2, lane, acc);
            ks_compute(B, kq, Bs, nt - 1, lane, acc);
          }
          bstamp(a, layer, ph, 3);
          // the partial of (block, slice), zeros from a slice without columns, to the block's owner
          if (kq.q < a.str_oct && kq.blk < kq.nblk && (lane & 15) < m) {
            tagged_t* dst = a.ppart + ((long)((kq.blk * kq.S + kq.s) * 4 + kg) * m + (lane & 15)) * 4;
#pragma unroll
            for (int r = 0; r < 4; ++r) st_tag(dst + r, acc[r], wtag);
          }
          acc = f32x4{0.f, 0.f, 0.f, 0.f};
          bstamp(a, layer, ph, 7);
          // ---- residual products: x += W v (+ bias) on the 16 rows this workgroup owns; what leaves is x times the gain
          // of the norm that follows, as bf16 pairs, and this workgroup's share of every message's sum of squares (every
          // workgroup's, also without rows: see the top of the file).  One lane per (message, row pair), which adds the S
          // partials in slice order.
          tagged_t* xn_out = ph == PH_OPROJ ? a.xn[1] : a.xn[0];
          tagged_t* ssq_out = ph == PH_OPROJ ? a.ssq[1] : a.ssq[0];
          tagged_t* ssum_out = ph == PH_OPROJ ? a.ssum[1] : a.ssum[0];
          const int j = tid >> 3, p = tid & 7, r0 = wg * 16 + 2 * p;
          if (j < m) {
            float s2 = 0.f, s1 = 0.f;
            if (wg < kq.nblk) {
              const tagged_t* srcp = a.ppart + (long)wg * kq.S * (16 * m);
              const uint32_t off = (uint32_t)((p >> 1) * m + j) * 32u + (uint32_t)(p & 1) * 16u;
              float d0 = 0.f, d1 = 0.f;
              auto add = [&](auto n_const) __attribute__((always_inline)) {
                constexpr int NS = decltype(n_const)::value;
                tagged_t raw[2 * NS];                                // slices past the last repeat it
                poll_words(raw, [&](int k, uint32_t z) { return word_at(srcp + min(k >> 1, kq.S - 1) * (16 * m) + (k & 1), off + z); }, wtag, a.spin_limit, a.err);
#pragma unroll
                for (int k = 0; k < NS; ++k) { d0 += k < kq.S ? tag_value(raw[2 * k]) : 0.f; d1 += k < kq.S ? tag_value(raw[2 * k + 1]) : 0.f; }
              };
              if (kq.S <= 8) add(std::integral_constant<int, 8>()); else add(std::integral_constant<int, 16>());
              if (r0 < g.N) {
                float* xr = xres + 2 * p * 16 + j;
                const float x0 = xr[0] + d0 + ops.b0, x1 = xr[16] + d1 + ops.b1;
                xr[0] = x0; xr[16] = x1;
                if (last) {
                  store_kind(sl.out[j], a.act_kind, r0, x0); store_kind(sl.out[j], a.act_kind, r0 + 1, x1);
                } else {
                  st_pair(xn_out + (r0 >> 1) * m + j, pack_bf16x2((x0 - rcen[j]) * ops.g0, (x1 - rcen[j]) * ops.g1), wtag);
                  s2 = x0 * x0 + x1 * x1; s1 = x0 + x1;
                }
              }
            }
            if (!last) publish_sums(s2, s1, p, ssq_out + j * nwg + wg, ln ? ssum_out + j * nwg + wg : nullptr, wtag);
          }
        }
        if (ph == PH_QKV || ph == PH_UP) {
          __syncthreads();                                           // every wavefront's partial products are in LDS
          bstamp(a, layer, ph, 4);
        }

        // ---- epilogue of the normed products: one thread per (block, row pair or quad, message)
        if (ph == PH_QKV) {
          for (int e = tid; e < n_items; e += kStepThreads) {
            const EpiItem it = epi_item(e, m, a.m_magic, n_sh);
            const int j = it.j, p = it.p, lb = it.lb;
            const int r0 = block_row(g, lb * nwg + wg, p), r1 = r0 + (a.h >> 1);
            float v0 = part_sum(part, lb, p, j) * rscale[j], v1 = part_sum(part, lb, p + half, j) * rscale[j];
            if (ln) { v0 += ops.n[2] - rshift[j] * ops.n[0]; v1 += ops.n[3] - rshift[j] * ops.n[1]; }
            v0 += ops.b0; v1 += ops.b1;
            const int head = r0 >> (31 - __builtin_clz(a.h)), i = r0 & (a.h - 1);
            if (sl.rope[j] && head < a.H + a.K) {
              const float t0 = v0 * ops.g0 - v1 * ops.g1, t1 = v0 * ops.g1 + v1 * ops.g0;
              v0 = t0; v1 = t1;
            }
            char* base = a.slot0 + (long)j * a.slot_stride;
            if (head < a.H) {
              tagged_t* q = (tagged_t*)(base + a.off_q);
              st_tag(q + r0, v0, wtag); st_tag(q + r1, v1, wtag);
            } else {
              // the cache row is for later launches (plain stores); this launch's attention takes the same
              // rounded values from the tagged copy
              const bool is_v = head >= a.H + a.K;
              const int kvh = head - a.H - (is_v ? a.K : 0);
              WT* dst = (WT*)Lv.kv + sl.kv_off[j] + (long)(kvh * 2 + (is_v ? 1 : 0)) * a.pt_h + i;
              Storage<WT>::put(dst, v0); Storage<WT>::put(dst + (a.h >> 1), v1);
              tagged_t* kn = (tagged_t*)(base + a.off_knew) + (long)(is_v ? a.K * a.h : 0) + kvh * a.h + i;
              st_tag(kn, bf16_to_f32(f32_to_bf16(v0)), wtag); st_tag(kn + (a.h >> 1), bf16_to_f32(f32_to_bf16(v1)), wtag);
            }
            if (e + kStepThreads < n_items) ops = epi_ops(a, Lv, g, sl, nc, ph, last, e + kStepThreads, n_items, n_sh, wg, nwg);
          }
        } else if (ph == PH_UP) {
          if (a.mlp_kind == MDI_MLP_SWIGLU) {
            // rows (4q .. 4q + 3) = (gate_f, up_f, gate_f+1, up_f+1): one lane of every wavefront's result holds all four
            for (int e = tid; e < n_items; e += kStepThreads) {
              const EpiItem it = epi_item(e, m, a.m_magic, n_sh);
              const int j = it.j, qd = it.p, lb = it.lb;
              const int r0 = (lb * nwg + wg) * R + 4 * qd;
              if (r0 < g.N) {
                const float* pp = part + ((lb * kStepWaves) << 8) + (((qd << 4) + j) << 2);
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < kStepWaves; ++w) { const f32x4 t = *reinterpret_cast<const f32x4*>(pp + (w << 8)); v += t; }
                const float rs = rscale[j];
                v *= rs;
                if (ln) {
                  const float sh = rshift[j];
                  v.x += nc[N + r0] - sh * nc[r0]; v.y += nc[N + r0 + 1] - sh * nc[r0 + 1];
                  v.z += nc[N + r0 + 2] - sh * nc[r0 + 2]; v.w += nc[N + r0 + 3] - sh * nc[r0 + 3];
                }
                const float u0 = silu_f(v.x) * v.y, u1 = silu_f(v.z) * v.w;
                st_pair(ub_l + (r0 >> 2) * m + j, pack_bf16x2(u0, u1), wtag);
              }
            }
          } else {
            const bool tanh_form = a.mlp_kind == MDI_MLP_GELU_TANH;
            for (int e = tid; e < n_items; e += kStepThreads) {
              const EpiItem it = epi_item(e, m, a.m_magic, n_sh);
              const int j = it.j, p = it.p, lb = it.lb;
              const int r0 = (lb * nwg + wg) * R + 2 * p;
              if (r0 < g.N) {
                float v0 = part_sum(part, lb, 2 * p, j) * rscale[j], v1 = part_sum(part, lb, 2 * p + 1, j) * rscale[j];
                if (ln) { v0 += ops.n[2] - rshift[j] * ops.n[0]; v1 += ops.n[3] - rshift[j] * ops.n[1]; }
                v0 += ops.b0; v1 += ops.b1;
                st_pair(ub_l + (r0 >> 1) * m + j, pack_bf16x2(tanh_form ? gelu_tanh_f(v0) : gelu_erf_f(v0), tanh_form ? gelu_tanh_f(v1) : gelu_erf_f(v1)), wtag);
              }
              if (e + kStepThreads < n_items) ops = epi_ops(a, Lv, g, sl, nc, ph, last, e + kStepThreads, n_items, n_sh, wg, nwg);
            }
          }
        }
      }

      // ---- the partial products and the attention's records in LDS have been read
      bstamp(a, layer, ph, 5);
      __syncthreads();
      bstamp(a, layer, ph, 6);
      if (s_flag[kFailed]) return;                                   // a bounded wait expired: everybody else's will, too
    }
  }
}

}  // namespace step_w8

bool step_batch_allow_lds(size_t lds) {
  using namespace step_w8;
  const void* const kernels[] = {(const void*)k_step_batch<1, false>, (const void*)k_step_batch<2, false>, (const void*)k_step_batch<4, false>,
                                 (const void*)k_step_batch<4, true>};
  for (const void* k : kernels)
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return false;
  return true;
}

void launch_step_batch(hipStream_t s, int G, bool scores_on_mfma, size_t lds, const BatchArgs& a) {
  using namespace step_w8;
  const dim3 grid(a.nwg), block(kStepThreads);
  if (G == 4 && scores_on_mfma) hipLaunchKernelGGL((k_step_batch<4, true>), grid, block, lds, s, a);
  else if (G == 4) hipLaunchKernelGGL((k_step_batch<4, false>), grid, block, lds, s, a);
  else if (G == 2) hipLaunchKernelGGL((k_step_batch<2, false>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((k_step_batch<1, false>), grid, block, lds, s, a);
}

}  // namespace mdi

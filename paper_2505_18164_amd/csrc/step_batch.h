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
//   * One set of workgroups, all messages in lockstep: of eight wavefronts, or of four where the messages' vectors are short
//     (batch_plan in mdi_api.hip: one wavefront per SIMD executes a phase boundary's instructions without taking turns).
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
//     wavefronts of a workgroup split the block's columns among them and their partial 16 x 16 results are
//     added in LDS in wavefront order (deterministic, no float atomics).  RoPE partners (i, i + h/2) and SwiGLU
//     partners (gate_f, up_f) sit in the same block, so the epilogue of a row pair needs no other workgroup.
//   * What a phase boundary costs beyond the exchange is instructions: the two wavefronts of a SIMD issue theirs in turn.
//     With one body for all norms, MLPs and phases a wavefront executed 700 scalar and 800 vector instructions per phase,
//     and 300 to 430 scalar registers lived in lanes of vector registers.  Now norm and MLP kind are template arguments,
//     every phase is code of its own that loads what it needs of the arguments when it starts (55 to 89 such lanes here, in
//     k_step 38 to 48 with eight wavefronts and 75 to 113 with four), words are requested two at a time through buffer
//     descriptors and without branches, and a wavefront polls as one.  With that, with requests that no hidden wait holds up,
//     and with workgroups of four wavefronts, per call: 4 layers of GPT-2 with 3 messages 199 -> 140 us, TinyLlama starter with
//     4 634 -> 572, 8 layers of the 7B shape with 8 1027 -> 956, of the 8B shape with 16 and 6144 positions 1502 -> 1390; one
//     message (k_step): 4 fp32 GPT-2 layers with output layers 202 -> 149, 8 of the 7B shape 762 -> 697.
//   * Vectors that feed a product cross workgroups as bf16 PAIRS with the writing phase's counter in one 8-byte
//     word, already multiplied by the gain of the RMSNorm that follows (1/rms is applied to the finished products;
//     the sum of squares travels as one partial per workgroup and message).  Bytes exchanged per message are half
//     those of k_step's (float, counter) words, which matters now that 16 messages share a pass.  A vector kind is
//     ONE array for the whole launch, laid out for the loads of the matrix instruction's second operand (vec_word), and no
//     line carries room for messages the launch does not have.
//   * The residual stream never leaves the workgroup that owns its rows: it stays in LDS for the whole launch.
//   * Products whose input is the d-sized normalised vector (QKV, MLP up) keep each wavefront's column slice of all
//     messages in registers for all the blocks of the phase; the others (output projection, MLP down: one block per
//     workgroup at the benchmark shapes, a long inner dimension) split the inner dimension among workgroups, so
//     that a workgroup reads a fraction of the vectors, and exchange 16 x 16 partial results (split, below).
// Needs bf16 storage and widths that are multiples of 32; other shapes keep one pass per message.  With LayerNorm the vectors still travel as x * gain: the mean and the norm's bias enter the finished
// products through two precomputed vectors per matrix (W g and W b), see BatchArgs.
//
// step_batch_ln*.hip and step_batch_rms*.hip compile it for one norm each (MDI_BATCH_LN), and for workgroups of eight and (_w4) of
// four wavefronts (MDI_STEP_WAVES).
#include "step_mfma.h"

namespace mdi {
namespace MDI_STEP_CAT(step_w, MDI_STEP_WAVES) {

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
// Waits until both words of all of a thread's pieces carry the counter `tag`; ask() asks for the pieces again.
template <int N, typename ASK>
__device__ __forceinline__ void await_two(u32x4 (&raw)[N], const ASK& ask, bool live, unsigned tag, int spin_limit, int* err) {
  poll_while([&]() {
    uint32_t bad = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) bad |= (raw[i].y ^ tag) | (raw[i].w ^ tag);
    return live && bad != 0;
  }, ask, spin_limit, err);
}
// Eight column steps of 16 weight rows as the matrix instruction's first operand: lane (i = l mod 16, kg = l div 16) takes
// 16 bytes of row i.  off: the lane's offset; `uniform`: the first row's and column's; n: steps there are.
// Always eight loads, so that the compiler can tell how many are on their way; those past the last step read nothing.  (Two
// cases, one of them without the choice per step, make it copy what the first has loaded, and wait for it.)
__device__ __forceinline__ void w_issue(Tile& t, Buffer b, uint32_t off, uint32_t uniform, int n) {
  uniform = __builtin_amdgcn_readfirstlane(n > 0 ? uniform : 0u);   // (what lies outside is told by off + uniform not exceeding 32 bits)
#pragma unroll
  for (int s = 0; s < 8; ++s) t.r[s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)((s < n ? off : kNowhere) + s * 64), (int)uniform, 0));
}
__device__ __forceinline__ f32x4 mac(const u32x4& w, const u32x4& v, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, v), acc, 0, 0, 0);
}

constexpr int kWatchWords = 2048;
constexpr int kTiles = 2;              // weight tiles a wavefront has on their way
constexpr int kResSteps = 16;          // column steps a wavefront can keep: widths up to 8 * 16 * 32 = 4096
// Eight steps of a normed product, the second operand in registers; n as in w_issue.
template <int HALF>
__device__ __forceinline__ void res_compute(const Tile& t, const u32x4 (&Bv)[kResSteps], int n, f32x4& acc) {
  if (n >= 8) {
#pragma unroll
    for (int s = 0; s < 8; ++s) acc = mac(t.r[s], Bv[HALF * 8 + s], acc);
  } else {
#pragma unroll
    for (int s = 0; s < 7; ++s)
      if (s < n) acc = mac(t.r[s], Bv[HALF * 8 + s], acc);
  }
}
// Eight steps of a split product, the second operand in LDS as [group of 8 columns][message ^ (group mod 16)]; vb: the
// lane's byte offset of step s = 0 .. 3 of every four.
__device__ __forceinline__ void ks_compute(const Tile& t, const char* Bs, const uint32_t (&vb)[4], int n, f32x4& acc) {
  auto v = [&](int s) __attribute__((always_inline)) { return *reinterpret_cast<const u32x4*>(Bs + vb[s & 3] + (s >> 2) * 4096); };
  if (n >= 8) {
#pragma unroll
    for (int s = 0; s < 8; ++s) acc = mac(t.r[s], v(s), acc);
  } else {
#pragma unroll
    for (int s = 0; s < 7; ++s)
      if (s < n) acc = mac(t.r[s], v(s), acc);
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

// Where pair `pair` of message j stands in an exchange vector: [step of 16 pairs][half][group][message][pair of the half],
// a group being the 4 pairs (8 columns) that a lane of the matrix instruction takes and a half two of them.  So what the
// lanes of a wavefront ask for with one instruction - a half of a step, 16 bytes a lane - is one contiguous piece of memory.
// With the 4 pairs of a group next to each other, 32 bytes a lane in two instructions, each instruction touched all lines of
// the step and used half of every one.
__device__ __forceinline__ int vec_word(int pair, int j, int m) {
  return ((((((pair >> 4) << 1) + ((pair >> 1) & 1)) * 4 + ((pair >> 2) & 3)) * m + j) << 1) + (pair & 1);
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
      st_pair(S.ob + vec_word((head * h + e) >> 1, S.msg, S.n_msg), pack_bf16x2(o0 / l, o1 / l), wtag);
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
    st_pair(S.ob + vec_word((head * h + e) >> 1, S.msg, S.n_msg), pack_bf16x2(o0 / l, o1 / l), wtag);
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
  const void* in[kMaxBatch];
  void* out[kMaxBatch];
  long kv_off[kMaxBatch];
  long tok[kMaxBatch];
  int pos[kMaxBatch], item_lo[kMaxBatch];
};

// Element `row` of message j's input vector (the token's embedding plus learned position, or the previous stage's activation).
__device__ __forceinline__ float batch_input(const BatchArgs& a, const BatchLds& sl, int j, int row) {
  if (a.in_kind == IN_TOKEN) {
    float v = bf16_to_f32(((const MDI_GLOBAL bf16_t*)a.wte)[sl.tok[j] * a.d + row]);
    if (a.wpe) v += bf16_to_f32(((const MDI_GLOBAL bf16_t*)a.wpe)[(long)sl.pos[j] * a.d + row]);
    return v;
  }
  return bf16_to_f32(((const MDI_GLOBAL bf16_t*)sl.in[j])[row]);
}

// Sums over the eight lanes of a message's row pairs, published by the first of them.  Workgroup wg's share is word wg of a
// message's row; the words from nwg to the row's end are published too, as zeros, so that readers need not tell them apart.
__device__ __forceinline__ void publish_sum(float v, int p, tagged_t* row, int wg, int nwg, unsigned tag) {
  v = dpp_add<kDppXor1, 0xF>(v); v = dpp_add<kDppXor2, 0xF>(v); v = dpp_add<kDppHalfMirror, 0xF>(v);
  if (p == 0)
    for (int w = wg; w < kBatchWgs; w += nwg) st_tag(row + w, w == wg ? v : 0.f, tag);
}

// G query heads per attention work item; kScoresOnMfma: see Attn4 (G = 4).
template <int G, bool kScoresOnMfma, bool kLn, bool kSwiglu>
__global__ __launch_bounds__(kStepThreads) __attribute__((amdgpu_waves_per_eu(kStepWaves / 4, kStepWaves / 4))) void k_step_batch(BatchArgs a0) {
  typedef bf16_t WT;
  extern __shared__ float smem[];
  __shared__ BatchLds sl;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = blockIdx.x, nwg = a0.nwg, m = a0.m;
  int* s_flag = lds_flag();
  float* rscale = smem + 32;                     // [16] 1/rms (LayerNorm: 1/std) of every message's vector in the normed products
  float* rshift = smem + 64;                     // [16] LayerNorm: (mean - centre) / std of every message's vector
  float* rcen = smem + 80;                       // [16] LayerNorm: the centre the vectors are published around (see below)
  float* xres = smem + kBatchLdsXres;            // residual rows this workgroup owns: [16 rows][16 messages]
  float* part = smem + kBatchLdsPart;            // the wavefronts' partial products [block][wavefront][lane][4]; attention scratch

  if (threadIdx.x == 0) s_flag[kFailed] = 0;
  if ((int)threadIdx.x < m) {                    // a lane per message
    const int j = threadIdx.x;
    const BatchArgs& a = args_again<BatchArgs>();
    const MDI_GLOBAL BatchSlot& S = *(const MDI_GLOBAL BatchSlot*)&a.s[j];
    sl.in[j] = S.in; sl.out[j] = S.act_out; sl.kv_off[j] = S.kv_tok_off; sl.pos[j] = S.pos; sl.item_lo[j] = S.item_lo;
    sl.tok[j] = a.in_kind == IN_TOKEN ? checked_token(S.in, 0, a.vocab, a.err) : 0;
    if (wg == 0 && S.table_entry) *S.table_entry = S.new_page;      // for later launches: no position before the newest lies on a page that starts now
    rcen[j] = 0.f;
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
  if constexpr (kLn) {
    const int lane = threadIdx.x & 63;
    for (int j = wave; j < m; j += kStepWaves) {
      float u = 0.f;
      for (int r0 = lane; r0 < a0.d; r0 += 512) {    // eight loads in flight
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = batch_input(a0, sl, j, min(r0 + 64 * k, a0.d - 1));
#pragma unroll
        for (int k = 0; k < 8; ++k) u += r0 + 64 * k < a0.d ? v[k] : 0.f;
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) u += __shfl_xor(u, off, 64);
      if (lane == 0) rcen[j] = u / (float)a0.d;
    }
    __syncthreads();
  }
  {
    // item (message j, row pair p) of the block of 16 rows this workgroup owns: eight neighbouring lanes share a message
    const BatchArgs& a = args_again<BatchArgs>();
    const int e = threadIdx.x, j = e >> 3, p = e & 7, r0 = wg * 16 + 2 * p;
    if (e < 8 * m) {
      float s2 = 0.f, s1 = 0.f;
      if (r0 < a.d) {
        const float x0 = batch_input(a, sl, j, r0), x1 = batch_input(a, sl, j, r0 + 1);
        float* xr = xres + 2 * p * 16 + j;
        xr[0] = x0; xr[16] = x1;
        const MDI_GLOBAL float* gain = (const MDI_GLOBAL float*)a.l0.ln1_g;
        st_pair(a.xn[0] + vec_word(r0 >> 1, j, m), pack_bf16x2((x0 - rcen[j]) * gain[r0], (x1 - rcen[j]) * gain[r0 + 1]), a.epoch0);
        s2 = x0 * x0 + x1 * x1; s1 = x0 + x1;
      }
      publish_sum(s2, p, a.ssq[0] + j * kBatchWgs, wg, nwg, a.epoch0);
      if constexpr (kLn) publish_sum(s1, p, a.ssum[0] + j * kBatchWgs, wg, nwg, a.epoch0);
    }
  }
  __syncthreads();

  // The page numbers of this workgroup's first attention item's first two tiles: the same in every layer, and in every layer
  // a round trip before the first key can be asked for.
  constexpr int kPages = kScoresOnMfma ? 1 : kTile;
  int page0A[kPages] = {}, page0B[kPages] = {};
  auto item_of = [&](int item, int& slot) __attribute__((always_inline)) {
    const BatchArgs& a = args_again<BatchArgs>();
    const int lane = threadIdx.x & 63;
    slot = __popcll(__ballot(lane < m && item >= sl.item_lo[min(lane, m - 1)])) - 1;
    return item - a.s[slot].item_lo;
  };
  if (wg < a0.n_items) {
    const BatchArgs& a = args_again<BatchArgs>();
    int slot;
    const int at = item_of(wg, slot), lane = threadIdx.x & 63;
    const BatchView V = view_of(a, slot, a.ob);
    const AttnGeo ga = make_attn_geo<WT, G>(a, V, at, wave, lane);
    if constexpr (kScoresOnMfma) {
      Attn4 s4;
      s4.n_t = max(ga.s1p - ga.s0 + 15, 0) >> 4;
      page0A[0] = attn4_page(ga, s4, V, 0, wave); page0B[0] = attn4_page(ga, s4, V, 1, wave);
    } else {
      attn_pages(page0A, ga, a, V, 0, wave); attn_pages(page0B, ga, a, V, 1, wave);
    }
  }

  const int ks_q = wg / a0.str_S, ks_s = wg - ks_q * a0.str_S;
  long w_off = 0, kv_off = 0, nc_off = 0;        // bytes from the first layer's matrices / pages / corrections to this layer's
  unsigned epoch = a0.epoch0;                    // what the phase that runs expects its input's words to carry; it writes epoch + 1

#pragma nounroll
  for (int layer = 0; layer < a0.n_layer; ++layer) {
    // Every kind of phase keeps its registers to itself (tiles in flight, the second operand, attention state are
    // declared inside it and given a value on every path), so that the compiler sees them dead elsewhere.
    // Each first issues the requests that depend on nothing another workgroup writes; they are on their way
    // while the words of the phase before arrive.  The epilogue's own operands (gains, biases, angles) are among
    // them: a thread keeps those of its first item, fetched again they would cost a round trip at the phase's end.
    // Per-lane addresses and epilogue indexes do not change from phase to phase; computed once outside the loops they
    // would occupy dozens of registers for the whole launch, so they are derived from a thread index the compiler cannot see
    // through and are recomputed where they are used.

    // ---- a product whose second operand stays in registers: this wavefront's column slice of every message, as
    // published, bf16 pairs of x * gain.
    auto normed = [&](auto ph_const) __attribute__((always_inline)) -> bool {
      constexpr int ph = decltype(ph_const)::value;
      constexpr bool up = ph == PH_UP, quads = up && kSwiglu;
      const BatchArgs& a = args_again<BatchArgs>();
      const BatchProduct& P = a.pr[ph == PH_QKV ? 0 : 2];
      const unsigned wtag = epoch + 1;
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, kg = lane >> 4, n = lane & 15;
      bstamp(a, layer, ph, 0);
      const int R = P.R, half = R >> 1, r_sh = R == 16 ? 4 : 3, rb = P.row_bytes, N = P.N;
      const int nb = P.nb_q + (wg < P.nb_r ? 1 : 0);               // this workgroup's blocks: block lb * nwg + wg of the matrix
      // The columns are cut into one slice per wavefront; which wavefront takes which slice rotates with the workgroup,
      // so that at any moment the workgroups read different parts of the messages' vectors (every workgroup walks the
      // same vectors: in step they would all queue up at the same few memory channels).
      const int slice = (wave + wg) & (kStepWaves - 1), ks0 = slice * a.res_c, nks = max(0, min(a.res_c, (a.d >> 5) - ks0));
      // Row of the matrix that row i (< R) of a block stands for.  QKV: R/2 consecutive rows of a head's first half followed by
      // their RoPE partners in the second half (head sizes are powers of two); otherwise row block * R + i.
      const int hh_sh = 30 - __builtin_clz(a.h);                    // log2(h / 2)
      auto first_row = [&](int block) __attribute__((always_inline)) {
        if (up) return block << r_sh;
        const int hsh = r_sh - 1, bsh = hh_sh - hsh;                // log2 of the rows a block takes of a half head, of the blocks per head
        return ((block >> bsh) << (hh_sh + 1)) + ((block & ((1 << bsh) - 1)) << hsh);
      };
      // ---- requests
      const Buffer sqb = buffer_at(up ? a.ssq[1] : a.ssq[0]), smb = buffer_at(kLn ? (up ? a.ssum[1] : a.ssum[0]) : nullptr);
      const bool long_vec = (a.d >> 1) * m > kWatchWords;
      uint32_t gate = 0;                                            // (the counter alone: half a loaded pair left unused is reused, and waited for)
      auto ask_gate = [&]() __attribute__((always_inline)) {
        gate = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(sqb, (int)fresh(long_vec && tid < kBatchWgs ? (uint32_t)tid * 8u + 4u : kNowhere), 0, kAgentScope);
      };
      ask_gate();
      // the sums: 32 threads per message (16 in a workgroup of four wavefronts), all words at once
      constexpr int kSumThreads = kStepThreads / kMaxBatch, kSumPieces = kBatchWgs / 2 / kSumThreads;
      static_assert(kStepThreads >= kBatchWgs, "a thread for every word that is watched");
      const int sj = tid / kSumThreads, sc = tid % kSumThreads;
      const bool sums = sj < m;
      const uint32_t s_off = sums ? (uint32_t)(sj * kBatchWgs + 2 * sc) * 8u : kNowhere;
      u32x4 sq[kSumPieces], sm[kSumPieces];
      auto ask_sq = [&]() __attribute__((always_inline)) {
        const uint32_t o = fresh(s_off);
#pragma unroll
        for (int k = 0; k < kSumPieces; ++k) sq[k] = ld_two(sqb, o + k * kSumThreads * 16, 0);
      };
      auto ask_sm = [&]() __attribute__((always_inline)) {
        const uint32_t o = fresh(s_off);
#pragma unroll
        for (int k = 0; k < kSumPieces; ++k) sm[k] = ld_two(smb, o + k * kSumThreads * 16, 0);
      };
      ask_sq();
      if constexpr (kLn) ask_sm();
      // the epilogue's items: (block, message, row pair or quad of rows), the latter neighbours
      constexpr int kQ = quads ? 1 : 0;
      const int n_sh = r_sh - 1 - kQ, n_items = (nb << n_sh) * m;
      struct Item { int j, p, lb, r0, r1; };
      auto item_at = [&](int e) __attribute__((always_inline)) {
        Item it;
        const int x = e >> n_sh;
        it.p = e & ((1 << n_sh) - 1);
        it.lb = (int)__umulhi((unsigned)x, a.m_magic);             // x / m, see BatchArgs
        it.j = x - it.lb * m;
        const int f = first_row(it.lb * nwg + wg);
        it.r0 = up ? f + ((2 << kQ) * it.p) : f + it.p;
        it.r1 = up ? it.r0 + 1 : it.r0 + (2 << hh_sh >> 1);
        return it;
      };
      struct Ops { float c, s, b0, b1, n[4]; };
      const Buffer biasb = buffer_at(P.bias ? (const char*)P.bias + w_off : nullptr);
      // LayerNorm corrections of this phase's product: [W g | W b], N floats each (QKV's first, then the up product's)
      const float* ncp = kLn ? (const float*)((const char*)a.nc0 + nc_off) + (up ? 2 * a.pr[0].N : 0) : nullptr;
      const Buffer n0b = buffer_at(ncp), n1b = buffer_at(kLn ? ncp + N : nullptr);
      // The table of angles may be longer than a descriptor reaches (2^31 bytes are 4 million positions of heads of 128), so
      // its entries are loaded by address.  Without a table: any 8 bytes, not used.
      const MDI_GLOBAL u32x2* angles = (const MDI_GLOBAL u32x2*)(a.rope ? (const void*)a.rope : P.W);
      const long angle_mask = a.rope ? -1L : 0L;
      auto ops_of = [&](const Item& it, bool own) __attribute__((always_inline)) {
        Ops o{};
        if constexpr (quads) return o;
        const uint32_t o0 = own ? (uint32_t)it.r0 * 4u : kNowhere, o1 = own ? (uint32_t)it.r1 * 4u : kNowhere;
        o.b0 = ld_f32(biasb, o0); o.b1 = ld_f32(biasb, o1);
        if constexpr (!up) {
          const u32x2 cs = angles[(((long)sl.pos[it.j] << hh_sh) + (it.r0 & ((1 << hh_sh) - 1))) & angle_mask];   // (no item: item 0's)
          o.c = __uint_as_float(cs.x); o.s = __uint_as_float(cs.y);
        }
        if constexpr (kLn) { o.n[0] = ld_f32(n0b, o0); o.n[1] = ld_f32(n0b, o1); o.n[2] = ld_f32(n1b, o0); o.n[3] = ld_f32(n1b, o1); }
        return o;
      };
      Ops ops{};
      if constexpr (!quads) {
        const Item it = item_at(tid < n_items ? tid : 0);
        ops = ops_of(it, tid < n_items && it.r1 < N);
      }
      // The vectors: steps of 32 columns, 32 bytes per lane and step, eight steps at a time; steps past the slice repeat its
      // last one (the second four read nothing if the slice has no more than four).
      const bool two = nks > 8, half8 = nks > 4;                    // two tiles per block, else one
      const Buffer vb = buffer_at(up ? a.xn[1] : a.xn[0]);
      const bool has = n < m && nks > 0;
      const uint32_t v_off = has ? (uint32_t)(kg * m + n) * 16u : kNowhere;
      const uint32_t v_step = (uint32_t)m * 128u, v_base = (uint32_t)ks0 * v_step;
      u32x4 raw[16];
      auto ask_vec = [&](int k0) __attribute__((always_inline)) {
        const uint32_t o = fresh(v_off), o4 = half8 ? o : kNowhere;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t u = v_base + (uint32_t)max(min(k0 + k, nks - 1), 0) * v_step;
          raw[2 * k] = ld_two(vb, k < 4 ? o : o4, u); raw[2 * k + 1] = ld_two(vb, k < 4 ? o : o4, u + (v_step >> 1));
        }
      };
      auto await_vec = [&](int k0) __attribute__((always_inline)) {
        poll_while([&]() {
          uint32_t bad = 0, bad4 = 0;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            bad |= (raw[k].y ^ epoch) | (raw[k].w ^ epoch);
            bad4 |= (raw[8 + k].y ^ epoch) | (raw[8 + k].w ^ epoch);
          }
          return has && (bad | (half8 ? bad4 : 0u)) != 0;
        }, [&]() { ask_vec(k0); }, a.spin_limit, a.err);
      };
      ask_vec(0);
      // the first two tiles of weights
      Tile T[kTiles];
      const Buffer wb = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)P.W + w_off), 0, (int)P.bytes, 0x00020000);
      const int wi = n & (R - 1);
      const uint32_t w_lane = (uint32_t)((up ? wi : (wi & (half - 1)) + (wi >= half ? 1 << hh_sh : 0)) * rb + (kg << 4));
      auto issue = [&](Tile& t, int lb, int h8) __attribute__((always_inline)) {
        w_issue(t, wb, w_lane, (uint32_t)(first_row(lb * nwg + wg) * rb + ks0 * 64 + h8 * 512), lb < nb ? nks - 8 * h8 : 0);
      };
#pragma unroll
      for (int k = 0; k < kTiles; ++k) issue(T[k], two ? k >> 1 : k, two ? k & 1 : 0);
      bstamp(a, layer, ph, 1);
      // ---- Vectors of more than kWatchWords words are looked at only after every workgroup's first sum of
      // squares (which it stores last) is there: 256 workgroups that watch 32 KB each crowd out the stores they wait
      // for (TinyLlama, 4 messages: 629 us, ungated 644; the 7B shape with 8: 979 and 975).
      if (long_vec) {
        if (wave < kBatchWgs / 64) poll_while([&]() { return gate != epoch; }, ask_gate, a.spin_limit, a.err);
        __syncthreads();
      }
      float sum2 = 0.f, sum1 = 0.f;                                 // this thread's share of its message's sums
      await_two(sq, ask_sq, sums, epoch, a.spin_limit, a.err);
      if constexpr (kLn) await_two(sm, ask_sm, sums, epoch, a.spin_limit, a.err);
#pragma unroll
      for (int k = 0; k < kSumPieces; ++k) {
        sum2 += __uint_as_float(sq[k].x) + __uint_as_float(sq[k].z);
        if constexpr (kLn) sum1 += __uint_as_float(sm[k].x) + __uint_as_float(sm[k].z);
      }
      asm volatile("" : "+v"(sum2), "+v"(sum1));                    // (added up here: left to where they are used, the words stay in registers)
      u32x4 Bv[kResSteps];
      auto take = [&](auto first) __attribute__((always_inline)) {
        constexpr int k0 = decltype(first)::value;
        await_vec(k0);
#pragma unroll
        for (int k = 0; k < 8; ++k) Bv[k0 + k] = u32x4{raw[2 * k].x, raw[2 * k].z, raw[2 * k + 1].x, raw[2 * k + 1].z};
      };
      take(std::integral_constant<int, 0>());
      if (two) {
        ask_vec(8);
        take(std::integral_constant<int, 8>());
      } else {
#pragma unroll
        for (int k = 8; k < kResSteps; ++k) Bv[k] = Bv[0];
      }
      bstamp(a, layer, ph, 2);
      // ---- the stream: two tiles in flight, each multiplied while the other's rows arrive
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      f32x4* pw = reinterpret_cast<f32x4*>(part) + (wave << 6) + lane;
      auto put = [&](int lb) __attribute__((always_inline)) { pw[lb * (kStepWaves * 64)] = acc; acc = f32x4{0.f, 0.f, 0.f, 0.f}; };
      if (two) {
        constexpr int kD = kTiles / 2;                              // blocks on their way
        int lb = 0;
#pragma nounroll
        for (; lb + kD < nb; lb += kD) {
#pragma unroll
          for (int b = 0; b < kD; ++b) {
            res_compute<0>(T[2 * b], Bv, nks, acc);
            issue(T[2 * b], lb + b + kD, 0);
            res_compute<1>(T[2 * b + 1], Bv, nks - 8, acc);
            issue(T[2 * b + 1], lb + b + kD, 1);
            put(lb + b);
          }
        }
#pragma unroll
        for (int b = 0; b < kD; ++b)
          if (lb + b < nb) { res_compute<0>(T[2 * b], Bv, nks, acc); res_compute<1>(T[2 * b + 1], Bv, nks - 8, acc); put(lb + b); }
      } else {
        int lb = 0;
#pragma nounroll
        for (; lb + kTiles < nb; lb += kTiles) {
#pragma unroll
          for (int b = 0; b < kTiles; ++b) {
            res_compute<0>(T[b], Bv, nks, acc);
            issue(T[b], lb + b + kTiles, 0);
            put(lb + b);
          }
        }
#pragma unroll
        for (int b = 0; b < kTiles; ++b)
          if (lb + b < nb) { res_compute<0>(T[b], Bv, nks, acc); put(lb + b); }
      }
      bstamp(a, layer, ph, 3);
      // 1/rms of every message.  The shares of all workgroups have been seen before anything of this phase is stored
      // (see the top of the file).
      auto over_threads = [&](float v) __attribute__((always_inline)) {
        v = dpp_add<kDppXor1, 0xF>(v); v = dpp_add<kDppXor2, 0xF>(v); v = dpp_add<kDppHalfMirror, 0xF>(v); v = dpp_add<kDppMirror, 0xF>(v);
        return kSumThreads == 32 ? v + __shfl_xor(v, 16, 64) : v;
      };
      sum2 = over_threads(sum2);
      if constexpr (kLn) sum1 = over_threads(sum1);
      if (sums && sc == 0) {
        if constexpr (!kLn) {
          rscale[sj] = 1.f / sqrtf(sum2 / (float)a.d + a.eps);
        } else {
          const float mean = sum1 / (float)a.d;
          const float rstd = 1.f / sqrtf(fmaxf(sum2 / (float)a.d - mean * mean, 0.f) + a.eps);
          rscale[sj] = rstd; rshift[sj] = rstd * (mean - rcen[sj]);
          rcen[sj] = mean;                                          // what the next norm's vector is published around
        }
      }
      loads_done();
      __syncthreads();                                              // every wavefront's partial products are in LDS
      bstamp(a, layer, ph, 4);
      // ---- epilogue: one thread per (block, message, row pair or quad)
      for (int e = tid; e < n_items; e += kStepThreads) {
        const Item it = item_at(e);
        const int j = it.j, p = it.p, lb = it.lb, r0 = it.r0, r1 = it.r1;
        if (quads) {
          // rows (4q .. 4q + 3) = (gate_f, up_f, gate_f+1, up_f+1): one lane of every wavefront's result holds all four
          if (r0 >= N) continue;
          const float* pp = part + ((lb * kStepWaves) << 8) + (((p << 4) + j) << 2);
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int w = 0; w < kStepWaves; ++w) { const f32x4 t = *reinterpret_cast<const f32x4*>(pp + (w << 8)); v += t; }
          v *= rscale[j];
          if constexpr (kLn) {
            const MDI_GLOBAL float* nc = (const MDI_GLOBAL float*)ncp;
            const float sh = rshift[j];
            v.x += nc[N + r0] - sh * nc[r0]; v.y += nc[N + r0 + 1] - sh * nc[r0 + 1];
            v.z += nc[N + r0 + 2] - sh * nc[r0 + 2]; v.w += nc[N + r0 + 3] - sh * nc[r0 + 3];
          }
          st_pair(a.ub + vec_word(r0 >> 2, j, m), pack_bf16x2(silu_f(v.x) * v.y, silu_f(v.z) * v.w), wtag);
          continue;
        }
        if (up && r0 >= N) continue;
        if (e != tid) ops = ops_of(it, r1 < N);
        float v0 = part_sum(part, lb, up ? 2 * p : p, j) * rscale[j], v1 = part_sum(part, lb, up ? 2 * p + 1 : p + half, j) * rscale[j];
        if constexpr (kLn) { v0 += ops.n[2] - rshift[j] * ops.n[0]; v1 += ops.n[3] - rshift[j] * ops.n[1]; }
        v0 += ops.b0; v1 += ops.b1;
        if (up) {
          const bool tanh_form = a.mlp_kind == MDI_MLP_GELU_TANH;
          st_pair(a.ub + vec_word(r0 >> 1, j, m), pack_bf16x2(tanh_form ? gelu_tanh_f(v0) : gelu_erf_f(v0), tanh_form ? gelu_tanh_f(v1) : gelu_erf_f(v1)), wtag);
          continue;
        }
        const int head = r0 >> (hh_sh + 1), i = r0 & ((2 << hh_sh) - 1);
        if (a.rope && head < a.H + a.K) {
          const float t0 = v0 * ops.c - v1 * ops.s, t1 = v0 * ops.s + v1 * ops.c;
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
          MDI_GLOBAL WT* dst = (MDI_GLOBAL WT*)((char*)a.l0.kv + kv_off) + sl.kv_off[j] + (long)(kvh * 2 + (is_v ? 1 : 0)) * a.pt_h + i;
          dst[0] = f32_to_bf16(v0); dst[1 << hh_sh] = f32_to_bf16(v1);
          tagged_t* kn = (tagged_t*)(base + a.off_knew) + (is_v ? a.K * a.h : 0) + kvh * a.h + i;
          st_tag(kn, bf16_to_f32(f32_to_bf16(v0)), wtag); st_tag(kn + (1 << hh_sh), bf16_to_f32(f32_to_bf16(v1)), wtag);
        }
      }
      // ---- the partial products in LDS have been read
      bstamp(a, layer, ph, 5);
      __syncthreads();
      bstamp(a, layer, ph, 6);
      epoch = wtag;
      return __builtin_amdgcn_readfirstlane(s_flag[kFailed]) == 0;    // (else a bounded wait expired: everybody else's will, too)
    };

    // ---- attention: one work item = (message, head group, context split); items dealt round-robin
    auto attention = [&]() __attribute__((always_inline)) -> bool {
      constexpr int ph = PH_ATTN;
      const BatchArgs& a = args_again<BatchArgs>();
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63;
      const void* kv = (const char*)a.l0.kv + kv_off;
      bstamp(a, layer, ph, 0);
      for (int item = wg; item < a.n_items; item += nwg) {
        if (item != wg) __syncthreads();                            // the records in LDS have been read
        int slot;
        const int at = item_of(item, slot);
        const BatchView V = view_of(a, slot, a.ob);
        const AttnGeo ga = make_attn_geo<WT, G>(a, V, at, wave, lane);
        AttnState<WT, G> st;
        AttnAsk<WT> ask;
        Tile A, B;
        attn_ask<WT, G>(ask, ga, a, V, wave, tid);
        if constexpr (kScoresOnMfma) {
          Attn4 s4;
          s4.n_t = max(ga.s1p - ga.s0 + 15, 0) >> 4;
          int pgA = page0A[0], pgB = page0B[0];
          if (item != wg) { pgA = attn4_page(ga, s4, V, 0, wave); pgB = attn4_page(ga, s4, V, 1, wave); }
          attn4_issue(A, pgA, ga, s4, a, V, kv, 0, wave, lane); attn4_issue(B, pgB, ga, s4, a, V, kv, 1, wave, lane);
          if (item == wg) bstamp(a, layer, ph, 1);
          attn_begin<WT, G>(st, ask, ga, a, V, part, wave, epoch, tid);
          if (item == wg) bstamp(a, layer, ph, 2);
          attn4_stream(s4, st, A, B, pgA, pgB, ga, a, V, kv, wave, lane, part);
        } else {
          int pgA[kTile], pgB[kTile];
#pragma unroll
          for (int k = 0; k < kTile; ++k) { pgA[k] = page0A[k % kPages]; pgB[k] = page0B[k % kPages]; }
          if (item != wg) { attn_pages(pgA, ga, a, V, 0, wave); attn_pages(pgB, ga, a, V, 1, wave); }
          attn_issue<WT>(A, pgA, ga, a, V, kv, 0, wave); attn_issue<WT>(B, pgB, ga, a, V, kv, 1, wave);
          if (item == wg) bstamp(a, layer, ph, 1);
          attn_begin<WT, G>(st, ask, ga, a, V, part, wave, epoch, tid);
          if (item == wg) bstamp(a, layer, ph, 2);
          const int nte = ((ga.n_k + kTile - 1) / kTile + 1) & ~1;
          attn_stream<WT, G>(st, A, B, pgA, pgB, ga, a, V, kv, nte, wave, part);
        }
        loads_done();
        if (item == wg) bstamp(a, layer, ph, 3);
        attn_to_lds<WT, G>(st, ga, a.h, part, wave);
        attn_finish_pairs<G>(ga, a, V, part, s_flag, epoch, tid);
      }
      // ---- the records in LDS have been read
      bstamp(a, layer, ph, 5);
      __syncthreads();
      bstamp(a, layer, ph, 6);
      ++epoch;
      return __builtin_amdgcn_readfirstlane(s_flag[kFailed]) == 0;
    };

    // ---- a product whose inner dimension is split among workgroups.  Every workgroup used to read the whole
    // vector of all messages for its one block of rows: 256 copies of it through the dies' L2s, twice the bytes of
    // the matrix itself in the MLP down projection.  Here workgroup (q, s) takes column slice s of the q-th group of row
    // blocks, one block per wavefront: it reads 1 / S of the vector - once, validated, into LDS, from
    // where its wavefronts take the matrix instruction's second operand - and hands the 16 x 16 partial result
    // of every block, as tagged words, to the workgroup that owns the block's residual rows, which adds the S partials
    // in slice order.
    auto split = [&](auto ph_const) __attribute__((always_inline)) -> bool {
      constexpr int ph = decltype(ph_const)::value;
      constexpr bool down = ph == PH_DOWN;
      const BatchArgs& a = args_again<BatchArgs>();
      const BatchProduct& P = a.pr[down ? 3 : 1];
      const unsigned wtag = epoch + 1;
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, kg = lane >> 4, n = lane & 15;
      bstamp(a, layer, ph, 0);
      const int rb = P.row_bytes, S = a.str_S, c = a.str_c[down ? 1 : 0], nblk = (a.d + 15) >> 4;
      const int ktot = rb >> 6, k0 = min(ks_s * c, ktot), nk = ks_q < a.str_groups ? max(0, min(c, ktot - ks_s * c)) : 0;   // column steps of the slice
      const int blk = ks_q * kStepWaves + wave;                     // this wavefront's block
      const bool has = ks_q < a.str_groups && blk < nblk, live = has && nk > 0;
      // the slice of every message's vector to LDS, by pieces of four columns of one message (see vec_word)
      const Buffer vb = buffer_at(down ? a.ub : a.ob);
      const int n_pieces = nk * 8 * m;
      const uint32_t v_base = (uint32_t)k0 * (uint32_t)m * 128u;
      constexpr int kAsk = 4;                                       // pieces of a thread that are asked for together
      u32x4 raw[2][kAsk];
      auto ask = [&](u32x4 (&r)[kAsk], int u) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kAsk; ++k) {
          const int uk = u + k * kStepThreads;
          r[k] = ld_two(vb, fresh(uk < n_pieces ? (uint32_t)uk * 16u : kNowhere), v_base);
        }
      };
      ask(raw[0], tid);
      ask(raw[1], tid + kAsk * kStepThreads);
      // the rows this workgroup owns: what their epilogue needs
      const int j = tid >> 3, p = tid & 7, r0 = wg * 16 + 2 * p;
      const bool mine = j < m && r0 < a.d, last = down && layer == a.n_layer - 1;
      const uint32_t o0 = mine ? (uint32_t)r0 * 4u : kNowhere;
      const Buffer biasb = buffer_at(P.bias ? (const char*)P.bias + w_off : nullptr);
      const Buffer gainb = buffer_at(last ? nullptr : down ? (const char*)a.l0.ln1_g + w_off + a.w_stride : (const char*)a.l0.ln2_g + w_off);
      auto two_at = [&](Buffer b) __attribute__((always_inline)) { return __builtin_amdgcn_raw_buffer_load_b64(b, (int)o0, 0, 0); };
      const u32x2 bias = two_at(biasb), gain = two_at(gainb);
      // weights
      Tile T[kTiles];
      const Buffer wb = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)P.W + w_off), 0, (int)P.bytes, 0x00020000);
      const uint32_t w_lane = (uint32_t)(n * rb + (kg << 4)), w_base = (uint32_t)(blk * 16 * rb + k0 * 64);
      auto issue = [&](Tile& t, int ti) __attribute__((always_inline)) { w_issue(t, wb, w_lane, w_base + ti * 512, live ? nk - ti * 8 : 0); };
#pragma unroll
      for (int k = 0; k < kTiles; ++k) issue(T[k], k);
      bstamp(a, layer, ph, 1);
      char* Bs = reinterpret_cast<char*>(part);
      auto stage = [&](u32x4 (&r)[kAsk], int u) __attribute__((always_inline)) {
        if (u - tid >= n_pieces) return;                            // uniform
        poll_while([&]() {
          bool bad = false;
#pragma unroll
          for (int k = 0; k < kAsk; ++k) bad |= u + k * kStepThreads < n_pieces && ((r[k].y ^ epoch) | (r[k].w ^ epoch)) != 0;
          return bad;
        }, [&]() { ask(r, u); }, a.spin_limit, a.err);
#pragma unroll
        for (int k = 0; k < kAsk; ++k) {
          const int uk = u + k * kStepThreads, x = (int)__umulhi((unsigned)uk, a.m_magic), nm = uk - x * m;   // x: (step, half, group)
          const int gi = ((x >> 3) << 2) + (x & 3);
          if (uk < n_pieces) *reinterpret_cast<u32x2*>(Bs + gi * 256 + ((nm ^ (gi & 15)) << 4) + ((x >> 2) & 1) * 8) = u32x2{r[k].x, r[k].z};
        }
      };
      for (int u = tid;;) {
        stage(raw[0], u);
        if (u - tid + 2 * kAsk * kStepThreads < n_pieces) ask(raw[0], u + 2 * kAsk * kStepThreads);
        stage(raw[1], u + kAsk * kStepThreads);
        u += 2 * kAsk * kStepThreads;
        if (u - tid >= n_pieces) break;
        ask(raw[1], u + kAsk * kStepThreads);
      }
      __syncthreads();
      bstamp(a, layer, ph, 2);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      if (live) {                                                   // uniform per wavefront
        uint32_t vl[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) { const int gi = s * 4 + kg; vl[s] = (uint32_t)(gi * 256 + ((n ^ gi) << 4)); }
        const char* bs = Bs;
        const int nt = (nk + 7) >> 3;
        int t = 0;
#pragma nounroll
        for (; t + kTiles < nt; t += kTiles) {
#pragma unroll
          for (int k = 0; k < kTiles; ++k) { ks_compute(T[k], bs + k * 8192, vl, 8, acc); issue(T[k], t + k + kTiles); }
          bs += kTiles * 8192;
        }
#pragma unroll
        for (int k = 0; k < kTiles; ++k) ks_compute(T[k], bs + k * 8192, vl, nk - (t + k) * 8, acc);
      }
      bstamp(a, layer, ph, 3);
      loads_done();
      // the partial of (block, slice), zeros from a slice without columns, to the block's owner
      const Buffer pb = buffer_at(a.ppart);
      {
        const uint32_t o = has && n < m ? (uint32_t)(kg * m + n) * 32u : kNowhere, u = has ? (uint32_t)((blk * S + ks_s) * m) * 128u : 0u;
        st_two(pb, o, u, acc[0], acc[1], wtag); st_two(pb, o + 16, u, acc[2], acc[3], wtag);
      }
      bstamp(a, layer, ph, 7);
      // ---- residual products: x += W v (+ bias) on the 16 rows this workgroup owns; what leaves is x times the gain
      // of the norm that follows, as bf16 pairs, and this workgroup's share of every message's sum of squares (every
      // workgroup's, also without rows: see the top of the file).  One lane per (message, row pair), which adds the S
      // partials in slice order.
      if (j < m) {
        float s2 = 0.f, s1 = 0.f;
        if (wg < nblk) {
          const uint32_t off = (uint32_t)((p >> 1) * m + j) * 32u + (uint32_t)(p & 1) * 16u;
          float d0 = 0.f, d1 = 0.f;
          for (int k0s = 0; k0s < S; k0s += 8) {
            u32x4 r[8];                                             // slices past the last repeat it
            auto ask_parts = [&]() __attribute__((always_inline)) {
              const uint32_t o = fresh(off);
#pragma unroll
              for (int k = 0; k < 8; ++k) r[k] = ld_two(pb, o, (uint32_t)((wg * S + min(k0s + k, S - 1)) * m) * 128u);
            };
            ask_parts();
            await_two(r, ask_parts, true, wtag, a.spin_limit, a.err);
#pragma unroll
            for (int k = 0; k < 8; ++k) { d0 += k0s + k < S ? __uint_as_float(r[k].x) : 0.f; d1 += k0s + k < S ? __uint_as_float(r[k].z) : 0.f; }
          }
          if (mine) {
            float* xr = xres + 2 * p * 16 + j;
            const float x0 = xr[0] + d0 + __uint_as_float(bias.x), x1 = xr[16] + d1 + __uint_as_float(bias.y);
            xr[0] = x0; xr[16] = x1;
            if (last) {
              MDI_GLOBAL bf16_t* y = (MDI_GLOBAL bf16_t*)sl.out[j] + r0;
              y[0] = f32_to_bf16(x0); y[1] = f32_to_bf16(x1);
            } else {
              st_pair((down ? a.xn[0] : a.xn[1]) + vec_word(r0 >> 1, j, m),
                      pack_bf16x2((x0 - rcen[j]) * __uint_as_float(gain.x), (x1 - rcen[j]) * __uint_as_float(gain.y)), wtag);
              s2 = x0 * x0 + x1 * x1; s1 = x0 + x1;
            }
          }
        }
        if (!last) {
          publish_sum(s2, p, (down ? a.ssq[0] : a.ssq[1]) + j * kBatchWgs, wg, nwg, wtag);
          if constexpr (kLn) publish_sum(s1, p, (down ? a.ssum[0] : a.ssum[1]) + j * kBatchWgs, wg, nwg, wtag);
        }
      }
      // ---- the vector's slice in LDS has been read
      bstamp(a, layer, ph, 5);
      __syncthreads();
      bstamp(a, layer, ph, 6);
      epoch = wtag;
      return __builtin_amdgcn_readfirstlane(s_flag[kFailed]) == 0;
    };

    if (!normed(std::integral_constant<int, PH_QKV>())) return;
    if (!attention()) return;
    if (!split(std::integral_constant<int, PH_OPROJ>())) return;
    if (!normed(std::integral_constant<int, PH_UP>())) return;
    if (!split(std::integral_constant<int, PH_DOWN>())) return;
    w_off += a0.w_stride; kv_off += a0.kv_stride; nc_off += 4 * a0.nc_stride;
  }
}

}  // namespace step_w<waves>

namespace MDI_STEP_CAT(step_w, MDI_STEP_WAVES) {
template <bool kLn, bool kSwiglu> const void* step_batch_kernel(int G, bool scores_on_mfma) {
  if (G == 4) return scores_on_mfma ? (const void*)k_step_batch<4, true, kLn, kSwiglu> : (const void*)k_step_batch<4, false, kLn, kSwiglu>;
  return G == 2 ? (const void*)k_step_batch<2, false, kLn, kSwiglu> : (const void*)k_step_batch<1, false, kLn, kSwiglu>;
}
}  // namespace step_w<waves>

// The kernel of a norm: G query heads per attention work item, their scores on the matrix cores (G = 4) or not, MLP kind.
template <> const void* step_batch_kernel<MDI_STEP_WAVES, MDI_BATCH_LN>(int G, bool scores_on_mfma, bool swiglu) {
  return swiglu ? MDI_STEP_CAT(step_w, MDI_STEP_WAVES)::step_batch_kernel<MDI_BATCH_LN, true>(G, scores_on_mfma) : MDI_STEP_CAT(step_w, MDI_STEP_WAVES)::step_batch_kernel<MDI_BATCH_LN, false>(G, scores_on_mfma);
}

}  // namespace mdi

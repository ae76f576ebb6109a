// Causal attention of a first visit (all T prompt positions of a sample at once; Alg. 1 round 0,
// Alg. 2 "first iteration") on the matrix cores: bf16 operands, fp32 scores, softmax and output
// accumulation.
//
// Everything is computed transposed, S^T = K Q^T and O^T = V^T P^T, because of where the matrix
// core leaves its results: with v_mfma_f32_32x32x16_bf16, register r of lane l is element
// (row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32).  In the transposed products a column is a
// query, so each lane owns one query: its running maximum, its sum and the rescaling of its output
// are plain per-lane scalars (lanes l and l + 32 share a query and exchange two numbers per block of
// keys), and P^T leaves the first product in exactly the register layout the second one wants as
// its B operand, without any data movement.  The values are needed with the key index
// contiguous (A operand of V^T P^T): they lie in LDS as they lie in memory, and ds_read_b64_tr_b16 transposes four keys x
// sixteen channels on the way to the registers.
//
// Keys and values are read where they live, in the sample's cache pages, those of this call as well as those of earlier
// pieces of the visit.  (Two kernels per layer and call used to lay them out for this one, values transposed: 10 us of a
// layer's 480 at 1024 positions of the 7B shape, 26 of 223 in pieces of 256: visits of 1024 3.63 -> 3.56 ms, in four
// pieces 7.16 -> 6.41 ms, 333 of TinyLlama 1.15 -> 1.07 ms, 6000 of the 8B shape 22.0 -> 22.4 ms on one machine.
// Transposing in registers on the way into LDS: 531 us a layer of 6000 positions, 490 as it is.)
#include "device_utils.h"
#include "visit_internal.h"

namespace mdi {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int BK = kFlashKeys;   // keys per step
constexpr float kRaise = 8.f;    // how far (in powers of two) a score may exceed its query's reference

typedef short i16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 read_transposed(const bf16_t* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)p));
}

// 2^x as the hardware gives it (the scores carry log2 e, see the launch)
__device__ __forceinline__ float exp2f_raw(float x) { return __builtin_amdgcn_exp2f(x); }

// A workgroup is NG groups of WQ wavefronts that work on the same 32 WQ queries; group g takes the key blocks
// NG i + g.  With more groups the longest workgroup (the last queries, which see every key) has fewer steps in a
// row and a SIMD holds two wavefronts; the groups' running (maximum, sum, output) are folded through LDS at the end,
// group 0 first, so the result does not depend on timing.  With one, two workgroups share a compute unit and nothing
// keeps them in step: one multiplies while the other takes exponentials.
// Where the chip is not full, a step takes 2.7 us whether a SIMD holds one wavefront or two (a chain of products, maxima,
// exponentials and products): what helps is fewer steps in a row and more workgroups, not less work in one.  (Bringing a
// head's keys and values into the L2 of the die beforehand: nothing.)
//
// What bounds it: a block of 64 keys is 32 matrix instructions (about 1000 cycles of a SIMD), half as much again on the vector
// ALUs (32 scores per lane: maximum, exponential, sum, conversion), and 32 KiB of LDS reads per wavefront, which take as long
// as the matrix instructions when all four SIMDs ask.
// 6000 positions of the 8B shape: 500 us a layer with a mask (four instructions a score) and a subtraction in every block and
// a rescaling wherever any of a wavefront's 32 queries found a new maximum, which is most blocks; 379 us (0.78 PFLOP/s) with
// the mask in the last blocks only, scores that come out relative, and a rescaling when it is needed.  1024 positions of the
// 7B shape 33 -> 28, pieces of 256 23 -> 20 us.  Heads that share keys on one die give 20 of it.
template <int HD, int NG, int WQ>
__global__ __launch_bounds__(WQ * 64 * NG, 2) void k_flash_prefill(FlashArgs a) {
  constexpr int BQ = 32 * WQ, GT = 64 * WQ;  // queries of a workgroup, threads of a group
  constexpr int KS = HD + 8;            // LDS row stride of a key (elements): 16 bytes of padding spread the rows over the banks
  constexpr int VR = HD + 32;           // LDS row stride of a key's values: 16 dwords past a multiple of 64 (heads of 64: 48), so that the
                                        // eight keys x 32 channels of a transposing read touch every bank twice
  constexpr int HT = HD / 32;           // 32-channel tiles of the output
  extern __shared__ __attribute__((aligned(16))) unsigned char flash_smem[];
  constexpr int KV = BK * KS + BK * VR;                 // elements of a key block and its values
  constexpr int NB = NG == 4 ? 1 : 2;                   // blocks per group: two of four groups would not fit

  const int tid = threadIdx.x & (GT - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // position inside the group
  const int grp = threadIdx.x / GT;
  bf16_t* bufs = (bf16_t*)flash_smem + grp * NB * KV;
  // Workgroups are handed to the eight compute dies in turn, each with an L2 of its own: a die takes heads that follow
  // each other (they share their keys), longest rows first.
  const int n_qb = (a.T + BQ - 1) / BQ, per_die = (n_qb * a.H + 7) >> 3, idx = (blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
  if (idx >= n_qb * a.H) return;
  const int head = idx / n_qb, qb = n_qb - 1 - (idx - head * n_qb), kvh = head / (a.H / a.K);
  const int q0 = qb * BQ, qw0 = q0 + 32 * wave;
  const int col = lane & 31, half = lane >> 5;
  const int query = qw0 + col;
  const long HH = (long)a.H * HD;

  // this lane's query as B operand of K Q^T: elements [16 ks + 8 half, + 8) for every step ks
  bf16x8 qf[HD / 16];
  {
    const bf16_t* qp = a.q + (long)min(query, a.T - 1) * HH + (long)head * HD + 8 * half;
#pragma unroll
    for (int ks = 0; ks < HD / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
  }

  f32x16 o[HT];
#pragma unroll
  for (int i = 0; i < HT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  // Scores are kept relative to m, the query's reference: the products start from -m, so nothing is subtracted afterwards.
  // m is the maximum of the first block and is raised only when a score exceeds it by more than kRaise: a softmax's weights
  // may be scaled by any number, and 2^8 costs neither bf16 nor fp32 a digit (the largest weight is no longer 1, which bf16 holds
  // exactly: the sum makes up for it, see below).  A score counted from -m is rounded like m, which
  // near m is what it is rounded like by itself.  Where a block raises m from much further below zero than the score that
  // raises it (the first keys 2^26 powers of two down, or lower than -1e30) its products start from zero once more.
  // 6000 positions of the 8B shape, scores that grow by 12 powers of two a block for a quarter of the queries: 444 us against
  // 402 with no raises (once more in every block that raises: 558 against 412; the case left out: 448 against 402).
  float m = -1e30f, l = 0.f;
  bool first = true;                                             // no block yet: scores are counted from zero
  f32x16 neg_m;
#pragma unroll
  for (int r = 0; r < 16; ++r) neg_m[r] = 0.f;

  const int p0 = a.p0;                                           // position of query 0: keys 0 .. p0 + query are visible
  const int n_keys = p0 + a.T, n_kb = min((p0 + q0 + BQ + BK - 1) / BK, (n_keys + BK - 1) / BK); // key blocks any query of this workgroup may see
  const int n_it = (n_kb + NG - 1) / NG;                         // steps: block NG it + grp each

  // Staging: the next block's keys and values travel global -> registers during the arithmetic, its page numbers a block
  // ahead of that.  A thread moves channels 8 oct .. + 7 of KU keys of a block.  Keys past the last repeat
  // it (no query sees them, but they are finite), a group whose last step has no block re-reads the last key.
  constexpr int KU = HD / (8 * WQ);
  const int oct = tid % (HD / 8), ku = tid / (HD / 8);
  u32x4 kreg[KU], vreg[KU];
  int pg[KU];
  auto key_in = [&](int j) __attribute__((always_inline)) { return ku + j * (GT * 8 / HD); };
  auto key_of = [&](int kb, int j) __attribute__((always_inline)) { return min(kb * BK + key_in(j), n_keys - 1); };
  auto page_of = [&](int pos) __attribute__((always_inline)) { return a.pt_sh >= 0 ? pos >> a.pt_sh : (int)__umulhi((unsigned)pos, a.pt_magic); };
  const bool block_page = a.pt_sh >= 6;                          // a block of 64 keys lies in one page
  auto pages = [&](int kb) __attribute__((always_inline)) {
    if (block_page) {
      int at = min(kb * BK, n_keys - 1) >> a.pt_sh;
      asm volatile("" : "+v"(at));                               // a vector load: behind a scalar one every read of LDS would have to wait for it
      pg[0] = a.table[at];
    } else {
#pragma unroll
      for (int j = 0; j < KU; ++j) pg[j] = a.table[page_of(key_of(kb, j))];
    }
  };
  auto fetch = [&](int kb) __attribute__((always_inline)) {
    if (block_page) {                                            // uniform base, 32-bit lane offsets
      const int page = __builtin_amdgcn_readfirstlane(pg[0]);
      const char* kp = (const char*)(a.pool + ((long)page * a.K + kvh) * 2 * a.pt * HD);
      const char* vp = kp + (long)a.pt * HD * 2;
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        const uint32_t off = (uint32_t)((key_of(kb, j) & (a.pt - 1)) * HD + 8 * oct) * 2u;
        kreg[j] = *reinterpret_cast<const u32x4*>(kp + off);
        vreg[j] = *reinterpret_cast<const u32x4*>(vp + off);
      }
      pages(kb + NG);
      return;
    }
#pragma unroll
    for (int j = 0; j < KU; ++j) {
      const int pos = key_of(kb, j);
      const bf16_t* kp = a.pool + (((long)pg[j] * a.K + kvh) * 2 * a.pt + (pos - page_of(pos) * a.pt)) * HD + 8 * oct;
      kreg[j] = *reinterpret_cast<const u32x4*>(kp);
      vreg[j] = *reinterpret_cast<const u32x4*>(kp + (long)a.pt * HD);
    }
    pages(kb + NG);
  };
  auto stash = [&](bf16_t* Ks) __attribute__((always_inline)) {
    bf16_t* Vs = Ks + BK * KS;
#pragma unroll
    for (int j = 0; j < KU; ++j) {
      *reinterpret_cast<u32x4*>(Ks + key_in(j) * KS + 8 * oct) = kreg[j];
      *reinterpret_cast<u32x4*>(Vs + key_in(j) * VR + 8 * oct) = vreg[j];
    }
  };

  pages(grp);
  // Of every 16 lanes, lane j names key j / 4 and channels 4 (j mod 4) .. + 3 and receives channel j of the four keys.
  const int v_lane = (4 * half + ((lane & 15) >> 2)) * VR + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

  fetch(grp);
  stash(bufs);
  __syncthreads();
  for (int it = 0; it < n_it; ++it) {
    const int kb = NG * it + grp;
    const bf16_t* Ks = bufs + (NB == 2 ? it & 1 : 0) * KV;
    const bf16_t* Vs = Ks + BK * KS;
    if (it + 1 < n_it) fetch(kb + NG);
    const int k0 = kb * BK;
    if (kb < n_kb && k0 <= p0 + qw0 + 31) {                      // else: no block, or this wavefront's queries see none of these keys

      // ---- S^T = K Q^T: two tiles of 32 keys x 32 queries, counted from `start`
      f32x16 s[2];
      float top;
      auto scores = [&](const f32x16& start) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          s[t] = start;
          const bf16_t* kr = Ks + (32 * t + col) * KS + 8 * half;
#pragma unroll
          for (int ks = 0; ks < HD / 16; ++ks)
            s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kr + 16 * ks), qf[ks], s[t], 0, 0, 0);
        }
        // ---- causal mask (the last blocks only) and the lane's share of the row statistics (row of S = column here = this
        //      lane's query)
        if (k0 + BK - 1 > p0 + qw0) {
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (k0 + 32 * t + 8 * (r >> 2) + 4 * half + (r & 3) > p0 + query) s[t][r] = -1e30f;
        }
        top = -1e30f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) top = fmaxf(top, s[t][r]);
      };
      scores(neg_m);
      if (first || __any(top > kRaise)) {
        float base = first ? 0.f : m;
        if (!first && __any(top > kRaise && m < -16.f - 2.f * fabsf(m + top))) {
          // a reference much further below zero than the score, which has lost digits: once more without it
          asm volatile("" ::: "memory");                         // (or the keys would be kept in registers for this)
          f32x16 zero;
#pragma unroll
          for (int r = 0; r < 16; ++r) zero[r] = 0.f;
          scores(zero);
          base = 0.f;
        }
        first = false;
        top = fmaxf(top, __shfl_xor(top, 32, 64));               // both lanes of a query raise alike
        const float to = fmaxf(m, base + top), by = to - base, alpha = exp2f_raw(m - to);
        m = to;
        l *= alpha;
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[i][r] *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s[0][r] -= by; s[1][r] -= by; neg_m[r] = -m; }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[t][r] = exp2f_raw(s[t][r]);

      // ---- O^T += V^T P^T.  Step (t, pp) contracts keys [32 t + 16 pp, + 16); inside a step this half of the
      // wavefront supplies keys {0..3, 8..11} + 4 half, which is what registers 8 pp .. 8 pp + 7 of tile t hold.  The sum takes the
      // weights as they are multiplied, rounded to bf16: what one key dominates is then that key's value, whatever its weight
      // (1600 positions of such scores: 2.61e-3 from 64 bits, 2.71e-3 with the sum of the others; two weights an instruction
      // take no longer than one, and the instruction's fp32 sum over 6000 of them is as close as additions, 2e-6).  The two
      // lanes of a query keep separate sums until the end.
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int pp = 0; pp < 2; ++pp) {
          bf16x8 pf;
#pragma unroll
          for (int j = 0; j < 8; ++j) pf[j] = (__bf16)s[t][8 * pp + j];
#pragma unroll
          for (int j = 0; j < 8; j += 2) l = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[j], pf[j + 1]}, bf16x2{(__bf16)1.f, (__bf16)1.f}, l, false);
#pragma unroll
          for (int i = 0; i < HT; ++i) {
            const bf16_t* vr = Vs + v_lane + (32 * t + 16 * pp) * VR + 32 * i;
            const u32x2 lo = read_transposed(vr), hi = read_transposed(vr + 8 * VR);
            const u32x4 vf = {lo.x, lo.y, hi.x, hi.y};
            o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf), pf, o[i], 0, 0, 0);
          }
        }
    }
    if (NB == 1) __syncthreads();
    if (it + 1 < n_it) stash(bufs + (NB == 2 ? (it + 1) & 1 : 0) * KV);   // over a block which everybody has left
    __syncthreads();
  }

  // ---- fold the groups: the others hand their states to group 0 through LDS (the K/V area, no longer needed);
  //      element j of thread t at [j][t], so that a wavefront's accesses are consecutive
  if constexpr (NG > 1) {
    float* fold = (float*)flash_smem + (grp > 0 ? grp - 1 : 0) * (HT * 16 + 2) * GT;
    if (grp > 0) {
#pragma unroll
      for (int i = 0; i < HT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) fold[(i * 16 + r) * GT + tid] = o[i][r];
      fold[(HT * 16) * GT + tid] = m;
      fold[(HT * 16 + 1) * GT + tid] = l;
    }
    __syncthreads();
    if (grp > 0) return;
    for (int g = 1; g < NG; ++g, fold += (HT * 16 + 2) * GT) {
      const float m1 = fold[(HT * 16) * GT + tid], l1 = fold[(HT * 16 + 1) * GT + tid];
      const float mn = fmaxf(m, m1);
      const float a0 = exp2f_raw(m - mn), a1 = exp2f_raw(m1 - mn);   // group 0 has seen key 0; of a group that saw none m = -1e30 and nothing stays
      l = l * a0 + l1 * a1;
      m = mn;
#pragma unroll
      for (int i = 0; i < HT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] = o[i][r] * a0 + fold[(i * 16 + r) * GT + tid] * a1;
    }
  }

  l += __shfl_xor(l, 32, 64);
  if (query < a.T) {
    const float inv = 1.f / l;
    bf16_t* op = a.out + (long)query * HH + (long)head * HD;
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {                              // four consecutive channels: 32 i + 8 g + 4 half + 0..3
        const uint32_t w0 = (uint32_t)f32_to_bf16(o[i][4 * g] * inv) | ((uint32_t)f32_to_bf16(o[i][4 * g + 1] * inv) << 16);
        const uint32_t w1 = (uint32_t)f32_to_bf16(o[i][4 * g + 2] * inv) | ((uint32_t)f32_to_bf16(o[i][4 * g + 3] * inv) << 16);
        *reinterpret_cast<u32x2*>(op + 32 * i + 8 * g + 4 * half) = u32x2{w0, w1};
      }
  }
}

template <int HD, int NG, int WQ>
constexpr size_t flash_lds_bytes() {
  // two key blocks and their values per group, one of four; the fold at the end needs HD / 2 + 2 floats per thread of the
  // groups but one
  const size_t kv = (size_t)NG * (NG == 4 ? 1 : 2) * BK * (HD + 8 + HD + 32) * sizeof(bf16_t);
  const size_t fold = NG > 1 ? (size_t)(NG - 1) * (HD / 2 + 2) * 64 * WQ * sizeof(float) : 0;
  return kv > fold ? kv : fold;
}
template <int HD, int NG, int WQ>
bool allow_flash() {                                             // 64 KiB is what a kernel gets by default
  constexpr size_t lds = flash_lds_bytes<HD, NG, WQ>();
  return lds <= 64 * 1024 || hipFuncSetAttribute((const void*)k_flash_prefill<HD, NG, WQ>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
}
template <int HD, int NG, int WQ>
void launch_flash(hipStream_t s, const FlashArgs& a) {
  const int items = (a.T + 32 * WQ - 1) / (32 * WQ) * a.H;
  hipLaunchKernelGGL((k_flash_prefill<HD, NG, WQ>), dim3(8 * ((items + 7) / 8)), dim3(64 * WQ * NG), (flash_lds_bytes<HD, NG, WQ>()), s, a);
}
template <int HD>
void launch_flash_heads(hipStream_t s, const FlashArgs& a) {
  const FlashPlan p = plan_flash(a.T, a.p0, a.H);
  if (p.groups == 1) launch_flash<HD, 1, 4>(s, a);
  else if (p.groups == 4) launch_flash<HD, 4, 2>(s, a);
  else if (p.waves == 4) launch_flash<HD, 2, 4>(s, a);
  else launch_flash<HD, 2, 2>(s, a);
}

}  // namespace

bool flash_supported(int dtype, int h) { return dtype == MDI_BF16 && (h == 64 || h == 128); }

bool allow_flash_lds() {
  return allow_flash<64, 1, 4>() && allow_flash<64, 2, 4>() && allow_flash<64, 2, 2>() && allow_flash<64, 4, 2>() && allow_flash<128, 1, 4>() && allow_flash<128, 2, 4>() &&
         allow_flash<128, 2, 2>() && allow_flash<128, 4, 2>();
}

void launch_flash_prefill(hipStream_t s, const FlashArgs& a) {
  if (a.h == 128) launch_flash_heads<128>(s, a); else launch_flash_heads<64>(s, a);
}

}  // namespace mdi

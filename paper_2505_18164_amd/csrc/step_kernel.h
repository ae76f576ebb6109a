// Decode steps of a whole partition as ONE persistent kernel launch.
//
// A later visit of a sample (Sec. III-D) pushes a single position through every
// local layer; each layer is five dependent matrix-vector / attention phases whose
// inputs are full vectors produced by the previous phase.  Launching them as
// separate kernels leaves the memory system idle at every boundary (drain, launch,
// ramp-up).  Here workgroups stay resident for the whole launch - one of eight
// wavefronts per compute unit for a launch that carries one message, two of four
// wavefronts for a launch that carries the queued messages of several samples
// (Sec. III-A: the input queue; Sec. III-C: several samples in flight).  In the
// latter a set of workgroups takes its messages in turn inside every phase and
// two sets share each compute unit, so that the serial part of one message's
// phase boundary (vector staging, cross-wavefront sums, epilogue) runs
// under other messages' weight streams; every message still makes its own pass
// over the weights.
//
//   * there is no grid-wide barrier.  Everything that crosses workgroups (x, q, o, u, attention partials, the newest K/V
//     row) is written and read with cache-coherent (sc1, agent scope) stores and loads, each value with the counter of
//     the phase that wrote it in the same 8-byte word, and readers reload until the counter is the expected one.
//     Nothing is overwritten that is still being read, because every phase needs all of the one before: who stores x in
//     the output projection has read all of o, so every head's attention is done, so every workgroup with QKV rows has
//     stored them, after it read x; who stores x in the down projection has read all of u, so all have read x for it;
//     and q, u, o are written a layer after they were read.  (A workgroup without rows in a product does not read its
//     vector.)  Phase counters watched before the data cost 3.2 us a phase; the data alone take 1.65 us from store to
//     store (2048 words, 256 workgroups), and for the longest vectors too, waiting for the counters first was slower
//     (7B shape, one message: 795 against 757 us).  What is left of the counters paces the two sets of workgroups.
//   * weight and KV-cache addresses do not depend on activations, so every
//     wavefront keeps two register tiles of 16-byte loads in flight and issues the
//     first two of a phase before the phase's vector is there - but after it has
//     asked for that vector's first words, which loads return in order.
//   * the rows a workgroup owns in a phase form one flat sequence of (row pair,
//     1-KiB chunk) items dealt round-robin to its wavefronts.  At any moment the
//     workgroup therefore reads consecutive KiB of a row pair (DRAM sees a few
//     wide sequential streams instead of thousands of narrow ones), and the
//     wavefronts stay balanced whatever the shape.  A wavefront's share of a pair
//     goes to an LDS slot of its own; slots are summed in wavefront order
//     (deterministic, no float atomics; the order depends on the number of
//     wavefronts, which is why launches of one and of several messages may differ
//     in the last bits).
//   * in a launch with two sets of workgroups, each workgroup compares once per
//     phase the work it has left with that of the other set and takes the higher
//     wave priority when it has more: left alone, the set that was dispatched
//     first is served first by a compute unit's memory pipeline and finishes a
//     fifth earlier.
//
// Every spin is bounded: a wait of more than `spin_limit` polls raises the
// partition's error word, the other waits of that workgroup end with it, and the
// workgroup leaves at the end of the phase at the latest.  What it stored in that phase is
// worthless (the error word says so); everybody who needs its words later
// expires in the same way.
//
// step_w4*.hip and step_w8*.hip compile it for workgroups of four and of eight wavefronts (MDI_STEP_WAVES) and one storage
// type each (MDI_STEP_TYPE, and its name in the launcher's: MDI_STEP_TYPE_NAME).
#include "step_impl.h"

namespace mdi {
namespace MDI_STEP_CAT(step_w, MDI_STEP_WAVES) {

// Norm and MLP kind are template arguments and every phase is code of its own, see k_step_batch.
template <typename WT, int G, bool kLn, bool kSwiglu>
__global__ __launch_bounds__(kStepThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_step(StepArgs a0) {
  constexpr bool kOne = kStepWaves == 8;           // one message, one set of workgroups
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a set of nwg workgroups takes its messages in turn inside every phase; two sets share the compute units
  const int nwg = a0.nwg, wg = kOne ? blockIdx.x : blockIdx.x % nwg;
  const int set = kOne ? 0 : (int)blockIdx.x / nwg;
  const int slot_lo = kOne ? 0 : a0.set_lo[set], slot_hi = kOne ? 1 : a0.set_lo[set + 1];
  float* part = lds_part();
  float* xs = lds_vec(a0.part_floats);
  float* red = lds_red();
  int* s_flag = lds_flag();

  if (threadIdx.x == 0) s_flag[kFailed] = 0;
  if (wg == 0 && (int)threadIdx.x < a0.n_slots) {
    const MDI_GLOBAL StepSlot& S = *(const MDI_GLOBAL StepSlot*)&args_again<StepArgs>().s[threadIdx.x];
    if (S.table_entry) *S.table_entry = S.new_page;
  }
  __syncthreads();

  float acc0 = 0.f, acc1 = 0.f;
  // requested while finishing the previous (message, phase): the head of the next one's input vector
  VecAsk vec;
  bool early = false;
  int layer = 0;
  long w_off = 0, kv_off = 0;                      // bytes from the first layer's matrices / pages to this layer's

  // what phase `ph` of message N reads: asked for by this thread's first pieces (the launch's own input is not exchanged)
  auto ask_for = [&](auto ph_const, const StepArgs& a, const StepSlot& N, long at, int tid) __attribute__((always_inline)) {
    constexpr int ph = decltype(ph_const)::value;
    if constexpr (ph != PH_ATTN) {
      const float* gain = kLn || ph == PH_OPROJ || ph == PH_DOWN ? nullptr : (const float*)((const char*)(ph == PH_QKV ? a.l0.ln1_g : a.l0.ln2_g) + at);
      vec_ask(vec, ph == PH_OPROJ ? N.o : ph == PH_DOWN ? N.u : N.xres, ph == PH_OPROJ ? a.H * a.h : ph == PH_DOWN ? a.F : a.d, gain, tid);
    }
  };

  // The page numbers of the first two tiles of attention: the same in every layer, and in every layer a round trip before the
  // first key can be asked for.  (Several messages: their streams cover it.)
  int page0A[kTile] = {}, page0B[kTile] = {};
  if constexpr (kOne) {
    const StepArgs& a = args_again<StepArgs>();
    const AttnGeo ga = make_attn_geo<WT, G>(a, a.s[0], wg, wave, threadIdx.x & 63);
    attn_pages(page0A, ga, a, a.s[0], 0, wave); attn_pages(page0B, ga, a, a.s[0], 1, wave);
  }

  auto phase = [&](auto ph_const) __attribute__((always_inline)) -> bool {
    constexpr int ph = decltype(ph_const)::value;
    constexpr bool normed = ph == PH_QKV || ph == PH_UP, resid = ph == PH_OPROJ || ph == PH_DOWN, fused_rms = normed && !kLn;
#pragma nounroll
    for (int slot = slot_lo; slot < slot_hi; ++slot) {
      // Messages alternate inside a phase: while this message's input vector makes its round trip,
      // the memory system is still busy with the other message's stream, and by the time a message reaches its
      // next phase every workgroup has long finished its previous one.
      const StepArgs& a = args_again<StepArgs>();
      const StepSlot& S = a.s[kOne ? 0 : slot];
      const unsigned epoch = S.epoch0 + (unsigned)(layer * 5 + ph);
      stamp(a, S, layer, ph, 0);
      // per-thread addresses are recomputed in every phase (see k_step_batch)
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63;
      // requests for the next (message, phase), answered while this phase is being finished: with two messages
      // alternating, what the next one needs was published a whole phase ago
      auto early_requests = [&]() __attribute__((always_inline)) {
        if constexpr (!kOne) {
          early = false;
          if (slot_hi - slot_lo > 1) {
            if (slot + 1 < slot_hi) {
              if (!(ph == PH_QKV && layer == 0)) { ask_for(ph_const, a, a.s[slot + 1], w_off, tid); early = ph != PH_ATTN; }
            } else if (ph != PH_DOWN) {
              ask_for(std::integral_constant<int, (ph + 1) % 5>(), a, a.s[slot_lo], w_off, tid); early = ph + 1 != PH_ATTN;
            } else if (layer + 1 < a.n_layer) {
              ask_for(std::integral_constant<int, 0>(), a, a.s[slot_lo], w_off + a.w_stride, tid); early = true;
            }
          }
        }
      };
      // Two sets share a compute unit's memory pipeline, and the hardware serves the older wavefronts (the set
      // that was dispatched first) or the higher priority first; left alone, one set finishes a fifth earlier
      // and the other runs the rest of the launch on half the wavefronts.  So the set that is behind takes the
      // higher priority, phase by phase: work left, in (message, phase) units; the set with more of it goes first.
      // (Launches of one message leave the counters behind: before the other set's first phase they say nothing.)
      unsigned other_done = 0u;
      const bool pace = !kOne && a.n_sets == 2 && slot == slot_lo;
      if (pace) {
        const StepSlot& O = a.s[a.set_lo[set ^ 1]];                // the other set's first message
        other_done = __hip_atomic_load((const MDI_GLOBAL unsigned*)O.flags + wg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - O.epoch0;
      }
      auto take_pace = [&]() __attribute__((always_inline)) {
        if (!pace) return;
        const int total = a.n_layer * 5, seen = min(max(__builtin_amdgcn_readfirstlane((int)other_done), 0), total);
        const int left = (total - (layer * 5 + ph)) * (slot_hi - slot_lo);
        const int other_left = (total - seen) * (a.set_lo[2 - set] - a.set_lo[1 - set]);
        if (left > other_left || (left == other_left && set == 1)) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
      };

      if constexpr (ph == PH_ATTN) {
        // ---- attention over the sample's pages -----------------------------------------------------
        const void* kv = (const char*)a.l0.kv + kv_off;
        const AttnGeo ga = make_attn_geo<WT, G>(a, S, wg, wave, lane);
        AttnState<WT, G> st;
        AttnAsk<WT> ask;
        Tile A, B;
        int pgA[kTile], pgB[kTile];                  // page numbers of the tiles that go into A and B next
        attn_ask<WT, G>(ask, ga, a, S, wave, tid);
        if constexpr (kOne) {
#pragma unroll
          for (int k = 0; k < kTile; ++k) { pgA[k] = page0A[k]; pgB[k] = page0B[k]; }
        } else {
          attn_pages(pgA, ga, a, S, 0, wave); attn_pages(pgB, ga, a, S, 1, wave);
        }
        attn_issue<WT>(A, pgA, ga, a, S, kv, 0, wave); attn_issue<WT>(B, pgB, ga, a, S, kv, 1, wave);
        stamp(a, S, layer, ph, 1);
        take_pace();
        attn_begin<WT, G>(st, ask, ga, a, S, xs, wave, epoch, tid);
        stamp(a, S, layer, ph, 2);
        const int nte = ((ga.n_k + kTile - 1) / kTile + 1) & ~1;
        attn_stream<WT, G>(st, A, B, pgA, pgB, ga, a, S, kv, nte, wave, xs);
        loads_done();
        stamp(a, S, layer, ph, 3);
        early_requests();
        attn_to_lds<WT, G>(st, ga, a.h, xs, wave);
        attn_finish<G>(ga, a, S, xs, s_flag, epoch, tid);
      } else {
        // ---- a GEMV phase ----------------------------------------------------------------------------
        const Geo g = make_geo<WT, ph == PH_QKV>(a.pr[ph == PH_QKV ? 0 : ph - 1], w_off, wg, nwg, wave, a.h);
        const bool first = ph == PH_QKV && layer == 0;
        if (g.n_pl > 0 || first) {                   // who has no rows in a product reads nothing for it either
          // The head of the input vector is asked for first: loads return in order, and the workgroup that everybody
          // waits for finds it there at once instead of behind its weights.
          if (!(first || early)) ask_for(ph_const, a, S, w_off, tid);
          const Buffer xb = buffer_at(S.xres);
          FinOps ops = fin_ops<ph, kSwiglu>(g, a, S, w_off, tid);
          // residual phases: this thread's own rows of x
          const uint32_t x_off = resid && tid < g.n_pl ? (uint32_t)ops.r0 * 8u : kNowhere;
          tagged_t x0 = ld_word(xb, x_off), x1 = ld_word(xb, resid && ops.r0 + 1 < g.N ? x_off + 8u : kNowhere);
          // then this phase's first two tiles: their addresses depend on nothing another workgroup writes
          Tile A, B;
          Cursor ci = cursor_start(g), cc = ci;              // where the loads and the multiplications are
          gemv_issue(A, g, ci, lane); gemv_issue(B, g, ci, lane);
          stamp(a, S, layer, ph, 1);
          take_pace();
          for (int i = tid; i < g.n_pl * 2 * kStepWaves; i += kStepThreads) part[i] = 0.f;
          const int n = ph == PH_OPROJ ? a.H * a.h : ph == PH_DOWN ? a.F : a.d;
          const float* gain = (const float*)((const char*)(ph == PH_QKV ? a.l0.ln1_g : a.l0.ln2_g) + w_off);
          float share;                                 // of the sum of squares (RMSNorm) or of the sum
          if (first) {
            share = stage_input<WT, kLn>(a, S, xs, gain, make_geo<WT, false>(a.pr[1], 0, wg, nwg, wave, a.h), epoch, tid);
          } else {
            share = stage_coherent<fused_rms>(vec, ph == PH_OPROJ ? S.o : ph == PH_DOWN ? S.u : S.xres, n, xs, gain, epoch, a.spin_limit, a.err, tid);
          }
          // zeros behind the vector up to a whole 64-lane chunk (the host sizes the LDS for it): see gemv_compute
          for (int i = g.units * Storage<WT>::kVec + tid; i < g.cpp * 64 * Storage<WT>::kVec; i += kStepThreads) xs[i] = 0.f;
          float row_scale = 1.f;                       // 1/rms when the norm is folded into the epilogue
          if constexpr (fused_rms) {
            row_scale = 1.f / sqrtf(step_sum(share, red, tid) / (float)a.d + a.eps);
          } else {
            if constexpr (normed) {
              const float* b = ph == PH_QKV ? a.l0.ln1_b : a.l0.ln2_b;
              layer_norm(xs, a.d, share, a.eps, buffer_at(gain), buffer_at(b ? (const char*)b + w_off : nullptr), red, tid);
            }
            __syncthreads();
          }
          if (__builtin_amdgcn_readfirstlane(s_flag[kFailed])) return false;
          stamp(a, S, layer, ph, 2);

          const int nte = ((g.n_k + kTile - 1) / kTile + 1) & ~1;
#pragma nounroll
          for (int t = 2; t < nte; t += 2) {
            gemv_compute<WT, true>(A, g, t - 2, cc, wave, lane, xs, part, acc0, acc1);
            gemv_issue(A, g, ci, lane);
            gemv_compute<WT, true>(B, g, t - 1, cc, wave, lane, xs, part, acc0, acc1);
            gemv_issue(B, g, ci, lane);
          }
          if (nte) {                                   // (the last two tiles: nothing more to ask for)
            gemv_compute<WT, true>(A, g, nte - 2, cc, wave, lane, xs, part, acc0, acc1);
            gemv_compute<WT, true>(B, g, nte - 1, cc, wave, lane, xs, part, acc0, acc1);
          }
          loads_done();
          stamp(a, S, layer, ph, 3);
          early_requests();
          __syncthreads();                             // all wavefronts' partials are in LDS
          stamp(a, S, layer, ph, 4);
          gemv_finish<WT, ph, kSwiglu>(g, layer, a, S, (char*)a.l0.kv + kv_off, part, row_scale, x0, x1, ops, w_off, epoch, tid);
        } else {
          early = false;
        }
      }

      // ---- this workgroup is done with the phase ------------------------------------------------------
      stamp(a, S, layer, ph, 5);
      __syncthreads();
      stamp(a, S, layer, ph, 6);
      if (__builtin_amdgcn_readfirstlane(s_flag[kFailed])) return false;
      if (!kOne && a.n_sets == 2 && tid == 0) __hip_atomic_store((MDI_GLOBAL unsigned*)S.flags + wg, epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return true;
  };

#pragma nounroll
  for (; layer < a0.n_layer; ++layer) {
    if (!phase(std::integral_constant<int, PH_QKV>())) return;
    if (!phase(std::integral_constant<int, PH_ATTN>())) return;
    if (!phase(std::integral_constant<int, PH_OPROJ>())) return;
    if (!phase(std::integral_constant<int, PH_UP>())) return;
    if (!phase(std::integral_constant<int, PH_DOWN>())) return;
    w_off += a0.w_stride; kv_off += a0.kv_stride;
  }
}

template <typename WT, int G>
static void launch_step_t(hipStream_t s, int nwg, size_t lds, const StepArgs& a) {
  const dim3 grid(nwg * a.n_sets), block(kStepThreads);
  const bool ln = a.norm_kind == MDI_NORM_LAYERNORM, swiglu = a.mlp_kind == MDI_MLP_SWIGLU;
  if (ln && swiglu) hipLaunchKernelGGL((k_step<WT, G, true, true>), grid, block, lds, s, a);
  else if (ln) hipLaunchKernelGGL((k_step<WT, G, true, false>), grid, block, lds, s, a);
  else if (swiglu) hipLaunchKernelGGL((k_step<WT, G, false, true>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((k_step<WT, G, false, false>), grid, block, lds, s, a);
}
// G = query heads per attention work item: the host asks for 1 or 2 (larger groups were measured slower)
template <typename WT>
static void launch_step_t(hipStream_t s, int G, int nwg, size_t lds, const StepArgs& a) {
  if (G == 2) launch_step_t<WT, 2>(s, nwg, lds, a); else launch_step_t<WT, 1>(s, nwg, lds, a);
}

}  // namespace step_w<waves>

void MDI_STEP_CAT(MDI_STEP_CAT(launch_step_w, MDI_STEP_WAVES), MDI_STEP_TYPE_NAME)(hipStream_t s, int G, int nwg, size_t lds, const StepArgs& a) {
  MDI_STEP_CAT(step_w, MDI_STEP_WAVES)::launch_step_t<MDI_STEP_TYPE>(s, G, nwg, lds, a);
}

}  // namespace mdi

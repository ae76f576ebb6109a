// Which kernels a first visit runs on.  Host code without HIP, so that tests can ask which ones a set of sizes reaches.
#pragma once

#include <algorithm>
#include <cstddef>

#include "mdi.h"

namespace mdi {

// ---- Products: the tile shape, and into how many pieces the inner dimension is cut so that few positions still fill the chip
// (kernel: gemm_impl.h; the shapes' wavefronts and rings: gemm_bf16.hip, gemm_f32.hip).
constexpr int kMaxKSplits = 16;
struct GemmPlan { int shape, S; };

// What plan_shape goes by: a round of workgroups (`round` per compute unit) takes steps * us + fixed, a last round that is
// a fraction f full part + (1 - part) f of that, and no product is faster than its weights arrive (tbps).  All are fitted
// to measured times; `round` too, which is not how many workgroups a compute unit holds (64 x 32: two by their LDS, 4 fitted).
// (Matrices beyond the fitted ones, 57344 x 8192: 256 x 256 reaches 4.0 TB/s, 256 positions in 235 us, and 256 x 128 5.3, 128
// positions in 177.  With the fit's 2.7 and 4.2 these went to 256 x 128, 269 us, and 128 x 128, 204.  At the sizes of the models
// here the choices are the same.)
struct Shape { int BN, BT, round; float us, fixed, part, tbps; };
constexpr Shape kShapesBf16[] = {
    {256, 256, 1, 1.393f, 14.28f, 0.79f, 4.0f}, {192, 256, 1, 1.157f, 12.86f, 0.96f, 2.8f}, {256, 192, 1, 1.090f, 11.22f, 0.77f, 2.5f},
    {192, 192, 1, 0.911f, 11.80f, 0.83f, 2.8f}, {256, 128, 1, 0.873f, 11.18f, 0.72f, 5.2f}, {192, 128, 1, 0.717f, 7.06f, 0.82f, 4.5f},
    {128, 192, 1, 0.726f, 6.68f, 0.71f, 3.8f},  {128, 128, 1, 0.576f, 6.24f, 0.70f, 5.1f},  {96, 128, 1, 0.451f, 5.59f, 0.78f, 4.7f},
    {128, 64, 1, 0.382f, 4.43f, 0.82f, 6.9f},   {64, 96, 2, 0.496f, 6.00f, 0.50f, 4.7f},    {64, 64, 2, 0.419f, 5.08f, 0.58f, 4.9f},
    {64, 32, 4, 0.546f, 7.38f, 0.34f, 5.0f}};
constexpr Shape kShapesF32[] = {{64, 32, 4, 1.055f, 2.36f, 0.29f, 4.5f}, {64, 64, 1, 0.578f, 1.37f, 1.0f, 4.5f}};

inline GemmPlan plan_shape(const Shape* shapes, int n_shapes, int elem_bytes, int compute_units, int T, int N, int Kd, size_t part_floats) {
  const double n_cu = compute_units > 0 ? compute_units : 256;
  const int nk = (elem_bytes * Kd + 127) >> 7;
  GemmPlan best{0, 1};
  double best_us = 1e30;
  for (int i = 0; i < n_shapes; ++i) {
    const Shape& sh = shapes[i];
    if (elem_bytes == 2 && sh.BT == 32 && T > 32) continue;   // a second position tile would read the weights again
    const double tiles = (double)((T + sh.BT - 1) / sh.BT) * ((N + sh.BN - 1) / sh.BN);
    for (int S = 1; S <= kMaxKSplits && S <= nk; ++S) {
      const int per = (nk + S - 1) / S;
      if ((nk + per - 1) / per != S) continue;                // no split without a step
      if (S > 1 && (size_t)S * T * N > part_floats) break;
      const double u = tiles * S / (n_cu * sh.round), full = (double)(long)u, f = u - full;
      double us = (full + (f > 0 ? sh.part + (1 - sh.part) * f : 0)) * (per * sh.us + sh.fixed);
      us = std::max(us, (double)elem_bytes * N * Kd / (sh.tbps * 1e6));
      if (S > 1) us += (double)S * T * N * 4.0 / 4.5e6;       // the partial results are read again (4.5 TB/s)
      if (us < best_us) { best_us = us; best = GemmPlan{i, S}; }
    }
  }
  return best;
}
// part_floats = room for partial results, 0 forbids a split
inline GemmPlan plan_gemm(int dtype, int n_cu, int T, int N, int Kd, size_t part_floats) {
  return dtype == MDI_BF16 ? plan_shape(kShapesBf16, (int)(sizeof(kShapesBf16) / sizeof(Shape)), 2, n_cu, T, N, Kd, part_floats)
                           : plan_shape(kShapesF32, (int)(sizeof(kShapesF32) / sizeof(Shape)), 4, n_cu, T, N, Kd, part_floats);
}

// ---- Causal attention on the matrix cores (kernel: attn_prefill.hip): groups of wavefronts per workgroup, and wavefronts of a
// group, 32 queries each.
constexpr int kFlashKeys = 64;         // keys of a step
struct FlashPlan { int groups, waves; };
// The numbers of workgroups are those of 256 compute units.
inline FlashPlan plan_flash(int T, int p0, int H) {
  const int items = (T + 127) / 128 * H;
  // Many workgroups: one group each.  us a layer of one / two groups: 1024 positions of the 7B shape (256 items of 128
  // queries) 34 / 29, 1280 (320) 44 / 38, 1536 (384) 55 / 53, 2048 (512) 78 / 85; TinyLlama 1500 (384) 34.5 / 34.
  // So does a single block of keys, which a second group could only wait for: 64 positions of the 7B shape 6.0 / 7.6, TinyLlama 4.1 / 4.8.
  if (items >= 384 || p0 + T <= kFlashKeys) return {1, 4};
  // As many items as would leave half the chip idle: 64 queries a workgroup, 128 / 64 queries: 256 positions of the 7B shape
  // 12.4 / 10.1, 512 (128 items) 18.1 / 16.0, 768 (192) 22.9 / 29.2; TinyLlama 500 (128) 11.3 / 9.6, 750 (192) 14.7 / 17.1.
  // Between the two it depends on more than the number of items: 160 of the 7B shape, 520 positions 20.4 / 19.8, 576 18.8 / 18.6,
  // 640 20.4 / 24.1; TinyLlama 11.9 / 11.0, 12.4 / 11.6, 13.4 / 14.6; 16 heads of 64, 1100 positions (144) 19.1 / 14.8, 1400
  // (176) 23.2 / 17.6.
  if (items > 128) return {2, 4};
  // Many keys on average: four groups.  Two / four: 256 positions behind 0, 256, 512, ... 1792 of the 8B shape 9.7 / 10.6,
  // 15.1 / 14.2, 20.6 / 18.4, ... 47.4 / 37.9; 512 of the 7B shape behind none 16.0 / 16.7, TinyLlama 256 6.5 / 6.5.
  return {p0 + T / 2 >= 320 ? 4 : 2, 2};
}

}  // namespace mdi

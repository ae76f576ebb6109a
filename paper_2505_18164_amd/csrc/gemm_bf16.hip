// First-visit products with bf16 storage: tile shapes and their choice (kernel: gemm_impl.h).
#include "gemm_impl.h"

namespace mdi {
namespace {

// index, BN, BT, wavefronts WN x WT, ring depths.  The figures are fitted to 14000 measured (T, N, Kd, shape, splits) over
// the shapes of all the models here, T from 1 to 6000; going by them takes 2.6 % more time than picking the best
// measured one each time.  Against the eight shapes that stood here before (without 256 x 192, 192 x 192, 128 x 192, 96 x 128
// and 64 x 96): 6 % less on average; most where the number of positions leaves the last round of larger tiles nearly empty
// (6000 x 4096 x 14336 677 -> 552 us: 512 tiles of 256 x 192 are two rounds, 384 of 256 x 256 one and a half), and where a
// product of few positions did not fill the chip (256 x 12288 x 4096 43 -> 38, 333 x 2560 x 2048 15.8 -> 12.9).
// 256 x 256 and 256 x 192 as 4 x 2 wavefronts: the residual epilogue of 2 x 4 spills (6000 x 4096 x 14336 on 256 x 256 tiles 876
// against 656 us).  Four wavefronts of 128 x 128 each, a third less LDS traffic: 5 to 20 % slower, nothing hides a wavefront's waits.
#define MDI_GEMM_SHAPES(X) \
  X(0, 256, 256, 4, 2, 3, 2) X(1, 192, 256, 2, 4, 3, 2) X(2, 256, 192, 4, 2, 3, 2) X(3, 192, 192, 2, 4, 3, 3) X(4, 256, 128, 2, 4, 3, 3) \
  X(5, 192, 128, 2, 4, 4, 4) X(6, 128, 192, 2, 4, 4, 4) X(7, 128, 128, 2, 4, 4, 4) X(8, 96, 128, 1, 4, 4, 4) X(9, 128, 64, 4, 2, 4, 4) \
  X(10, 64, 96, 2, 2, 4, 4) X(11, 64, 64, 2, 2, 4, 4) X(12, 64, 32, 2, 2, 6, 6)
constexpr int kShapes = 13;
constexpr Shape kShape[kShapes] = {
    {256, 256, 1, 1.393f, 14.28f, 0.79f, 2.7f}, {192, 256, 1, 1.157f, 12.86f, 0.96f, 2.8f}, {256, 192, 1, 1.090f, 11.22f, 0.77f, 2.5f},
    {192, 192, 1, 0.911f, 11.80f, 0.83f, 2.8f}, {256, 128, 1, 0.873f, 11.18f, 0.72f, 4.2f}, {192, 128, 1, 0.717f, 7.06f, 0.82f, 4.5f},
    {128, 192, 1, 0.726f, 6.68f, 0.71f, 3.8f},  {128, 128, 1, 0.576f, 6.24f, 0.70f, 5.1f},  {96, 128, 1, 0.451f, 5.59f, 0.78f, 4.7f},
    {128, 64, 1, 0.382f, 4.43f, 0.82f, 6.9f},   {64, 96, 2, 0.496f, 6.00f, 0.50f, 4.7f},    {64, 64, 2, 0.419f, 5.08f, 0.58f, 4.9f},
    {64, 32, 4, 0.546f, 7.38f, 0.34f, 5.0f}};

template <int EPI>
void launch_epi(hipStream_t s, int shape, const GemmArgs& a) {
  switch (shape) {
#define X(I, BN, BT, WN, WT, NBW, NBA) case I: launch_shape<bf16_t, EPI, BN, BT, WN, WT, NBW, NBA>(s, a); break;
    MDI_GEMM_SHAPES(X)
#undef X
  }
}

template <int EPI>
bool allow_epi() {
#define X(I, BN, BT, WN, WT, NBW, NBA) && allow_shape<bf16_t, EPI, BN, BT, WN, WT, NBW, NBA>()
  return true MDI_GEMM_SHAPES(X);
#undef X
}

}  // namespace

GemmPlan plan_gemm_bf16(int n_cu, int T, int N, int Kd, size_t part_floats) { return plan_shape(kShape, kShapes, 2, n_cu, T, N, Kd, part_floats); }

bool allow_gemm_lds_bf16() {
  return allow_epi<GEPI_QKV>() && allow_epi<GEPI_RESID>() && allow_epi<GEPI_PART>() && allow_epi<GEPI_SWIGLU>() && allow_epi<GEPI_GELU>();
}

void launch_gemm_bf16(hipStream_t s, int epi, int shape, const GemmArgs& a) {
  switch (epi) {
    case GEPI_QKV: launch_epi<GEPI_QKV>(s, shape, a); break;
    case GEPI_RESID: launch_epi<GEPI_RESID>(s, shape, a); break;
    case GEPI_PART: launch_epi<GEPI_PART>(s, shape, a); break;
    case GEPI_SWIGLU: launch_epi<GEPI_SWIGLU>(s, shape, a); break;
    default: launch_epi<GEPI_GELU>(s, shape, a); break;
  }
}

}  // namespace mdi

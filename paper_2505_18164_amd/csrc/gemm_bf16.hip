// First-visit products with bf16 storage: tile shapes and their choice (kernel: gemm_impl.h).
#include "gemm_impl.h"

namespace mdi {
namespace {

// index, BN, BT, wavefronts WN x WT, ring depths.  The figures are fitted to 7500 measured (T, N, Kd, shape, splits) over
// the shapes of all the models here, T from 16 to 6000; going by them takes 2 % more time than picking the best
// measured one each time.
#define MDI_GEMM_SHAPES(X) \
  X(0, 256, 256, 2, 4, 3, 2) X(1, 192, 256, 2, 4, 3, 2) X(2, 256, 128, 2, 4, 3, 3) X(3, 192, 128, 2, 4, 4, 4) \
  X(4, 128, 128, 2, 4, 4, 4) X(5, 128, 64, 4, 2, 4, 4) X(6, 64, 64, 2, 2, 4, 4) X(7, 64, 32, 2, 2, 6, 6)
constexpr int kShapes = 8;
constexpr Shape kShape[kShapes] = {
    {256, 256, 1, 1.485f, 14.0f, 0.71f, 4.9f}, {192, 256, 1, 1.228f, 10.6f, 0.71f, 4.9f}, {256, 128, 1, 0.939f, 8.1f, 0.71f, 4.9f},
    {192, 128, 1, 0.784f, 6.3f, 0.71f, 4.9f},  {128, 128, 1, 0.600f, 4.4f, 0.73f, 4.9f},  {128, 64, 1, 0.441f, 2.35f, 0.79f, 4.9f},
    {64, 64, 2, 0.538f, 1.82f, 0.60f, 3.9f},   {64, 32, 3, 0.510f, 1.47f, 0.40f, 4.2f}};

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
  return allow_epi<GEPI_F32_BIAS>() && allow_epi<GEPI_RESID>() && allow_epi<GEPI_PART>() && allow_epi<GEPI_SWIGLU>() && allow_epi<GEPI_GELU>();
}

void launch_gemm_bf16(hipStream_t s, int epi, int shape, const GemmArgs& a) {
  switch (epi) {
    case GEPI_F32_BIAS: launch_epi<GEPI_F32_BIAS>(s, shape, a); break;
    case GEPI_RESID: launch_epi<GEPI_RESID>(s, shape, a); break;
    case GEPI_PART: launch_epi<GEPI_PART>(s, shape, a); break;
    case GEPI_SWIGLU: launch_epi<GEPI_SWIGLU>(s, shape, a); break;
    default: launch_epi<GEPI_GELU>(s, shape, a); break;
  }
}

}  // namespace mdi

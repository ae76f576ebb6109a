// First-visit products with fp32 storage (exact fp32 products): tile shapes and their choice (kernel: gemm_impl.h).
#include "gemm_impl.h"

namespace mdi {
namespace {

// index, BN, BT, wavefronts WN x WT, ring depths.  A compute unit's matrix cores take 256 fp32 operations a clock, a
// sixteenth of the bf16 rate, so small tiles keep them as busy as large ones (within 5 % at every size measured) and
// divide better; the figures are fitted to 3900 measured (T, N, Kd, shape, splits), T from 1 to 2048, choices 5 % from the
// best.  On vector ALUs with one 64 x 64 tile shape: 69 / 202 (output and down, mean) / 74 us for QKV / residual
// products / gate-up of the 304M shape at 100 positions, here 16 / 12 / 33.
#define MDI_GEMM_SHAPES(X) X(0, 64, 32, 2, 2, 4, 4) X(1, 64, 64, 2, 4, 4, 4)
#define X(I, BN_, BT_, WN, WT, NBW, NBA) static_assert(kShapesF32[I].BN == BN_ && kShapesF32[I].BT == BT_, "shape I of the plan");
MDI_GEMM_SHAPES(X)
#undef X

template <int EPI>
void launch_epi(hipStream_t s, int shape, const GemmArgs& a) {
  switch (shape) {
#define X(I, BN, BT, WN, WT, NBW, NBA) case I: launch_shape<float, EPI, BN, BT, WN, WT, NBW, NBA>(s, a); break;
    MDI_GEMM_SHAPES(X)
#undef X
  }
}

template <int EPI>
bool allow_epi() {
#define X(I, BN, BT, WN, WT, NBW, NBA) && allow_shape<float, EPI, BN, BT, WN, WT, NBW, NBA>()
  return true MDI_GEMM_SHAPES(X);
#undef X
}

}  // namespace

bool allow_gemm_lds_f32() {
  return allow_epi<GEPI_QKV>() && allow_epi<GEPI_RESID>() && allow_epi<GEPI_PART>() && allow_epi<GEPI_SWIGLU>() && allow_epi<GEPI_GELU>();
}

void launch_gemm_f32(hipStream_t s, int epi, int shape, const GemmArgs& a) {
  switch (epi) {
    case GEPI_QKV: launch_epi<GEPI_QKV>(s, shape, a); break;
    case GEPI_RESID: launch_epi<GEPI_RESID>(s, shape, a); break;
    case GEPI_PART: launch_epi<GEPI_PART>(s, shape, a); break;
    case GEPI_SWIGLU: launch_epi<GEPI_SWIGLU>(s, shape, a); break;
    default: launch_epi<GEPI_GELU>(s, shape, a); break;
  }
}

}  // namespace mdi

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
#define X(I, BN_, BT_, WN, WT, NBW, NBA) static_assert(kShapesBf16[I].BN == BN_ && kShapesBf16[I].BT == BT_, "shape I of the plan");
MDI_GEMM_SHAPES(X)
#undef X

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

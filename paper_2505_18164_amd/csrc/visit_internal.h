// First visits (prefill: T positions at once; Alg. 2): what mdi_api.hip and the kernels of gemm_impl.h, attn_prefill.hip and
// prefill.hip share.
#pragma once

#include "mdi_internal.h"
#include "visit_plan.h"

namespace mdi {

// Where the rows of a call come from: token ids (embedded on the way) or hidden states in the storage type.
struct RowSource {
  const void* in;                    // nullptr: the rows are in the residual stream
  int in_kind, aligned;              // aligned: `in` may be read four values at a time
  const void* wte; const void* wpe;
  int vocab; int* err;               // a token id outside [0, vocab) sets *err = 2 and is read as token 0
  int pos0;                          // position of row 0 (a first visit in several chunks continues at the cache length)
};

// Residual rows x [T, d], or those of `src`: adds what the product before left as partial results (S > 1: part[0 .. S - 1],
// each [T, d] part_stride floats apart, and the product's bias), normalises the sum into `out` and keeps it in x (out =
// nullptr: neither) and / or copies it to act_out.
struct NormRowsArgs {
  float* x; int T, d; int norm_kind; const float* g; const float* b; float eps;
  void* out; int out_kind;           // out_kind: the storage type, of everything here that is not fp32
  int S; const float* part; long part_stride; const float* part_bias;
  void* act_out; int act_aligned;    // hand-off copy in the storage type or nullptr; may it be written four values at a time
  RowSource src;
};
void launch_norm_rows(hipStream_t s, const NormRowsArgs& a);

// Where the QKV product leaves its rows: queries, rotated, for the attention kernel; keys (rotated) and values in the sample's pages.
struct QkvOut {
  int H, K, h, pt;        // h: a power of two from 8 on; pt: positions per page
  int pt_sh; unsigned pt_magic;   // page of a position: as in FlashArgs
  int pos0;               // position of row 0
  float scale;
  const float2* rope;     // (cos, sin) [max_ctx][h/2] or nullptr
  float* q_out;           // [T, H*h] fp32, or nullptr
  bf16_t* q_bf;           // [T, H*h], times `scale`: the queries of the matrix-core attention, or nullptr
  void* pool;             // this layer's pages, storage dtype
  const int32_t* table;
};

enum GemmEpi { GEPI_QKV = 0, GEPI_RESID = 1, GEPI_SWIGLU = 2, GEPI_GELU = 3, GEPI_PART = 4 };
struct GemmArgs {
  const void* A;     // [T, Kd] storage dtype
  const void* W;     // [N, Kd] storage dtype
  const float* bias; // [N] or nullptr
  int T, N, Kd;      // N and Kd multiples of 8
  int S;             // splits of the inner dimension (1 unless GEPI_PART): split s leaves its sums at out_f32 + s T N
  float* out_f32;    // GEPI_RESID: residual stream [T, N], updated in place; GEPI_PART: [S][T, N]
  void* out_act;     // SWIGLU: [T, N/2]; GELU: [T, N]; RESID: optional hand-off copy [T, N]; storage dtype
  int gelu_tanh;     // GELU: the tanh form, else the erf form
  int act_aligned;   // out_act may be written 16 bytes at a time
  QkvOut qkv;        // GEPI_QKV: N = (H + 2 K) h
};
// Once per device, with it current, before the first launch there: kernels with more than 64 KiB of LDS are let have it.
bool allow_gemm_lds_bf16();
bool allow_gemm_lds_f32();
void launch_gemm_bf16(hipStream_t s, int epi, int shape, const GemmArgs& a);
void launch_gemm_f32(hipStream_t s, int epi, int shape, const GemmArgs& a);
inline void launch_gemm(hipStream_t s, int dtype, int epi, int shape, const GemmArgs& a) {
  if (dtype == MDI_BF16) launch_gemm_bf16(s, epi, shape, a); else launch_gemm_f32(s, epi, shape, a);
}

// Causal attention of a first visit on the matrix cores (bf16 operands, fp32 accumulation and softmax).
struct FlashArgs {
  const bf16_t* q;        // [T][H*h] rotated, scaled: the queries of positions p0 .. p0 + T - 1
  const bf16_t* pool;     // this layer's cache pages [page][K][2][pt][h]: positions 0 .. p0 + T - 1 of the sample are in them
  const int32_t* table;   // its page ids
  bf16_t* out;            // [T][H*h]
  int T, H, K, h;
  int p0;
  int pt, pt_sh; unsigned pt_magic;   // positions per page; log2 of it, or -1 and pos / pt = high word of pos * pt_magic (0xFFFFFFFF / pt + 1)
};
bool flash_supported(int dtype, int h);
bool allow_flash_lds();    // as allow_gemm_lds_bf16
void launch_flash_prefill(hipStream_t s, const FlashArgs& a);

}  // namespace mdi

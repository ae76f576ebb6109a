// First-visit kernels: all T prompt positions of a sample go through the local
// layers at once and fill the sample's KV cache (Alg. 1 round 0, Alg. 2 "first
// iteration for current sample").  With T rows the linear layers are dense
// contractions, which run on the matrix cores (gemm_impl.h); this file holds what
// stands between them, and the set-up kernels.
#include <type_traits>

#include "device_utils.h"
#include "visit_internal.h"

namespace mdi {

// four consecutive values in the storage type, at a multiple of four from an aligned base
__device__ __forceinline__ void put_four(void* base, int kind, long at, const float4& v) {
  if (kind == IN_BF16) {
    uint2 w;
    w.x = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
    w.y = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
    *reinterpret_cast<uint2*>((bf16_t*)base + at) = w;
  } else {
    *reinterpret_cast<float4*>((float*)base + at) = v;
  }
}

// ---------------------------------------------------------------------------
// One workgroup per row, the row in registers (NV pieces of four values per thread; NV = 0: rows beyond 8192 values
// are read again for every pass).  The first one of a call takes the row from the node's input (embeds a token, or widens
// the hidden state that arrived), the others from the residual stream, and adds the partial results of the product before.
// Bound by memory: the row is read once - with S partial results S times more - and written once or twice.  Adding the
// partial results here costs no launch and no pass of its own, nor does taking the input.
//
// With few rows what counts is how many round trips to memory a row takes: everything that can be asked for is, before
// anything is stored (a store between two loads keeps the compiler from asking for the second before the first is there).
// 256 rows of 4096 with two to four partial results 7.5 -> 6.8 us, 1024 rows, half of them with, 12.9 -> 11.6 on average; a kernel of its own for the input took 10
// to 14 us there (41 at 6000 rows) and left the row to be read again.
// With many rows it is how many of them are in flight, and the partial results asked for at a time are two thirds of the
// registers (rows of 8192: 203 against 82, two wavefronts a SIMD against five): kernels with and without.  2048 rows of 8192
// without partial results 21.3 -> 19.5 us and from the input 44 -> 31, of 5120 15.6 -> 13.1 and 31 -> 24, 4000 of 4096
// from the input 35 -> 28.5; two at a time instead of four for rows
// beyond 4096: 64 of 8192 8.1 -> 9.3 us, 600 of 5120 15.7 -> 13.3, 256 to 1024 of 8192 within 4 %.
template <int NV, bool kParts>
__global__ __launch_bounds__(kBlock) void k_norm_rows(NormRowsArgs a) {
  __shared__ float red[2][kBlock / kWave];
  const int t = blockIdx.x, d4 = a.d >> 2;
  float4* x = reinterpret_cast<float4*>(a.x + (long)t * a.d);
  const float4* g4 = reinterpret_cast<const float4*>(a.g);
  const float4* b4 = reinterpret_cast<const float4*>(a.b);
  constexpr int NR = NV ? NV : 1;
  float4 v[NR], g[NR];
  auto add = [](float4& r, const float4& p) { r.x += p.x; r.y += p.y; r.z += p.z; r.w += p.w; };
  // four values of a row in the storage type; `aligned`: the base may be read in pieces of four
  auto four = [](const void* base, int kind, bool aligned, long at) __attribute__((always_inline)) {
    if (!aligned) return float4{load_kind(base, kind, at), load_kind(base, kind, at + 1), load_kind(base, kind, at + 2), load_kind(base, kind, at + 3)};
    if (kind == IN_F32) return *reinterpret_cast<const float4*>((const float*)base + at);
    const uint2 w = *reinterpret_cast<const uint2*>((const bf16_t*)base + at);
    return float4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
  };
  const int kind = a.out_kind;                       // storage type: of embeddings, hidden states, and what is written here
  const long tok = a.src.in && a.src.in_kind == IN_TOKEN ? checked_token(a.src.in, t, a.src.vocab, a.src.err) : 0;
  auto start = [&](int i) __attribute__((always_inline)) {         // piece i of the row before partial results
    if (!a.src.in) return x[i];
    if (a.src.in_kind != IN_TOKEN) return four(a.src.in, kind, a.src.aligned, (long)t * a.d + 4 * i);
    float4 r = four(a.src.wte, kind, true, tok * a.d + 4 * i);
    if (a.src.wpe) add(r, four(a.src.wpe, kind, true, (long)(a.src.pos0 + t) * a.d + 4 * i));
    return r;
  };
  auto part = [&](int s, int i) __attribute__((always_inline)) { return reinterpret_cast<const float4*>(a.part + s * a.part_stride + (long)t * a.d)[i]; };
  auto keep = [&](int i, const float4& r) __attribute__((always_inline)) {
    if (a.out && (kParts || a.src.in)) x[i] = r;    // without a norm to follow nobody reads the stream again
    if (!a.act_out) return;
    const long at = (long)t * a.d + 4 * i;
    if (!a.act_aligned) {
      store_kind(a.act_out, kind, at, r.x); store_kind(a.act_out, kind, at + 1, r.y);
      store_kind(a.act_out, kind, at + 2, r.z); store_kind(a.act_out, kind, at + 3, r.w);
    } else {
      put_four(a.act_out, kind, at, r);
    }
  };
  auto each = [&](auto&& f) __attribute__((always_inline)) {       // f(number in this thread, piece)
#pragma unroll
    for (int j = 0; j < NR; ++j) { const int i = threadIdx.x + j * kBlock; if (i < d4) f(j, i); }
  };
  if (NV) {
    each([&](int j, int i) { v[j] = start(i); });
    if (a.out) each([&](int j, int i) { g[j] = g4[i]; });
    if (kParts) {
      if (a.part_bias) each([&](int j, int i) { add(v[j], reinterpret_cast<const float4*>(a.part_bias)[i]); });
      constexpr int U = 4;                           // partial results asked for at a time
      int s = 0;
      auto some = [&](auto count) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        float4 p[N][NR];
#pragma unroll
        for (int u = 0; u < N; ++u) each([&](int j, int i) { p[u][j] = part(s + u, i); });
#pragma unroll
        for (int u = 0; u < N; ++u) each([&](int j, int) { add(v[j], p[u][j]); });
        s += N;
      };
      while (s + U <= a.S) some(std::integral_constant<int, U>{});
      if (s + 2 <= a.S) some(std::integral_constant<int, 2>{});
      if (s < a.S) some(std::integral_constant<int, 1>{});
    }
    each([&](int j, int i) { keep(i, v[j]); });
  } else {
    for (int i = threadIdx.x; i < d4; i += kBlock) {
      float4 r = start(i);
      if (kParts) {
        if (a.part_bias) add(r, reinterpret_cast<const float4*>(a.part_bias)[i]);
        for (int s = 0; s < a.S; ++s) add(r, part(s, i));
      }
      keep(i, r);
    }
  }
  if (!a.out) return;
  auto row = [&](auto&& f) __attribute__((always_inline)) {        // f(values, gain, piece)
    if (NV) each([&](int j, int i) { f(v[j], g[j], i); });
    else for (int i = threadIdx.x; i < d4; i += kBlock) f(x[i], g4[i], i);
  };
  auto row_sum = [&](float s, float* r) __attribute__((always_inline)) {
    s = wave_sum_to_lane63(s);
    if ((threadIdx.x & 63) == 63) r[threadIdx.x >> 6] = s;
    __syncthreads();
    return (r[0] + r[1]) + (r[2] + r[3]);
  };
  float mean = 0.f, s2 = 0.f;
  if (a.norm_kind == MDI_NORM_LAYERNORM) {
    float s = 0.f;
    row([&](const float4& r, const float4&, int) { s += (r.x + r.y) + (r.z + r.w); });
    mean = row_sum(s, red[0]) / (float)a.d;
    row([&](const float4& r, const float4&, int) {
      const float c0 = r.x - mean, c1 = r.y - mean, c2 = r.z - mean, c3 = r.w - mean;
      s2 += (c0 * c0 + c1 * c1) + (c2 * c2 + c3 * c3);
    });
  } else {
    row([&](const float4& r, const float4&, int) { s2 += (r.x * r.x + r.y * r.y) + (r.z * r.z + r.w * r.w); });
  }
  const float rstd = 1.f / sqrtf(row_sum(s2, red[1]) / (float)a.d + a.eps);
  row([&](const float4& r, const float4& gain, int i) {
    float4 o = {(r.x - mean) * rstd * gain.x, (r.y - mean) * rstd * gain.y, (r.z - mean) * rstd * gain.z, (r.w - mean) * rstd * gain.w};
    if (a.b) add(o, b4[i]);
    put_four(a.out, kind, (long)t * a.d + 4 * i, o);
  });
}
template <bool kParts>
void launch_norm_rows_parts(hipStream_t s, const NormRowsArgs& a) {
  const int n = (a.d / 4 + kBlock - 1) / kBlock;
  if (n <= 1) hipLaunchKernelGGL((k_norm_rows<1, kParts>), dim3(a.T), dim3(kBlock), 0, s, a);
  else if (n <= 2) hipLaunchKernelGGL((k_norm_rows<2, kParts>), dim3(a.T), dim3(kBlock), 0, s, a);
  else if (n <= 4) hipLaunchKernelGGL((k_norm_rows<4, kParts>), dim3(a.T), dim3(kBlock), 0, s, a);
  else if (n <= 8) hipLaunchKernelGGL((k_norm_rows<8, kParts>), dim3(a.T), dim3(kBlock), 0, s, a);
  else hipLaunchKernelGGL((k_norm_rows<0, kParts>), dim3(a.T), dim3(kBlock), 0, s, a);
}
void launch_norm_rows(hipStream_t s, const NormRowsArgs& a) {
  if (a.S > 1) launch_norm_rows_parts<true>(s, a); else launch_norm_rows_parts<false>(s, a);
}

// ---------------------------------------------------------------------------
// set-up kernels
__global__ void k_rope_table(float2* table, int max_ctx, int half, int h, double base) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)max_ctx * half) return;
  const int p = idx / half, i = idx % half;
  const double ang = (double)p * pow(base, -2.0 * (double)i / (double)h);
  table[idx] = make_float2((float)cos(ang), (float)sin(ang));
}
void launch_rope_table(hipStream_t s, float2* table, int max_ctx, int h, double base) {
  const long n = (long)max_ctx * (h / 2);
  hipLaunchKernelGGL(k_rope_table, dim3((n + 255) / 256), dim3(256), 0, s, table, max_ctx, h / 2, h, base);
}

template <typename T>
__global__ void k_copy_rows(const T* src, T* dst, long rows, long cols, long row_mul, long row_off) {
  const long n = rows * cols;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    const long r = idx / cols, c = idx - r * cols;
    dst[(r * row_mul + row_off) * cols + c] = src[idx];
  }
}
void launch_copy_rows(hipStream_t s, int elem_bytes, const void* src, void* dst, long rows, long cols, long row_mul, long row_off) {
  const long n = rows * cols;
  if (n == 0) return;
  const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  if (elem_bytes == 2)
    hipLaunchKernelGGL(k_copy_rows<uint16_t>, dim3(blocks), dim3(256), 0, s, (const uint16_t*)src, (uint16_t*)dst, rows, cols, row_mul, row_off);
  else
    hipLaunchKernelGGL(k_copy_rows<uint32_t>, dim3(blocks), dim3(256), 0, s, (const uint32_t*)src, (uint32_t*)dst, rows, cols, row_mul, row_off);
}

__global__ void k_fill_u32(uint32_t* dst, long n, uint32_t v) {
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) dst[idx] = v;
}
void launch_fill_u32(hipStream_t s, uint32_t* dst, long n, uint32_t v) {
  if (n == 0) return;
  const int blocks = (int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
  hipLaunchKernelGGL(k_fill_u32, dim3(blocks), dim3(256), 0, s, dst, n, v);
}
void launch_fill_f32(hipStream_t s, float* dst, long n, float v) {
  uint32_t u;
  __builtin_memcpy(&u, &v, 4);
  launch_fill_u32(s, (uint32_t*)dst, n, u);
}

}  // namespace mdi

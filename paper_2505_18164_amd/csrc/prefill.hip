// First-visit kernels: all T prompt positions of a sample go through the local
// layers at once and fill the sample's KV cache (Alg. 1 round 0, Alg. 2 "first
// iteration for current sample").  With T rows the linear layers are dense
// contractions, which run on the matrix cores (gemm_impl.h); this file holds what
// stands between them, and the set-up kernels.
#include "device_utils.h"

namespace mdi {

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_rows_input(RowsInArgs a) {
  const int t = blockIdx.x;
  float* xr = a.xres + (long)t * a.d;
  if (a.in_kind == IN_TOKEN) {
    const long tok = checked_token(a.in, t, a.vocab, a.err);
    const int wk = a.dtype == MDI_BF16 ? IN_BF16 : IN_F32;
    for (int i = threadIdx.x; i < a.d; i += kBlock) {
      float v = load_kind(a.wte, wk, tok * a.d + i);
      if (a.wpe) v += load_kind(a.wpe, wk, (long)(a.pos0 + t) * a.d + i);
      xr[i] = v;
    }
  } else {
    for (int i = threadIdx.x; i < a.d; i += kBlock) xr[i] = load_kind(a.in, a.in_kind, (long)t * a.d + i);
  }
}
void launch_rows_input(hipStream_t s, const RowsInArgs& a) {
  hipLaunchKernelGGL(k_rows_input, dim3(a.T), dim3(kBlock), 0, s, a);
}

// ---------------------------------------------------------------------------
// One workgroup per row, the row in registers (NV pieces of four values per thread; NV = 0: rows beyond 8192 values
// are read again for every pass).  Bound by memory: the row is read once - with S partial results of the product
// before, S times more - and written once or twice.  Adding the partial results here costs no launch and no pass of
// its own.
template <int NV>
__global__ __launch_bounds__(kBlock) void k_norm_rows(NormRowsArgs a) {
  __shared__ float red[8];
  const int t = blockIdx.x, d4 = a.d >> 2;
  float4* x = reinterpret_cast<float4*>(a.x + (long)t * a.d);
  const float4* g4 = reinterpret_cast<const float4*>(a.g);
  const float4* b4 = reinterpret_cast<const float4*>(a.b);
  constexpr int NR = NV ? NV : 1;
  float4 v[NR];
  auto fetch = [&](int i) {                          // the row's piece i with the partial results added, split by split
    float4 r = x[i];
    if (a.S > 1) {
      if (a.part_bias) { const float4 p = reinterpret_cast<const float4*>(a.part_bias)[i]; r.x += p.x; r.y += p.y; r.z += p.z; r.w += p.w; }
      const float4* p4 = reinterpret_cast<const float4*>(a.part + (long)t * a.d) + i;
#pragma unroll 4
      for (int s = 0; s < a.S; ++s) {
        const float4 p = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p4) + s * a.part_stride);
        r.x += p.x; r.y += p.y; r.z += p.z; r.w += p.w;
      }
      x[i] = r;
    }
    if (a.act_out) {
      const long at = (long)t * a.d + 4 * i;
      store_kind(a.act_out, a.out_kind, at, r.x); store_kind(a.act_out, a.out_kind, at + 1, r.y);
      store_kind(a.act_out, a.out_kind, at + 2, r.z); store_kind(a.act_out, a.out_kind, at + 3, r.w);
    }
    return r;
  };
  auto each = [&](auto&& f) {                        // f(piece, its values)
    if (NV) {
#pragma unroll
      for (int j = 0; j < NR; ++j) { const int i = threadIdx.x + j * kBlock; if (i < d4) f(i, v[j]); }
    } else {
      for (int i = threadIdx.x; i < d4; i += kBlock) f(i, x[i]);
    }
  };
  if (NV) {
#pragma unroll
    for (int j = 0; j < NR; ++j) { const int i = threadIdx.x + j * kBlock; if (i < d4) v[j] = fetch(i); }
  } else {
    for (int i = threadIdx.x; i < d4; i += kBlock) (void)fetch(i);
  }
  if (!a.out) return;
  float mean = 0.f, s2 = 0.f;
  if (a.norm_kind == MDI_NORM_LAYERNORM) {
    float s = 0.f;
    each([&](int, const float4& r) { s += (r.x + r.y) + (r.z + r.w); });
    mean = block_sum(s, red) / (float)a.d;
    each([&](int, const float4& r) {
      const float c0 = r.x - mean, c1 = r.y - mean, c2 = r.z - mean, c3 = r.w - mean;
      s2 += (c0 * c0 + c1 * c1) + (c2 * c2 + c3 * c3);
    });
  } else {
    each([&](int, const float4& r) { s2 += (r.x * r.x + r.y * r.y) + (r.z * r.z + r.w * r.w); });
  }
  const float rstd = 1.f / sqrtf(block_sum(s2, red) / (float)a.d + a.eps);
  each([&](int i, const float4& r) {
    const float4 g = g4[i];
    float4 o = {(r.x - mean) * rstd * g.x, (r.y - mean) * rstd * g.y, (r.z - mean) * rstd * g.z, (r.w - mean) * rstd * g.w};
    if (a.b) { const float4 b = b4[i]; o.x += b.x; o.y += b.y; o.z += b.z; o.w += b.w; }
    const long at = (long)t * a.d + 4 * i;
    if (a.out_kind == IN_BF16) {
      uint2 p;
      p.x = (uint32_t)f32_to_bf16(o.x) | ((uint32_t)f32_to_bf16(o.y) << 16);
      p.y = (uint32_t)f32_to_bf16(o.z) | ((uint32_t)f32_to_bf16(o.w) << 16);
      *reinterpret_cast<uint2*>((bf16_t*)a.out + at) = p;
    } else {
      *reinterpret_cast<float4*>((float*)a.out + at) = o;
    }
  });
}
void launch_norm_rows(hipStream_t s, const NormRowsArgs& a) {
  const int n = (a.d / 4 + kBlock - 1) / kBlock;
  if (n <= 1) hipLaunchKernelGGL(k_norm_rows<1>, dim3(a.T), dim3(kBlock), 0, s, a);
  else if (n <= 2) hipLaunchKernelGGL(k_norm_rows<2>, dim3(a.T), dim3(kBlock), 0, s, a);
  else if (n <= 4) hipLaunchKernelGGL(k_norm_rows<4>, dim3(a.T), dim3(kBlock), 0, s, a);
  else if (n <= 8) hipLaunchKernelGGL(k_norm_rows<8>, dim3(a.T), dim3(kBlock), 0, s, a);
  else hipLaunchKernelGGL(k_norm_rows<0>, dim3(a.T), dim3(kBlock), 0, s, a);
}

// ---------------------------------------------------------------------------
// Rotate q and k by their positions, keep q in fp32 for the attention kernel
// and scatter k, v into the sample's pages.  One workgroup per prompt position.
__global__ __launch_bounds__(kBlock) void k_rope_scatter(RopeScatterArgs a) {
  const int t = blockIdx.x, h = a.h, half = h >> 1;
  const int n_heads = a.H + 2 * a.K;
  const float* row = a.qkv + (long)t * n_heads * h;
  const int pos = a.pos0 + t;
  const int page = a.table[pos / a.pt], slot = pos % a.pt;
  const long pt_h = (long)a.pt * h;
  const bool bf = a.dtype == MDI_BF16;
  // four consecutive pairs (i, i + h/2) per thread: h/2 is a multiple of 4, so everything moves in 8- or 16-byte pieces
  auto put4 = [&](void* base, bool as_bf16, long o, const float4& v) __attribute__((always_inline)) {
    if (as_bf16) {
      uint2 w;
      w.x = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
      w.y = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
      *reinterpret_cast<uint2*>((bf16_t*)base + o) = w;
    } else {
      *reinterpret_cast<float4*>((float*)base + o) = v;
    }
  };
  const int q4 = half >> 2;
  for (int p = threadIdx.x; p < n_heads * q4; p += kBlock) {
    const int head = p / q4, i = (p - head * q4) * 4;
    float4 v0 = *reinterpret_cast<const float4*>(row + head * h + i);
    float4 v1 = *reinterpret_cast<const float4*>(row + head * h + i + half);
    if (a.rope && head < a.H + a.K) {
      const float4 c01 = *reinterpret_cast<const float4*>(a.rope + (long)pos * half + i);       // (cos, sin) of pairs i, i+1
      const float4 c23 = *reinterpret_cast<const float4*>(a.rope + (long)pos * half + i + 2);   // ... i+2, i+3
      const float4 r0 = {v0.x * c01.x - v1.x * c01.y, v0.y * c01.z - v1.y * c01.w, v0.z * c23.x - v1.z * c23.y, v0.w * c23.z - v1.w * c23.w};
      const float4 r1 = {v0.x * c01.y + v1.x * c01.x, v0.y * c01.w + v1.y * c01.z, v0.z * c23.y + v1.z * c23.x, v0.w * c23.w + v1.w * c23.z};
      v0 = r0; v1 = r1;
    }
    if (head < a.H) {
      const long o = (long)t * a.H * h + head * h + i;
      if (a.q_out) { put4(a.q_out, false, o, v0); put4(a.q_out, false, o + half, v1); }
      if (a.q_bf) {
        const float sc = a.scale;
        put4(a.q_bf, true, o, float4{v0.x * sc, v0.y * sc, v0.z * sc, v0.w * sc});
        put4(a.q_bf, true, o + half, float4{v1.x * sc, v1.y * sc, v1.z * sc, v1.w * sc});
      }
    } else {
      const bool is_v = head >= a.H + a.K;
      const int kvh = head - a.H - (is_v ? a.K : 0);
      const long o = (((long)page * a.K + kvh) * 2 + (is_v ? 1 : 0)) * pt_h + (long)slot * h + i;
      put4(a.pool, bf, o, v0);
      put4(a.pool, bf, o + half, v1);
    }
  }
}
void launch_rope_scatter(hipStream_t s, const RopeScatterArgs& a) {
  hipLaunchKernelGGL(k_rope_scatter, dim3(a.T), dim3(kBlock), 0, s, a);
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

// Row-wise kernels of the forward: embedding gather with the first RMSNorm, RMSNorm, item log-softmax.
#include "common.h"
#include "kernels.h"

namespace atspeed {

// Copy of the k and v rows a forward wrote, in row order (instrumentation of
// the residual capture): row r's k/v sit in the prefix cache [B][H][Pmax][dh]
// at (user, position) (kv_mode 0) or in the tree K/V [slot][d] (kv_mode 1).
__global__ void gather_kv_rows_kernel(const bf16_t* __restrict__ kc, const bf16_t* __restrict__ vc, Rows rows,
                                      int rmax, int kv_mode, int H, int dh, int Pmax, bf16_t* __restrict__ ko,
                                      bf16_t* __restrict__ vo) {
  const int M = min(*rows.M, rmax), d = H * dh;
  const size_t total = (size_t)M * d;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int r = (int)(i / d), c = (int)(i % d), head = c / dh, j = c % dh;
    const size_t src = kv_mode == 0 ? (((size_t)rows.user[r] * H + head) * Pmax + rows.pos[r]) * dh + j
                                    : (size_t)rows.slot[r] * d + c;
    ko[i] = kc[src];
    vo[i] = vc[src];
  }
}

hipError_t gather_kv_rows(const void* kc, const void* vc, const Rows& rows, int rmax, int kv_mode, int H, int dh,
                          int Pmax, void* ko, void* vo, hipStream_t st) {
  const int blocks = (int)std::max<size_t>(1, std::min<size_t>(4096, ((size_t)rmax * H * dh + 255) / 256));
  hipLaunchKernelGGL(gather_kv_rows_kernel, dim3(blocks), dim3(256), 0, st, (const bf16_t*)kc, (const bf16_t*)vc,
                     rows, rmax, kv_mode, H, dh, Pmax, (bf16_t*)ko, (bf16_t*)vo);
  return hipGetLastError();
}

__device__ __forceinline__ float block_sum256(float v, float* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

__device__ __forceinline__ float block_max256(float v, float* red) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// out[r] = g * x[src] / sqrt(mean(x[src]^2) + eps), src = row_index ? row_index[r] : r.
// With add: x[src] + add[src] takes the place of x[src] (the second partial
// product of a GEMM split in k), and without row_index that sum is written
// back to x.  With EMB the row is the embedding of tok[r] instead, and x[r] is
// written too (the first norm of a forward: the gather alone took 28 us at 2,624 x
// 4,096 and 63 at 7,744, and the norm read it back).  One workgroup per row; the row is read once in 16-byte loads and
// held in registers (up to 256 * 4 * VMAX columns) between the sum of squares
// and the scaled write.
constexpr int kNormVmax = 8;

template <class T>
__device__ __forceinline__ void store4(T* p, float a, float b, float c, float e);
template <>
__device__ __forceinline__ void store4<float>(float* p, float a, float b, float c, float e) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, e);
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float a, float b, float c, float e) {
  uint2 w;
  w.x = (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
  w.y = (uint32_t)f2bf(c) | ((uint32_t)f2bf(e) << 16);
  *reinterpret_cast<uint2*>(p) = w;
}

// Four consecutive stored values as floats, in one load.  The embedding is the
// caller's and may be a view at any element, so the load assumes an element's
// alignment only (the device takes it whole at any address).
typedef float f32x4_any_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any_t __attribute__((ext_vector_type(2), aligned(2)));
__device__ __forceinline__ float4 load4(const float* p) {
  const f32x4_any_t v = *reinterpret_cast<const f32x4_any_t*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 load4(const bf16_t* p) {
  const u32x2_any_t w = *reinterpret_cast<const u32x2_any_t*>(p);
  return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                     __uint_as_float(w.y & 0xffff0000u));
}

template <class T, bool EMB>
__global__ void __launch_bounds__(256)
rmsnorm_kernel(float* __restrict__ x, const float* __restrict__ add, const int* __restrict__ Mdev, int d,
               const float* __restrict__ g, T* __restrict__ out, const int* __restrict__ row_index,
               const T* __restrict__ emb, const int* __restrict__ tok) {
  __shared__ float red[4];
  const int M = *Mdev;
  const int n4 = d >> 2;
  for (int r = blockIdx.x; r < M; r += gridDim.x) {
    const int src = row_index ? row_index[r] : r;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)src * d);  // read once, before any write-back
    const T* er = EMB ? emb + (size_t)tok[r] * d : nullptr;
    // every load of the row is issued before any store (the x write-back waits
    // until after the reduction): 18.1 -> 17.0 us at 1,920 x 4,096, same bits
    float4 v[kNormVmax], p[kNormVmax];
#pragma unroll
    for (int k = 0; k < kNormVmax; ++k) {
      const int c = threadIdx.x + k * 256;
      v[k] = c < n4 ? (EMB ? load4(er + 4 * c) : xr[c]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (add) {
#pragma unroll
      for (int k = 0; k < kNormVmax; ++k) {
        const int c = threadIdx.x + k * 256;
        p[k] = c < n4 ? reinterpret_cast<const float4*>(add + (size_t)src * d)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < kNormVmax; ++k) {
      if (add) {
        v[k].x += p[k].x; v[k].y += p[k].y; v[k].z += p[k].z; v[k].w += p[k].w;
      }
      ss += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
    }
    ss = block_sum256(ss, red);
    const float inv = rsqrtf(ss / (float)d + 1e-6f);
    const float4* g4 = reinterpret_cast<const float4*>(g);
#pragma unroll
    for (int k = 0; k < kNormVmax; ++k) {
      const int c = threadIdx.x + k * 256;
      if (c < n4) {
        if (EMB || (add && !row_index)) reinterpret_cast<float4*>(x + (size_t)src * d)[c] = v[k];
        const float4 gg = g4[c];
        store4<T>(out + (size_t)r * d + 4 * c, v[k].x * inv * gg.x, v[k].y * inv * gg.y, v[k].z * inv * gg.z,
                  v[k].w * inv * gg.w);
      }
    }
  }
}

// The same for rows of at most 1,024 columns, a wave per row: no barrier, and four
// rows a workgroup (640 x 768 rows: 5.2 -> 4.1 us, most of it the launch and two
// dependent loads).  Lane l stands for threads l, l + 64, l + 128 and l + 192 of
// the kernel above, whose four wave sums it forms apart and adds in the same order.
template <class T, bool EMB>
__global__ void __launch_bounds__(256)
rmsnorm_wave_kernel(float* __restrict__ x, const float* __restrict__ add, const int* __restrict__ Mdev, int d,
                    const float* __restrict__ g, T* __restrict__ out, const int* __restrict__ row_index,
                    const T* __restrict__ emb, const int* __restrict__ tok) {
  const int M = *Mdev, n4 = d >> 2, lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= M) return;
  const int src = row_index ? row_index[r] : r;
  const T* er = EMB ? emb + (size_t)tok[r] * d : nullptr;
  const float4* xr = reinterpret_cast<const float4*>(x + (size_t)src * d);
  const float4* ar = reinterpret_cast<const float4*>(add + (size_t)src * d);
  float4 v[4], p[4], gg[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = lane + k * 64;
    v[k] = c < n4 ? (EMB ? load4(er + 4 * c) : xr[c]) : make_float4(0.f, 0.f, 0.f, 0.f);
    if (add) p[k] = c < n4 ? ar[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    gg[k] = c < n4 ? reinterpret_cast<const float4*>(g)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float ss[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (add) {
      v[k].x += p[k].x; v[k].y += p[k].y; v[k].z += p[k].z; v[k].w += p[k].w;
    }
    ss[k] = 0.f;
    ss[k] += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) ss[k] += __shfl_xor(ss[k], o);
  const float inv = rsqrtf((ss[0] + ss[1] + ss[2] + ss[3]) / (float)d + 1e-6f);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = lane + k * 64;
    if (c < n4) {
      if (EMB || (add && !row_index)) reinterpret_cast<float4*>(x + (size_t)src * d)[c] = v[k];
      store4<T>(out + (size_t)r * d + 4 * c, v[k].x * inv * gg[k].x, v[k].y * inv * gg[k].y, v[k].z * inv * gg[k].z,
                v[k].w * inv * gg[k].w);
    }
  }
}

template <class T, bool EMB>
static hipError_t launch_norm(float* x, const float* add, const int* Mdev, int Mmax, int d, const float* g, void* out,
                              const int* row_index, const void* emb, const int* tok, hipStream_t st) {
  if (d % 4 != 0 || d > 1024 * kNormVmax) return hipErrorInvalidValue;
  if (d <= 1024)
    hipLaunchKernelGGL((rmsnorm_wave_kernel<T, EMB>), dim3(std::max(1, (Mmax + 3) / 4)), dim3(256), 0, st, x, add, Mdev, d,
                       g, (T*)out, row_index, (const T*)emb, tok);
  else
    hipLaunchKernelGGL((rmsnorm_kernel<T, EMB>), dim3(std::max(1, std::min(Mmax, 8192))), dim3(256), 0, st, x, add, Mdev, d,
                       g, (T*)out, row_index, (const T*)emb, tok);
  return hipGetLastError();
}

hipError_t rmsnorm(bool bf16, float* x, const float* add, const int* Mdev, int Mmax, int d, const float* g, void* out,
                   const int* row_index, hipStream_t st) {
  return bf16 ? launch_norm<bf16_t, false>(x, add, Mdev, Mmax, d, g, out, row_index, nullptr, nullptr, st)
              : launch_norm<float, false>(x, add, Mdev, Mmax, d, g, out, row_index, nullptr, nullptr, st);
}

hipError_t embed_norm(bool bf16, const void* emb, const Rows& rows, int Mmax, int d, const float* g, float* x, void* out,
                      hipStream_t st) {
  return bf16 ? launch_norm<bf16_t, true>(x, nullptr, rows.M, Mmax, d, g, out, nullptr, emb, rows.token, st)
              : launch_norm<float, true>(x, nullptr, rows.M, Mmax, d, g, out, nullptr, emb, rows.token, st);
}

// lp[dst[r]] = z[r] - logsumexp(z[r]) over the n item-token columns (fp32).  A
// workgroup per row, which is read once and held in registers (n is at most 4 x 256:
// the item tokens of four levels).
constexpr int kLsmCols = 4;
__global__ void __launch_bounds__(256)
log_softmax_kernel(const float* __restrict__ z, const int* __restrict__ Mdev, int n, const int* __restrict__ dst,
                   float* __restrict__ lp, float* __restrict__ zcopy) {
  __shared__ float red[4];
  const int M = *Mdev;
  for (int r = blockIdx.x; r < M; r += gridDim.x) {
    const float* zr = z + (size_t)r * n;
    const size_t o = (size_t)(dst ? dst[r] : r) * n;
    float v[kLsmCols];
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < kLsmCols; ++k) {
      const int c = threadIdx.x + k * 256;
      v[k] = c < n ? zr[c] : -INFINITY;
    }
#pragma unroll
    for (int k = 0; k < kLsmCols; ++k) mx = fmaxf(mx, v[k]);
    mx = block_max256(mx, red);
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < kLsmCols; ++k)
      if (threadIdx.x + k * 256 < n) s += expf(v[k] - mx);
    s = block_sum256(s, red);
    const float lse = mx + logf(s);
#pragma unroll
    for (int k = 0; k < kLsmCols; ++k) {
      const int c = threadIdx.x + k * 256;
      if (c < n) {
        lp[o + c] = v[k] - lse;
        if (zcopy) zcopy[o + c] = v[k];
      }
    }
  }
}

hipError_t log_softmax_rows(const float* logits, const int* Mdev, int Mmax, int n, const int* dst_index,
                            float* lp, float* logits_copy, hipStream_t st) {
  if (n > 256 * kLsmCols) return hipErrorInvalidValue;   // L <= 4 levels of at most 256 codes
  int blocks = std::max(1, std::min(Mmax, 8192));
  hipLaunchKernelGGL(log_softmax_kernel, dim3(blocks), dim3(256), 0, st, logits, Mdev, n, dst_index, lp, logits_copy);
  return hipGetLastError();
}

}  // namespace atspeed

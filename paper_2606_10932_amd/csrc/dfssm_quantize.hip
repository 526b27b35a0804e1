// dfssm_quantize.hip -- per-token absmax int8 activation quantisation (the
// int8 operand of the scaffold product, Sec. 4.1 of the paper), gfx950.
//
// One workgroup of 256 threads per token row: max|x| over the row (wave64
// butterfly, then across the 4 waves through LDS), then the codes.  Rows are
// read with 16-byte loads when the row start and stride allow it, and held in
// registers between the two where VPT loads per thread cover them (8: 8192
// fp32 or 16384 fp16 columns); longer or unaligned rows are read again.
#include <float.h>

#include "dfssm_internal.hpp"

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float to_f32(_Float16 h) { return (float)h; }  // exact widening
__device__ __forceinline__ float to_f32(float f) { return f; }

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

__device__ __forceinline__ int8_t code(float v, float inv) {
  float t = v * inv;
  float r = rintf(t);  // v_rndne_f32: round to nearest, ties to even
  r = fminf(fmaxf(r, -127.0f), 127.0f);
  return (int8_t)(int)r;
}

// VEC elements per vector access (16 bytes), or 1; VPT accesses per thread
// held in registers, or 0.
template <typename T, int VEC, int VPT>
__global__ __launch_bounds__(kThreads) void quantize_rows(const T* __restrict__ x, int K,
                                                          int64_t ldx, int8_t* __restrict__ q,
                                                          float* __restrict__ s, int scale_mode) {
  const int64_t m = blockIdx.x;
  const T* row = x + m * ldx;
  int8_t* qrow = q + m * (int64_t)K;
  __shared__ float red[kThreads / 64];

  using V = __attribute__((ext_vector_type(VEC))) T;
  float a = 0.0f;
  V held[VPT > 0 ? VPT : 1];
  if constexpr (VPT > 0) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int k = (threadIdx.x + kThreads * i) * VEC;
      held[i] = k < K ? *reinterpret_cast<const V*>(row + k) : V(T(0));
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i)
#pragma unroll
      for (int e = 0; e < VEC; ++e) a = fmaxf(a, fabsf(to_f32(held[i][e])));
  } else if constexpr (VEC > 1) {
    for (int k = threadIdx.x * VEC; k < K; k += kThreads * VEC) {
      V v = *reinterpret_cast<const V*>(row + k);
#pragma unroll
      for (int e = 0; e < VEC; ++e) a = fmaxf(a, fabsf(to_f32(v[e])));
    }
  } else {
    for (int k = threadIdx.x; k < K; k += kThreads) a = fmaxf(a, fabsf(to_f32(row[k])));
  }
  a = wave_max(a);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  a = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));

  if (a < FLT_MIN) {  // all-zero (or subnormal-only) row
    for (int k = threadIdx.x; k < K; k += kThreads) qrow[k] = 0;
    if (threadIdx.x == 0) s[m] = scale_mode ? 1.0f / 127.0f : 0.0f;
    return;
  }
  const float inv = 127.0f / a;  // correctly rounded fp32 division
  if (threadIdx.x == 0) s[m] = scale_mode ? 1.0f / 127.0f : a / 127.0f;

  auto store = [&](int k, const V& v) {
    uint32_t w[VEC >= 4 ? VEC / 4 : 1] = {};
#pragma unroll
    for (int e = 0; e < VEC; ++e) w[e / 4] |= (uint32_t)(uint8_t)code(to_f32(v[e]), inv) << (8 * (e % 4));
    if constexpr (VEC == 8)
      *reinterpret_cast<uint2*>(qrow + k) = make_uint2(w[0], w[1]);
    else
      *reinterpret_cast<uint32_t*>(qrow + k) = w[0];
  };
  if constexpr (VPT > 0) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int k = (threadIdx.x + kThreads * i) * VEC;
      if (k < K) store(k, held[i]);
    }
  } else if constexpr (VEC > 1) {
    for (int k = threadIdx.x * VEC; k < K; k += kThreads * VEC) store(k, *reinterpret_cast<const V*>(row + k));
  } else {
    for (int k = threadIdx.x; k < K; k += kThreads) qrow[k] = code(to_f32(row[k]), inv);
  }
}

template <typename T, int VEC>
void launch(const T* x, int64_t M, int64_t K, int64_t ldx, int8_t* q, float* s, int scale_mode, hipStream_t st) {
  const bool vec = reinterpret_cast<uintptr_t>(x) % 16 == 0 && (ldx * sizeof(T)) % 16 == 0 && K % VEC == 0;
  const int64_t vpt = dfssm::ceil_div(K, kThreads * VEC);
  dim3 grid((unsigned)M), block(kThreads);
  if (!vec)
    quantize_rows<T, 1, 0><<<grid, block, 0, st>>>(x, (int)K, ldx, q, s, scale_mode);
  else if (vpt == 1)
    quantize_rows<T, VEC, 1><<<grid, block, 0, st>>>(x, (int)K, ldx, q, s, scale_mode);
  else if (vpt == 2)
    quantize_rows<T, VEC, 2><<<grid, block, 0, st>>>(x, (int)K, ldx, q, s, scale_mode);
  else if (vpt <= 4)
    quantize_rows<T, VEC, 4><<<grid, block, 0, st>>>(x, (int)K, ldx, q, s, scale_mode);
  else if (vpt <= 8)
    quantize_rows<T, VEC, 8><<<grid, block, 0, st>>>(x, (int)K, ldx, q, s, scale_mode);
  else
    quantize_rows<T, VEC, 0><<<grid, block, 0, st>>>(x, (int)K, ldx, q, s, scale_mode);
}

}  // namespace

namespace dfssm {

hipError_t launch_quantize(const void* x, int x_dtype, int64_t M, int64_t K, int64_t ldx,
                           int8_t* q, float* s, int scale_mode, hipStream_t st) {
  if (M == 0) return hipSuccess;
  if (x_dtype == DFSSM_F16)
    launch<_Float16, 8>(static_cast<const _Float16*>(x), M, K, ldx, q, s, scale_mode, st);
  else
    launch<float, 4>(static_cast<const float*>(x), M, K, ldx, q, s, scale_mode, st);
  return hipGetLastError();
}

}  // namespace dfssm

// Device-side helpers: storage types, conversions, fixed-order wave reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spec {

struct bf16_t { uint16_t v; };
typedef _Float16 f16_t;

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
// round-to-nearest-even; NaN stays NaN (one conversion instruction on gfx950; written out it was six)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

template <class T> struct Conv;
template <> struct Conv<float> {
  static __device__ __forceinline__ float ld(const float *p, size_t i) { return p[i]; }
  static __device__ __forceinline__ void st(float *p, size_t i, float f) { p[i] = f; }
  static __device__ __forceinline__ float round(float f) { return f; }
};
template <> struct Conv<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t *p, size_t i) { return bf16_bits_to_f32(p[i].v); }
  static __device__ __forceinline__ void st(bf16_t *p, size_t i, float f) { p[i].v = f32_to_bf16_bits(f); }
  static __device__ __forceinline__ float round(float f) { return bf16_bits_to_f32(f32_to_bf16_bits(f)); }
};
template <> struct Conv<f16_t> {
  static __device__ __forceinline__ float ld(const f16_t *p, size_t i) { return (float)p[i]; }
  static __device__ __forceinline__ void st(f16_t *p, size_t i, float f) { p[i] = (f16_t)f; }
  static __device__ __forceinline__ float round(float f) { return (float)(f16_t)f; }
};

// Operand type of the matrix-core GEMMs, for bf16 and fp16 models alike: fp16 has three more
// significand bits than bf16, and an fp32 activation rounded once to fp16 carries the layer as
// accurately as a bf16 high part plus a bf16 low part at half the matrix work.  Weights of bf16
// models are held as fp16 times a power of two per matrix (exact, see the packing kernel);
// activations beyond the fp16 range saturate.
typedef f16_t op_t;
__device__ __forceinline__ op_t to_op(float f) {
  f = f > 65504.f ? 65504.f : (f < -65504.f ? -65504.f : f);  // NaN passes through
  return (op_t)f;
}

// to_op that also counts the values it had to clamp (sat: a device counter, or null)
__device__ __forceinline__ op_t to_op_counted(float f, unsigned int *sat) {
  if (sat && (f > 65504.f || f < -65504.f)) atomicAdd(sat, 1u);
  return to_op(f);
}

// Activations that feed a matrix-core GEMM are stored in the order the B operand is loaded:
// 16-row x 32-k tiles of 1 KB, tile (m/16, k/32) at ((m/16) * KT + k/32), inside a tile lane
// 16*((k%32)/8) + m%16 owns 8 consecutive k.  Element index of X[m][k] for a row length of 32*KT:
__host__ __device__ __forceinline__ size_t xpack_index(int m, int k, int KT) {
  return ((((size_t)(m >> 4) * KT + (k >> 5)) * 64 + (((k & 31) >> 3) << 4) + (m & 15)) << 3) + (k & 7);
}

// Butterfly sum over the 64 lanes of a wave: every lane ends with the same value and
// the order of additions is fixed by the lane numbers alone.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// (value, index) arg-max combine: larger value wins, equal values -> lower index.
__device__ __forceinline__ void argmax_combine(float &v, int &i, float ov, int oi) {
  if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
}
__device__ __forceinline__ void wave_argmax(float &v, int &i) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    float ov = __shfl_xor(v, o, 64);
    int oi = __shfl_xor(i, o, 64);
    argmax_combine(v, i, ov, oi);
  }
}

// Arg-max over the n_part partials of row src by a block of 256 threads; all of them return it.
// Trips to memory are what this costs (2000 partials of a 32000-token head): eight partials a thread in flight, the
// clamped ones repeating the last, instead of one after the other.  7B width, 4 layers, one sequence, seven draft
// steps and a verification: 765 -> 748 us a round; six sequences, five draft steps: 863 -> 847.
__device__ __forceinline__ int block_argmax_partials(const float *__restrict__ pv, const int32_t *__restrict__ pi, size_t src, int n_part, int V) {
  __shared__ float shv[4];
  __shared__ int shi[4];
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  for (int t0 = threadIdx.x; t0 < n_part; t0 += 2048) {
    float v[8];
    int id[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const size_t at = src * n_part + min(t0 + 256 * i, n_part - 1);
      v[i] = pv[at]; id[i] = pi[at];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) argmax_combine(bv, bi, v[i], id[i]);
  }
  wave_argmax(bv, bi);
  if ((threadIdx.x & 63) == 0) { shv[threadIdx.x >> 6] = bv; shi[threadIdx.x >> 6] = bi; }
  __syncthreads();
  bv = shv[0]; bi = shi[0];
  for (int w = 1; w < 4; ++w) argmax_combine(bv, bi, shv[w], shi[w]);
  return bi < 0 || bi >= V ? 0 : bi;
}

}  // namespace spec

#define SPEC_DISPATCH_DTYPE(dtype, T, ...)                                   \
  do {                                                                       \
    if ((dtype) == SPEC_DTYPE_F32) { typedef float T; __VA_ARGS__; }         \
    else if ((dtype) == SPEC_DTYPE_BF16) { typedef spec::bf16_t T; __VA_ARGS__; } \
    else { typedef spec::f16_t T; __VA_ARGS__; }                             \
  } while (0)

// Shared by the matrix-core GEMM kernels: operand types, the one MFMA instruction, and the
// tile epilogues (the layer's element-wise work on finished fp32 tiles).
#pragma once
#include "spec_internal.h"
#include "device_utils.h"
#include "mfma_gemm.h"

// No implicit fusing of multiplies and adds (see kernels_gemm_mfma.hip).
#pragma clang fp contract(off)

namespace spec {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_v;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_v;
typedef __attribute__((ext_vector_type(4))) float f32x4_v;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_v;

// The one instruction: D(16x16 fp32) += A(16x32 fp16) * B(32x16 fp16).
struct Mfma16 {
  static __device__ __forceinline__ f32x4_v run(u32x4_v a, u32x4_v b, f32x4_v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_v, a), __builtin_bit_cast(f16x8_v, b), c,
                                                  0, 0, 0);
  }
};

// Folded norm, consumer side: the sum of squares of a row of activations is taken from the fp16 operand
// fragments the GEMM reads anyway.  In the B operand lane (c, g) holds elements 8g .. 8g+7 of row c of a
// 32-k step: a lane adds its eight squares to a running fp32 sum, two at a time in ascending k (the two-element
// dot-product instruction: four instead of sixteen operations per fragment), one chain per k-slice from zero; the
// slices are added in slice order per lane, then the four lane groups of a row as (g0 + g1) + (g2 + g3).  Every
// GEMM kernel follows exactly this order, so the value depends on the row alone.
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_v;
// (the pairs are taken from the fragment cast as a whole: a bit cast of one element of a vector, x[i], compiles to a
// read of element 0 whatever i)
__device__ __forceinline__ float frag_ssq(u32x4_v x, float s) {
  const f16x8_v h = __builtin_bit_cast(f16x8_v, x);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f16x2_v p = {h[2 * i], h[2 * i + 1]};
    s = __builtin_amdgcn_fdot2(p, p, s, false);
  }
  return s;
}
// the same chain for the plain sum of the row (folded LayerNorm: the mean)
__device__ __forceinline__ float frag_sum(u32x4_v x, float s) {
  const f16x8_v h = __builtin_bit_cast(f16x8_v, x);
  const f16x2_v one = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f16x2_v p = {h[2 * i], h[2 * i + 1]};
    s = __builtin_amdgcn_fdot2(p, one, s, false);
  }
  return s;
}
// folded LayerNorm: per-lane slice-ordered sums of squares and sums -> 1 / std and mean of the lane's row (lane groups
// combined as below; variance as mean of squares minus squared mean, in fp32)
__device__ __forceinline__ void row_ln_from_lane(float ssq, float sum, int d, float eps, float &rinv, float &mean) {
  ssq += __shfl_xor(ssq, 16, 64);
  ssq += __shfl_xor(ssq, 32, 64);
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  mean = sum / (float)d;
  const float var = fmaxf(ssq / (float)d - mean * mean, 0.f);
  rinv = 1.0f / sqrtf(var + eps);
}
// per-lane slice-ordered sum -> 1 / rms of the lane's row (all four lanes of a row get the same bits)
__device__ __forceinline__ float row_inv_from_lane_ssq(float t, int d, float eps) {
  t += __shfl_xor(t, 16, 64);
  t += __shfl_xor(t, 32, 64);
  return 1.0f / sqrtf(t / (float)d + eps);
}

// Values on their way to a GEMM operand: rounded to fp16, clamped to its range, every clamp counted in *sat (or not,
// sat null); NaN passes through.  One test of the largest magnitude covers the group: clamping is the rare case.
template <int N>
__device__ __forceinline__ void to_op_group(const float (&x)[N], op_t (&o)[N], unsigned int *sat) {
  float big = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) big = fmaxf(big, fabsf(x[i]));
  if (big > 65504.f) {
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = to_op_counted(x[i], sat);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = (op_t)x[i];
  }
}

// The same for the MT row tiles of a strip (rows that do not exist are left out), one test for all of them, the same for the
// wave: the clamping and counting then stay off the path that the others take (tile by tile the branches were most of an epilogue:
// with this, the products' own code per kind of model and the rows of h ahead, a prefill of 64 prompts at the 7B width 11.24 -> 11.03 ms).
template <int MT, int N>
__device__ __forceinline__ void to_op_strip(const float (&x)[MT][N], const bool (&live)[MT], op_t (&o)[MT][N], unsigned int *sat) {
  float big = 0.f;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float b = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) b = fmaxf(b, fabsf(x[mt][i]));
    big = fmaxf(big, live[mt] ? b : 0.f);
  }
  if (__builtin_expect(__any(big > 65504.f), 0)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (live[mt]) {
#pragma unroll
        for (int i = 0; i < N; ++i) o[mt][i] = to_op_counted(x[mt][i], sat);
      }
  } else {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < N; ++i) o[mt][i] = (op_t)x[mt][i];
  }
}

// h[m][n..n+3] += v (scaled, biased): the residual update of one lane's four outputs; o4 = the updated values
// rounded to the next GEMM's operand type (also written to x_out in fragment order when that is set).
// o: the values of h, b4: the bias (if there is one)
__device__ __forceinline__ void residual_update(const GemmArgs &a, f32x4_v v, int n, int m, op_t (&o4)[4], float4 o, const float4 &b4) {
  v[0] *= a.out_scale; v[1] *= a.out_scale; v[2] *= a.out_scale; v[3] *= a.out_scale;  // exact: a power of two
  if (a.bias) { v[0] += b4.x; v[1] += b4.y; v[2] += b4.z; v[3] += b4.w; }
  float4 *p = (float4 *)(a.h + (size_t)m * a.N + n);
  o.x += v[0]; o.y += v[1]; o.z += v[2]; o.w += v[3];
  *p = o;
  if (a.x_out) {  // the next GEMM's activations: the updated row, rounded to fp16
    const float x4[4] = {o.x, o.y, o.z, o.w};
    to_op_group(x4, o4, a.sat);
    *(uint2 *)((op_t *)a.x_out + xpack_index(m, n, a.N >> 5)) = *(const uint2 *)o4;
  }
}

__device__ __forceinline__ void residual_update(const GemmArgs &a, f32x4_v v, int n, int m, op_t (&o4)[4]) {
  float4 b4;
  if (a.bias) b4 = *(const float4 *)(a.bias + n);
  residual_update(a, v, n, m, o4, *(const float4 *)(a.h + (size_t)m * a.N + n), b4);
}

// EPI_LOGITS: where row m of the logits is dumped, if it is
__device__ __forceinline__ float *logits_row(const GemmArgs &a, int m) {
  if (!a.logits) return nullptr;
  if (a.logit_step <= 1) return a.logits + (size_t)m * a.N;
  return m % a.logit_step == a.logit_step - 1 ? a.logits + (size_t)(m / a.logit_step) * a.N : nullptr;
}
// ... and four consecutive outputs v of column n on (a multiple of four) into it, in one store where all rows allow it
__device__ __forceinline__ void dump_logits(const GemmArgs &a, float *row, int n, f32x4_v v) {
  if ((a.N & 3) == 0 && ((uintptr_t)a.logits & 15) == 0) {
    if (n < a.N) *(f32x4_v *)(row + n) = v;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n + i < a.N) row[n + i] = v[i];
  }
}
// EPI_LOGITS: the four lane groups' candidates for row m -> partial p of the row (lowest index wins ties)
__device__ __forceinline__ void row_argmax_out(const GemmArgs &a, float bv, int bi, int m, int p, bool live, int g) {
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    const float ov = __shfl_xor(bv, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    argmax_combine(bv, bi, ov, oi);
  }
  if (live && g == 0) {
    a.part_val[(size_t)m * a.n_part + p] = bv;
    a.part_idx[(size_t)m * a.n_part + p] = bi;
  }
}

// gate / (1 + exp(-gate)) * up.  The quotient from the reciprocal and one correction by its remainder instead of the compiler's division,
// which scales its operands against overflow first (the divisor is at least 1): five instructions for ten.  It is not always the
// rounded quotient (one in some millions is its neighbour), and for gates below -87.3, where the reciprocal is below the smallest
// normal float, it may be -0 instead of less than 1e-36 in magnitude, which is 0 as fp16 whatever `up` is, up to 1e28.
__device__ __forceinline__ float swiglu(float gate, float up) {
  const float den = 1.0f + __expf(-gate), r = __builtin_amdgcn_rcpf(den), q = gate * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-den, q, gate), r, q), den, gate) * up;  // (the fix-up: infinities and NaN)
}

// The sequence (row group) m / q_rows of row m without an integer division: a float product, made exact by one step
// either way.
__device__ __forceinline__ int row_group(int m, int q_rows, float inv_q) {
  int b = (int)(((float)m + 0.5f) * inv_q);
  b += ((b + 1) * q_rows <= m) ? 1 : 0;
  b -= (b * q_rows > m) ? 1 : 0;
  return b;
}

// ------------------------------------------------------------------------- epilogues
// One finished 16x16 tile: this lane holds stored rows n .. n+3 (n = 16*nt + 4g) of
// activation row m.  The element-wise work of the layer happens here, on fp32 sums.
// rinv: 1 / rms of row m when the norm in front of this GEMM is folded into it, else 1.
// What it reads from memory can be asked for ahead (fetch_tile_operands), while the sums are still on their way.
struct TileOperands {
  float4 b4, w4;  // bias; row sums of the weights (folded LayerNorm)
  float4 h;       // EPI_RESIDUAL
  float4 cs;      // EPI_QKV: (cos, sin) of the two rotary pairs
  int pos, seq;   // EPI_QKV: the row's position and sequence
  int region, cc, hh;  // EPI_QKV: 0 q, 1 k, 2 v; the strip's first column there, and its head
};
// EPI_QKV, pos: the row's position, if it is here already
template <int EPI>
__device__ __forceinline__ TileOperands fetch_tile_operands(const GemmArgs &a, int nt, int m, int g, const int *pos = nullptr) {
  TileOperands t;
  t.b4 = t.w4 = t.h = t.cs = make_float4(0.f, 0.f, 0.f, 0.f);
  t.pos = -1; t.seq = t.region = t.cc = t.hh = 0;
  const int n = nt * 16 + 4 * g;
  if (nt >= a.NT) return t;
  if (a.bias) t.b4 = *(const float4 *)(a.bias + n);
  if (EPI == EPI_RESIDUAL) {
    if (m < a.M && n < a.N) t.h = *(const float4 *)(a.h + (size_t)m * a.N + n);
    return t;
  }
  if (a.wsum) t.w4 = *(const float4 *)(a.wsum + n);
  if (EPI == EPI_QKV && m < a.M && n < a.N) {
    t.pos = pos ? *pos : a.row_pos[m];
    t.seq = row_group(m, a.q_rows, 1.0f / (float)a.q_rows);
    if (a.grp_seq) t.seq = a.grp_seq[t.seq];  // prefill passes only
    // No per-lane integer division (it would be most of this epilogue).  A strip of 16 stored rows lies
    // inside one head of one of q, k, v (d and hd are multiples of 16), and the strip number is the same for
    // the whole wave: its place is scalar arithmetic.
    const int base = __builtin_amdgcn_readfirstlane(nt) * 16;
    t.region = base / a.d; t.cc = base - t.region * a.d; t.hh = t.cc / a.hd;
    const int e = t.cc - t.hh * a.hd + 4 * g;
    if (t.region < 2 && a.rope && t.pos >= 0) t.cs = *(const float4 *)(a.rope + (size_t)t.pos * (a.hd >> 1) + (e >> 1));
  }
  return t;
}
template <class T, int EPI>
__device__ __forceinline__ void tile_epilogue(const GemmArgs &a, f32x4_v v, int nt, int m, int g, float rinv, float mean, const TileOperands &t) {
  if (nt >= a.NT) return;
  const int n = nt * 16 + 4 * g;
  if (EPI == EPI_RESIDUAL) {
    op_t o4[4];
    if (m < a.M && n < a.N) residual_update(a, v, n, m, o4, t.h, t.b4);
    return;
  }
  if (a.wsum) {  // folded LayerNorm: take the mean's share out, in the packed weights' units
    const float4 ws = t.w4;
    v[0] -= mean * ws.x; v[1] -= mean * ws.y; v[2] -= mean * ws.z; v[3] -= mean * ws.w;
  }
  v[0] *= a.out_scale; v[1] *= a.out_scale; v[2] *= a.out_scale; v[3] *= a.out_scale;  // exact: a power of two
  v[0] *= rinv; v[1] *= rinv; v[2] *= rinv; v[3] *= rinv;
  if (a.bias) { v[0] += t.b4.x; v[1] += t.b4.y; v[2] += t.b4.z; v[3] += t.b4.w; }
  const bool live = m < a.M;

  if (EPI == EPI_QKV) {
    if (live && n < a.N) {
      const int region = t.region, hh = t.hh, cc = t.cc + 4 * g, e = cc - hh * a.hd;
      const int pos = t.pos, b = t.seq;
      if (region < 2) {
        float r0 = v[0], r1 = v[1], r2 = v[2], r3 = v[3];
        if (a.rope && pos >= 0) {
          r0 = v[0] * t.cs.x - v[1] * t.cs.y; r1 = v[1] * t.cs.x + v[0] * t.cs.y;
          r2 = v[2] * t.cs.z - v[3] * t.cs.w; r3 = v[3] * t.cs.z + v[2] * t.cs.w;
        }
        if (region == 0) {  // queries stay fp32: they are never cached, and the attention kernel feeds them at full width
          *(float4 *)((float *)a.q + (size_t)m * a.d + cc) = make_float4(r0, r1, r2, r3);
        } else if (pos >= 0) {
          T o4[4];
          Conv<T>::st(o4, 0, r0); Conv<T>::st(o4, 1, r1); Conv<T>::st(o4, 2, r2); Conv<T>::st(o4, 3, r3);
          *(uint2 *)((T *)a.kc + kv_k_index(a.L_pad, a.H, a.hd, KV_KUNIT16, b, hh, pos, e)) = *(const uint2 *)o4;
        }
      } else if (pos >= 0) {
        T *vc = (T *)a.vc;
#pragma unroll
        for (int i = 0; i < 4; ++i) Conv<T>::st(vc, kv_v_index(a.L_pad, a.H, a.hd, b, hh, pos, e + i), v[i]);
      }
    }
  } else if (EPI == EPI_SWIGLU) {
    const int j = n >> 1;  // stored rows n..n+3 = gate_j, up_j, gate_{j+1}, up_{j+1}
    if (live && j < a.f) {
      const float r2[2] = {swiglu(v[0], v[1]), swiglu(v[2], v[3])};
      op_t o2[2];
      to_op_group(r2, o2, a.sat);
      const size_t at = xpack_index(m, j, a.f >> 5);
      *(uint32_t *)((op_t *)a.act + at) = *(const uint32_t *)o2;
    }
  } else if (EPI == EPI_RELU) {
    if (live && n < a.N) {
      float r4[4];
      op_t o4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) r4[i] = v[i] > 0.f ? v[i] : 0.f;
      to_op_group(r4, o4, a.sat);
      const size_t at = xpack_index(m, n, a.N >> 5);
      *(uint2 *)((op_t *)a.act + at) = *(const uint2 *)o4;
    }
  } else {  // EPI_LOGITS: optional dump, per-strip arg-max partial (lowest index wins ties)
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    float *dump = live ? logits_row(a, m) : nullptr;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n + i < a.N) argmax_combine(bv, bi, v[i], n + i);
    if (dump) dump_logits(a, dump, n, v);
    row_argmax_out(a, bv, bi, m, nt, live, g);
  }
}
template <class T, int EPI>
__device__ __forceinline__ void tile_epilogue(const GemmArgs &a, f32x4_v v, int nt, int m, int g, float rinv = 1.0f, float mean = 0.f) {
  tile_epilogue<T, EPI>(a, v, nt, m, g, rinv, mean, fetch_tile_operands<EPI>(a, nt, m, g));
}

// Four lanes 4k .. 4k+3 hold four 16-bit values each: lane 4k+i returns value i of all four lanes, in lane order.
__device__ __forceinline__ uint2 quad_transpose(uint2 v, int lane) {
  auto swap = [](uint32_t x, auto perm) {  // lane exchange inside the quad
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(perm)::value, 0xf, 0xf, true);
  };
  // halves: even lanes keep values 0, 1 (and take the odd neighbour's), odd lanes 2, 3 -> x = (value a: lanes l, l+1), y = (value a+1)
  const bool odd = lane & 1, high = lane & 2;
  const uint32_t give = odd ? v.x : v.y, keep = odd ? v.y : v.x;
  const uint32_t got = swap(give, std::integral_constant<int, 0xB1>{});  // quad_perm 1,0,3,2
  const uint32_t lo = odd ? got : keep, hi = odd ? keep : got;            // the even lane's pair, the odd lane's pair
  uint32_t x = (lo & 0xffffu) | (hi << 16), y = (lo >> 16) | (hi & 0xffff0000u);
  // even lanes now hold values 0 (x) and 1 (y) of two lanes, odd lanes values 2 and 3; lanes 0, 1 keep x of both pairs
  // of lanes, lanes 2, 3 keep y
  const uint32_t give2 = high ? x : y, keep2 = high ? y : x;
  const uint32_t got2 = swap(give2, std::integral_constant<int, 0x4E>{});  // quad_perm 2,3,0,1
  uint2 r = high ? make_uint2(got2, keep2) : make_uint2(keep2, got2);
  // lane 0: value 0, lane 1: value 2, lane 2: value 1, lane 3: value 3 -> put 1 and 2 in their places
  r.x = swap(r.x, std::integral_constant<int, 0xD8>{});  // quad_perm 0,2,1,3
  r.y = swap(r.y, std::integral_constant<int, 0xD8>{});
  return r;
}

// The epilogue of a wave's NBW x MTW finished tiles (strips nt0 .., row tiles mtile0 ..): per output the arithmetic of
// tile_epilogue, with what depends on the row alone fetched once per row and every load ahead of the strip that uses
// it.  Tile by tile, the chain row position -> rotary entry -> store costs two memory latencies per tile: at 256 x 192
// outputs per workgroup the QKV epilogue took 37 us, as much as 30 % of the launch.
template <class T, int EPI, int MTW, int NBW>
__device__ __forceinline__ void wave_epilogue(const GemmArgs &a, f32x4_v (&acc)[NBW][MTW], int nt0, int mtile0, int lane,
                                              const float (&rinv)[MTW], const float (&mean)[MTW]) {
  const int c = lane & 15, g = lane >> 4;
  bool live[MTW];
#pragma unroll
  for (int mt = 0; mt < MTW; ++mt) live[mt] = (mtile0 + mt) * 16 + c < a.M;
  const bool lnx = a.wsum != nullptr;
  // (acc - mean * wsum) * scale * rinv + bias of the four outputs of a tile
  auto finish = [&](f32x4_v v, int mt, const float4 &b4, const float4 &w4, auto lnx, auto bias) {
    if (EPI != EPI_RESIDUAL && lnx) {
      v[0] -= mean[mt] * w4.x; v[1] -= mean[mt] * w4.y; v[2] -= mean[mt] * w4.z; v[3] -= mean[mt] * w4.w;
    }
    v[0] *= a.out_scale; v[1] *= a.out_scale; v[2] *= a.out_scale; v[3] *= a.out_scale;  // exact: a power of two
    if (EPI != EPI_RESIDUAL) { v[0] *= rinv[mt]; v[1] *= rinv[mt]; v[2] *= rinv[mt]; v[3] *= rinv[mt]; }
    if (bias) { v[0] += b4.x; v[1] += b4.y; v[2] += b4.z; v[3] += b4.w; }
    return v;
  };
  // What a model has is the same for the launch: the usual combinations get code of their own (tile by tile the tests, or the
  // additions behind a select, are as many instructions as the rest of `finish`).
  auto with_kind = [&](auto body) {
    if (!a.bias && (EPI == EPI_RESIDUAL || !lnx)) body(std::false_type{}, std::false_type{});
    else if (EPI == EPI_RESIDUAL) body(std::false_type{}, std::true_type{});
    else if (a.bias && lnx) body(std::true_type{}, std::true_type{});
    else body(lnx, a.bias != nullptr);
  };
  float4 b4[NBW], w4[NBW];
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb) {
    const int n = min(nt0 + nb, a.NT - 1) * 16 + 4 * g;
    if (a.bias) b4[nb] = *(const float4 *)(a.bias + n);
    if (EPI != EPI_RESIDUAL && lnx) w4[nb] = *(const float4 *)(a.wsum + n);
  }
  if (EPI == EPI_LOGITS) {  // optional dump; one arg-max partial per row for all strips of the wave
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
      const int m = (mtile0 + mt) * 16 + c;
      float *dump = live[mt] ? logits_row(a, m) : nullptr;
      float bv = -INFINITY;
      int bi = 0x7fffffff;
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
        const f32x4_v v = finish(acc[nb][mt], mt, b4[nb], w4[nb], lnx, a.bias != nullptr);
        const int n = (nt0 + nb) * 16 + 4 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < a.N) argmax_combine(bv, bi, v[i], n + i);
        if (dump) dump_logits(a, dump, n, v);
      }
      row_argmax_out(a, bv, bi, m, nt0 / NBW, live[mt], g);
    }
  } else if (EPI == EPI_SWIGLU || EPI == EPI_RELU) {
    // fragment order: a strip of 16 outputs (8 after SwiGLU) is 512 (256) consecutive bytes of its row tile
    const size_t tile_bytes = (size_t)(EPI == EPI_SWIGLU ? a.f : a.N) * 32;
    const unsigned in_row = c * 16 + (EPI == EPI_SWIGLU ? g * 4 : (g >> 1) * 256 + (g & 1) * 8);
    auto row = [&](int nb, int mt) {  // a row tile's place is the same for the wave
      return (unsigned char *)a.act + ((size_t)(mtile0 + mt) * tile_bytes + (size_t)(nt0 + nb) * (EPI == EPI_SWIGLU ? 256 : 512)) + in_row;
    };
    with_kind([&](auto ln, auto bias) {
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
        if (nt0 + nb >= a.NT) break;
        constexpr int N = EPI == EPI_SWIGLU ? 2 : 4;
        float r[MTW][N];
        op_t o[MTW][N];
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
          const f32x4_v v = finish(acc[nb][mt], mt, b4[nb], w4[nb], ln, bias);
#pragma unroll
          for (int i = 0; i < N; ++i) {
            if constexpr (EPI == EPI_SWIGLU) r[mt][i] = swiglu(v[2 * i], v[2 * i + 1]);
            else r[mt][i] = v[i] > 0.f ? v[i] : 0.f;
          }
        }
        to_op_strip(r, live, o, a.sat);
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt)
          if (live[mt]) {
            if constexpr (EPI == EPI_SWIGLU) *(uint32_t *)row(nb, mt) = *(const uint32_t *)o[mt];
            else *(uint2 *)row(nb, mt) = *(const uint2 *)o[mt];
          }
      }
    });
  } else if (EPI == EPI_RESIDUAL) {
    // DEPTH strips' rows of h in flight: one strip at a time is a memory latency per strip (256 x 192 outputs took 16 us, beside 78 for the
    // steps of a k of 4096; 4096 x 4096 at 6592 rows 299 -> 290 us)
    constexpr int DEPTH = NBW < 3 ? NBW : 3;
    float4 o[DEPTH][MTW];
    // a row tile's place is the same for the wave, a lane's in it the same for all row tiles: few registers for addresses
    const unsigned h_lane = (unsigned)(c * a.N + 4 * g) * 4, x_lane = c * 16 + (g >> 1) * 256 + (g & 1) * 8;
    auto h_at = [&](int nb, int mt) { return (float4 *)((unsigned char *)a.h + ((size_t)(mtile0 + mt) * 16 * a.N + (size_t)(nt0 + nb) * 16) * 4 + h_lane); };
    auto load_h = [&](int nb) {
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt)
        if (live[mt] && nt0 + nb < a.NT) o[nb % DEPTH][mt] = *h_at(nb, mt);
    };
#pragma unroll
    for (int nb = 0; nb < DEPTH; ++nb) load_h(nb);
    with_kind([&](auto ln, auto bias) {
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
        if (nt0 + nb >= a.NT) break;
        float x4[MTW][4];
        op_t o4[MTW][4];
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
          const f32x4_v v = finish(acc[nb][mt], mt, b4[nb], w4[nb], ln, bias);
          const float4 h4 = o[nb % DEPTH][mt];
          x4[mt][0] = h4.x + v[0]; x4[mt][1] = h4.y + v[1]; x4[mt][2] = h4.z + v[2]; x4[mt][3] = h4.w + v[3];
          if (live[mt]) *h_at(nb, mt) = make_float4(x4[mt][0], x4[mt][1], x4[mt][2], x4[mt][3]);
        }
        if (nb + DEPTH < NBW) load_h(nb + DEPTH);
        if (a.x_out) {
          to_op_strip(x4, live, o4, a.sat);
#pragma unroll
          for (int mt = 0; mt < MTW; ++mt)
            if (live[mt])
              *(uint2 *)((unsigned char *)a.x_out + ((size_t)(mtile0 + mt) * a.N * 32 + (size_t)(nt0 + nb) * 512) + x_lane) = *(const uint2 *)o4[mt];
        }
      }
    });
  } else {  // EPI_QKV
    // A strip of 16 stored rows lies inside one head of one of q, k, v: its place is scalar arithmetic.  What depends on
    // the row (cache rows of its sequence and position) is worked out once per row tile.
    const int first = __builtin_amdgcn_readfirstlane(nt0) * 16;
    int region = first / a.d, cc0 = first - region * a.d;
    const int half = a.hd >> 1, hd_shift = a.hd == 128 ? 7 : 6;
    const float inv_q = 1.0f / (float)a.q_rows;
    int pos[MTW];
    T *krow[MTW], *vrow[MTW];
    bool quads[MTW];  // same for the wave: every four rows of the tile hold four consecutive positions of one sequence from a
                      // multiple of four on, as the passes of a prefill do; their values are then stored together
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) pos[mt] = live[mt] ? a.row_pos[(mtile0 + mt) * 16 + c] : -1;
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
      int b = row_group((mtile0 + mt) * 16 + c, a.q_rows, inv_q);
      if (a.grp_seq && live[mt]) b = a.grp_seq[b];
      const size_t seq0 = (size_t)b * a.H * a.L_pad * a.hd;
      const int p0 = max(pos[mt], 0);
      krow[mt] = (T *)a.kc + kv_k_index(a.L_pad, a.H, a.hd, KV_KUNIT16, b, 0, p0, 0);
      vrow[mt] = (T *)a.vc + seq0 + (size_t)(p0 / KV_VBLOCK) * a.hd * KV_VBLOCK + p0 % KV_VBLOCK;
      quads[mt] = (a.q_rows & 3) == 0 && __all(pos[mt] >= 0 && (pos[mt] & 3) == (lane & 3) && pos[mt] == __shfl(pos[mt], lane & ~3, 64) + (lane & 3));
    }
    float4 cs[2][MTW];  // (cos, sin) of the two rotary pairs: this strip's and the next one's
    auto load_cs = [&](int nb, int cc) {  // column cc of q or k
      const float2 *tab = a.rope + (((cc & (a.hd - 1)) + 4 * g) >> 1);
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) cs[nb & 1][mt] = *(const float4 *)(tab + (size_t)max(pos[mt], 0) * half);
    };
    if (a.rope && region < 2) load_cs(0, cc0);
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
      if (nt0 + nb >= a.NT) break;
      const int next_cc0 = cc0 + 16 == a.d ? 0 : cc0 + 16, next_region = cc0 + 16 == a.d ? region + 1 : region;
      if (nb + 1 < NBW && a.rope && next_region < 2) load_cs(nb + 1, next_cc0);
      const int hh = cc0 >> hd_shift, e = (cc0 & (a.hd - 1)) + 4 * g;
      const size_t head = (size_t)hh * a.L_pad * a.hd;
      if (region < 2) {
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
          const f32x4_v v = finish(acc[nb][mt], mt, b4[nb], w4[nb], lnx, a.bias != nullptr);
          float r0 = v[0], r1 = v[1], r2 = v[2], r3 = v[3];
          if (a.rope && pos[mt] >= 0) {
            const float4 t = cs[nb & 1][mt];
            r0 = v[0] * t.x - v[1] * t.y; r1 = v[1] * t.x + v[0] * t.y;
            r2 = v[2] * t.z - v[3] * t.w; r3 = v[3] * t.z + v[2] * t.w;
          }
          if (region == 0) {  // queries stay fp32 (see tile_epilogue)
            if (live[mt]) *(float4 *)((float *)a.q + (size_t)((mtile0 + mt) * 16 + c) * a.d + cc0 + 4 * g) = make_float4(r0, r1, r2, r3);
          } else {
            T o4[4];
            Conv<T>::st(o4, 0, r0); Conv<T>::st(o4, 1, r1); Conv<T>::st(o4, 2, r2); Conv<T>::st(o4, 3, r3);
            if (pos[mt] >= 0) *(uint2 *)(krow[mt] + head + (e >> 3) * (8 * KV_KBLOCK) + (e & 7)) = *(const uint2 *)o4;
          }
        }
      } else {
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
          const f32x4_v v = finish(acc[nb][mt], mt, b4[nb], w4[nb], lnx, a.bias != nullptr);
          T o4[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) Conv<T>::st(o4, i, v[i]);
          if (quads[mt]) {  // four rows of one element per lane: their positions are neighbours in the cache
            const uint2 o = quad_transpose(*(const uint2 *)o4, lane);
            *(uint2 *)(vrow[mt] - (lane & 3) + head + (size_t)(e + (lane & 3)) * KV_VBLOCK) = o;
          } else if (pos[mt] >= 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) vrow[mt][head + (size_t)(e + i) * KV_VBLOCK] = o4[i];
          }
        }
      }
      region = next_region; cc0 = next_cc0;
    }
  }
}

}  // namespace spec

// fp32 models on the matrix cores: v_mfma_f32_16x16x4_f32, fp32 operands and sums throughout.
//
//   Y^T[n][m] = sum_k W[n][k] * X[m][k]        W: weights [N][K], X: activations [M][K], both fp32
//
// Packed weights: 16-row x 16-k tiles of 1 KB; lane 16g + r of a wave owns W[n0 + r][k0 + 4g .. k0 + 4g + 3], so a wave
// streams a strip as one linear run of 16-byte loads, and element e of the lanes' quadruples is the operand of one
// instruction (which four k an instruction takes is free as long as W and X agree).  X is read the same way straight
// from its rows.
//
// Order of every sum: K is cut into KS equal slices (gemm_ks_for); inside a slice each 16-k block is two chains of two
// instructions, their sum is added to the slice's total in ascending k, the slices in order.  It is a function of K
// alone: neither the number of rows nor the tiling changes a bit, so a sequence's tokens do not depend on batch size or
// speculation length.  Short chains keep the rounding error at the level of a 64-lane partial sum with a butterfly.
//
// Against the generic kernels (norm, product, rotary + append, attention, activation as nine launches a layer; one wave
// per output and four rows): verification of 8 sequences x 5 rows at d_model 1024, 4 layers 2679 -> 307 us, logits'
// error against 64 bits 7.2e-7 -> 6.7e-7 (266 us since); a d_model 256 target with its 128 draft, 12 rounds 4.7 -> 2.2 ms, 2.4e-7 both.
#include "spec_internal.h"
#include "device_utils.h"
#include <algorithm>

#pragma clang fp contract(off)

namespace spec {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// ------------------------------------------------------------------------- set-up
// hd 64 or 128: the attention kernel's accumulators; d_model is then a multiple of 16 as well
bool fp32_supported(const spec_model_desc &D, int dtype) {
  const int hd = D.d_model / D.n_heads;
  return dtype == SPEC_DTYPE_F32 && (hd == 64 || hd == 128) && D.d_ffn % 16 == 0;
}

static size_t al256s(size_t b) { return (b + 255) & ~(size_t)255; }
static size_t pad16(size_t n) { return (n + 15) / 16 * 16; }

size_t fp32_packed_bytes(const spec_model_desc &D, int L_max) {
  const size_t d = D.d_model, f = D.d_ffn, kf = D.ffn_kind == SPEC_FFN_SWIGLU ? 2 : 1;
  const size_t layer = 4 * al256s(d * 4) + al256s(3 * d * d * 4) + al256s(d * d * 4) + al256s(kf * f * d * 4) + al256s(d * f * 4) +
                       al256s(3 * d * 4) + al256s(kf * f * 4) + 2 * al256s(d * 4);
  return al256s((size_t)D.vocab * d * 4) + al256s((size_t)D.max_pos * d * 4) + 2 * al256s(d * 4) + al256s(pad16(D.vocab) * d * 4) +
         al256s((size_t)L_max * (d / D.n_heads / 2) * sizeof(float2)) + layer * (size_t)D.n_layers;
}

// Source row of stored row n.  mode 0: as it is; mode 1: q | k | v stacked, q and k rows pair-interleaved inside a head
// (a rotary pair is then lane-local in the epilogue, and in the cache's element order); mode 2: gate and up alternate.
__device__ __forceinline__ const float *src_row(int mode, int n, int K, int d, int hd, const float *s0, const float *s1, const float *s2) {
  if (mode == 0) return s0 + (size_t)n * K;
  if (mode == 2) return ((n & 1) ? s1 : s0) + (size_t)(n >> 1) * K;
  const int region = n / d, c = n % d, hh = c / hd;
  int e = c % hd;
  if (region < 2) e = (e & 1) ? (e >> 1) + (hd >> 1) : (e >> 1);
  return (region == 0 ? s0 : region == 1 ? s1 : s2) + (size_t)(hh * hd + e) * K;
}

// gain: the norm in front, folded into the columns (or null)
__global__ void k_pack_f32(int mode, int N, int K, int d, int hd, const float *__restrict__ s0, const float *__restrict__ s1,
                           const float *__restrict__ s2, const float *__restrict__ gain, f32x4 *__restrict__ dst, size_t total) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int lane = (int)(idx & 63), KT = K / 16;
  const size_t tile = idx >> 6;
  const int n = (int)(tile / KT) * 16 + (lane & 15), k = (int)(tile % KT) * 16 + (lane >> 4) * 4;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (n < N) {
    const float *r = src_row(mode, n, K, d, hd, s0, s1, s2) + k;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gain ? r[e] * gain[k + e] : r[e];
  }
  dst[idx] = v;
}
__global__ void k_pack_bias_f32(int mode, int N, int d, int hd, const float *__restrict__ s0, const float *__restrict__ s1,
                                const float *__restrict__ s2, float *__restrict__ dst) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n < N) dst[n] = *src_row(mode, n, 1, d, hd, s0, s1, s2);
}

static void *bump32(void *&cursor, size_t bytes) {
  void *p = cursor;
  cursor = (char *)cursor + al256s(bytes);
  return p;
}
static const void *take32(const void *src, size_t bytes, void *&cursor, hipStream_t st) {
  if (!src) return nullptr;
  void *dst = bump32(cursor, bytes);
  generic_copy(src, dst, bytes, st);
  return dst;
}
static const void *pack32(int mode, int N, int K, int d, int hd, const void *s0, const void *s1, const void *s2, const void *gain,
                          void *&cursor, hipStream_t st) {
  const size_t total = pad16(N) * K / 4;
  void *dst = bump32(cursor, total * 16);
  hipLaunchKernelGGL(k_pack_f32, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, mode, N, K, d, hd, (const float *)s0,
                     (const float *)s1, (const float *)s2, (const float *)gain, (f32x4 *)dst, total);
  return dst;
}
static const void *bias32(int mode, int N, int d, int hd, const void *s0, const void *s1, const void *s2, void *&cursor, hipStream_t st) {
  void *dst = bump32(cursor, (size_t)N * 4);
  hipLaunchKernelGGL(k_pack_bias_f32, dim3((N + 255) / 256), dim3(256), 0, st, mode, N, d, hd, (const float *)s0, (const float *)s1,
                     (const float *)s2, (float *)dst);
  return dst;
}

// RMS norms are folded: gain in the packed weights, 1 / rms in the epilogue of the product behind the norm.  LayerNorms
// run as a kernel of their own.
void fp32_setup_model(spec_ctx *c, Model &m, const spec_weights *w, void *&cursor, hipStream_t st) {
  const spec_model_desc &D = m.desc;
  const int d = D.d_model, f = D.d_ffn, hd = m.hd;
  const bool ln = D.norm_kind == SPEC_NORM_LAYER, hb = D.has_bias != 0, swi = D.ffn_kind == SPEC_FFN_SWIGLU;
  m.tok_emb = take32(w->d_tok_emb, (size_t)D.vocab * d * 4, cursor, st);
  m.pos_emb = D.pos_kind == SPEC_POS_LEARNED ? take32(w->d_pos_emb, (size_t)D.max_pos * d * 4, cursor, st) : nullptr;
  m.final_norm_w = take32(w->d_final_norm_w, (size_t)d * 4, cursor, st);
  m.final_norm_b = ln ? take32(w->d_final_norm_b, (size_t)d * 4, cursor, st) : nullptr;
  m.lm_head = pack32(0, D.vocab, d, d, hd, w->d_lm_head, nullptr, nullptr, ln ? nullptr : m.final_norm_w, cursor, st);
  m.rope = nullptr;
  if (D.pos_kind == SPEC_POS_ROPE) {
    float2 *tab = (float2 *)bump32(cursor, (size_t)c->run.L_max * (hd / 2) * sizeof(float2));
    launch_rope_table(c->run.L_max, hd, D.rope_theta, tab, st);
    m.rope = tab;
  }
  for (int l = 0; l < D.n_layers; ++l) {
    const void *const *T = w->layer_tensors + (size_t)l * SPEC_T_COUNT;
    LayerW &L = m.layers[l];
    L.attn_norm_w = take32(T[SPEC_T_ATTN_NORM_W], (size_t)d * 4, cursor, st);
    L.attn_norm_b = ln ? take32(T[SPEC_T_ATTN_NORM_B], (size_t)d * 4, cursor, st) : nullptr;
    L.ffn_norm_w = take32(T[SPEC_T_FFN_NORM_W], (size_t)d * 4, cursor, st);
    L.ffn_norm_b = ln ? take32(T[SPEC_T_FFN_NORM_B], (size_t)d * 4, cursor, st) : nullptr;
    const void *g1 = ln ? nullptr : L.attn_norm_w, *g2 = ln ? nullptr : L.ffn_norm_w;
    L.wqkv = pack32(1, 3 * d, d, d, hd, T[SPEC_T_WQ], T[SPEC_T_WK], T[SPEC_T_WV], g1, cursor, st);
    L.wo = pack32(0, d, d, d, hd, T[SPEC_T_WO], nullptr, nullptr, nullptr, cursor, st);
    L.w13 = swi ? pack32(2, 2 * f, d, d, hd, T[SPEC_T_W1], T[SPEC_T_W3], nullptr, g2, cursor, st)
                : pack32(0, f, d, d, hd, T[SPEC_T_W1], nullptr, nullptr, g2, cursor, st);
    L.w2 = pack32(0, d, f, d, hd, T[SPEC_T_W2], nullptr, nullptr, nullptr, cursor, st);
    L.bqkv = hb ? bias32(1, 3 * d, d, hd, T[SPEC_T_BQ], T[SPEC_T_BK], T[SPEC_T_BV], cursor, st) : nullptr;
    L.bo = hb ? bias32(0, d, d, hd, T[SPEC_T_BO], nullptr, nullptr, cursor, st) : nullptr;
    L.b13 = hb && !swi ? bias32(0, f, d, hd, T[SPEC_T_B1], nullptr, nullptr, cursor, st) : nullptr;
    L.b2 = hb && !swi ? bias32(0, d, d, hd, T[SPEC_T_B2], nullptr, nullptr, cursor, st) : nullptr;
  }
}

// ------------------------------------------------------------------------- products
struct F32Gemm {
  const f32x4 *W;
  const float *bias, *X;
  int M, N, NT, KT, KS;    // NT: 16-row strips of W, KT: 16-k steps
  int x_mul, x_off;        // output row m reads X row m * x_mul + x_off
  int passes, groups;
  int fold;                // X is un-normed: multiply by 1 / rms of the row
  float eps;
  float *out;              // EPI_RESIDUAL: h, EPI_QKV: q, EPI_SWIGLU / EPI_RELU: act, EPI_LOGITS: logits or null
  float *part_val;         // EPI_LOGITS: arg-max partials [M][NT]
  int32_t *part_idx;
  int ldo;
  float *kc, *vc;          // EPI_QKV
  const int32_t *row_pos, *grp_seq;
  const float2 *rope;
  int q_rows, d, hd, H, L_pad;
};

template <int EPI>
__device__ __forceinline__ void f32_epilogue(const F32Gemm &a, f32x4 v, int nt, int m, int g, float rinv) {
  const int n = nt * 16 + 4 * g;
  if (a.fold) v *= rinv;
  if (EPI == EPI_LOGITS) {  // the strip's arg-max (lowest index wins ties), and the logits where they are wanted
    float bv = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < a.N) argmax_combine(bv, bi, v[e], n + e);
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      argmax_combine(bv, bi, ov, oi);
    }
    if (m >= a.M || nt >= a.NT) return;
    if (g == 0) {
      a.part_val[(size_t)m * a.NT + nt] = bv;
      a.part_idx[(size_t)m * a.NT + nt] = bi;
    }
    if (!a.out || n >= a.N) return;
    float *p = a.out + (size_t)m * a.ldo + n;
    if ((a.N & 3) == 0 && ((uintptr_t)a.out & 15) == 0) *(f32x4 *)p = v;
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) p[e] = v[e];
    }
    return;
  }
  if (m >= a.M || n >= a.N) return;
  if (a.bias) v += *(const f32x4 *)(a.bias + n);
  if (EPI == EPI_RESIDUAL) {
    f32x4 *p = (f32x4 *)(a.out + (size_t)m * a.ldo + n);
    *p = *p + v;
  } else if (EPI == EPI_SWIGLU) {
    float2 r;
    r.x = v[0] / (1.0f + expf(-v[0])) * v[1];
    r.y = v[2] / (1.0f + expf(-v[2])) * v[3];
    *(float2 *)(a.out + (size_t)m * a.ldo + (n >> 1)) = r;
  } else if (EPI == EPI_RELU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    *(f32x4 *)(a.out + (size_t)m * a.ldo + n) = v;
  } else {  // EPI_QKV
    const int region = n / a.d, cc = n - region * a.d, hh = cc / a.hd, e0 = cc - hh * a.hd;
    const int pos = a.row_pos[m];
    if (region < 2) {
      if (a.rope && pos >= 0) {
        const float4 t = *(const float4 *)(a.rope + (size_t)pos * (a.hd >> 1) + (e0 >> 1));  // (cos, sin) of two pairs
        const float x0 = v[0] * t.x - v[1] * t.y, y0 = v[1] * t.x + v[0] * t.y;
        const float x1 = v[2] * t.z - v[3] * t.w, y1 = v[3] * t.z + v[2] * t.w;
        v = (f32x4){x0, y0, x1, y1};
      }
      if (region == 0) { *(f32x4 *)(a.out + (size_t)m * a.d + cc) = v; return; }
    }
    if (pos < 0) return;
    const int grp = m / a.q_rows, b = a.grp_seq ? a.grp_seq[grp] : grp;
    if (region == 1) *(f32x4 *)(a.kc + kv_k_index(a.L_pad, a.H, a.hd, KV_KUNIT32, b, hh, pos, e0)) = v;
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e) a.vc[kv_v_index(a.L_pad, a.H, a.hd, b, hh, pos, e0 + e)] = v[e];
    }
  }
}

// LDS of a workgroup: a finished tile per slice, strip and row tile, and behind them the slices' sums of squares per row.
// With eight slices of eight tiles that is above the 64 KB a kernel has without asking (fp32_prepare).
constexpr size_t f32_lds(int KS, int MT, int NB) { return (size_t)KS * (NB * MT * 1024 + MT * 16 * 4); }

// Workgroup = KS waves, one k-slice each, over NB strips of W and MT row tiles of X; the slices meet in LDS.  Bound by the latencies of a
// wave's loads (few rows; a slice has K / 128 steps, up to K / 16 where that is odd) or by the matrix cores (2 x 4 tiles: 256 cycles of MFMA per unit and step
// against 96 cycles of L2 reads; 4 x 4 spills); operands of the next steps are in flight while the present ones are multiplied.
// (A wave per strip over all of k, the rows through LDS, was slower everywhere but for the head at 1 to 5 rows: 8192 x 1024 at 40 rows 44
// us against 15.6, 32000 x 1024 55 and 53.)
template <int MT, int NB, int EPI, bool DEEP>
__global__ __launch_bounds__(512, 2) void k_gemm_f32(F32Gemm a) {
  extern __shared__ float red[];  // [KS][NB * MT][256], then [KS][MT * 16]: f32_lds()
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, g = lane >> 4;
  const int KS = a.KS;
  float *ssq_s = red + (size_t)KS * (NB * MT * 256);
  int G = blockIdx.x, pass = 0;
  if (a.passes > 1) {  // all row passes of a strip group on one XCD: its L2 serves the weights again
    const int rest = (int)blockIdx.x >> 3;
    pass = rest % a.passes;
    G = (rest / a.passes) * 8 + ((int)blockIdx.x & 7);
  }
  if (G >= a.groups) return;
  const int nt0 = G * NB, m_base = pass * (MT * 16), K = a.KT * 16;
  const int kt_per = a.KT / KS, kt0 = w * kt_per, kt1 = kt0 + kt_per;

  // Addresses: what is the same for the wave in scalars, a lane's part in 32 bits (no registers for addresses beside the batches).
  const unsigned char *Wp[NB], *Xp[MT];
  unsigned x_off[MT];
  const unsigned w_off = lane * 16;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) Wp[nb] = (const unsigned char *)a.W + (size_t)min(nt0 + nb, a.NT - 1) * a.KT * 1024;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row0 = min(m_base + mt * 16, a.M - 1), row = min(row0 + c, a.M - 1);
    Xp[mt] = (const unsigned char *)a.X + ((size_t)row0 * a.x_mul + a.x_off) * K * 4;
    x_off[mt] = (unsigned)((row - row0) * a.x_mul * K + 4 * g) * 4;
  }

  f32x4 acc[NB][MT];
  float ssq[MT];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    ssq[mt] = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb][mt] = zero;
  }
  // Steps in two batches of U, the loads of one in flight while the other is multiplied.  DEEP: inside the loop every load is
  // unconditional (behind a branch the compiler waits, where it joins, for all loads under way), and the multiplies stay
  // in order, so that few of their intermediate sums take registers beside the batches.
  constexpr int U = DEEP ? 4 : NB + MT >= 5 ? 1 : NB + MT >= 3 ? 2 : 4;  // (DEEP: at most three tiles)
  f32x4 wf[2][U][NB], xf[2][U][MT];
  auto load = [&](f32x4 (&wd)[U][NB], f32x4 (&xd)[U][MT], int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(kt + u, kt1 - 1);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) wd[u][nb] = __builtin_nontemporal_load((const f32x4 *)(Wp[nb] + (size_t)k * 1024 + w_off));
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xd[u][mt] = *(const f32x4 *)(Xp[mt] + (size_t)k * 64 + x_off[mt]);
    }
  };
  auto mul = [&](const f32x4 (&wd)[U][NB], const f32x4 (&xd)[U][MT], int steps) {  // the first `steps` of a batch, the same for the wave
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u >= steps) break;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const f32x4 lo = mfma4(wd[u][nb][1], xd[u][mt][1], mfma4(wd[u][nb][0], xd[u][mt][0], zero));
          const f32x4 hi = mfma4(wd[u][nb][3], xd[u][mt][3], mfma4(wd[u][nb][2], xd[u][mt][2], zero));
          acc[nb][mt] += lo + hi;
        }
        if (DEEP) __builtin_amdgcn_sched_barrier(0);
      }
      if (EPI != EPI_RESIDUAL) {  // (without a test: used or not, a.fold says; a branch here costs the batches their registers)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int e = 0; e < 4; ++e) ssq[mt] = fmaf(xd[u][mt][e], xd[u][mt][e], ssq[mt]);
      }
    }
  };
  load(wf[0], xf[0], kt0);
  if (DEEP) {
    int left = __builtin_amdgcn_readfirstlane(kt_per), kt = kt0;
    for (; left > 2 * U; left -= 2 * U, kt += 2 * U) {
      load(wf[1], xf[1], kt + U);
      __builtin_amdgcn_sched_barrier(0);
      mul(wf[0], xf[0], U);
      load(wf[0], xf[0], kt + 2 * U);
      __builtin_amdgcn_sched_barrier(0);
      mul(wf[1], xf[1], U);
    }
    if (left > U) {
      load(wf[1], xf[1], kt + U);
      __builtin_amdgcn_sched_barrier(0);
      mul(wf[0], xf[0], U);
      mul(wf[1], xf[1], left - U);
    } else {
      mul(wf[0], xf[0], left);
    }
  } else {
    for (int kt = kt0; kt < kt1; kt += 2 * U) {
      if (kt + U < kt1) load(wf[1], xf[1], kt + U);
      mul(wf[0], xf[0], kt1 - kt);
      if (kt + U >= kt1) break;
      if (kt + 2 * U < kt1) load(wf[0], xf[0], kt + 2 * U);
      mul(wf[1], xf[1], kt1 - kt - U);
    }
  }

  if (a.fold) {  // the row's sum of squares: the four k-quarters of a slice here, the slices in order behind the barrier
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float t = ssq[mt];
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      if (g == 0) ssq_s[w * (MT * 16) + mt * 16 + c] = t;
    }
  }
  float rinv[MT];
  auto finish_rinv = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      rinv[mt] = 1.f;
      if (!a.fold) continue;
      const float *p = ssq_s + mt * 16 + c;
      float t = p[0];
      if (KS == 8) {  // (all reads ahead of the additions)
        float q[8];
#pragma unroll
        for (int s = 1; s < 8; ++s) q[s] = p[s * (MT * 16)];
#pragma unroll
        for (int s = 1; s < 8; ++s) t += q[s];
      } else {
        for (int s = 1; s < KS; ++s) t += p[s * (MT * 16)];
      }
      rinv[mt] = 1.0f / sqrtf(t / (float)K + a.eps);
    }
  };
  constexpr int TILES = NB * MT;
#pragma unroll
  for (int t = 0; t < TILES; ++t) *(f32x4 *)&red[((size_t)(w * TILES + t) * 64 + lane) * 4] = acc[t / MT][t % MT];
  __syncthreads();
  finish_rinv();
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    if (t % KS != w) continue;
    const f32x4 *p = (const f32x4 *)red + t * 64 + lane;
    f32x4 v = p[0];
    if (KS == 8) {
      f32x4 q[8];
#pragma unroll
      for (int s = 1; s < 8; ++s) q[s] = p[s * TILES * 64];
#pragma unroll
      for (int s = 1; s < 8; ++s) v += q[s];
    } else {
      for (int s = 1; s < KS; ++s) v += p[s * TILES * 64];
    }
    f32_epilogue<EPI>(a, v, nt0 + t / MT, m_base + (t % MT) * 16 + c, g, rinv[t % MT]);
  }
}

// blocks < 0: preparation pass.  DEEP where the workgroups leave a CU to one or two and a wave's chain of memory latencies is what
// counts: no more than two of one tile to a CU, one of two or three tiles (us without / with: 8192 x 1024 at 1 row 9.5 / 8.4, 1024 x
// 4096 11.2 / 9.3, 3072 x 1024 at 40 rows as 3 x 1 11.8 / 11.2; but 32000 x 1024 at 1 row 30.5 / 32.3, 8192 x 1024 at 40 as 3 x 2 15.6 / 16.3).
template <int MT, int NB, int EPI>
static void f32_launch(const F32Gemm &a, int blocks, int n_cu, hipStream_t st) {
  constexpr bool CAN = MT * NB <= 3;
  const size_t lds = f32_lds(a.KS, MT, NB);
  if (blocks < 0)
    (void)hipFuncSetAttribute((const void *)k_gemm_f32<MT, NB, EPI, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)f32_lds(8, MT, NB));
  else if (CAN && blocks <= (MT * NB == 1 ? 2 : 1) * n_cu)
    hipLaunchKernelGGL((k_gemm_f32<MT, NB, EPI, CAN>), dim3(blocks), dim3(a.KS * 64), lds, st, a);
  else
    hipLaunchKernelGGL((k_gemm_f32<MT, NB, EPI, false>), dim3(blocks), dim3(a.KS * 64), lds, st, a);
}

template <int MT, int NB>
static void f32_launch_epi(const F32Gemm &a, int epi, int blocks, int n_cu, hipStream_t st) {
  switch (epi) {
    case EPI_RESIDUAL: f32_launch<MT, NB, EPI_RESIDUAL>(a, blocks, n_cu, st); break;
    case EPI_QKV: f32_launch<MT, NB, EPI_QKV>(a, blocks, n_cu, st); break;
    case EPI_SWIGLU: f32_launch<MT, NB, EPI_SWIGLU>(a, blocks, n_cu, st); break;
    case EPI_RELU: f32_launch<MT, NB, EPI_RELU>(a, blocks, n_cu, st); break;
    default: f32_launch<MT, NB, EPI_LOGITS>(a, blocks, n_cu, st); break;
  }
}

static void f32_launch_shape(const F32Gemm &a, int MT, int NB, int epi, int blocks, int n_cu, hipStream_t st) {
  switch (MT * 8 + NB) {
    case 9: f32_launch_epi<1, 1>(a, epi, blocks, n_cu, st); break;
    case 10: f32_launch_epi<1, 2>(a, epi, blocks, n_cu, st); break;
    case 12: f32_launch_epi<1, 4>(a, epi, blocks, n_cu, st); break;
    case 17: f32_launch_epi<2, 1>(a, epi, blocks, n_cu, st); break;
    case 18: f32_launch_epi<2, 2>(a, epi, blocks, n_cu, st); break;
    case 20: f32_launch_epi<2, 4>(a, epi, blocks, n_cu, st); break;
    case 25: f32_launch_epi<3, 1>(a, epi, blocks, n_cu, st); break;
    case 26: f32_launch_epi<3, 2>(a, epi, blocks, n_cu, st); break;
    case 28: f32_launch_epi<3, 4>(a, epi, blocks, n_cu, st); break;
    case 33: f32_launch_epi<4, 1>(a, epi, blocks, n_cu, st); break;
    default: f32_launch_epi<4, 2>(a, epi, blocks, n_cu, st); break;
  }
}

// once per context, with its device current: more than 64 KB of LDS for the shapes with eight tiles
void fp32_prepare() {
  const F32Gemm a{};
  for (int epi : {(int)EPI_RESIDUAL, (int)EPI_QKV, (int)EPI_SWIGLU, (int)EPI_RELU, (int)EPI_LOGITS}) {
    f32_launch_shape(a, 2, 4, epi, -1, 0, nullptr);
    f32_launch_shape(a, 3, 4, epi, -1, 0, nullptr);
    f32_launch_shape(a, 4, 2, epi, -1, 0, nullptr);
  }
}

// Strips and row tiles per workgroup (neither changes a result): the compute unit with the most workgroups sets the
// time (gate-up of d_model 1024 at 1328 rows: 585 us as 1 x 1, 370 us as 4 strips x 2 tiles).  Cycles per 16-k step of a workgroup:
// 16 per 1 KB fragment from L2, about three times that for weights the first time they are read (HBM), against 32 of the
// matrix cores per tile.
static long f32_cost(int M, int NT, int mt, int nb, int n_cu, bool by_xcd) {
  const long passes = (M + mt * 16 - 1) / (mt * 16), groups = (NT + nb - 1) / nb;
  // by_xcd: as the launch deals them, whole strip groups to an XCD when there are several row passes
  const long xcd_cu = std::max(1, n_cu / 8), per_cu = by_xcd && passes > 1 ? ((groups + 7) / 8 * passes + xcd_cu - 1) / xcd_cu : (groups * passes + n_cu - 1) / n_cu;
  return per_cu * (16 * nb * (2 + passes) / passes + 16 * mt + 32 * nb * mt);
}
static void f32_gemm(F32Gemm a, int epi, int n_cu, hipStream_t st) {
  if (a.M <= 0) return;
  int MT = 1, NB = 1;
  long best = -1;
  for (int mt = 1; mt <= 4; ++mt)
    for (int nb = 1; nb * mt <= 8 && nb <= 4; nb *= 2) {
      const long cost = f32_cost(a.M, a.NT, mt, nb, n_cu, false);
      if (best < 0 || cost < best) { best = cost; MT = mt; NB = nb; }
    }
  // Twelve tiles (one workgroup a CU, by its LDS) where that is estimated faster: one row pass (LM head 32000 x 1024 at 40 rows, whose
  // activations are fetched half as often as at 3 x 2: a verification of 8 sequences x 5 rows 304 -> 299 us); several, where
  // a look at the XCDs confirms it and it replaces 3 x 2 or 4 x 2 (qkv of d_model 1024 at 704 rows 86 -> 73 us, gate-up of 768 at
  // 848 rows 152 -> 128), or 2 x 4 with a share to save (over the products of d_model 512 to 1024 with k of up to 1024
  // 4 % faster, with longer k or less to save up to 3 % slower).  Elsewhere it loses: down of 768 at 784 rows, 12 groups on 8 XCDs, 64 -> 108 us as 3 x 4; the head at 72 rows, 1 x 4
  // keeps four workgroups a CU, 78 -> 103.
  if (MT == 3 || MT == 4 || NB == 4) {
    const bool once = a.M <= 48;
    const long twelve = f32_cost(a.M, a.NT, 3, 4, n_cu, !once), other = f32_cost(a.M, a.NT, MT, NB, n_cu, !once);
    if (once || MT >= 3 ? twelve < other : MT == 2 && 100 * twelve <= (a.KT <= 64 ? 98 : 93) * other) { MT = 3; NB = 4; }
  }
  a.passes = (a.M + MT * 16 - 1) / (MT * 16);
  a.groups = (a.NT + NB - 1) / NB;
  const int blocks = a.passes == 1 ? a.groups : (a.groups + 7) / 8 * 8 * a.passes;
  f32_launch_shape(a, MT, NB, epi, blocks, n_cu, st);
}

// ------------------------------------------------------------------------- attention
// Workgroup: up to 16 query rows of one row group, one head; eight waves take the 16-key tiles in turn (tile t belongs to
// wave t % 8 whatever the row), each with its own running maximum, and meet in LDS in wave order.  The scores' output
// layout (lane 16g + c: keys 4g .. 4g+3 of row c) is the operand layout of the product with V, and the cache's blocks of
// 8 positions make its quadruples 16-byte loads, so nothing is exchanged between lanes but the maxima.
// A row's result depends on its position and its sequence's cache alone: tiles beyond its position leave it unchanged.
template <int HD>
__global__ __launch_bounds__(512) void k_attn_f32(int q_rows, int chunks, const int32_t *__restrict__ grp_seq, int H, int L_pad,
                                                  const float *__restrict__ q, const int32_t *__restrict__ row_pos,
                                                  const float *__restrict__ kc, const float *__restrict__ vc, float *__restrict__ out) {
  constexpr int NI = HD / 16;
  __shared__ f32x4 so[8][4][64];
  __shared__ float smx[8][16], ssum[8][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  const int grp = blockIdx.x / chunks, r0 = (blockIdx.x % chunks) * 16, nr = min(16, q_rows - r0), hh = blockIdx.y, d = H * HD;
  const int b = grp_seq ? grp_seq[grp] : grp;
  const size_t m = (size_t)grp * q_rows + r0 + min(c, nr - 1);
  const int pos = c < nr ? row_pos[m] : -1;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const f32x4 *qp = (const f32x4 *)(q + m * d + (size_t)hh * HD) + g;
  f32x4 qf[NI], acc[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) { qf[i] = qp[4 * i]; acc[i] = zero; }
  const size_t head = ((size_t)b * H + hh) * L_pad * HD;
  const float scale = 1.0f / sqrtf((float)HD);
  float mx = -INFINITY, sum = 0.f;
  f32x4 kf[NI], vf[NI];
  auto fetch = [&](int k0) {
    const f32x4 *kp = (const f32x4 *)(kc + head) + (size_t)((k0 + c) / KV_KBLOCK) * HD + 4 * g + c % KV_KBLOCK;
    const f32x4 *vp = (const f32x4 *)(vc + head + ((size_t)((k0 >> 3) + (g >> 1)) * HD + c) * 8 + (g & 1) * 4);
#pragma unroll
    for (int i = 0; i < NI; ++i) kf[i] = kp[16 * i];
#pragma unroll
    for (int i = 0; i < NI; ++i) vf[i] = vp[32 * i];
  };
  // the first tile is asked for before the rows' positions are here (inside the cache, if behind the last key)
  fetch(min(w * 16, L_pad - 16));
  int last = pos;
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
  for (int k0 = w * 16; k0 <= last; k0 += 128) {
    if (k0 >= 128) fetch(k0);
    f32x4 s0 = zero, s1 = zero;
#pragma unroll
    for (int i = 0; i < NI; i += 2)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 = mfma4(kf[i][e], qf[i][e], s0);
        s1 = mfma4(kf[i + 1][e], qf[i + 1][e], s1);
      }
    const int key = k0 + 4 * g;
    f32x4 p = s0 + s1;
    float tm = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = key + e <= pos ? p[e] * scale : -INFINITY;
      tm = fmaxf(tm, p[e]);
    }
    tm = fmaxf(tm, __shfl_xor(tm, 16, 64));
    tm = fmaxf(tm, __shfl_xor(tm, 32, 64));
    const float mn = fmaxf(mx, tm), ms = mn == -INFINITY ? 0.f : mn, alpha = expf(mx - ms);
    mx = mn;
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = expf(p[e] - ms);
    sum = sum * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
    bool odd = false;  // values that a weight of zero does not take out
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      acc[i] *= alpha;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (key + e > last) vf[i][e] = 0.f;
        odd |= !(fabsf(vf[i][e]) < INFINITY);
      }
    }
    if (!__any(odd)) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i] = mfma4(vf[i][e], p[e], acc[i]);
    } else {  // row by row, without the keys behind the row
      for (int r = 0; r < nr; ++r) {
        const int pr = __shfl(pos, r, 64);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          f32x4 t = acc[i];
#pragma unroll
          for (int e = 0; e < 4; ++e) t = mfma4(key + e <= pr ? vf[i][e] : 0.f, p[e], t);
          if (c == r) acc[i] = t;
        }
      }
    }
  }
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  if (g == 0) { smx[w][c] = mx; ssum[w][c] = sum; }
  float f[8], inv = 0.f;
#pragma unroll
  for (int i0 = 0; i0 < NI; i0 += 4) {
    if (i0 > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) so[w][i][lane] = acc[i0 + i];
    __syncthreads();
    if (i0 == 0) {
      float mm = smx[0][c], L = 0.f;
#pragma unroll
      for (int s = 1; s < 8; ++s) mm = fmaxf(mm, smx[s][c]);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        f[s] = smx[s][c] == -INFINITY ? 0.f : expf(smx[s][c] - mm);
        L = fmaf(ssum[s][c], f[s], L);
      }
      inv = 1.0f / L;
    }
    if (w < 4 && c < nr) {
      f32x4 o = zero;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const f32x4 t = so[s][w][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = fmaf(t[e], f[s], o[e]);
      }
      o = pos < 0 ? zero : o * inv;
      *(f32x4 *)(out + m * d + (size_t)hh * HD + (i0 + w) * 16 + 4 * g) = o;
    }
  }
}

// ------------------------------------------------------------------------- one pass
static F32Gemm f32_args(const void *W, const void *bias, const void *X, int M, int N, int K) {
  F32Gemm a{};
  a.W = (const f32x4 *)W; a.bias = (const float *)bias; a.X = (const float *)X;
  a.M = M; a.N = N; a.NT = (N + 15) / 16; a.KT = K / 16; a.KS = gemm_ks_for(a.KT);
  a.x_mul = 1;
  return a;
}

void fp32_layer(spec_ctx *c, const Model &m, int layer, int B, int q_rows, int b0, const int32_t *grp_seq, hipStream_t st) {
  const spec_model_desc &D = m.desc;
  const int M = B * q_rows, d = D.d_model, f = D.d_ffn, H = D.n_heads, hd = m.hd;
  const LayerW &L = m.layers[layer];
  Workspace &ws = c->ws;
  const bool ln = D.norm_kind == SPEC_NORM_LAYER, swi = D.ffn_kind == SPEC_FFN_SWIGLU;
  const size_t area = (size_t)layer * m.kv_area_elems + (size_t)b0 * H * m.L_pad * hd;
  float *kc = (float *)m.kcache + area, *vc = (float *)m.vcache + area;
  auto behind_norm = [&](const void *W, const void *bias, int N, const void *gain, const void *nb) {
    if (ln) launch_norm(c, m, ws.h, gain, nb, ws.x, M, 0, st);
    F32Gemm a = f32_args(W, bias, ln ? ws.x : ws.h, M, N, d);
    a.fold = !ln; a.eps = D.norm_eps;
    return a;
  };
  {
    F32Gemm a = behind_norm(L.wqkv, L.bqkv, 3 * d, L.attn_norm_w, L.attn_norm_b);
    a.out = (float *)ws.q; a.kc = kc; a.vc = vc; a.row_pos = ws.row_pos; a.grp_seq = grp_seq; a.rope = m.rope;
    a.q_rows = q_rows; a.d = d; a.hd = hd; a.H = H; a.L_pad = m.L_pad;
    f32_gemm(a, EPI_QKV, c->n_cu, st);
  }
  {
    const int chunks = (q_rows + 15) / 16;
    hipLaunchKernelGGL((hd == 64 ? k_attn_f32<64> : k_attn_f32<128>), dim3(B * chunks, H), dim3(512), 0, st, q_rows, chunks, grp_seq, H,
                       m.L_pad, (const float *)ws.q, ws.row_pos, kc, vc, (float *)ws.attn);
  }
  {
    F32Gemm a = f32_args(L.wo, L.bo, ws.attn, M, d, d);
    a.out = ws.h; a.ldo = d;
    f32_gemm(a, EPI_RESIDUAL, c->n_cu, st);
  }
  {
    F32Gemm a = behind_norm(L.w13, L.b13, swi ? 2 * f : f, L.ffn_norm_w, L.ffn_norm_b);
    a.out = (float *)ws.act; a.ldo = f;
    f32_gemm(a, swi ? EPI_SWIGLU : EPI_RELU, c->n_cu, st);
  }
  {
    F32Gemm a = f32_args(L.w2, L.b2, ws.act, M, d, f);
    a.out = ws.h; a.ldo = d;
    f32_gemm(a, EPI_RESIDUAL, c->n_cu, st);
  }
}

// Final norm and LM head: all Mh rows of the pass, or (last_of_q > 0) the last row of each of Mh groups.
void fp32_head(spec_ctx *c, const Model &m, int Mh, int last_of_q, float *logits_or_null, int q, int arg_stride, int32_t *arg_out,
               HeadPartials *leave, hipStream_t st) {
  const spec_model_desc &D = m.desc;
  const bool ln = D.norm_kind == SPEC_NORM_LAYER;
  if (ln) launch_norm(c, m, c->ws.h, m.final_norm_w, m.final_norm_b, c->ws.x, Mh, last_of_q, st);
  F32Gemm a = f32_args(m.lm_head, nullptr, ln ? c->ws.x : c->ws.h, Mh, D.vocab, D.d_model);
  a.fold = !ln; a.eps = D.norm_eps;
  if (!ln && last_of_q > 0) { a.x_mul = last_of_q; a.x_off = last_of_q - 1; }
  a.out = logits_or_null; a.ldo = D.vocab; a.part_val = c->ws.head_part; a.part_idx = c->ws.head_part_idx;
  f32_gemm(a, EPI_LOGITS, c->n_cu, st);
  if (leave) *leave = {a.part_val, a.part_idx, 0, a.NT, D.vocab, arg_out, arg_stride};
  else launch_argmax_partials(a.part_val, a.part_idx, Mh, 0, a.NT, D.vocab, q, arg_stride, arg_out, st);
}

}  // namespace spec

// LM head of up to 32 activation rows over a short k (d_model 256 to 1024): a wave per 16-row strip of W.
//
// With eight k-slices of one to four 32-k steps the streaming kernel (kernels_gemm_mfma.hip) starts a workgroup of eight
// waves per strip that loads a few fragments a wave and spends its time starting, meeting in LDS and writing an arg-max
// partial: 32000 x 768 is 2000 such workgroups.  Here a wave owns whole strips: it asks for all of a strip's k at once,
// computes the eight slices' chains one after the other and adds each to the total, so nothing is exchanged between waves;
// the activations sit in LDS, one copy per workgroup, and the arg-max runs on in registers over the strips of a wave and
// in LDS over the waves, which leaves one partial per row and workgroup instead of one per strip.
//
// Bound by the weight stream behind a start (rows to LDS, their sums of squares) of about 5 us.  Between event pairs, us,
// streaming kernel / this, 16 rows: 32000 x 768 20.4 / 12.2, 50272 x 768 29.4 / 16.9, 32000 x 1024 22.0 / 15.4, 128000 x 512
// 57.6 / 22.2; 32 rows: 32000 x 768 18.3 / 16.3.  (Four row tiles beside a strip's 128 registers spill: 33 rows and more stay
// on the tiled kernel.)
//
// Same bits as the streaming kernel: the same instruction, every k-slice a chain from zero in ascending k, the slices added
// in order, the same arithmetic on the finished sums, the same sum-of-squares order for the folded norm.
#include "mfma_tiles.h"
#include <algorithm>

namespace spec {

#pragma clang fp contract(off)

constexpr int STRIP_WAVES = 8;
constexpr size_t strips_lds(int KT, int MT) { return (size_t)MT * KT * 1024 + STRIP_WAVES * MT * 16 * 8; }

// KTP: 32-k steps per slice.  MT: 16-row tiles of activations.  LN: the folded norm is a LayerNorm (and there is a bias).
template <int KTP, int MT, bool LN>
__global__ __launch_bounds__(512) void k_gemm_strips(GemmArgs a) {
  constexpr int KS = 8, KT = KS * KTP;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [MT][KT] fragments; behind them the waves' arg-max
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int m_tiles = (a.M + 15) >> 4, stride = (int)gridDim.x * STRIP_WAVES;
  int strip = (int)blockIdx.x * STRIP_WAVES + w;

  u32x4_v wf[KT];
  auto load_strip = [&](int s) {
    const u32x4_v *wp = (const u32x4_v *)a.W + (size_t)s * (KT * 64) + lane;
#pragma unroll
    for (int u = 0; u < KT; ++u) wf[u] = __builtin_nontemporal_load(wp + u * 64);
  };
  load_strip(min(strip, a.NT - 1));
  // activations: fragment f = mt * KT + kt by wave f % 8
  u32x4_v *xs = (u32x4_v *)smem;
  // Where a slice's reads start, made to depend on a sum of the slice before the last: the compiler would otherwise read all
  // fragments ahead of the strips, and spill them.
  auto slice_lane = [&](float before) {
    int l = lane;
    asm volatile("" : "+v"(l) : "v"(before));
    return l;
  };
#pragma unroll 4
  for (int i = 0; i < MT * KTP; ++i) {
    const int f = w + 8 * i, mt = f / KT;
    xs[f * 64 + lane] = ((const u32x4_v *)a.X)[((size_t)min(mt, m_tiles - 1) * KT + (f - mt * KT)) * 64 + lane];
  }
  __syncthreads();

  float rinv[MT], mean[MT], bv[MT];
  int bi[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    rinv[mt] = 1.0f; mean[mt] = 0.f; bv[mt] = -INFINITY; bi[mt] = 0x7fffffff;
    if (!a.fold_x) continue;
    float t = 0.f, ts = 0.f, before = mt > 0 ? rinv[mt - 1] : 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float q = 0.f, p = 0.f;
      const int l = slice_lane(before);
      before = t;
#pragma unroll
      for (int u = 0; u < KTP; ++u) {
        const u32x4_v x = xs[(mt * KT + s * KTP + u) * 64 + l];
        q = frag_ssq(x, q);
        if (LN) p = frag_sum(x, p);
      }
      t = s == 0 ? q : t + q;
      ts = s == 0 ? p : ts + p;
    }
    if (LN) row_ln_from_lane(t, ts, a.ss_d, a.ss_eps, rinv[mt], mean[mt]);
    else rinv[mt] = row_inv_from_lane_ssq(t, a.ss_d, a.ss_eps);
  }

  while (strip < a.NT) {
    const int n = strip * 16 + 4 * g;
    f32x4_v b4, w4;
    if (LN) { b4 = *(const f32x4_v *)(a.bias + n); w4 = *(const f32x4_v *)(a.wsum + n); }
    f32x4_v tot[MT];
    float before = 0.f, last = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      f32x4_v cur[MT];
      const int l = slice_lane(before);
      before = last;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) cur[mt] = (f32x4_v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = s * KTP; u < (s + 1) * KTP; ++u)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) cur[mt] = Mfma16::run(wf[u], xs[(mt * KT + u) * 64 + l], cur[mt]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        last = cur[mt][0];
        if (s == 0) tot[mt] = cur[mt];
        else { tot[mt][0] += cur[mt][0]; tot[mt][1] += cur[mt][1]; tot[mt][2] += cur[mt][2]; tot[mt][3] += cur[mt][3]; }
      }
    }
    strip += stride;
    if (strip < a.NT) load_strip(strip);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      f32x4_v v = tot[mt];
      if (LN) { v[0] -= mean[mt] * w4[0]; v[1] -= mean[mt] * w4[1]; v[2] -= mean[mt] * w4[2]; v[3] -= mean[mt] * w4[3]; }
      v[0] *= a.out_scale; v[1] *= a.out_scale; v[2] *= a.out_scale; v[3] *= a.out_scale;  // exact: a power of two
      v[0] *= rinv[mt]; v[1] *= rinv[mt]; v[2] *= rinv[mt]; v[3] *= rinv[mt];
      if (LN) { v[0] += b4[0]; v[1] += b4[1]; v[2] += b4[2]; v[3] += b4[3]; }
      const int m = mt * 16 + c;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (n + i < a.N) argmax_combine(bv[mt], bi[mt], v[i], n + i);
      float *dump = m < a.M ? logits_row(a, m) : nullptr;
      if (dump) dump_logits(a, dump, n, v);
    }
  }

  // the row's candidates: the four lane groups, then the waves (lowest index wins ties)
  float *sv = (float *)(smem + MT * KT * 1024);
  int *si = (int *)(sv + STRIP_WAVES * MT * 16);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float ov = __shfl_xor(bv[mt], o, 64);
      const int oi = __shfl_xor(bi[mt], o, 64);
      argmax_combine(bv[mt], bi[mt], ov, oi);
    }
    if (g == 0) { sv[(w * MT + mt) * 16 + c] = bv[mt]; si[(w * MT + mt) * 16 + c] = bi[mt]; }
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m < a.M) {
    float v = sv[m];
    int i = si[m];
#pragma unroll
    for (int s = 1; s < STRIP_WAVES; ++s) argmax_combine(v, i, sv[s * MT * 16 + m], si[s * MT * 16 + m]);
    a.part_val[(size_t)m * a.n_part + blockIdx.x] = v;
    a.part_idx[(size_t)m * a.n_part + blockIdx.x] = i;
  }
}

// blocks < 0: preparation pass (more than 64 KB of LDS)
template <int KTP, int MT, bool LN>
static void strips_launch(const GemmArgs &a, int blocks, hipStream_t st) {
  constexpr size_t lds = strips_lds(8 * KTP, MT);
  if (blocks < 0) (void)hipFuncSetAttribute((const void *)k_gemm_strips<KTP, MT, LN>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  else hipLaunchKernelGGL((k_gemm_strips<KTP, MT, LN>), dim3(blocks), dim3(STRIP_WAVES * 64), lds, st, a);
}
template <int KTP>
static void strips_launch_mt(const GemmArgs &a, int MT, bool ln, int blocks, hipStream_t st) {
  if (MT == 1) ln ? strips_launch<KTP, 1, true>(a, blocks, st) : strips_launch<KTP, 1, false>(a, blocks, st);
  else ln ? strips_launch<KTP, 2, true>(a, blocks, st) : strips_launch<KTP, 2, false>(a, blocks, st);
}
static void strips_launch_k(const GemmArgs &a, int KTP, int MT, bool ln, int blocks, hipStream_t st) {
  if (KTP == 1) strips_launch_mt<1>(a, MT, ln, blocks, st);
  else if (KTP == 2) strips_launch_mt<2>(a, MT, ln, blocks, st);
  else if (KTP == 3) strips_launch_mt<3>(a, MT, ln, blocks, st);
  else strips_launch_mt<4>(a, MT, ln, blocks, st);
}

// Where the weights are enough to hide the start: up to 16 rows from four strips a CU on (streaming / this, us: 16384 x 512
// 11.2 / 8.4, 16384 x 1024 13.6 / 12.0, but 8192 x 1024 8.9 / 11.3 and 12000 x 1024 11.9 / 11.6), with two row tiles from
// seven on (32000 x 1024 20.6 / 19.6, but 16384 x 768 11.6 / 13.6).
bool gemm_takes_strips(const GemmArgs &a) {
  const int n_cu = a.n_cu > 0 ? a.n_cu : 256;
  return a.M > 0 && a.M <= 32 && a.KS == 8 && a.KT <= 32 && a.NT >= (a.M <= 16 ? 4 : 7) * n_cu && !(a.tune & 0xff) && (a.wsum != nullptr) == (a.bias != nullptr);
}
int gemm_strips_partials(const GemmArgs &a) {  // workgroups: one a CU
  return std::min(a.n_cu > 0 ? a.n_cu : 256, (a.NT + STRIP_WAVES - 1) / STRIP_WAVES);
}
void launch_gemm_strips(GemmArgs a, hipStream_t st) {
  a.n_part = gemm_strips_partials(a);
  strips_launch_k(a, a.KT / 8, a.M <= 16 ? 1 : 2, a.wsum != nullptr, a.n_part, st);
}
void gemm_strips_prepare() {
  const GemmArgs a{};
  for (int ktp = 1; ktp <= 4; ++ktp)
    for (int mt : {1, 2})
      for (bool ln : {false, true}) strips_launch_k(a, ktp, mt, ln, -1, nullptr);
}

}  // namespace spec

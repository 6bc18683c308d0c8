// Speculative sampling: the non-greedy form of the acceptance step (Sec. 2 describes speculative decoding and
// cites this rule for sampling; Alg. 1 itself is greedy).
//
//   q_j = softmax(draft logits of step j / T),  p_j = softmax(target logits of row j / T)
//   keep proposal t_j  if  u * q_j[t_j] < p_j[t_j];  at the first j that fails, emit one token drawn from
//   max(0, p_j - q_j) (normalised) and stop;  if all are kept, emit one token drawn from the next target row.
// Proposals that come from no distribution (a table) count as point masses: q_j[t_j] = 1.
// A draw from weights w with a uniform number u is the smallest index whose cumulative weight exceeds u * sum(w).
//
// The kernels here only replace the "greedy tokens of the target" by tokens chosen so that the unchanged
// longest-matching-prefix rule reproduces the outcome: entry j is t_{j+1} while proposals are kept, the drawn token
// at the first rejection (never equal to the rejected proposal: its residual weight is zero), the bonus draw
// behind s kept proposals.  Commit, roll-back, end token and budgets then work as in the greedy case.
//
// One workgroup per row (proposal draws) or per place of a round (verification; large rounds: several places in turn).  A
// wave owns a contiguous segment of the vocabulary and walks it 256 logits at a time, four per lane; lanes, then waves are
// added in a fixed order by every thread alike, so a draw depends on the row alone.
//
// Bound by latency and by reading rows twice (from L2 the second time): a row of 32000 logits is 128 KB, a place needs two of
// them, and 22 us for that are about 5 bytes per clock and CU, well below what a CU can take from memory.  While
// they fit the chip, all places of a round are therefore decided at once, each as if its round reached it (draws behind
// the first rejection are thrown away by k_sample_seal), so that the rows stream through B * (s + 1) CUs instead of one
// after the other through B; a row is read once for maximum and sum together, and once more (from L2) where a token is
// drawn from it.  A thread with a contiguous chunk of its own (loads 512 bytes apart across a wave), a pass for each of
// maximum and sum, and a sequence's places in turn took 87 us for 64 sequences x 4 places of 32000 logits with draft rows;
// this takes 26 us (30 with a test for -inf and for the end beside every exponential: what is left of a place is about
// equal parts waiting for loads and exponentials).  Larger rounds take places in turn (workgroups_per_sequence).
#include "spec_internal.h"
#include "device_utils.h"
#include <algorithm>
#include <limits>
#include <type_traits>

namespace spec {

#pragma clang fp contract(off)

constexpr int SMP_STEP = 256;   // logits per wave and step: a float4 per lane

// this wave's part of the row: [k0, end), k0 a multiple of SMP_STEP (empty: end <= k0)
struct Seg { int k0, end; };
template <int W>
__device__ __forceinline__ Seg my_seg(int V) {
  const int per = ((V - 1) / (W * SMP_STEP) + 1) * SMP_STEP;
  const int k0 = (int)(threadIdx.x >> 6) * per;
  return Seg{k0, V - k0 < per ? V : k0 + per};
}

// z[k .. k+3] (k a multiple of four), -inf from `end` on.  VEC: one 16-byte load, for V a multiple of four and rows
// aligned to 16 bytes; the launch chooses.  The addresses are clamped into the row instead of branched around, so that
// the loads of several steps can be in flight together.
template <bool VEC>
__device__ __forceinline__ void load4z(const float *__restrict__ z, int k, int V, int end, float (&o)[4]) {
  constexpr float fill = -INFINITY;
  if (VEC) {
    const float4 v = *(const float4 *)(z + min(k, V - 4));
    const bool in = k < end;  // V and every segment's end are multiples of four here
    o[0] = in ? v.x : fill; o[1] = in ? v.y : fill; o[2] = in ? v.z : fill; o[3] = in ? v.w : fill;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = z[min(k + i, V - 1)];
      o[i] = k + i < end ? v : fill;
    }
  }
}
// U steps of z[k ..]: as load4z, without its clamps and selects where all of them lie before `end`
template <bool VEC, int U>
__device__ __forceinline__ void load_steps(const float *__restrict__ z, int k, int lane4, int V, int end, float (&v)[U][4]) {
  if (VEC && k + U * SMP_STEP <= end) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const float4 t = *(const float4 *)(z + k + i * SMP_STEP + lane4);
      v[i][0] = t.x; v[i][1] = t.y; v[i][2] = t.z; v[i][3] = t.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < U; ++i) load4z<VEC>(z, k + i * SMP_STEP + lane4, V, end, v[i]);
  }
}
// How a kernel loads its rows, LD: bit 0 for 16-byte loads, above it the steps whose loads are in flight together (single loads
// need four addresses a step).  with_loads chooses.
constexpr bool ld_vec(int LD) { return LD & 1; }
constexpr int ld_steps(int LD) { return LD >> 1; }

// Exclusive prefix over the waves of one value per wave, *total = the sum over the workgroup: added in wave order, the
// same bits in every thread.  sh: W floats.
template <int W>
__device__ __forceinline__ float waves_prefix(float v, float *sh, float *total) {
  const int wv = threadIdx.x >> 6;
  __syncthreads();  // sh may still be read by the previous user
  if ((threadIdx.x & 63) == 0) sh[wv] = v;
  __syncthreads();
  float before = 0.f, all = 0.f;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    if (i == wv) before = all;
    all += sh[i];
  }
  *total = all;
  return before;
}

// maximum of a row, the same in every thread
template <int W, int LD>
__device__ __forceinline__ float row_max(const float *__restrict__ z, int V, float *sh) {
  const Seg g = my_seg<W>(V);
  const int lane4 = (threadIdx.x & 63) * 4;
  constexpr int U = ld_steps(LD);
  float lm = -INFINITY;
#pragma unroll 1
  for (int k = g.k0; k < g.end; k += U * SMP_STEP) {
    float v[U][4];
    load_steps<ld_vec(LD), U>(z, k, lane4, V, g.end, v);
#pragma unroll
    for (int i = 0; i < U; ++i) lm = fmaxf(fmaxf(lm, v[i][0]), fmaxf(fmaxf(v[i][1], v[i][2]), v[i][3]));
  }
  lm = wave_max(lm);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = lm;
  __syncthreads();
  float m = sh[0];
#pragma unroll
  for (int i = 1; i < W; ++i) m = fmaxf(m, sh[i]);
  return m;
}

// Running (maximum, sum of exp((z - maximum) * inv_T)).  -inf counts as weight 0 also while the maximum is -inf.
__device__ __forceinline__ float rescaled(float Z, float m, float m_new, float inv_T) {
  return m == -INFINITY ? Z : Z * __expf((m - m_new) * inv_T);
}
template <int U>
__device__ __forceinline__ void stats_step(const float (&v)[U][4], float inv_T, float &m, float &Z) {
  float mn = m;
#pragma unroll
  for (int i = 0; i < U; ++i) mn = fmaxf(fmaxf(mn, v[i][0]), fmaxf(fmaxf(v[i][1], v[i][2]), v[i][3]));
  // the exponential of -inf is 0 by itself, but for a maximum that is -inf too
  const float base = mn == -INFINITY ? 0.f : mn;
  float ls = 0.f;
#pragma unroll
  for (int i = 0; i < U; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) ls += __expf((v[i][e] - base) * inv_T);
  Z = rescaled(Z, m, mn, inv_T) + ls;
  m = mn;
}

// Maximum and sum of exp((z - max) * inv_T) of a target row and, PAIR, of a draft row, the same bits in every thread
// (a row of -inf alone has no distribution: its sum is NaN).  sh: 4 * W floats.
struct RowStats { float m, Z; };
template <int W, int LD, bool PAIR>
__device__ __forceinline__ void row_stats(const float *__restrict__ zp, const float *__restrict__ zq, int V, float inv_T,
                                          float *sh, RowStats &p, RowStats &q) {
  const Seg g = my_seg<W>(V);
  const int lane4 = (threadIdx.x & 63) * 4, wv = threadIdx.x >> 6;
  constexpr int U = ld_steps(LD);
  float mp = -INFINITY, Zp = 0.f, mq = -INFINITY, Zq = 0.f;
#pragma unroll 1
  for (int k = g.k0; k < g.end; k += U * SMP_STEP) {
    float v[U][4], w[U][4];
    load_steps<ld_vec(LD), U>(zp, k, lane4, V, g.end, v);
    if (PAIR) load_steps<ld_vec(LD), U>(zq, k, lane4, V, g.end, w);
    stats_step<U>(v, inv_T, mp, Zp);
    if (PAIR) stats_step<U>(w, inv_T, mq, Zq);
  }
  const float wmp = wave_max(mp), wZp = wave_sum(rescaled(Zp, mp, wmp, inv_T));
  float wmq = 0.f, wZq = 0.f;
  if (PAIR) { wmq = wave_max(mq); wZq = wave_sum(rescaled(Zq, mq, wmq, inv_T)); }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    sh[wv] = wmp; sh[W + wv] = wZp;
    if (PAIR) { sh[2 * W + wv] = wmq; sh[3 * W + wv] = wZq; }
  }
  __syncthreads();
  auto combine = [&](const float *s) {
    RowStats r{s[0], 0.f};
#pragma unroll
    for (int i = 1; i < W; ++i) r.m = fmaxf(r.m, s[i]);
#pragma unroll
    for (int i = 0; i < W; ++i) r.Z += rescaled(s[W + i], s[i], r.m, inv_T);
    if (r.m == -INFINITY) r.Z = __builtin_nanf("");
    return r;
  };
  p = combine(sh);
  if (PAIR) q = combine(sh + 2 * W);
}

// Draw with u from the weights w4(k, lane4, end, out) -> weights of the lane's four tokens of W4::UNROLL steps from k on (zero
// from `end` on): every thread returns the same index.  *total_out: the sum of all weights.
template <int W, class W4>
__device__ __forceinline__ int block_draw(int V, W4 w4, float u, float *sh, int *sh_i, float *total_out = nullptr) {
  const Seg g = my_seg<W>(V);
  const int lane = threadIdx.x & 63, lane4 = lane * 4, wv = threadIdx.x >> 6;
  constexpr int U = W4::UNROLL;
  float local = 0.f;
#pragma unroll 1
  for (int k = g.k0; k < g.end; k += U * SMP_STEP) {
    float w[U][4];
    w4(k, lane4, g.end, w);
#pragma unroll
    for (int i = 0; i < U; ++i) local += (w[i][0] + w[i][1]) + (w[i][2] + w[i][3]);
  }
  local = wave_sum(local);
  float total;
  const float excl = waves_prefix<W>(local, sh, &total);
  if (threadIdx.x == 0) *sh_i = -1;
  if (total_out) *total_out = total;
  float x = u * total;
  if (!(x < total)) x = total * 0.99999994f;  // u < 1, but the product may round up to the total
  __syncthreads();
  // the owner of x: the last wave with weight whose prefix does not exceed x (the prefixes come from sums in
  // different associations, so "prefix <= x < prefix + local" could leave a hair's gap between neighbours)
  if (lane == 0 && local > 0.f && excl <= x) atomicMax(sh_i, wv);
  __syncthreads();
  const int owner = *sh_i;
  __syncthreads();
  if (wv == owner) {
    float run = excl;
    int pick = -1, last = -1;  // wave-wide pick; this lane's last token with weight
    constexpr int UW = U > 4 ? 4 : U;
    // as in the sum, the loads of several steps are in flight together: one step after the other, each waiting for its rows, the
    // walk took half a microsecond more (64 sequences x 4 places 26.7 -> 26.2)
#pragma unroll 1
    for (int k = g.k0; k < g.end && pick < 0; k += UW * SMP_STEP) {
      float w[UW][4];
      w4(k, lane4, g.end, w);
#pragma unroll
      for (int s = 0; s < UW; ++s) {
        if (pick >= 0) break;
        const int kl = k + s * SMP_STEP + lane4;
        const float mine = (w[s][0] + w[s][1]) + (w[s][2] + w[s][3]);
        float inc = mine;  // inclusive prefix over the lanes, added pairwise by doubling distances
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const float up = __shfl_up(inc, o, 64);
          if (lane >= o) inc += up;
        }
        int own = -1;  // the first of this lane's tokens whose cumulative weight exceeds x, or the nearest one with weight
        float c = run + (inc - mine);
        bool past = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          c += w[s][i];
          if (w[s][i] > 0.f) {
            last = kl + i;
            if (!past || own < 0) own = kl + i;
          }
          past |= c > x;
        }
        const unsigned long long hit = __ballot(mine > 0.f && run + inc > x);
        if (hit) pick = __shfl(own, __ffsll(hit) - 1, 64);
        run += __shfl(inc, 63, 64);
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
    if (lane == 0) *sh_i = pick >= 0 ? pick : last;  // the walk may end a hair below x: then the segment's last token
  } else if (owner < 0 && threadIdx.x == 0) {
    *sh_i = 0;  // all weights zero or not finite: the lowest index, as the greedy rule does for a row of NaNs
  }
  __syncthreads();
  return *sh_i;
}

// weights exp((z - m) * inv_T) of a row, optionally with one token removed; -inf behind the end makes the zeros there
template <int W, int LD>
struct ExpW {
  static constexpr int UNROLL = ld_steps(LD);
  const float *z; int V; float m, inv_T; int drop;
  template <int U>
  __device__ __forceinline__ void operator()(int k, int lane4, int end, float (&w)[U][4]) const {
    load_steps<ld_vec(LD), U>(z, k, lane4, V, end, w);
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) w[s][i] = __expf((w[s][i] - m) * inv_T);
    if ((unsigned)(drop - k) < (unsigned)(U * SMP_STEP)) {
#pragma unroll
      for (int s = 0; s < U; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k + s * SMP_STEP + lane4 + i == drop) w[s][i] = 0.f;
    }
  }
};
// residual weights max(0, p - q) of a target and a draft row
template <int W, int LD>
struct ResidW {
  static constexpr int UNROLL = ld_steps(LD) > 1 ? ld_steps(LD) / 2 : 1;  // two rows a step
  ExpW<W, LD> p, q; float ip, iq;
  template <int U>
  __device__ __forceinline__ void operator()(int k, int lane4, int end, float (&w)[U][4]) const {
    float b[U][4];
    p(k, lane4, end, w); q(k, lane4, end, b);
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) { const float r = w[s][i] * ip - b[s][i] * iq; w[s][i] = r > 0.f ? r : 0.f; }
  }
};

__device__ __forceinline__ float uniform_at(const float *__restrict__ u, const int32_t *__restrict__ n, int b, int off,
                                            int u_rows, int kind) {
  // with lengths: a table [B][u_rows][3] indexed by the absolute position of the token the number decides;
  // without: [B][u_rows][3] indexed by the row of the round
  const int row = n ? min(n[b] + off, u_rows - 1) : off;
  return u[((size_t)b * u_rows + row) * 3 + kind];
}

// One proposal per sequence: a draw from softmax(logits[b] / T).  out[b * out_stride].
template <int W, int LD>
__global__ __launch_bounds__(W * 64) void k_sample_rows(const float *__restrict__ logits, int V, float inv_T,
                                                             const float *__restrict__ u, const int32_t *__restrict__ n,
                                                             int off, int u_rows, int32_t *__restrict__ out, int out_stride) {
  __shared__ float sh[W];
  __shared__ int sh_i;
  const int b = blockIdx.x;
  const float *z = logits + (size_t)b * V;
  const float m = row_max<W, LD>(z, V, sh);  // a draw needs the maximum only: its own pass over the row adds the weights up
  const float uu = n ? uniform_at(u, n, b, off, u_rows, 0) : u[b];
  const int tok = block_draw<W>(V, ExpW<W, LD>{z, V, m, inv_T, -1}, uu, sh, &sh_i);
  if (threadIdx.x == 0) out[(size_t)b * out_stride] = tok;
}

// Place j of a round, decided as if the round reached it: t_{j+1} if the proposal is kept, -1 - (the drawn token) if it is
// rejected; the same in every thread.  zq: the draft's row, null for a point-mass proposal.
template <int W, int LD>
__device__ __forceinline__ int decide_place(const float *__restrict__ zp, const float *__restrict__ zq, int V, float inv_T,
                                            int tj, float ua, float us, float *sh, int *sh_i) {
  RowStats p, q;
  const bool valid = tj >= 0 && tj < V;
  int res;
  if (zq) {
    row_stats<W, LD, true>(zp, zq, V, inv_T, sh, p, q);
    const float pt = valid ? __expf((zp[tj] - p.m) * inv_T) * (1.0f / p.Z) : 0.f;
    const float qt = valid ? __expf((zq[tj] - q.m) * inv_T) * (1.0f / q.Z) : 1.f;
    if (ua * qt < pt) {
      res = tj;
    } else {
      const ExpW<W, LD> wp{zp, V, p.m, inv_T, -1};
      float total;
      res = block_draw<W>(V, ResidW<W, LD>{wp, ExpW<W, LD>{zq, V, q.m, inv_T, -1}, 1.0f / p.Z, 1.0f / q.Z}, us, sh, sh_i, &total);
      // p = q everywhere leaves no residual (not reachable with u < 1 and a valid proposal): draw from p
      if (!(total > 0.f)) res = block_draw<W>(V, wp, us, sh, sh_i);
      res = -1 - res;
    }
  } else {
    row_stats<W, LD, false>(zp, nullptr, V, inv_T, sh, p, q);
    const float pt = valid ? __expf((zp[tj] - p.m) * inv_T) * (1.0f / p.Z) : 0.f;
    if (ua < pt) res = tj;
    else res = -1 - block_draw<W>(V, ExpW<W, LD>{zp, V, p.m, inv_T, valid ? tj : -1}, us, sh, sh_i);
  }
  return res;
}
// The bonus draw, for a round that keeps every proposal: needs the row's maximum only.
template <int W, int LD>
__device__ __forceinline__ int bonus_draw(const float *__restrict__ zp, int V, float inv_T, float us, float *sh, int *sh_i) {
  const float m = row_max<W, LD>(zp, V, sh);
  return block_draw<W>(V, ExpW<W, LD>{zp, V, m, inv_T, -1}, us, sh, sh_i);
}

// Verification, a workgroup per (sequence, place j), places 0 .. s_b: a[b][j] = decide_place, or the bonus draw at place s_b.
// k_sample_seal does the rest.
//   tl: target logits, row b * (s + 1) + j;  dl: draft logits of step j + 1 at ((size_t)j * d_rows + b) * V, or null
template <int W, int LD>
__global__ __launch_bounds__(W * 64) void k_sample_verify(const float *__restrict__ tl, const float *__restrict__ dl,
                                                          int d_rows, int b0, int s, int V, float inv_T,
                                                          const int32_t *__restrict__ t, int t_stride,
                                                          const int32_t *__restrict__ seq_s,
                                                          const float *__restrict__ u, const int32_t *__restrict__ n,
                                                          int u_rows, int32_t *__restrict__ a, int a_stride) {
  __shared__ float sh[4 * W];
  __shared__ int sh_i;
  const int b = b0 + blockIdx.x / (s + 1), j = blockIdx.x % (s + 1);
  const int sb = seq_s ? min(s, max(0, seq_s[b])) : s;
  if (j > sb) return;
  const float *zp = tl + ((size_t)b * (s + 1) + j) * V;
  const float us = uniform_at(u, n, b, j, u_rows, 2);
  if (j == sb) {
    const int tok = bonus_draw<W, LD>(zp, V, inv_T, us, sh, &sh_i);
    if (threadIdx.x == 0) a[(size_t)b * a_stride + j] = tok;
    return;
  }
  const int res = decide_place<W, LD>(zp, dl ? dl + ((size_t)j * d_rows + b) * V : nullptr, V, inv_T, t[(size_t)b * t_stride + j],
                                       uniform_at(u, n, b, j, u_rows, 1), us, sh, &sh_i);
  if (threadIdx.x == 0) a[(size_t)b * a_stride + j] = res;
}

// The same with `per` <= s workgroups to a sequence: workgroup i of them takes the places i, i + per, ... up to s_b in
// turn and stops at the first it rejects.  Every place before the round's first rejection is then decided (a place is
// left out only behind a rejection of its own workgroup); k_sample_seal ignores what lies behind.
template <int W, int LD, bool DRAFT>
__global__ __launch_bounds__(W * 64) void k_sample_verify_turns(const float *__restrict__ tl, const float *__restrict__ dl,
                                                                int d_rows, int b0, int per, int s, int V, float inv_T,
                                                                const int32_t *__restrict__ t, int t_stride,
                                                                const int32_t *__restrict__ seq_s,
                                                                const float *__restrict__ u, const int32_t *__restrict__ n,
                                                                int u_rows, int32_t *__restrict__ a, int a_stride) {
  __shared__ float sh[4 * W];
  __shared__ int sh_i;
  const int b = b0 + blockIdx.x / per;
  const int sb = seq_s ? min(s, max(0, seq_s[b])) : s;
  for (int j = blockIdx.x % per; j <= sb; j += per) {
    const float *zp = tl + ((size_t)b * (s + 1) + j) * V, *zq = DRAFT ? dl + ((size_t)j * d_rows + b) * V : nullptr;
    const bool bonus = j == sb;
    const int tj = bonus ? 0 : t[(size_t)b * t_stride + j];
    const float ua = uniform_at(u, n, b, j, u_rows, 1), us = uniform_at(u, n, b, j, u_rows, 2);
    const int res = bonus ? bonus_draw<W, LD>(zp, V, inv_T, us, sh, &sh_i) : decide_place<W, LD>(zp, zq, V, inv_T, tj, ua, us, sh, &sh_i);
    if (threadIdx.x == 0) a[(size_t)b * a_stride + j] = res;
    if (res < 0) break;
  }
}

// Ends every sequence's round at its first rejection: that place gets its drawn token, the places behind it -1.  For the
// stand-alone entry point (accepted given, no seq_s) also the count and the emitted tokens, by the longest-prefix rule.
// 16 lanes per sequence, one per place: a round has at most 16.
__global__ __launch_bounds__(64) void k_sample_seal(int B, int s, const int32_t *__restrict__ seq_s, int32_t *__restrict__ a,
                                                    int a_stride, const int32_t *__restrict__ t, int32_t *__restrict__ accepted,
                                                    int32_t *__restrict__ emitted) {
  const int lane = threadIdx.x, j = lane & 15, b = blockIdx.x * 4 + (lane >> 4);
  const bool on = b < B;
  const int sb = on ? (seq_s ? min(s, max(0, seq_s[b])) : s) : -1;
  int32_t *ab = a + (size_t)(on ? b : 0) * a_stride;
  int v = j <= sb ? ab[j] : 0;
  const unsigned rej = (unsigned)(__ballot(v < 0) >> (lane & 48)) & 0xffffu;
  const int first = rej ? __ffs(rej) - 1 : 16;
  if (j >= first) {
    v = j == first ? -1 - v : -1;
    if (on && j <= s) ab[j] = v;
  }
  if (!accepted) return;
  const bool stop = j >= s || (on && t[(size_t)b * s + j] != v);
  const unsigned stops = (unsigned)(__ballot(stop) >> (lane & 48)) & 0xffffu;
  const int l = __ffs(stops) - 1;  // place s always stops
  if (!on || j > s) return;
  if (j == 0) accepted[b] = l;
  emitted[(size_t)b * (s + 1) + j] = j <= l ? v : -1;
}

// 1 / T as the kernels take it, never 0: the zero weight of a masked token, and of what lies behind a row's end, is the
// exponential of -inf * inv_T, and T = inf (every token alike) would make that the one of -inf * 0.  The smallest positive
// float leaves finite logits their weight of 1 there (3.4e38 * 1.4e-45 = 5e-7).
static float inverse_temperature(float T) { return std::max(1.0f / T, std::numeric_limits<float>::denorm_min()); }

static bool rows_vec(const float *z, int V) { return (V & 3) == 0 && ((uintptr_t)z & 15) == 0; }

// Waves per workgroup, by the vocabulary alone (a draw's sums then still depend on nothing but the row): 4 up to 8192
// logits, where 16 have too little to do and large rounds pay for starting and meeting them, 16 beyond, where 4 need more
// trips to memory than a small round can hide.  4 / 16 waves, us: 4096 rows of 1000 logits 12 / 37, 1024 of 6000 11 / 18, 16 of
// 6000 the same; 16 rows of 16000 14 / 10.
static bool narrow_rows(int V) { return V <= 8192; }

// f(waves per workgroup, LD) for rows of V logits.  Four steps in flight a wave of a narrow workgroup, eight of a wide one, but no more
// than a wave's segment has: steps behind its end cost their exponentials (64 draws from 1000 logits 4.8 us with four, 4.1 with
// one; from 2000 5.1, 4.5 with two; sums and draws stay the same bits).
template <class F>
static void with_loads(int V, bool vec, F f) {
  auto go = [&](auto W, auto vec_ld, auto single_ld) { vec ? f(W, vec_ld) : f(W, single_ld); };
  using std::integral_constant;
  constexpr integral_constant<int, 4> four{};
  if (!narrow_rows(V)) go(integral_constant<int, 16>{}, integral_constant<int, 8 * 2 + 1>{}, integral_constant<int, 2 * 2>{});
  else if (V <= 4 * SMP_STEP) go(four, integral_constant<int, 1 * 2 + 1>{}, integral_constant<int, 1 * 2>{});
  else if (V <= 8 * SMP_STEP) go(four, integral_constant<int, 2 * 2 + 1>{}, integral_constant<int, 2 * 2>{});
  else go(four, integral_constant<int, 4 * 2 + 1>{}, integral_constant<int, 2 * 2>{});
}

void launch_sample_rows(const float *logits, int rows, int V, float temperature, const float *u, const int32_t *n, int off,
                        int u_rows, int32_t *out, int out_stride, hipStream_t st) {
  if (rows <= 0) return;
  with_loads(V, rows_vec(logits, V), [&](auto W_, auto LD_) {
    constexpr int W = decltype(W_)::value, LD = decltype(LD_)::value;
    hipLaunchKernelGGL((k_sample_rows<W, LD>), dim3(rows), dim3(W * 64), 0, st, logits, V, inverse_temperature(temperature), u, n, off, u_rows,
                       out, out_stride);
  });
}
// How many workgroups share the places of a sequence's round.  A workgroup per place reads rows behind the first rejection
// for nothing, which is free only while the chip has room: `slots` is the workgroups it works on at a time (one of 16 waves
// per CU; four of 4 waves).
//   point-mass proposals: what fits the slots, so that rounds that end at once cost one place each.
//   proposals with a draft row (kept more often): as few as take no more turns, if every proposal is kept, than a workgroup
//   per place would.
// A workgroup per sequence with the older kernel / a workgroup per place / this, us, draft rows where (d), 32000 logits:
//   256 sequences x 9 places, 1.4 kept (d) 189 / 185 / 94, all kept (d) 230 / 129 / 126, none kept 32 / 131 / 20
//   1024 x 9, 1.4 kept (d) 585 / 681 / 243, all kept (d) 932 / 439 / 425, none kept 91 / 498 / 64
//   128 x 9, 1.2 kept (d) 185 / 101 / 59, all kept (d) 202 / 67 / 66, none kept 30 / 71 / 20
//   1024 x 9 of 1000 logits, 1.6 kept (d) 45 / 267 / 38, none kept 17 / 212 / 18
static int workgroups_per_sequence(int B, int s, bool draft, int slots) {
  if (!draft) return std::min(s + 1, std::max(1, slots / B));
  auto turns = [&](int per) { return ((int64_t)B * per + slots - 1) / slots * ((s + per) / per); };
  int per = 1;
  while (per < s + 1 && turns(per) > turns(s + 1)) ++per;
  return per;
}

void launch_sample_verify(const float *tl, const float *dl, int d_rows, int B, int s, int V, float temperature,
                          const int32_t *t, int t_stride, const int32_t *seq_s, const float *u, const int32_t *n, int u_rows,
                          int32_t *a, int a_stride, hipStream_t st, int32_t *accepted, int32_t *emitted) {
  if (B <= 0) return;
  const bool vec = rows_vec(tl, V) && (!dl || rows_vec(dl, V)), narrow = narrow_rows(V);
  const float inv_T = inverse_temperature(temperature);
  const int per = workgroups_per_sequence(B, s, dl != nullptr, narrow ? 1024 : 256);
  const int per_launch = (1 << 21) / per;  // a grid holds less than 2^32 threads
  for (int64_t b0 = 0; b0 < B; b0 += per_launch) {
    const int nb = (int)std::min<int64_t>(per_launch, B - b0);
    with_loads(V, vec, [&](auto W_, auto LD_) {
      constexpr int W = decltype(W_)::value, LD = decltype(LD_)::value;
      if (per == s + 1)
        hipLaunchKernelGGL((k_sample_verify<W, LD>), dim3(nb * per), dim3(W * 64), 0, st, tl, dl, d_rows, (int)b0, s, V, inv_T,
                           t, t_stride, seq_s, u, n, u_rows, a, a_stride);
      else
        hipLaunchKernelGGL((dl ? k_sample_verify_turns<W, LD, true> : k_sample_verify_turns<W, LD, false>), dim3(nb * per), dim3(W * 64), 0,
                           st, tl, dl, d_rows, (int)b0, per, s, V, inv_T, t, t_stride, seq_s, u, n, u_rows, a, a_stride);
    });
  }
  hipLaunchKernelGGL(k_sample_seal, dim3((B - 1) / 4 + 1), dim3(64), 0, st, B, s, seq_s, a, a_stride, t, accepted, emitted);
}

}  // namespace spec

using namespace spec;

extern "C" int spec_sample_tokens(void *hip_stream, const float *d_logits, int32_t rows, int32_t vocab, float temperature,
                                  const float *d_uniforms, int32_t *d_tokens) {
  if (rows < 0 || vocab < 1) return fail_noctx(SPEC_ERR_INVALID_ARG, "spec_sample_tokens: rows=%d vocab=%d", rows, vocab);
  if (!(temperature > 0.f)) return fail_noctx(SPEC_ERR_INVALID_ARG, "spec_sample_tokens: temperature must be positive");
  if (rows == 0) return SPEC_OK;
  if (!d_logits || !d_uniforms || !d_tokens) return fail_noctx(SPEC_ERR_INVALID_ARG, "spec_sample_tokens: null pointer");
  if (rows > 65535 * 16) return fail_noctx(SPEC_ERR_CAPACITY, "spec_sample_tokens: rows=%d beyond 1048560", rows);
  launch_sample_rows(d_logits, rows, vocab, temperature, d_uniforms, nullptr, 0, 1, d_tokens, 1, (hipStream_t)hip_stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail_noctx(SPEC_ERR_HIP, "spec_sample_tokens: %s", hipGetErrorString(e));
  return SPEC_OK;
}

extern "C" int spec_sample_accept(void *hip_stream, const float *d_target_logits, const float *d_draft_logits,
                                  const int32_t *d_proposals, const float *d_uniforms, int32_t B, int32_t s, int32_t vocab,
                                  float temperature, int32_t *d_chosen, int32_t *d_accepted, int32_t *d_emitted) {
  if (B < 0 || s < 0 || vocab < 1) return fail_noctx(SPEC_ERR_INVALID_ARG, "spec_sample_accept: B=%d s=%d vocab=%d", B, s, vocab);
  if (!(temperature > 0.f)) return fail_noctx(SPEC_ERR_INVALID_ARG, "spec_sample_accept: temperature must be positive");
  if (s > 15) return fail_noctx(SPEC_ERR_CAPACITY, "spec_sample_accept: s=%d beyond 15", s);
  if (B == 0) return SPEC_OK;
  if (!d_target_logits || !d_uniforms || !d_chosen || !d_accepted || !d_emitted || (s > 0 && !d_proposals))
    return fail_noctx(SPEC_ERR_INVALID_ARG, "spec_sample_accept: null pointer");
  hipStream_t st = (hipStream_t)hip_stream;
  launch_sample_verify(d_target_logits, d_draft_logits, B, B, s, vocab, temperature, d_proposals, s, nullptr, d_uniforms, nullptr,
                       s + 1, d_chosen, s + 1, st, d_accepted, d_emitted);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail_noctx(SPEC_ERR_HIP, "spec_sample_accept: %s", hipGetErrorString(e));
  return SPEC_OK;
}

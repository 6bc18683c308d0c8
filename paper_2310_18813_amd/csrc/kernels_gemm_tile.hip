// GEMM for more than 32 activation rows, where its estimated time beats the streaming kernel's.
//
// The streaming kernel covers 64 rows per pass and re-streams the weights for every pass.
// Here one workgroup holds up to 256 rows of a group of weight strips, so a weight byte is
// fetched once per up to 256 rows, and both operands reach the waves through LDS:
//
//   workgroup = 8 waves = 2 (strip halves) x 4 (row quarters); wave tile = NBW strips x MTW
//   16-row tiles; workgroup tile = 2*NBW strips x 4*MTW row tiles.
//   Per 32-k step the workgroup needs 2*NBW weight fragments and 4*MTW activation
//   fragments of 1 KB each.  Weights and activations are both stored in fragment order in
//   global memory, so a fragment is one 16-byte load per lane that goes straight to LDS, several
//   steps ahead, and the waves read it back with one conflict-free 16-byte LDS load per lane.
//
// Wide outputs (QKV, gate-up / fc1, LM head) walk all of k in one workgroup.  Narrow outputs (the
// residual GEMMs, N = d_model) would leave most CUs idle that way: there each workgroup takes
// one k-slice of its tile (EPI_PARTIAL) and k_partial_reduce adds the slices in slice order.
//
// Results are bit-identical to the streaming kernel: the same instruction, every k-slice a
// chain of MFMAs from zero in ascending k, the slices added in order, the same epilogue code.
#include "mfma_tiles.h"
#include <algorithm>
#include <cmath>

namespace spec {

#pragma clang fp contract(off)

// One fragment of 1 KB from `base` (uniform) straight to LDS byte offset `lds` (uniform), lane l's 16 bytes at 16 l.
// Written out because the compiler, which would have to assume that every LDS read depends on such a load, waits for
// all of them in front of each read; here the waits are placed by hand (vmcnt before the barrier that publishes a slot).
// NT: non-temporally
template <bool NT>
__device__ __forceinline__ void load_frag_to_lds(const unsigned char *base, unsigned lane_off, unsigned lds) {
  if (NT) asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
  else asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
}
// the same for all lanes (mask -1, uniform) or for none (0); counted by vmcnt either way
__device__ __forceinline__ void load_frag_to_lds_masked(const unsigned char *base, unsigned lane_off, unsigned lds, int mask) {
  asm volatile("s_mov_b32 exec_lo, %3\n\ts_mov_b32 exec_hi, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1" ::"{m0}"(lds),
               "v"(lane_off), "s"(base), "s"(mask) : "memory");
}
// -1 if x is negative, else 0, in a scalar register (written out: the compiler may make a per-lane select of a mask)
__device__ __forceinline__ int sign_mask(int x) {
  int m;
  asm("s_ashr_i32 %0, %1, 31" : "=s"(m) : "s"(x) : "scc");
  return m;
}
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "wait count field");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int N, int R>
__device__ __forceinline__ void wait_loads_and_reads() {
  static_assert(N >= 0 && N < 64 && R >= 0 && R < 16, "wait count fields");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)" ::"n"(N), "n"(R) : "memory");
}

// Fragments of one 32-k step of a workgroup, and the ring of LDS slots that hold one step each: as deep as LDS allows,
// since the loads in flight are what the small tiles, which stream weights for few rows, are bound by.
template <int MTW, int NBW> struct TileShape {
  static constexpr int NBG = 2 * NBW, MTG = 4 * MTW, FRAGS = NBG + MTG;
  static constexpr int SLOT = FRAGS * 1024;
  static constexpr int FIT = 160 / FRAGS;
  static constexpr int RING = FIT > 16 ? 16 : FIT;
  static constexpr size_t LDS = (size_t)RING * SLOT;
  static_assert(RING >= 4, "a step being read, the next one, the one being freed, and one in flight");
};

__host__ __device__ constexpr bool tile_takes_row_sums(int MTW) { return MTW == 1; }

// activation fragments of the next step whose reads go out behind the first nb strips of a step: none behind the last
// strip, since the next step needs them all at once
__host__ __device__ constexpr int x_reads_upto(int nb, int MTW, int NBW) { return nb >= NBW - 1 ? MTW : nb * MTW / (NBW - 1); }
// pins the instruction order of a step: strip by strip MTW multiplies, then its weight fragment's read and its share of
// the MTW activation fragments' reads
template <int MTW, int NBW, int NB = 0>
__device__ __forceinline__ void pin_step() {
  if constexpr (NB < NBW) {
    __builtin_amdgcn_sched_group_barrier(0x008, MTW, 0);                                             // MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, 1 + x_reads_upto(NB + 1, MTW, NBW) - x_reads_upto(NB, MTW, NBW), 0);  // LDS reads
    pin_step<MTW, NBW, NB + 1>();
  }
}

// NORM: what is folded in front (0 nothing, 1 RMS norm, 2 LayerNorm).  T: the cache's type (EPI_QKV only).
// LOADS: LOADS_PASSES several row passes; else a single one, so that no other workgroup reads a weight: LOADS_NT loads them
// non-temporally.  (With several row passes that takes them out of the L2 for the next workgroup: loads alone, 22016 x 4096 at 6592
// rows 632 -> 711 us.)  LOADS_KEPT does not: weights that fit the memory-side cache are there from the last pass (two layers
// of d_model 1536 with an LM head of 32000, 211 MB: the head at 72 rows 22.9 us, non-temporally 24.7; 14 layers of it 25.7 and
// 24.3).  fast_weights_kept says which.
enum TileLoads { LOADS_PASSES, LOADS_NT, LOADS_KEPT };
template <class T, int MTW, int NBW, int EPI, int NORM, int LOADS>
__global__ __launch_bounds__(512, 2) void k_gemm_tile(GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using S = TileShape<MTW, NBW>;
  constexpr int NBG = S::NBG, MTG = S::MTG, FRAGS = S::FRAGS, SLOT = S::SLOT, RING = S::RING;
  constexpr bool ONCE = LOADS != LOADS_PASSES, NT = LOADS == LOADS_NT;
  // Fragments a wave fetches per step, between its multiplies.  ONCE: LW strips and LX row tiles, and of the W_REST strips and
  // X_REST tiles left over the first and the last waves one each.  Else strips and tiles in one row, w, w + 8, ..., and in the
  // last place the waves without a fragment issue a load without lanes, so that all waves count alike.  Such a load takes a
  // place among the loads a CU keeps in flight like any other, and those are what a launch of few rows is bound by (10
  // fragments of 36 rows were 16 loads: gate-up 22016 x 4096 40.0 -> 35.1 us; 12 of 64 rows 16: 46.0 -> 40.3); with several
  // row passes the branches around the rest cost more than it gains (776 rows, 5120 wide, a layer +4 %).  The rest goes out in
  // front of a step's multiplies, with one row tile per wave behind them (80 rows of 20480 x 5120 50.6 and 52.7, 36 rows of
  // 22016 x 4096 38.1 and 35.1).
  constexpr int LW = ONCE ? NBG / 8 : 0, W_REST = ONCE ? NBG % 8 : 0, LX = MTG / 8, X_REST = ONCE ? MTG % 8 : 0;
  constexpr int LPW = ONCE ? LW + LX : (FRAGS + 7) / 8;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = w & 1, wm = w >> 1;
  const int c = lane & 15, g = lane >> 4;
  constexpr bool PARTIAL = EPI == EPI_PARTIAL;
  int G, pass, slice_id = 0;
  if (!PARTIAL && a.passes == 1) { G = blockIdx.x; pass = 0; }
  else if (PARTIAL && a.KS == 8) {
    // one k-slice per workgroup, and one k-slice per XCD (workgroups are dealt round-robin to the 8 XCDs): all
    // workgroups on an XCD read the same k-slice of the activations, which its L2 then fetches once for the chip
    const int id = blockIdx.x, rest = id >> 3;
    slice_id = id & 7;
    pass = rest % a.passes;
    G = rest / a.passes;
  } else if (PARTIAL) {
    // one k-slice per workgroup, slice by slice; all row passes of a strip group on one XCD
    const int id = blockIdx.x, gpx = (a.groups + 7) >> 3;
    int rest = id >> 3;
    slice_id = rest / (gpx * a.passes);
    rest %= gpx * a.passes;
    pass = rest % a.passes;
    G = (rest / a.passes) * 8 + (id & 7);
  } else {
    // The tiles in blocks of up to 8 row passes, strip group by strip group, one eighth of that row to each XCD (workgroups are
    // dealt round-robin to the 8 XCDs): the 32 workgroups an XCD runs at a time are 8 passes x 4 groups and share both
    // operands in its L2, and none has more than an eighth of all tiles, rounded up.  (Strip groups dealt to the XCDs whole, with all
    // their passes, left XCDs with a group more than others: 4096 x 11008 at 1328 rows, 11 groups, 218 -> 138 us, 20480 x 5120
    // at 784 rows 221 -> 195, 6592 rows of the 7B width's four products -1.5 to -2.6 %.)  a.whole_groups: dealt whole after all.
    const bool whole = EPI == EPI_QKV && a.whole_groups;
    const int id = blockIdx.x, row = whole ? (a.groups + 7) >> 3 : a.groups, total = row * a.passes, per = whole ? total : (total + 7) >> 3, at = id >> 3;
    const int tile = whole ? at : (id & 7) * per + at;
    if (at >= per || tile >= total) return;
    const int blk = tile / (row * 8), rest = tile - blk * row * 8, in_blk = min(8, a.passes - blk * 8);
    pass = blk * 8 + rest % in_blk;
    G = whole ? rest / in_blk * 8 + (id & 7) : rest / in_blk;
  }
  G = __builtin_amdgcn_readfirstlane(G);
  pass = __builtin_amdgcn_readfirstlane(pass);
  slice_id = __builtin_amdgcn_readfirstlane(slice_id);
  if (G >= a.groups) return;
  const int kt_per = a.KT / a.KS;
  const int KTL = PARTIAL ? kt_per : a.KT;          // steps of this workgroup
  const int kt_lo = PARTIAL ? slice_id * kt_per : 0;  // first k-tile
  const int nt0 = G * NBG;
  const int mtile0 = pass * MTG;
  const int m_tiles = (a.M + 15) >> 4;

  // Fragment f of a step (and its place in the slot): f < NBG weight strip nt0 + f; else activation tile f - NBG.
  const bool w_rest = W_REST > 0 && w < W_REST, x_rest = X_REST > 0 && w >= 8 - X_REST;
  auto frag_of = [&](int i) {
    if (!ONCE) return min(w + 8 * i, FRAGS - 1);
    if (i < LPW) return i < LW ? w + 8 * i : NBG + w + 8 * (i - LW);
    return i == LPW ? min(w + 8 * LW, NBG - 1) : NBG + min(8 * LX + max(w - (8 - X_REST), 0), MTG - 1);
  };
  const unsigned char *src[LPW + 2];
#pragma unroll
  for (int i = 0; i < LPW + 2; ++i) {
    const int f = frag_of(i);
    const size_t row = f < NBG ? (size_t)min(nt0 + f, a.NT - 1) : (size_t)min(mtile0 + f - NBG, m_tiles - 1);
    src[i] = (const unsigned char *)(f < NBG ? a.W : a.X) + (row * a.KT + kt_lo) * 1024;
  }
  const unsigned lane_off = lane * 16;
  const int last_mask = sign_mask(w - (FRAGS - 8 * (LPW - 1)));  // !ONCE: the waves with an LPW-th fragment
  // this wave's fragments at byte k of their rows into the slot at `lds`
  auto fetch1 = [&](int i, size_t k, unsigned lds) {
    if (ONCE && i < LW) load_frag_to_lds<NT>(src[i] + k, lane_off, lds + (w + 8 * i) * 1024);
    else if (ONCE) load_frag_to_lds<false>(src[i] + k, lane_off, lds + (NBG + w + 8 * (i - LW)) * 1024);
    else if (i < LPW - 1 || FRAGS % 8 == 0) load_frag_to_lds<false>(src[i] + k, lane_off, lds + (w + 8 * i) * 1024);
    else load_frag_to_lds_masked(src[i] + k, lane_off, lds + (w + 8 * i) * 1024, last_mask);
  };
  auto fetch_rest = [&](size_t k, unsigned lds) {
    if (w_rest) load_frag_to_lds<NT>(src[LPW] + k, lane_off, lds + (8 * LW + w) * 1024);
    if (x_rest) load_frag_to_lds<false>(src[LPW + 1] + k, lane_off, lds + (NBG + 8 * LX + w - (8 - X_REST)) * 1024);
  };
  // step kt of this wave's fragments into ring position `at`; beyond the end the last step is fetched again: nobody
  // reads it, and no wait count depends on where the end lies
  auto fetch_k = [&](int kt) { return (size_t)min(kt, KTL - 1) * 1024; };
  auto fetch_lds = [&](int at) { return (unsigned)(at * SLOT); };

  f32x4_v cur[NBW][MTW], tot[NBW][MTW];
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
      cur[nb][mt] = (f32x4_v){0.f, 0.f, 0.f, 0.f};
      tot[nb][mt] = (f32x4_v){0.f, 0.f, 0.f, 0.f};
    }

  // Folded norm.  With one row tile per wave the row sums of squares (and the plain sums of a LayerNorm) come from the
  // operand fragments inside the loop, beside the multiplies (frag_ssq: per lane, one chain per k-slice, slices added in
  // order).  With more they hold up the multiplies of a step, which all waves start together: 7 to 18 us per launch at
  // 80 to 256 rows (whichever wave tile), against the 5 us of k_row_inv_x, which then has run before.
  constexpr bool INLOOP = NORM != 0 && tile_takes_row_sums(MTW);
  float ssq_cur[MTW], ssq_tot[MTW], sum_cur[MTW], sum_tot[MTW];
#pragma unroll
  for (int mt = 0; mt < MTW; ++mt) ssq_cur[mt] = ssq_tot[mt] = sum_cur[mt] = sum_tot[mt] = 0.f;

  // Fragments in registers.  A weight fragment takes the next step's behind its last multiply; the activation
  // fragments, which every strip multiplies, alternate between two sets.  The reads then spread evenly over the
  // multiplies of a step (the CU's LDS queue is short: read in a burst at the end of the step, with all waves in
  // phase behind the barrier, they cost as much time as the multiplies).
  u32x4_v wf[NBW], xa[MTW], xb[MTW];
  const unsigned char *w_base = smem + lane * 16 + wn * NBW * 1024, *x_base = smem + lane * 16 + (NBG + wm * MTW) * 1024;
  auto rd = [](const unsigned char *p) { return *(const u32x4_v *)p; };

  auto slice_end = [&]() {  // the slice's chains join the running totals, in slice order (a chain that starts from +0 never
#pragma unroll               // ends at -0: adding the first one to +0 keeps its bits)
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) {
        tot[nb][mt][0] += cur[nb][mt][0]; tot[nb][mt][1] += cur[nb][mt][1];
        tot[nb][mt][2] += cur[nb][mt][2]; tot[nb][mt][3] += cur[nb][mt][3];
      }
    if (INLOOP) {
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) { ssq_tot[mt] += ssq_cur[mt]; sum_tot[mt] += sum_cur[mt]; }
    }
  };
  // One step: the multiplies of the fragments at hand (x), strip by strip, and the reads of the next step's (xn) from
  // ring position `at`; the fetches of a later step (offset fk, to flds) go out between them.
  // `first`: the first step of a k-slice, whose chains start from zero.
  auto step = [&](auto first, const u32x4_v (&x)[MTW], u32x4_v (&xn)[MTW], int at, size_t fk, unsigned flds) {
    constexpr bool FIRST = decltype(first)::value;
    const unsigned char *wp = w_base + at * SLOT, *xp = x_base + at * SLOT;
    if (MTW > 1) fetch_rest(fk, flds);
    if (INLOOP) {
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) {
        ssq_cur[mt] = frag_ssq(x[mt], FIRST ? 0.f : ssq_cur[mt]);
        if (NORM == 2) sum_cur[mt] = frag_sum(x[mt], FIRST ? 0.f : sum_cur[mt]);
      }
    }
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) {
        if (FIRST) cur[nb][mt] = Mfma16::run(wf[nb], x[mt], (f32x4_v){0.f, 0.f, 0.f, 0.f});
        else cur[nb][mt] = Mfma16::run(wf[nb], x[mt], cur[nb][mt]);
      }
      wf[nb] = rd(wp + nb * 1024);
#pragma unroll
      for (int mt = x_reads_upto(nb, MTW, NBW); mt < x_reads_upto(nb + 1, MTW, NBW); ++mt) xn[mt] = rd(xp + mt * 1024);
#pragma unroll
      for (int i = nb * LPW / NBW; i < (nb + 1) * LPW / NBW; ++i) fetch1(i, fk, flds);
    }
    pin_step<MTW, NBW>();
    if (MTW == 1) fetch_rest(fk, flds);
  };
  // A bare barrier, not __syncthreads(): the fence of the latter would wait for the loads in flight.
  // `left`: this wave's loads are done but for those of the last `left` steps; its LDS reads but for the READS of the
  // step it has just issued (LDS reads return in order).  The earlier ones, from the position that is fetched into behind
  // the barrier, have then arrived wherever the scheduler has put the multiplies that use them.
  constexpr int READS = NBW + MTW;
  auto publish = [&](auto left) {
    constexpr int L = decltype(left)::value;
    if (w_rest && x_rest) wait_loads_and_reads<L * (LPW + 2), READS>();
    else if (w_rest || x_rest) wait_loads_and_reads<L * (LPW + 1), READS>();
    else wait_loads_and_reads<L * LPW, READS>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // Step kt lives at ring position kt % RING.  At the top of step kt the registers hold (or await) its fragments, and
  // the barrier there says that step kt + 1 is in LDS.  Behind it every wave has the fragments of step kt - 1 in its
  // registers, whose position takes step kt + RING - 1.
  int at = 0, kt = 0;
  auto turn = [&](auto first, const u32x4_v (&x)[MTW], u32x4_v (&xn)[MTW]) {
    publish(std::integral_constant<int, RING - 3>{});
    const unsigned flds = fetch_lds(at == 0 ? RING - 1 : at - 1);
    at = at + 1 == RING ? 0 : at + 1;
    step(first, x, xn, at, fetch_k(kt + RING - 1), flds);
    ++kt;
  };
#pragma unroll
  for (int s = 0; s < RING - 1; ++s) {
#pragma unroll
    for (int i = 0; i < LPW; ++i) fetch1(i, fetch_k(s), fetch_lds(s));
    fetch_rest(fetch_k(s), fetch_lds(s));
  }
  publish(std::integral_constant<int, RING - 2>{});
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): with no scalar load left under way the waits on LDS reads in the loop are exact counts
#pragma unroll
  for (int mt = 0; mt < MTW; ++mt) xa[mt] = rd(x_base + mt * 1024);
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb) wf[nb] = rd(w_base + nb * 1024);
  while (kt < KTL) {  // a k-slice per round; the steps in pairs, since the activation fragments alternate
    turn(std::true_type{}, xa, xb);
    int left = kt_per - 1;
    for (; left > 1; left -= 2) {
      turn(std::false_type{}, xb, xa);
      turn(std::false_type{}, xa, xb);
    }
    if (left) {
      turn(std::false_type{}, xb, xa);
    } else {
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) xa[mt] = xb[mt];
    }
    slice_end();
  }
  wait_loads<0>();  // drain the over-fetched tail before the epilogue
  float rv[MTW], mv[MTW];  // 1 / rms (LayerNorm: 1 / std and mean) of this lane's rows
#pragma unroll
  for (int mt = 0; mt < MTW; ++mt) {
    rv[mt] = 1.0f; mv[mt] = 0.f;
    if (INLOOP) {
      if (NORM == 2) row_ln_from_lane(ssq_tot[mt], sum_tot[mt], a.ss_d, a.ss_eps, rv[mt], mv[mt]);
      else rv[mt] = row_inv_from_lane_ssq(ssq_tot[mt], a.ss_d, a.ss_eps);
    } else if (NORM != 0) {
      const int m = min((mtile0 + wm * MTW + mt) * 16 + c, a.M - 1);
      rv[mt] = a.rinv_ws[m];
      if (a.wsum) mv[mt] = a.mean_ws[m];
    }
  }
  if (PARTIAL) {  // the slice's chain as it is; k_partial_reduce adds the slices in order
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) {
        const int nt = nt0 + wn * NBW + nb, m = (mtile0 + wm * MTW + mt) * 16 + c, n = nt * 16 + 4 * g;
        if (nt < a.NT && m < a.M) *(f32x4_v *)(a.part + ((size_t)slice_id * a.part_rows + m) * a.N + n) = tot[nb][mt];
      }
  } else {
    wave_epilogue<T, PARTIAL ? EPI_RESIDUAL : EPI, MTW, NBW>(a, tot, nt0 + wn * NBW, mtile0 + wm * MTW, lane, rv, mv);
  }
}

// ((P_0 + P_1) + ...) + P_{KS-1} for four consecutive outputs; with eight slices all loads go out before the first add
__device__ __forceinline__ f32x4_v sum_slices(const float *__restrict__ p, size_t stride, int KS) {
  if (KS == 8) {
    f32x4_v q[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) q[s] = *(const f32x4_v *)(p + s * stride);
    f32x4_v v = q[0];
#pragma unroll
    for (int s = 1; s < 8; ++s) { v[0] += q[s][0]; v[1] += q[s][1]; v[2] += q[s][2]; v[3] += q[s][3]; }
    return v;
  }
  f32x4_v v = *(const f32x4_v *)p;
  for (int s = 1; s < KS; ++s) {
    const f32x4_v q = *(const f32x4_v *)(p + s * stride);
    v[0] += q[0]; v[1] += q[1]; v[2] += q[2]; v[3] += q[3];
  }
  return v;
}

// Second half of a split residual GEMM: out = ((P_0 + P_1) + ...) + P_{KS-1}, then the same epilogue as
// everywhere (scale, bias, h += out).  One thread per four consecutive outputs of a row.
__global__ __launch_bounds__(256) void k_partial_reduce(GemmArgs a) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int n4 = a.N >> 2;
  if (idx >= (size_t)a.M * n4) return;
  const int m = (int)(idx / n4), n = (int)(idx % n4) * 4;
  const float *p = a.part + (size_t)m * a.N + n;
  const size_t stride = (size_t)a.part_rows * a.N;
  tile_epilogue<f16_t, EPI_RESIDUAL>(a, sum_slices(p, stride, a.KS), n >> 4, m, (n & 15) >> 2);
}


// The same reduction, one workgroup per row, for the producer of the next GEMM's activations.  After the update the
// row's fp16-rounded values sit in LDS, and one thread per (k-slice of the next GEMM, lane group) adds their squares
// up exactly as that GEMM would take them from its operand fragments (frag_ssq: eight consecutive elements per 32-k
// step, ascending, one chain per k-slice); the slices are added in order, then the lane groups as
// row_inv_from_lane_ssq pairs them: a.rinv_ws[m] = 1 / rms of the row, the very bits k_row_inv_x would leave --
// which then need not run.  a.ssq_ks = the k-slices of the next GEMM (at most 8).
// A LayerNorm folded into the next GEMM (a.mean_ws set) wants the plain sums too, taken the same way (frag_sum):
// a.mean_ws[m] = the row's mean and a.rinv_ws[m] = 1 / std, as row_ln_from_lane computes them.
__global__ __launch_bounds__(1024) void k_partial_reduce_rows(GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char reduce_smem[];
  op_t *xs = (op_t *)reduce_smem;  // [N] fp16: the updated row as the next GEMM will read it
  __shared__ float ssq_s[8][4];
  const int m = blockIdx.x, n4 = a.N >> 2;
  const size_t stride = (size_t)a.part_rows * a.N;
  for (int i = threadIdx.x; i < n4; i += blockDim.x) {
    const int n = i * 4;
    const float *p = a.part + (size_t)m * a.N + n;
    op_t o4[4];
    residual_update(a, sum_slices(p, stride, a.KS), n, m, o4);
    *(uint2 *)(xs + n) = *(const uint2 *)o4;
  }
  __syncthreads();
  const int steps = (a.N >> 5) / a.ssq_ks;
  __shared__ float sum_s2[8][4];
  const bool lnx = a.mean_ws != nullptr;  // the next GEMM folds a LayerNorm: the plain sums and the mean as well
  if ((int)threadIdx.x < a.ssq_ks * 4) {
    const int w = threadIdx.x >> 2, g = threadIdx.x & 3;
    float s = 0.f, t = 0.f;
    for (int u = 0; u < steps; ++u) {
      const u32x4_v f = *(const u32x4_v *)(xs + (w * steps + u) * 32 + g * 8);
      s = frag_ssq(f, s);
      if (lnx) t = frag_sum(f, t);
    }
    ssq_s[w][g] = s;
    sum_s2[w][g] = t;
  }
  __syncthreads();
  if (threadIdx.x < 4) {  // one lane per lane group: the slices in order, then the pairs as the GEMM kernels add them
    const int g = threadIdx.x;
    float t = ssq_s[0][g], ts = sum_s2[0][g];
    for (int w = 1; w < a.ssq_ks; ++w) { t += ssq_s[w][g]; ts += sum_s2[w][g]; }
    t += __shfl_xor(t, 1, 64);
    t += __shfl_xor(t, 2, 64);
    ts += __shfl_xor(ts, 1, 64);
    ts += __shfl_xor(ts, 2, 64);
    if (g == 0) {
      if (lnx) {
        const float mean = ts / (float)a.ss_d, var = fmaxf(t / (float)a.ss_d - mean * mean, 0.f);
        a.rinv_ws[m] = 1.0f / sqrtf(var + a.ss_eps);
        a.mean_ws[m] = mean;
      } else {
        a.rinv_ws[m] = 1.0f / sqrtf(t / (float)a.ss_d + a.ss_eps);
      }
    }
  }
}

// 1 / rms of every row of the fp16 activations X, in exactly the order the GEMM kernels add the squares up
// themselves (frag_ssq): one workgroup per 16-row tile, wave w walks k-slice w, the slice sums meet in LDS and are
// added in slice order.  For the tiled kernel with more than one row tile per wave.
__global__ __launch_bounds__(512) void k_row_inv_x(const void *__restrict__ X, int M, int KT, int KS, int d, float eps,
                                                   float *__restrict__ rinv, float *__restrict__ mean_out) {
  __shared__ float ssq_s[8][64];
  __shared__ float sum_s[8][64];
  const bool lnx = mean_out != nullptr;  // folded LayerNorm: mean and 1 / std instead of 1 / rms
  float t = 0.f;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  const int tile = blockIdx.x, kt_per = KT / KS;
  const u32x4_v *xp = (const u32x4_v *)X + (size_t)tile * KT * 64 + lane;
  float s = 0.f;
  int kt = w * kt_per;
  const int kt1 = kt + kt_per;
  for (; kt + 8 <= kt1; kt += 8) {
    u32x4_v xf[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) xf[u] = xp[(size_t)(kt + u) * 64];
#pragma unroll
    for (int u = 0; u < 8; ++u) s = frag_ssq(xf[u], s);
    if (lnx) {
#pragma unroll
      for (int u = 0; u < 8; ++u) t = frag_sum(xf[u], t);
    }
  }
  for (; kt < kt1; ++kt) {
    const u32x4_v f = xp[(size_t)kt * 64];
    s = frag_ssq(f, s);
    if (lnx) t = frag_sum(f, t);
  }
  if (KS > 1) {
    ssq_s[w][lane] = s;
    sum_s[w][lane] = t;
    __syncthreads();
    s = ssq_s[0][lane];
    t = sum_s[0][lane];
    for (int i = 1; i < KS; ++i) { s += ssq_s[i][lane]; t += sum_s[i][lane]; }
  }
  float v, mean = 0.f;
  if (lnx) row_ln_from_lane(s, t, d, eps, v, mean);
  else v = row_inv_from_lane_ssq(s, d, eps);
  const int m = tile * 16 + c;
  if (w == 0 && g == 0 && m < M) {
    rinv[m] = v;
    if (lnx) mean_out[m] = mean;
  }
}

// blocks < 0: preparation pass (the kernel may use more than the default 64 KB of LDS)
template <class T, int MTW, int NBW, int EPI, int NORM>
static void launch_one(const GemmArgs &a, int blocks, hipStream_t st) {
  constexpr size_t lds = TileShape<MTW, NBW>::LDS;
  if (blocks < 0) {
    (void)hipFuncSetAttribute((const void *)k_gemm_tile<T, MTW, NBW, EPI, NORM, LOADS_PASSES>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipFuncSetAttribute((const void *)k_gemm_tile<T, MTW, NBW, EPI, NORM, LOADS_NT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipFuncSetAttribute((const void *)k_gemm_tile<T, MTW, NBW, EPI, NORM, LOADS_KEPT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  } else if (a.passes > 1) {
    hipLaunchKernelGGL((k_gemm_tile<T, MTW, NBW, EPI, NORM, LOADS_PASSES>), dim3(blocks), dim3(512), lds, st, a);
  } else if (a.w_kept) {
    hipLaunchKernelGGL((k_gemm_tile<T, MTW, NBW, EPI, NORM, LOADS_KEPT>), dim3(blocks), dim3(512), lds, st, a);
  } else {
    hipLaunchKernelGGL((k_gemm_tile<T, MTW, NBW, EPI, NORM, LOADS_NT>), dim3(blocks), dim3(512), lds, st, a);
  }
}

template <class T, int MTW, int NBW, int EPI>
static void launch_norm(const GemmArgs &a, int blocks, hipStream_t st) {
  if (tile_takes_row_sums(MTW) && a.wsum) launch_one<T, MTW, NBW, EPI, tile_takes_row_sums(MTW) ? 2 : 1>(a, blocks, st);
  else launch_one<T, MTW, NBW, EPI, 1>(a, blocks, st);
}

template <int MTW, int NBW>
static void launch_epi_tile(int dtype, const GemmArgs &a, int epi, int blocks, hipStream_t st) {
  switch (epi) {
    case EPI_QKV:
      if (dtype == SPEC_DTYPE_BF16) launch_norm<bf16_t, MTW, NBW, EPI_QKV>(a, blocks, st);
      else launch_norm<f16_t, MTW, NBW, EPI_QKV>(a, blocks, st);
      break;
    case EPI_SWIGLU: launch_norm<f16_t, MTW, NBW, EPI_SWIGLU>(a, blocks, st); break;
    case EPI_RELU: launch_norm<f16_t, MTW, NBW, EPI_RELU>(a, blocks, st); break;
    case EPI_LOGITS: launch_norm<f16_t, MTW, NBW, EPI_LOGITS>(a, blocks, st); break;
    case EPI_PARTIAL: launch_one<f16_t, MTW, NBW, EPI_PARTIAL, 0>(a, blocks, st); break;
    default: launch_one<f16_t, MTW, NBW, EPI_RESIDUAL, 0>(a, blocks, st); break;
  }
}

template <int MTW>
static void launch_nb_tile(int dtype, const GemmArgs &a, int NBW, int epi, int blocks, hipStream_t st) {
  if (NBW == 2) launch_epi_tile<MTW, 2>(dtype, a, epi, blocks, st);
  else if (NBW == 3) launch_epi_tile<MTW, 3>(dtype, a, epi, blocks, st);
  else if (NBW == 4) launch_epi_tile<MTW, 4>(dtype, a, epi, blocks, st);
  else launch_epi_tile<MTW, 6>(dtype, a, epi, blocks, st);
}

static void launch_shape(int dtype, const GemmArgs &a, int MTW, int NBW, int epi, int blocks, hipStream_t st) {
  if (MTW == 1) launch_nb_tile<1>(dtype, a, NBW, epi, blocks, st);
  else if (MTW == 2) launch_nb_tile<2>(dtype, a, NBW, epi, blocks, st);
  else if (MTW == 3) launch_nb_tile<3>(dtype, a, NBW, epi, blocks, st);
  else launch_nb_tile<4>(dtype, a, NBW, epi, blocks, st);
}

// Wave tile (MTW 16-row tiles x NBW strips) for a launch, and how long it takes, in us.  A workgroup occupies a CU, so
// a launch runs in rounds of n_cu workgroups.  Fitted to a sweep of all 16 shapes over 36 .. 8128 rows, seven weight
// matrices of the 7B, 13B and 33B widths, whole and split by k-slice (1300 launches; rms error 11 %): per step a
// constant for the meeting of the waves and the multiplies (us per tile) beside the fetches (us per KB), which overlap
// in part; per round the pipeline's filling and the epilogue; and no launch is faster than its weights stream from HBM.
// Over the sweep's 117 (matrix, row count) cells the shape it picked was 0.6 % slower than the best one, 11 % at worst.
// Three terms came later.  From a sweep of 36 .. 512 rows (14 matrices, 1412 launches): weights that several row passes read stream
// more slowly than those a single pass loads non-temporally, and the row sums of a folded norm, taken in the loop with one row
// tile per wave, cost a step 0.04 us; over its 162 cells the pick was then 0.8 % slower than the best (1.5 % before), 15360 x 5120 at
// 80 and 128 rows 50 -> 41 and 53 -> 46 us, 22016 x 4096 at 256 rows 63 -> 59, 12288 x 4096 at 80 rows 38 -> 33.  And larger wave
// tiles need k_row_inv_x in front, unless the producer has left the statistics: 3.5 us with its launch (without that term
// narrow products took it: 8192 x 1024 at 224 rows 12 -> 15 us).
enum Fold { FOLD_NONE, FOLD_WANTED, FOLD_LEFT };  // no norm folded in; its row statistics still to be taken; left by the producer
static Fold fold_of(const GemmArgs &a) { return !a.fold_x ? FOLD_NONE : a.stats_left ? FOLD_LEFT : FOLD_WANTED; }
constexpr int TILE_MT[4] = {1, 2, 3, 4}, TILE_NB[4] = {2, 3, 4, 6};
static double tile_us(int mt, int nb, int M, int NT, int n_cu, int steps, int wg_mult, double w_bytes, Fold fold) {
  const int passes = (M + 64 * mt - 1) / (64 * mt);
  int groups = (NT + 2 * nb - 1) / (2 * nb);
  // all workgroups of a strip group of a split launch of two or four k-slices share an XCD: the XCDs with one group more
  // set the time (2048 x 5504 at 320 rows, 11 groups x 20 workgroups: 42 us, where 32 groups x 8 take 25)
  if (wg_mult > 1 && wg_mult < 8) groups = (groups + 7) / 8 * 8;
  const int wgs = passes * groups * wg_mult;
  const int rounds = (wgs + n_cu - 1) / n_cu;
  const double mul = 0.0113 * mt * nb + (fold != FOLD_NONE && tile_takes_row_sums(mt) ? 0.04 : 0.0), load = 0.0087 * (2 * nb + 4 * mt);
  const double raw = rounds * (1.35 + 0.396 * mt * nb + steps * (0.066 + std::sqrt(mul * mul + load * load)));
  const double stats = fold == FOLD_WANTED && !tile_takes_row_sums(mt) ? 3.5 : 0.0;  // k_row_inv_x in front
  return 3.0 + stats + std::max(raw, w_bytes / (passes == 1 || wg_mult > 1 ? 5.3e6 : 3.5e6)) + 0.1 * raw;
}
static double choose_tile(int M, int NT, int n_cu, int steps, int wg_mult, double w_bytes, Fold fold, int &MTW, int &NBW) {
  double best = 0.0;
  for (int mt : TILE_MT)
    for (int nb : TILE_NB) {
      const double us = tile_us(mt, nb, M, NT, n_cu, steps, wg_mult, w_bytes, fold);
      if (best == 0.0 || us < best) { best = us; MTW = mt; NBW = nb; }
    }
  return best;
}

// Wave tile of the launch for these arguments; returns its estimate in us.  split: each workgroup takes one k-slice of
// its tile and a second kernel adds the slices (4.3 us, and 8 us per million outputs for the slices' way through memory).
static double tile_for(const GemmArgs &a, bool split, int &MTW, int &NBW) {
  const int n_cu = a.n_cu > 0 ? a.n_cu : 256, steps = split ? a.KT / a.KS : a.KT, wg_mult = split ? a.KS : 1;
  const double w_bytes = 1024.0 * a.NT * a.KT, second = split ? 4.3 + 7.9e-6 * a.M * a.N : 0.0;
  const int f_mt = a.tune & TUNE_TILE_MTW_MASK, f_nb = (a.tune >> TUNE_TILE_NBW_SHIFT) & 0xf;
  if (f_mt >= 1 && f_mt <= 4 && f_nb >= 2 && f_nb <= 6 && f_nb != 5) {  // test / tuning aid
    MTW = f_mt; NBW = f_nb;
    return second + tile_us(MTW, NBW, a.M, a.NT, n_cu, steps, wg_mult, w_bytes, fold_of(a));
  }
  MTW = 2; NBW = 2;
  return second + choose_tile(a.M, a.NT, n_cu, steps, wg_mult, w_bytes, fold_of(a), MTW, NBW);
}

// A launch of several rounds of workgroups ends in one that is partly empty, and a round of large wave tiles is long: the
// rows of that round can go to a second launch, whose wave tile suits what is left.  Returns how many of a.M rows the first
// launch takes (all of them unless two are estimated to save 3 %), and the second launch's wave tile.  One launch / two, us:
// 4096 x 11008 at 6592 and 4848 rows 628 / 583 and 426 / 409, 4096 x 4096 263 / 248 and 181 / 174, gate-up 22016 x 4096 at 6592
// and 776 rows 1078 / 1062 and 171 / 158, 15360 x 5120 at 784 rows 161 / 152, 6656 x 17920 at 4848 rows 1064 / 1035.
static int rows_of_first_launch(const GemmArgs &a, int epi, int MTW, int NBW, int &MTW2, int &NBW2) {
  const int n_cu = a.n_cu > 0 ? a.n_cu : 256, pass_rows = 64 * MTW;
  const int groups = (a.NT + 2 * NBW - 1) / (2 * NBW), passes = (a.M + pass_rows - 1) / pass_rows;
  // (not the LM head, whose partials are counted by strip group; nor where the rows' sums of squares are taken in the loop,
  // since the second launch's wave tile may want them from k_row_inv_x)
  if ((a.tune & 0xff) || epi == EPI_LOGITS || passes * groups <= n_cu || (a.fold_x && tile_takes_row_sums(MTW))) return a.M;
  const double w_bytes = 1024.0 * a.NT * a.KT;
  double best = 0.97 * tile_us(MTW, NBW, a.M, a.NT, n_cu, a.KT, 1, w_bytes, fold_of(a));
  const int rounds = (passes * groups + n_cu - 1) / n_cu;
  int first = a.M;
  for (int r = rounds - 1; r >= 1 && r >= rounds - 2; --r) {
    const int rows = r * n_cu / groups * pass_rows;
    if (rows <= 0 || rows >= a.M || (epi == EPI_QKV && rows % a.q_rows != 0)) continue;
    int mt = 2, nb = 2;
    const double rest = choose_tile(a.M - rows, a.NT, n_cu, a.KT, 1, w_bytes, a.fold_x ? FOLD_LEFT : FOLD_NONE, mt, nb);
    const double us = tile_us(MTW, NBW, rows, a.NT, n_cu, a.KT, 1, w_bytes, fold_of(a)) + rest;
    if (us < best) { best = us; first = rows; MTW2 = mt; NBW2 = nb; }
  }
  return first;
}
// the arguments of the same product for the rows from m0 on (a multiple of 16, and of q_rows where the epilogue is EPI_QKV)
static GemmArgs rows_from(GemmArgs a, int m0) {
  const size_t r = (size_t)m0;
  a.M -= m0;
  a.X = (const op_t *)a.X + r * a.KT * 32;
  if (a.h) a.h += r * a.N;
  if (a.x_out) a.x_out = (op_t *)a.x_out + r * a.N;
  if (a.act) a.act = (op_t *)a.act + r * (a.f > 0 ? a.f : a.N);
  if (a.rinv_ws) a.rinv_ws += r;
  if (a.mean_ws) a.mean_ws += r;
  if (a.row_pos) {
    a.row_pos += r;
    a.q = (float *)a.q + r * a.d;
    const size_t seqs = r / a.q_rows, elems = a.grp_seq ? 0 : seqs * a.H * a.L_pad * a.hd;
    if (a.grp_seq) a.grp_seq += seqs;
    a.kc = (char *)a.kc + 2 * elems;  // 16-bit caches
    a.vc = (char *)a.vc + 2 * elems;
  }
  return a;
}

// For the choice between the kernels: without the share of the row sums, which the streaming kernel's estimate has none of, but for
// QKV products over k beyond 3072, where it stands for the scattered stores behind a long k.  Streaming / tiled, us: QKV 12288 x 4096
// at 40 and 64 rows 28 / 30 and 30 / 33, but 9216 x 3072 at 64 27 / 25, 6144 x 2048 at 80 18 / 15; others 10240 x 2560 at 40 and 64
// rows 21 / 20 and 24 / 21, 12288 x 3072 at 64 27 / 24, 10240 x 5120 at 40 and 64 32 / 33 and 36 / 34, 2048 x 512 at 192 10 / 7.
double gemm_tile_us(GemmArgs a, int epi, bool split) {
  int MTW, NBW;
  if (epi != EPI_QKV || a.KT <= 96) a.fold_x = 0;
  return tile_for(a, split, MTW, NBW);
}

// With more than one row tile per wave the kernel reads 1 / rms of its rows from a.rinv_ws: the caller runs launch_row_inv_x first when this says so.
bool gemm_tile_wants_row_inv(const GemmArgs &a, int epi) {
  if (!a.fold_x || (epi != EPI_QKV && epi != EPI_SWIGLU && epi != EPI_RELU && epi != EPI_LOGITS)) return false;
  int MTW, NBW;
  tile_for(a, false, MTW, NBW);
  return !tile_takes_row_sums(MTW);
}
void launch_row_inv_x(const GemmArgs &a, hipStream_t st) {
  if (a.M <= 0) return;
  hipLaunchKernelGGL(k_row_inv_x, dim3((a.M + 15) / 16), dim3(a.KS * 64), 0, st, a.X, a.M, a.KT, a.KS, a.ss_d, a.ss_eps, a.rinv_ws,
                     a.wsum ? a.mean_ws : nullptr);
}

void gemm_tile_prepare() {
  GemmArgs a{};
  const float one = 1.f;
  for (int ln = 0; ln < 2; ++ln) {
    a.wsum = ln ? &one : nullptr;  // never read: selects the kernels with a LayerNorm
    for (int epi : {(int)EPI_RESIDUAL, (int)EPI_QKV, (int)EPI_SWIGLU, (int)EPI_RELU, (int)EPI_PARTIAL, (int)EPI_LOGITS})
      for (int mt : TILE_MT)
        for (int nb : TILE_NB)
          for (int dtype : {(int)SPEC_DTYPE_BF16, (int)SPEC_DTYPE_F16}) launch_shape(dtype, a, mt, nb, epi, -1, nullptr);
  }
}

// EPI_LOGITS: a wave leaves one arg-max partial per row for its NBW strips
int gemm_tile_head_partials(const GemmArgs &a) {
  int MTW, NBW;
  tile_for(a, false, MTW, NBW);
  return 2 * ((a.NT + 2 * NBW - 1) / (2 * NBW));
}

// The value strips of a decoding round's QKV product scatter a few rows over the cache, one channel at a time.  Dealt by eighths they
// end on two or three XCDs, which then finish last: as long as whole strip groups take no more rounds they go to the XCDs
// in turn (12288 x 4096 at 640 rows 89 us by eighths, 84 in turn, 19968 x 6656 at 1280 rows 327 and 309).  A prefill's values are
// written eight positions at a time: 19968 x 6656 at 8192 rows 1754 us by eighths, 1820 in turn.
static bool deal_whole_groups(const GemmArgs &a, int epi) {
  if (epi != EPI_QKV || a.grp_seq) return false;
  const int n_cu = a.n_cu > 0 ? a.n_cu : 256, xcd_cu = std::max(1, n_cu / 8);
  const int whole = (a.groups + 7) / 8 * a.passes, even = (a.groups * a.passes + 7) / 8;
  return (whole + xcd_cu - 1) / xcd_cu == (even + xcd_cu - 1) / xcd_cu;
}

static void launch_rows(int dtype, GemmArgs a, int epi, bool split, int MTW, int NBW, hipStream_t st) {
  a.n_part = 2 * ((a.NT + 2 * NBW - 1) / (2 * NBW));
  a.passes = (a.M + 64 * MTW - 1) / (64 * MTW);
  a.groups = (a.NT + 2 * NBW - 1) / (2 * NBW);
  a.whole_groups = !split && a.passes > 1 && deal_whole_groups(a, epi);
  const int blocks = split ? (a.KS == 8 ? a.groups * a.passes * 8 : ((a.groups + 7) / 8) * 8 * a.passes * a.KS)
                           : a.passes == 1 ? a.groups : a.whole_groups ? (a.groups + 7) / 8 * 8 * a.passes : (a.groups * a.passes + 7) / 8 * 8;
  launch_shape(dtype, a, MTW, NBW, split ? (int)EPI_PARTIAL : epi, blocks, st);
}

void launch_gemm_tile(int dtype, GemmArgs a, int epi, bool split, hipStream_t st) {
  int MTW, NBW, MTW2, NBW2;
  tile_for(a, split, MTW, NBW);
  const int first = split ? a.M : rows_of_first_launch(a, epi, MTW, NBW, MTW2, NBW2);
  if (first < a.M) {
    GemmArgs f = a;
    f.M = first;
    launch_rows(dtype, f, epi, false, MTW, NBW, st);
    launch_rows(dtype, rows_from(a, first), epi, false, MTW2, NBW2, st);
    return;
  }
  launch_rows(dtype, a, epi, split, MTW, NBW, st);
  if (split && a.ssq_ks > 0 && a.x_out) {
    const int rr_threads = std::min(1024, ((a.N >> 2) + 63) / 64 * 64);  // one float4 of outputs per thread where that fits
    hipLaunchKernelGGL(k_partial_reduce_rows, dim3(a.M), dim3(rr_threads), (size_t)a.N * sizeof(op_t), st, a);
  } else if (split) {
    const size_t total = (size_t)a.M * (a.N >> 2);
    hipLaunchKernelGGL(k_partial_reduce, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a);
  }
}

}  // namespace spec

// Kernels that move tokens and per-sequence state: pass assembly + embedding gather,
// norms, arg-max, acceptance/commit, proposal handling, reset/rewind, KV import/export.
#include "spec_internal.h"
#include "device_utils.h"
#include "mfma_tiles.h"

// No implicit fusing of multiplies and adds: which product a compiler folds into an FMA can
// differ between two instantiations of the same source, and results here must be bit-identical
// across launch shapes.  Fused operations are written out with fmaf where they are wanted.
#pragma clang fp contract(off)

namespace spec {

// four consecutive parameters with one load (index a multiple of 4 in an array aligned to four of them)
template <class T>
__device__ __forceinline__ void load4(const T *__restrict__ p, size_t i, float (&out)[4]) {
  struct alignas(sizeof(T) * 4) Quad { T v[4]; };
  const Quad q = *(const Quad *)(p + i);
#pragma unroll
  for (int k = 0; k < 4; ++k) out[k] = Conv<T>::ld(q.v, k);
}

// -------------------------------------------------------------------------
// Row assembly + embedding.  One block per row m = b*q + i.  Decides which token the
// row carries and at which absolute position (pos = -1 marks a dead row: no KV write,
// no attention, logits ignored), then gathers the embedding (plus the learned position
// row for OPT-shape models) into the fp32 residual stream.
// Verification rows follow Alg. 1's call LLM(S, t_1..t_s): pending token, then proposals.
// last: a draft head's arg-max whose second stage this kernel is, a launch less a draft step, inside spec_round only (a step called by
// itself has to leave its token).  Rounds of four target layers in steps one by one / through spec_round, us: 7B width, one sequence, seven
// draft steps 685 / 676, six sequences, five steps 688 / 682, 13B width, 16 sequences, four steps 1079 / 1074; twelve rounds of a
// d_model 256 target with its 128 draft, through spec_round without and with it, 2278 -> 2212.
// PREP (models whose RMS norm is folded into the GEMMs): the kernel also leaves what the first layer's QKV GEMM
// consumes, the fp16 copy of the row in fragment order (the GEMM takes 1 / rms of the row from those values).
template <class T, bool PREP>
__global__ __launch_bounds__(256) void k_assemble_embed(int kind, int q, int j, int s_max, int L_max, int vocab, int d,
                                 int learned_pos, const int32_t *__restrict__ grp_seq, const int32_t *__restrict__ grp_base, const int32_t *__restrict__ seq, const int32_t *__restrict__ n,
                                 const int32_t *__restrict__ kv_draft, int32_t *__restrict__ t, HeadPartials last, const int32_t *__restrict__ table, int fill,
                                 const int32_t *__restrict__ seq_s, const int32_t *__restrict__ P_b,
                                 const T *__restrict__ tok_emb, const T *__restrict__ pos_emb,
                                 int32_t *__restrict__ row_tok, int32_t *__restrict__ row_pos, float *__restrict__ h,
                                 op_t *__restrict__ x, unsigned int *__restrict__ sat) {
  // prefill: the table says which sequence a group of q rows belongs to and where it starts
  const int m = blockIdx.x, grp = m / q;
  const int b = grp_seq ? grp_seq[grp] : grp, i = m % q;
  int tok = 0, pos = -1;
  const int nb = n[b];
  // External proposals from a table, t_j = table[b][n_b + j - 1] (absolute position): the round's first pass leaves them for
  // the kernels behind it, which saves a launch a round (a round of 299 us takes 296).  Its own rows read the table.
  auto table_tok = [&](int jj) { return nb + jj < L_max ? table[(size_t)b * L_max + nb + jj] : 0; };
  if (table && i == 0)
    for (int jj = threadIdx.x; jj < fill; jj += blockDim.x) t[(size_t)b * s_max + jj] = table_tok(jj);
  // live or not, every sequence's token is written: t is what a draft step by itself leaves
  const bool take = last.val && i == q - 1;  // q is 1 in a draft step
  int newest = 0;
  if (take) {
    newest = block_argmax_partials(last.val, last.idx, last.row_step > 0 ? (size_t)b * last.row_step + last.row_step - 1 : (size_t)b, last.n_part, last.vocab);
    if (threadIdx.x == 0) last.out[(size_t)b * last.stride] = newest;
  }
  // a sequence with its own cap s_b on the speculation length: its rows for proposals beyond s_b are dead
  const int sb = seq_s ? max(0, seq_s[b]) : s_max;
  if (kind == PASS_VERIFY) {
    if (i <= sb) {
      pos = nb - 1 + i;
      tok = (i == 0) ? seq[(size_t)b * L_max + nb - 1] : take && last.proposes ? newest : table ? table_tok(i - 1) : t[(size_t)b * s_max + i - 1];
    }
  } else if (kind == PASS_DRAFT_FIRST) {
    int p = nb - j - q + i;  // j: positions the pass ends before n_b (catch-up passes of a draft cache far behind)
    if (p >= 0 && p >= kv_draft[b]) { pos = p; tok = seq[(size_t)b * L_max + p]; }
  } else if (kind == PASS_DRAFT_NEXT) {  // draft step j >= 2 yields t_j: wanted only up to s_b
    if (j <= sb) {
      pos = nb + j - 2;
      tok = take && last.proposes ? newest : t[(size_t)b * s_max + j - 2];
    }
  } else {  // PASS_PREFILL
    const int p = grp_base[grp] + i;
    if (p < P_b[b] - 1) { pos = p; tok = seq[(size_t)b * L_max + p]; }  // the sequence's own prompt length
  }
  if (pos >= L_max) pos = -1;  // cannot happen when the host checks hold; never write out of range
  tok = min(max(tok, 0), vocab - 1);
  if (threadIdx.x == 0) { row_tok[m] = tok; row_pos[m] = pos; }
  float *hr = h + (size_t)m * d;
  auto value = [&](int c) {
    float e = 0.f;
    if (pos >= 0) {
      e = Conv<T>::ld(tok_emb, (size_t)tok * d + c);
      if (learned_pos) e += Conv<T>::ld(pos_emb, (size_t)pos * d + c);
    }
    return e;
  };
  if (!PREP) {
    for (int c = threadIdx.x; c < d; c += blockDim.x) hr[c] = value(c);
    return;
  }
  // Four consecutive elements per thread (d is a multiple of 32), in one load from either table; 6592 rows of 4096
  // 85 -> 74 us; what is left is the fragment order's stores of 8 bytes.
  const int nv = d >> 2;
  for (int c = threadIdx.x; c < nv; c += 256) {
    float e[4] = {0.f, 0.f, 0.f, 0.f};
    if (pos >= 0) {
      load4(tok_emb, (size_t)tok * d + 4 * c, e);
      if (learned_pos) {
        float p[4];
        load4(pos_emb, (size_t)pos * d + 4 * c, p);
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] += p[k];
      }
    }
    *(float4 *)(hr + 4 * c) = make_float4(e[0], e[1], e[2], e[3]);
    op_t o4[4] = {to_op_counted(e[0], sat), to_op_counted(e[1], sat), to_op_counted(e[2], sat), to_op_counted(e[3], sat)};
    *(uint2 *)(x + xpack_index(m, 4 * c, d >> 5)) = *(const uint2 *)o4;
  }
}

void launch_assemble_embed(const spec_ctx *c, const Model &m, const PassArgs &pa, hipStream_t st) {
  const int M = pa.B * pa.q;
  const bool prefill = pa.kind == PASS_PREFILL;
  const bool prep = m.fast;  // the norms are folded into the GEMMs: they read fp16(h)
  SPEC_DISPATCH_DTYPE(c->run.dtype, T,
    hipLaunchKernelGGL((prep ? k_assemble_embed<T, true> : k_assemble_embed<T, false>), dim3(M), dim3(256), 0, st, (int)pa.kind, pa.q, pa.j,
                       c->run.s_max, c->run.L_max, m.desc.vocab, m.desc.d_model,
                       (int)(m.desc.pos_kind == SPEC_POS_LEARNED), prefill ? c->ws.grp_seq + pa.g0 : nullptr, prefill ? c->ws.grp_base + pa.g0 : nullptr,
                       c->st.seq + (size_t)pa.b0 * c->run.L_max,
                       c->st.n + pa.b0, c->drf.kv_len ? c->drf.kv_len + pa.b0 : nullptr,
                       c->st.t + (size_t)pa.b0 * c->run.s_max, pa.last, pa.fill > 0 ? c->prop_table + (size_t)pa.b0 * c->run.L_max : nullptr, pa.fill, c->seq_s ? c->seq_s + pa.b0 : nullptr, c->st.P_b + pa.b0,
                       (const T *)m.tok_emb, (const T *)m.pos_emb, c->ws.row_tok, c->ws.row_pos, c->ws.h,
                       (op_t *)c->ws.x, c->st.sat));
}

// -------------------------------------------------------------------------
// The row groups of a prefill: sequence by sequence, ceil((P_b - 1) / q) groups of q consecutive positions each, so that
// prompts of different lengths leave no dead rows but those of their own last group.  One workgroup; a thread owns a
// run of sequences, and a prefix sum over the runs says where its groups start.
__global__ __launch_bounds__(256) void k_prefill_groups(int B, int q, const int32_t *__restrict__ P_b, int32_t *__restrict__ grp_seq,
                                                        int32_t *__restrict__ grp_base) {
  __shared__ int sh[4];
  const int per = (B + 255) / 256, b0 = min(B, (int)threadIdx.x * per), b1 = min(B, b0 + per), lane = threadIdx.x & 63;
  int mine = 0;
  for (int b = b0; b < b1; ++b) mine += (P_b[b] - 1 + q - 1) / q;
  int inc = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(inc, o, 64);
    if (lane >= o) inc += up;
  }
  if (lane == 63) sh[threadIdx.x >> 6] = inc;
  __syncthreads();
  int at = inc - mine;
  for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) at += sh[w];
  for (int b = b0; b < b1; ++b)
    for (int base = 0; base < P_b[b] - 1; base += q, ++at) { grp_seq[at] = b; grp_base[at] = base; }
}
void launch_prefill_groups(const spec_ctx *c, int b0, int B, int q, hipStream_t st) {
  hipLaunchKernelGGL(k_prefill_groups, dim3(1), dim3(256), 0, st, B, q, c->st.P_b + b0, c->ws.grp_seq, c->ws.grp_base);
}

// -------------------------------------------------------------------------
// RMSNorm / LayerNorm of one row of the fp32 residual stream by a 256-thread workgroup (the models on the generic
// kernels: on the matrix-core path the norms live inside the GEMMs).  Statistics in fp32 with a fixed reduction tree
// (per-thread strided partial, wave butterfly, then the four wave results in order), so a row's result never depends
// on which other rows are in the pass.
__device__ __forceinline__ float block_sum_256(float v, float *sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Row held in registers: thread t owns the float4 groups t, t+256, ... (all loads issued
// before any arithmetic, so the kernel costs one memory round trip, not d/256 of them).
constexpr int NORM_MAX_V4 = 8;  // d <= 8192
// the gains and biases of the elements a thread owns (float4 groups t, t + 256, ...); zero where it owns none
template <class T>
__device__ __forceinline__ void norm_params(int kind, int d, const T *__restrict__ gain, const T *__restrict__ bias,
                                            float (&gn)[NORM_MAX_V4][4], float (&bs)[NORM_MAX_V4][4]) {
  const int nv = d >> 2;
#pragma unroll
  for (int i = 0; i < NORM_MAX_V4; ++i) {
    const int c = threadIdx.x + i * 256;
#pragma unroll
    for (int k = 0; k < 4; ++k) { gn[i][k] = 0.f; bs[i][k] = 0.f; }
    if (c < nv) {
      load4(gain, 4 * c, gn[i]);
      if (kind != SPEC_NORM_RMS) load4(bias, 4 * c, bs[i]);
    }
  }
}
// gn, bs: from norm_params, fetched by the caller as early as it can (their latency then passes behind other work)
template <class T>
__device__ __forceinline__ void norm_row(int kind, int d, float eps, const float4 *hr, const float (&gn)[NORM_MAX_V4][4],
                                         const float (&bs)[NORM_MAX_V4][4], int r, void *__restrict__ x, int pack_kt,
                                         unsigned int *__restrict__ sat, float *sh) {
  const int nv = d >> 2;
  float4 v[NORM_MAX_V4];
#pragma unroll
  for (int i = 0; i < NORM_MAX_V4; ++i) {
    const int c = threadIdx.x + i * 256;
    v[i] = c < nv ? hr[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float mean = 0.f, inv;
  if (kind == SPEC_NORM_RMS) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NORM_MAX_V4; ++i) {
      ss = fmaf(v[i].x, v[i].x, ss); ss = fmaf(v[i].y, v[i].y, ss);
      ss = fmaf(v[i].z, v[i].z, ss); ss = fmaf(v[i].w, v[i].w, ss);
    }
    ss = block_sum_256(ss, sh);
    inv = 1.0f / sqrtf(ss / (float)d + eps);
  } else {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NORM_MAX_V4; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    mean = block_sum_256(s, sh) / (float)d;
    float vs = 0.f;
#pragma unroll
    for (int i = 0; i < NORM_MAX_V4; ++i) {
      const int c = threadIdx.x + i * 256;
      if (c < nv) {
        float a0 = v[i].x - mean, a1 = v[i].y - mean, a2 = v[i].z - mean, a3 = v[i].w - mean;
        vs = fmaf(a0, a0, vs); vs = fmaf(a1, a1, vs); vs = fmaf(a2, a2, vs); vs = fmaf(a3, a3, vs);
      }
    }
    inv = 1.0f / sqrtf(block_sum_256(vs, sh) / (float)d + eps);
  }
#pragma unroll
  for (int i = 0; i < NORM_MAX_V4; ++i) {
    const int c = threadIdx.x + i * 256;
    if (c < nv) {
      const float e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
      float o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        o[k] = (e[k] - mean) * inv * gn[i][k];
        if (kind != SPEC_NORM_RMS) o[k] += bs[i][k];
      }
      if (pack_kt > 0) {
        // the consumer is a matrix-core GEMM: fp16 operands, rows stored in fragment order, where four consecutive
        // elements of a row are eight contiguous bytes
        op_t o4[4] = {to_op_counted(o[0], sat), to_op_counted(o[1], sat), to_op_counted(o[2], sat), to_op_counted(o[3], sat)};
        *(uint2 *)((op_t *)x + xpack_index(r, 4 * c, pack_kt)) = *(const uint2 *)o4;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) Conv<T>::st((T *)x, (size_t)r * d + 4 * c + k, o[k]);
      }
    }
  }
}

// -------------------------------------------------------------------------
// RMSNorm / LayerNorm over rows of the fp32 residual stream, output in the model dtype.
// One 256-thread block per output row; statistics in fp32 with a fixed reduction tree
// (per-thread strided partial, wave butterfly, then the four wave results in order), so a
// row's result never depends on which other rows are in the pass.
template <class T>
__global__ __launch_bounds__(256) void k_norm(int kind, int d, float eps, const float *__restrict__ h,
                                              const T *__restrict__ gain, const T *__restrict__ bias,
                                              int last_of_q, void *__restrict__ x,
                                              int pack_kt, unsigned int *__restrict__ sat) {
  __shared__ float sh[4];
  const int r = blockIdx.x;
  // last_of_q > 0: output row r is the last of input rows r * q .. r * q + q - 1 (the rows that need a token)
  const float4 *hr = (const float4 *)(h + (size_t)(last_of_q > 0 ? r * last_of_q + last_of_q - 1 : r) * d);
  // gains and biases are requested first, beside the row, so that their latency passes behind the reductions
  float gn[NORM_MAX_V4][4], bs[NORM_MAX_V4][4];
  norm_params<T>(kind, d, gain, bias, gn, bs);
  norm_row<T>(kind, d, eps, hr, gn, bs, r, x, pack_kt, sat, sh);
}

void launch_norm(const spec_ctx *c, const Model &m, const float *h, const void *gain, const void *bias, void *x,
                 int M, int last_of_q, hipStream_t st) {
  if (M <= 0) return;
  const int pack_kt = m.fast ? m.desc.d_model / 32 : 0;
  SPEC_DISPATCH_DTYPE(c->run.dtype, T,
    hipLaunchKernelGGL(k_norm<T>, dim3(M), dim3(256), 0, st, m.desc.norm_kind, m.desc.d_model, m.desc.norm_eps, h,
                       (const T *)gain, (const T *)bias, last_of_q, x, pack_kt, c->st.sat));
}

// -------------------------------------------------------------------------
// Greedy token per row (Alg. 1 prints "argmin"; Sec. 2 and the caption say the most
// probable token, so arg-max).  Lowest index wins ties.  Row m of the logits goes to
// out[(m / q) * out_stride + m % q].
__global__ void k_argmax_rows(const float *__restrict__ logits, int V, int q, int out_stride, int32_t *__restrict__ out) {
  __shared__ float shv[4];
  __shared__ int shi[4];
  const int m = blockIdx.x;
  const float *row = logits + (size_t)m * V;
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  for (int c = threadIdx.x; c < V; c += 256) argmax_combine(bv, bi, row[c], c);
  wave_argmax(bv, bi);
  if ((threadIdx.x & 63) == 0) { shv[threadIdx.x >> 6] = bv; shi[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) argmax_combine(bv, bi, shv[w], shi[w]);
    if (bi < 0 || bi >= V) bi = 0;
    out[(size_t)(m / q) * out_stride + m % q] = bi;
  }
}

void launch_argmax_rows(const float *logits, int M, int V, int q, int out_stride, int32_t *out, hipStream_t st) {
  if (M <= 0) return;
  hipLaunchKernelGGL(k_argmax_rows, dim3(M), dim3(256), 0, st, logits, V, q, out_stride, out);
}

// -------------------------------------------------------------------------
// -------------------------------------------------------------------------
// External proposals given for the round (those of a table are fetched by the round's first pass, k_assemble_embed).
__global__ void k_copy_proposals(int B, int s, int s_max, const int32_t *__restrict__ src, int32_t *__restrict__ t) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B * s) return;
  t[(size_t)(i / s) * s_max + i % s] = src[i];
}
void launch_copy_proposals(spec_ctx *c, const int32_t *d_tok, int s, hipStream_t st) {
  if (s <= 0) return;
  hipLaunchKernelGGL(k_copy_proposals, dim3((c->B * s + 255) / 256), dim3(256), 0, st, c->B, s, c->run.s_max, d_tok,
                     c->st.t);
}

// -------------------------------------------------------------------------
// Acceptance + commit, one thread per sequence (Sec. 2, Alg. 1): a proposal survives
// only while all earlier ones matched the target's greedy token; the target's token after
// the last survivor is appended.  Rollback is by length only: the K/V rows written for
// rejected positions stay in the cache and are overwritten by the next round.
// A sequence stops for good after gen_cap[b] emitted tokens: gen_max, or the count at which it emitted the end
// token eos (the tokens a round accepted behind an end token are dropped with it).
__global__ void k_accept(int B, int s, int s_max, int L_max, const int32_t *__restrict__ P_b, int32_t *__restrict__ gen_cap,
                         int eos, int draft_steps, const int32_t *__restrict__ seq_s,
                         const int32_t *__restrict__ t, const int32_t *__restrict__ a, int32_t *__restrict__ seq,
                         int32_t *__restrict__ n, int32_t *__restrict__ kv_draft, int32_t *__restrict__ l_last,
                         unsigned long long *__restrict__ hist, unsigned long long *__restrict__ counters) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b == 0) atomicAdd(&counters[1], 1ull);
  if (b >= B) return;
  const int n_old = n[b];
  const int gen = n_old - P_b[b];
  const int32_t *tb = t + (size_t)b * s_max;
  const int32_t *ab = a + (size_t)b * (s_max + 1);
  // with a cap per sequence only the first min(s, s_b) proposals were verified, and the draft ran
  // max(1, min(draft_steps, s_b)) live steps for this sequence
  const int sb = seq_s ? min(s, max(0, seq_s[b])) : s;
  if (seq_s && draft_steps > 0) draft_steps = max(1, min(draft_steps, sb));
  int l = 0;
  while (l < sb && tb[l] == ab[l]) ++l;
  const int cap = gen_cap[b];
  int take = min(l + 1, cap - gen);
  if (take < 0) take = 0;
  for (int i = 0; i < take; ++i) {
    const int32_t tok = (i < l) ? tb[i] : ab[l];
    seq[(size_t)b * L_max + n_old + i] = tok;
    if (tok == eos) { take = i + 1; gen_cap[b] = gen + take; }
  }
  const int n_new = n_old + take;
  n[b] = n_new;
  l_last[b] = l;
  if (draft_steps > 0 && kv_draft) {
    int kd = n_old + min(l, draft_steps - 1);
    kv_draft[b] = max(0, min(kd, n_new - 1));
  }
  if (gen < cap) {
    atomicAdd(&hist[l], 1ull);
    atomicAdd(&counters[0], (unsigned long long)take);
  }
}
void launch_accept(spec_ctx *c, int s, hipStream_t st) {
  hipLaunchKernelGGL(k_accept, dim3((c->B + 63) / 64), dim3(64), 0, st, c->B, s, c->run.s_max, c->run.L_max, c->st.P_b,
                     c->st.gen_cap, c->eos, c->draft_j, c->seq_s, c->st.t, c->st.a, c->st.seq, c->st.n, c->drf.kv_len, c->st.l_last,
                     c->st.hist, c->st.counters);
}

// -------------------------------------------------------------------------
// With a prompt: a new batch, every sequence P tokens long — or, ragged, prompt rows of stride P of which sequence
// b uses the first P_b[b] (already on the device).  Without: back to "prompts just given", every sequence to its
// own prompt length.
__global__ void k_state_reset(int B, int P, int ragged, int L_max, int s_max, int gen_max, const int32_t *__restrict__ prompt,
                              int32_t *__restrict__ seq, int32_t *__restrict__ n, int32_t *__restrict__ P_b,
                              int32_t *__restrict__ gen_cap,
                              int32_t *__restrict__ kv_draft,
                              int32_t *__restrict__ l_last, unsigned long long *__restrict__ hist,
                              unsigned long long *__restrict__ counters) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (prompt && i < B * P && (!ragged || i % P < P_b[i / P])) seq[(size_t)(i / P) * L_max + i % P] = prompt[i];
  if (i < B) {
    const int Pi = (prompt && !ragged) ? P : P_b[i];
    P_b[i] = Pi;
    gen_cap[i] = gen_max;
    n[i] = Pi; l_last[i] = 0;
    if (kv_draft) kv_draft[i] = Pi - 1;
  }
  if (i <= s_max) hist[i] = 0ull;
  if (i < 2) counters[i] = 0ull;
}
// One batch slot back to "prompt just given": its tokens, length, draft-cache length.  Counters and the
// accepted-length histogram belong to the whole batch and are left alone.
__global__ void k_state_admit(int P, int gen_max, const int32_t *__restrict__ prompt, int32_t *__restrict__ seq_b,
                              int32_t *__restrict__ n_b, int32_t *__restrict__ P_b_b, int32_t *__restrict__ gen_cap_b,
                              int32_t *__restrict__ kv_draft_b,
                              int32_t *__restrict__ l_last_b) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P) seq_b[i] = prompt[i];
  if (i == 0) { *n_b = P; *P_b_b = P; *gen_cap_b = gen_max; *l_last_b = 0; if (kv_draft_b) *kv_draft_b = P - 1; }
}
void launch_state_admit(spec_ctx *c, int b, const int32_t *d_prompt, int P, hipStream_t st) {
  hipLaunchKernelGGL(k_state_admit, dim3((P + 255) / 256), dim3(256), 0, st, P, c->run.gen_max, d_prompt,
                     c->st.seq + (size_t)b * c->run.L_max, c->st.n + b, c->st.P_b + b, c->st.gen_cap + b,
                     c->drf.kv_len ? c->drf.kv_len + b : nullptr, c->st.l_last + b);
}
void launch_state_reset(spec_ctx *c, const int32_t *d_prompt, int P_stride, bool ragged, hipStream_t st) {
  int work = c->B * P_stride;
  if (work < c->run.s_max + 1) work = c->run.s_max + 1;
  if (work < 2) work = 2;
  hipLaunchKernelGGL(k_state_reset, dim3((work + 255) / 256), dim3(256), 0, st, c->B, P_stride, (int)ragged, c->run.L_max,
                     c->run.s_max, c->run.gen_max, d_prompt, c->st.seq, c->st.n, c->st.P_b, c->st.gen_cap, c->drf.kv_len, c->st.l_last, c->st.hist,
                     c->st.counters);
}

// -------------------------------------------------------------------------
// KV import / export between the caller's [B][len][d_model] layout and the cache layout
// (keys pair-interleaved inside each head, values blocked by 8 positions).
// BLOCKED: keys in units of 16 bytes (else plain rows, kv_k_index's u = hd).
template <class T, bool BLOCKED>
__global__ void k_kv_convert(int import_, int B, int len, int H, int hd, int L_pad, T *__restrict__ kc,
                             T *__restrict__ vc, T *__restrict__ k_user, T *__restrict__ v_user) {
  const int d = H * hd;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)B * len * d) return;
  int c = (int)(i % d);
  size_t r = i / d;
  int pos = (int)(r % len), b = (int)(r / len);
  int hh = c / hd, e = c % hd;
  size_t ki = kv_k_index(L_pad, H, hd, BLOCKED ? (int)(16 / sizeof(T)) : hd, b, hh, pos, hd_interleave(e, hd));
  size_t vi = kv_v_index(L_pad, H, hd, b, hh, pos, e);
  if (import_) { kc[ki] = k_user[i]; vc[vi] = v_user[i]; }
  else { k_user[i] = kc[ki]; v_user[i] = vc[vi]; }
}
// The export of 16-bit rows to buffers aligned to 16 bytes: a thread takes eight channels at eight consecutive positions,
// where the cache has the values of a channel side by side, and the keys of eight pairs (two runs of four channels) of a
// row.  Element by element the scattered loads and stores were most of the time: 64 x 128 rows of 4096 116 -> 67 us (33 MB
// read at the rate they are written).  Workgroups of one wave, keys (blockIdx.y 0) and values (1) apart, so that a
// small export spreads over the CUs.
// Of a row of keys, neighbouring threads' units lie 64 bytes apart (kv_k_index).  So the wave loads them as they lie, a lane the positions lane % 4 and
// 4 + lane % 4 of every fourth unit (1 KB side by side at heads of 128), and the units change hands in LDS: 64 x 128 rows of 4096 75 -> 67.5 us, 5 x
// 2011 of 6656 146 -> 137, 777 of 5120 from memory 15.5 -> 13.7.  (Four positions at a time in half the LDS, that is more waves to a CU: 143 us.)
__global__ __launch_bounds__(64) void k_kv_export16(int B, int len, int H, int hd, int k_unit, int L_pad, const uint16_t *__restrict__ kc,
                                                     const uint16_t *__restrict__ vc, uint16_t *__restrict__ k_user,
                                                     uint16_t *__restrict__ v_user) {
  struct alignas(16) Eight { uint16_t v[8]; };
  __shared__ u32x4_v rows_s[8][66];  // [position][unit of the wave]; two more: the rows of a block are written without a bank conflict
  const int d = H * hd, nb = (len + KV_VBLOCK - 1) / KV_VBLOCK, n8 = d >> 3, lane = threadIdx.x;
  const size_t i = (size_t)blockIdx.x * 64 + lane, last = (size_t)B * nb * n8 - 1, at = min(i, last);
  const int c0 = (int)(at % n8) * 8;
  const size_t r = at / n8;
  const int p0 = (int)(r % nb) * KV_VBLOCK, b = (int)(r / nb), hh = c0 / hd, e0 = c0 - hh * hd, half = hd >> 1;
  const int rows = i <= last ? min(KV_VBLOCK, len - p0) : 0;
  const size_t row0 = ((size_t)b * len + p0) * d + (size_t)hh * hd;
  if (blockIdx.y) {
    uint16_t val[8][8];  // [channel][position]
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const Eight t = *(const Eight *)(vc + kv_v_index(L_pad, H, hd, b, hh, p0, e0 + e));
#pragma unroll
      for (int p = 0; p < 8; ++p) val[e][p] = t.v[p];
    }
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      Eight o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o.v[e] = val[e][p];
      if (p < rows) *(Eight *)(v_user + row0 + (size_t)p * d + e0) = o;
    }
    return;
  }
  // stored elements e0 .. e0 + 7 of a row: the pairs of channels e0 / 2 .. e0 / 2 + 3 and their partners
  const unsigned long long mine = kv_k_index(L_pad, H, hd, k_unit, b, hh, p0, e0);
  u32x4_v key[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint16_t *p = kc + __shfl(mine, 16 * k + (lane >> 2), 64) + (lane & 3) * k_unit;
    key[2 * k] = *(const u32x4_v *)p;
    key[2 * k + 1] = *(const u32x4_v *)(p + KV_KBLOCK * hd);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int j = 0; j < 2; ++j) rows_s[KV_KBLOCK * j + (lane & 3)][16 * k + (lane >> 2)] = key[2 * k + j];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    if (p >= rows) continue;
    const u32x4_v t = rows_s[p][lane];  // a word: a channel and its partner
    const size_t row = row0 + (size_t)p * d + (e0 >> 1);
    *(uint2 *)(k_user + row) = make_uint2((t[0] & 0xffff) | t[1] << 16, (t[2] & 0xffff) | t[3] << 16);
    *(uint2 *)(k_user + row + half) = make_uint2(t[0] >> 16 | (t[1] & 0xffff0000u), t[2] >> 16 | (t[3] & 0xffff0000u));
  }
}
void launch_kv_convert(spec_ctx *c, const Model &m, int layer, int B, int len, void *k, void *v, bool import_,
                       hipStream_t st) {
  size_t total = (size_t)B * len * m.desc.d_model;
  if (!total) return;
  size_t esz = dtype_bytes(c->run.dtype);
  char *kc = (char *)m.kcache + (size_t)layer * m.kv_area_elems * esz;
  char *vc = (char *)m.vcache + (size_t)layer * m.kv_area_elems * esz;
  // From 3 * 2^18 elements on: a thread's eight rows in turn take a microsecond or two longer than a launch of single elements, until
  // those are several to a lane of the chip; around the line there is little between them.  Elements / blocks, us: 16 rows of 4096 2.9 / 4.8, 64
  // rows of 6656 4.6 / 4.6, 128 rows of 5120 5.0 / 4.7, 64 x 16 rows of 768 5.4 / 4.9, 256 rows of 4096 6.5 / 4.9, 777 rows of 5120 17.3 / 9.6.
  if (!import_ && esz == 2 && total >= ((size_t)3 << 18) && m.hd % 16 == 0 && (((uintptr_t)k | (uintptr_t)v) & 15) == 0) {
    const size_t threads = (size_t)B * ((len + KV_VBLOCK - 1) / KV_VBLOCK) * (m.desc.d_model / 8);
    hipLaunchKernelGGL(k_kv_export16, dim3((unsigned)((threads + 63) / 64), 2), dim3(64), 0, st, B, len, m.desc.n_heads, m.hd, m.k_unit, m.L_pad,
                       (const uint16_t *)kc, (const uint16_t *)vc, (uint16_t *)k, (uint16_t *)v);
    return;
  }
  SPEC_DISPATCH_DTYPE(c->run.dtype, T,
    hipLaunchKernelGGL((m.k_unit == m.hd ? k_kv_convert<T, false> : k_kv_convert<T, true>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (int)import_, B, len, m.desc.n_heads, m.hd, m.L_pad, (T *)kc, (T *)vc, (T *)k, (T *)v));
}

}  // namespace spec

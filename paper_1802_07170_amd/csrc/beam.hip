// Beam search bookkeeping on the device (hyperparameter table: beam size 10, length penalty 0.6;
// the Settings section names the length normalisation of Wu et al. 2016).  The decoder runs on
// R = B * K rows, row r = b * K + s holding live hypothesis s of sentence b.  Per step:
//   beam_row_topk_kernel one workgroup per live row: log-sum-exp of its logits and its K best tokens;
//   beam_merge_kernel   one workgroup per sentence: the K best one-token extensions over all live
//                       hypotheses (equal scores: the lower (slot, token) pair first), finished
//                       hypotheses split off, history written;
//   beam_reorder_kernel the surviving hypotheses' decoder states and H_o move to their new rows, and
//                       the embeddings of their tokens become the next step's input.
// After the last step beam_finish_kernel walks the back-pointers of each sentence's best finished
// hypothesis.  Nothing returns to the host inside the loop.
#include "common.h"
#include "kernels.h"

namespace cmt {

// dst[i, r, 0:cols] = src[i, r / K, 0:cols] for r < R, zero rows for r in [R, Rp); i < n_outer.
// Row pitches in elements; cols * sizeof(T) is a multiple of 16.
template <typename T>
__global__ __launch_bounds__(128) void beam_expand_kernel(const T* __restrict__ src, int ld_src, int rows_src, T* __restrict__ dst,
                                                          int ld_dst, int R, int Rp, int K, int cols) {
  const int r = blockIdx.x, i = blockIdx.y;
  constexpr int VE = 16 / sizeof(T);
  const T* s = r < R ? src + ((size_t)i * rows_src + r / K) * ld_src : nullptr;
  T* d = dst + ((size_t)i * Rp + r) * ld_dst;
  for (int c = threadIdx.x * VE; c < cols; c += 128 * VE)
    *reinterpret_cast<uint4*>(d + c) = s ? *reinterpret_cast<const uint4*>(s + c) : make_uint4(0, 0, 0, 0);
}
void launch_beam_expand(int elem_bytes, const void* src, int ld_src, int rows_src, void* dst, int ld_dst, int n_outer, int R, int Rp,
                        int K, int cols, hipStream_t st) {
  dim3 grid(Rp, n_outer);
  if (elem_bytes == 2)
    hipLaunchKernelGGL(beam_expand_kernel<bf16_t>, grid, dim3(128), 0, st, (const bf16_t*)src, ld_src, rows_src, (bf16_t*)dst, ld_dst,
                       R, Rp, K, cols);
  else
    hipLaunchKernelGGL(beam_expand_kernel<float>, grid, dim3(128), 0, st, (const float*)src, ld_src, rows_src, (float*)dst, ld_dst, R,
                       Rp, K, cols);
}

// start of a search: one live hypothesis per sentence (slot 0, score 0, previous token bos)
__global__ __launch_bounds__(256) void beam_init_kernel(BeamState bs, int B, int Rp, int K, int bos, const int32_t* __restrict__ len_src,
                                                        int32_t* __restrict__ len_exp) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < Rp) {
    const int b = r / K, s = r - b * K;
    const bool real = b < B;
    bs.cum[r] = real && s == 0 ? 0.f : -INFINITY;
    bs.tok[r] = bos;
    bs.mask[r] = real && s == 0 ? 1.f : 0.f;
    len_exp[r] = real ? len_src[b] : 0;
  }
  if (r < B) { bs.nlive[r] = 1; bs.fin_score[r] = -INFINITY; bs.fin_step[r] = -1; bs.fin_par[r] = 0; bs.fin_tok[r] = 0; }
}
void launch_beam_init(const BeamState& bs, int B, int Rp, int K, int bos, const int32_t* len_src, int32_t* len_exp, hipStream_t st) {
  hipLaunchKernelGGL(beam_init_kernel, dim3((Rp + 255) / 256), dim3(256), 0, st, bs, B, Rp, K, bos, len_src, len_exp);
}

constexpr int BEAM_MAX = 16;
constexpr int BEAM_CAND_CAP = 1024;     // candidates a row's workgroup keeps in LDS

// (value, index) ordering: larger value first, then lower index
__device__ __forceinline__ bool beam_better(float v, int f, float bv, int bf) { return v > bv || (v == bv && f < bf); }

// Largest value of a wavefront, in every lane, by DPP moves: about a tenth of the time of six shuffles through LDS.
__device__ __forceinline__ float beam_wave_max(float v) {
#define STEP(ctrl, rows) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, rows, 0xf, false)))
  STEP(0x111, 0xf); STEP(0x112, 0xf); STEP(0x114, 0xf); STEP(0x118, 0xf);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16
  STEP(0x142, 0xa);                                                        // row_bcast15 into rows 1, 3
  STEP(0x143, 0xc);                                                        // row_bcast31 into rows 2, 3
#undef STEP
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// Workgroup-wide best (value, index) pair of NW wavefronts; every thread gets the result.
template <int NW>
__device__ __forceinline__ void beam_block_best(float& v, int& f, float* s_v, int* s_f) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(v, o, 64);
    const int of = __shfl_xor(f, o, 64);
    if (beam_better(ov, of, v, f)) { v = ov; f = of; }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();                                       // the previous round's readers are done
  if (lane == 0) { s_v[w] = v; s_f[w] = f; }
  __syncthreads();
  v = s_v[0]; f = s_f[0];
#pragma unroll
  for (int q = 1; q < NW; ++q)
    if (beam_better(s_v[q], s_f[q], v, f)) { v = s_v[q]; f = s_f[q]; }
}

// One workgroup per hypothesis row: log-sum-exp of the row's logits and its K best tokens (larger
// logit first, then lower token), written best first; entries beyond the row's candidates are
// (-inf, INT_MAX).  The K best of a row contain every extension of it that can be among the K best
// of its sentence (log-softmax is monotonic within a row).
//   pass 1: every thread's best value; the K-th best of one wavefront's 64 of them is a lower bound on the row's K-th
//           best logit, tau the largest of these bounds;
//   pass 2: sum of exp(z - max), and the elements >= tau are appended to a list in LDS;
//   then every list element counts how many are better: that is its place.  A list that overflows (many equal
//   logits) falls back to K rounds of a workgroup-wide arg-max over the row.
// The row stays in registers (NV 16-byte pieces per thread, all in flight at once) and memory is read once; NV = 0:
// each pass reads the row again, four pieces in flight.  What bounds it: the latency of the read and of the selection's
// chain, hence DPP instead of shuffles and counting instead of rounds (with reorder and merge, one sentence x 10 beams,
// 25 steps: 2.74 -> 2.32 ms per search).
// FAST (16-bit path): the hardware exponential in the log-sum-exp.
template <bool FAST, int NT, int NV>
__global__ __launch_bounds__(NT) void beam_row_topk_kernel(const float* __restrict__ z, int V, BeamState bs, int K) {
  constexpr int NW = NT / 64, G = NV ? NV : 4;
  __shared__ float s_v[NW];
  __shared__ int s_f[NW];
  __shared__ float s_sum[NW];
  __shared__ float s_cv[BEAM_CAND_CAP];
  __shared__ int s_ci[BEAM_CAND_CAP];
  __shared__ int s_n;
  const int r = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int b = r / K, slot = r - b * K;
  if (slot >= bs.nlive[b]) return;                       // dead row (uniform over the workgroup)
  const float* zr = z + (size_t)r * V;
  const int nv4 = V >> 2;                                // V is a multiple of 8
  float4 q[G];
  auto load = [&](int c0) {
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int c = c0 + NT * k;
      q[k] = c < nv4 ? *reinterpret_cast<const float4*>(zr + 4 * c) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
  };
  auto visit = [&](auto f) {                             // f(value, token) of this thread's elements
    int first = t;
    asm volatile("" : "+v"(first));                      // (opaque: token numbers are made on the spot, not kept in registers)
    for (int c0 = first; c0 < nv4; c0 += G * NT) {
      if (NV == 0) load(c0);
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const int c = c0 + NT * k;
        if (c < nv4) { f(q[k].x, 4 * c); f(q[k].y, 4 * c + 1); f(q[k].z, 4 * c + 2); f(q[k].w, 4 * c + 3); }
        __builtin_amdgcn_sched_barrier(0);               // (one piece at a time: registers)
      }
      if (NV) break;
    }
  };
  if (NV) load(t);
  if (t == 0) s_n = 0;
  float tv = -INFINITY;
  visit([&](float x, int) { tv = fmaxf(tv, x); });       // (a NaN is never the best)
  float mx = -INFINITY, tau = -INFINITY;
  {
    bool taken = false;
    for (int round = 0; round < K; ++round) {
      tau = beam_wave_max(taken ? -INFINITY : tv);       // -inf when fewer than K of its threads hold an element
      if (round == 0) mx = tau;
      const unsigned long long at = __ballot(!taken && tv == tau);
      if (at && lane == __ffsll(at) - 1) taken = true;
    }
  }
  if (lane == 0) { s_v[w] = tau; s_sum[w] = mx; }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) { tau = fmaxf(tau, s_v[i]); mx = fmaxf(mx, s_sum[i]); }
  __syncthreads();                                       // (s_sum is written again below)
  float e = 0.f;
  visit([&](float x, int token) {
    e += FAST ? __expf(x - mx) : expf(x - mx);
    if (x >= tau) {
      const int pos = atomicAdd(&s_n, 1);
      if (pos < BEAM_CAND_CAP) { s_cv[pos] = x; s_ci[pos] = token; }
    }
  });
  e = wave_sum(e);
  if (lane == 0) s_sum[w] = e;
  __syncthreads();
  if (t == 0) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) sum += s_sum[i];
    bs.row_lse[r] = mx + logf(sum);
  }
  const int n = s_n;
  float* const out_z = bs.cand_z + (size_t)r * BEAM_MAX;
  int32_t* const out_t = bs.cand_tok + (size_t)r * BEAM_MAX;
  if (n <= BEAM_CAND_CAP) {
    if (t >= n && t < K) { out_z[t] = -INFINITY; out_t[t] = 0x7fffffff; }
    for (int i = t; i < n; i += NT) {
      const float v = s_cv[i];
      const int f = s_ci[i];
      int place = 0;
#pragma unroll 8
      for (int k = 0; k < n; ++k) place += beam_better(s_cv[k], s_ci[k], v, f);
      if (place < K) { out_z[place] = v; out_t[place] = f; }
    }
    return;
  }
  // K rounds: the best element strictly after the previous winner in the (value, token) order
  float pv = INFINITY; int pi = -1;
  for (int round = 0; round < K; ++round) {
    float v = -INFINITY; int f = 0x7fffffff;
    visit([&](float x, int xi) {
      if ((x < pv || (x == pv && xi > pi)) && beam_better(x, xi, v, f)) { v = x; f = xi; }
    });
    beam_block_best<NW>(v, f, s_v, s_f);
    if (t == 0) { out_z[round] = v; out_t[round] = f; }
    pv = v; pi = f;
  }
}

// One workgroup per sentence: the K best one-token extensions over the candidates of its live rows
// (equal scores: the lower (slot, token) pair first), finished hypotheses split off, history written.
// Every candidate counts how many are better, then lane q of the first wavefront takes the q-th best: the chain of this
// launch is what it costs.
__global__ __launch_bounds__(256) void beam_merge_kernel(int V, BeamState bs, int K, int j, int max_len, int eos, float alpha) {
  __shared__ float s_cv[BEAM_MAX * BEAM_MAX];
  __shared__ int s_cf[BEAM_MAX * BEAM_MAX];
  __shared__ float s_winv[BEAM_MAX];
  __shared__ int s_winf[BEAM_MAX];
  const int b = blockIdx.x, t = threadIdx.x;
  // thread t holds candidate t % K of live row t / K (K * K <= 256); everything is requested at once, before it is known
  // which rows live
  const int row0 = b * K, slot = t / K, row = row0 + min(slot, K - 1);
  const int nl = bs.nlive[b];
  const float zc = bs.cand_z[(size_t)row * BEAM_MAX + t - slot * K], cum = bs.cum[row], lse = bs.row_lse[row];
  const int tok = bs.cand_tok[(size_t)row * BEAM_MAX + t - slot * K];
  const float fin_score = bs.fin_score[b];
  if (nl == 0) {                                         // the sentence is done (uniform over the workgroup)
    if (t < K) { bs.parent[row0 + t] = -1; bs.new_cum[row0 + t] = -INFINITY; }
    return;
  }
  float cv = -INFINITY; int cf = 0x7fffffff;
  if (slot < nl && tok != 0x7fffffff) { cv = (cum - lse) + zc; cf = slot * V + tok; }
  s_cv[t] = cv; s_cf[t] = cf;
  if (t < BEAM_MAX) { s_winv[t] = -INFINITY; s_winf[t] = 0; }
  __syncthreads();
  if (cv > -INFINITY) {                                  // (neither NaN nor an empty entry)
    int place = 0;
#pragma unroll 8
    for (int k = 0; k < nl * K; ++k) place += beam_better(s_cv[k], s_cf[k], cv, cf);
    if (place < K) { s_winv[place] = cv; s_winf[place] = cf; }
  }
  __syncthreads();
  if (t >= 64) return;
  // ---- split the winners into finished and live hypotheses ---------------------------------------------
  const float v = t < K ? s_winv[t] : -INFINITY;
  const int f = t < K ? s_winf[t] : 0;
  const int s = f / V, tk = f - s * V;
  const bool won = v > -INFINITY;                        // else fewer candidates than K
  const bool fin = won && (tk == eos || j == max_len - 1), live = won && !fin;
  const unsigned long long m_fin = __ballot(fin), m_live = __ballot(live);
  const int n_new = __popcll(m_live);
  if (live) {
    const int q = __popcll(m_live & ((1ull << t) - 1)), r = row0 + q;
    bs.new_cum[r] = v;
    bs.parent[r] = row0 + s;
    bs.new_tok[r] = tk;
    bs.hist_tok[(size_t)j * bs.hist_ld + r] = tk;
    bs.hist_par[(size_t)j * bs.hist_ld + r] = s;
  }
  if (t >= n_new && t < K) { bs.new_cum[row0 + t] = -INFINITY; bs.parent[row0 + t] = -1; }
  if (t == 0) bs.nlive[b] = n_new;
  if (m_fin) {
    const float norm = v / powf((5.f + (float)(j + 1)) / 6.f, alpha);
    float best = fin_score;
    int at = -1;
    for (unsigned long long m = m_fin; m; m &= m - 1) {
      const int q = __ffsll(m) - 1;
      const float x = __shfl(norm, q, 64);
      if (x > best) { best = x; at = q; }                // strict: the hypothesis finished first keeps a tie
    }
    if (t == at) { bs.fin_score[b] = best; bs.fin_step[b] = j; bs.fin_par[b] = s; bs.fin_tok[b] = tk; }
  }
}
void launch_beam_select(const float* z, int V, const BeamState& bs, int B, int K, int j, int max_len, int eos, float alpha,
                        hipStream_t st, int fast_exp) {
#define GO(NT, NV)                                                                                                  \
  do {                                                                                                              \
    if (fast_exp) hipLaunchKernelGGL((beam_row_topk_kernel<true, NT, NV>), dim3(B * K), dim3(NT), 0, st, z, V, bs, K); \
    else hipLaunchKernelGGL((beam_row_topk_kernel<false, NT, NV>), dim3(B * K), dim3(NT), 0, st, z, V, bs, K);      \
  } while (0)
  // Short rows, and rows for a chip's worth of workgroups, take 256 threads; fewer rows wait for their own chain, not for the
  // chip, and take 512.  Measured at V = 32000, whole searches, ms (256 threads reading twice | 512 | 512 with the row in
  // registers | 1024 in registers): one sentence of 10 rows 2.39 | 2.32 | 2.30 | 2.35, 64 sentences 14.90 | 15.00 | 15.01 | 15.09.
  if (V <= 4 * 256 * 8) GO(256, 8);
  else if (B * K >= 256) GO(256, 0);
  else if (V <= 4 * 512 * 16) GO(512, 16);
  else GO(512, 0);
#undef GO
  hipLaunchKernelGGL(beam_merge_kernel, dim3(B), dim3(256), 0, st, V, bs, K, j, max_len, eos, alpha);
}
// New row r takes the states of row parent[r] (or stays dead): blockIdx.y < L the h (T) and c (fp32) of that layer, L the H_o
// that becomes its input feed, L + 1 the embedding of its token and the scores, tokens and masks.  One part per
// workgroup: one workgroup for a whole row waits for its parts' loads one after the other, and a launch of its own for
// the embeddings is one more in the chain.
template <typename T>
__global__ __launch_bounds__(256) void beam_reorder_kernel(BeamReorder ro, BeamState bs, int H, int L) {
  const int r = blockIdx.x, l = blockIdx.y, t = threadIdx.x;
  const int pr = bs.parent[r];
  constexpr int VE = 16 / sizeof(T);
  auto copy = [&](const T* src, T* dst, T* dst_fm, int n, int k0, int nsteps) {   // dst_fm: 8 elements of one k chunk at a time
    for (int c = t * VE; c < n; c += 256 * VE) {
      const uint4 v = *reinterpret_cast<const uint4*>(src + c);
      *reinterpret_cast<uint4*>(dst + c) = v;
      if (sizeof(T) == 2 && dst_fm) *reinterpret_cast<uint4*>(dst_fm + fm_offset(r, k0 + c, nsteps)) = v;
    }
  };
  if (l == L + 1) {
    if (t == 0) { bs.cum[r] = bs.new_cum[r]; bs.mask[r] = pr >= 0 ? 1.f : 0.f; }
    if (pr < 0) return;
    const int tok = bs.new_tok[r];
    if (t == 0) bs.tok[r] = tok;
    copy((const T*)ro.table + (size_t)tok * ro.E, (T*)ro.x + (size_t)r * ro.ldho_dst, (T*)ro.ho_dst_fm, ro.E, 0, ro.ho_fm_nsteps);
    return;
  }
  if (pr < 0) return;
  if (l == L) {
    copy((const T*)ro.ho_src + (size_t)pr * ro.ldho_src, (T*)ro.ho_dst + (size_t)r * ro.ldho_dst, (T*)ro.ho_dst_fm, H, ro.ho_fm_k0,
         ro.ho_fm_nsteps);
    return;
  }
  const float* cs = ro.c_src[l] + (size_t)pr * H;
  float* cd = ro.c_dst[l] + (size_t)r * H;
  for (int c = t * 4; c < H; c += 256 * 4) *reinterpret_cast<float4*>(cd + c) = *reinterpret_cast<const float4*>(cs + c);
  copy((const T*)ro.h_src[l] + (size_t)pr * ro.ldh, (T*)ro.h_dst[l] + (size_t)r * ro.ldh, (T*)ro.h_dst_fm[l], H, 0, H >> 5);
}
void launch_beam_reorder(int prec, const BeamReorder& ro, const BeamState& bs, int R, int H, int L, hipStream_t st) {
  const dim3 grid(R, L + 2);
  if (prec) hipLaunchKernelGGL(beam_reorder_kernel<bf16_t>, grid, dim3(256), 0, st, ro, bs, H, L);
  else hipLaunchKernelGGL(beam_reorder_kernel<float>, grid, dim3(256), 0, st, ro, bs, H, L);
}

// one thread per sentence: walk the back-pointers of the best finished hypothesis
__global__ __launch_bounds__(64) void beam_finish_kernel(BeamState bs, int B, int K, int max_len, int pad, int32_t* __restrict__ out_ids,
                                                         int32_t* __restrict__ out_len, float* __restrict__ out_score) {
  const int b = blockIdx.x * 64 + threadIdx.x;
  if (b >= B) return;
  const int j = bs.fin_step[b];
  const int len = j + 1;
  int32_t* o = out_ids + (size_t)b * max_len;
  for (int q = 0; q < max_len; ++q) o[q] = pad;
  out_len[b] = len;
  out_score[b] = bs.fin_score[b];
  if (j < 0) { out_len[b] = 0; return; }
  o[j] = bs.fin_tok[b];
  int s = bs.fin_par[b];
  for (int q = j - 1; q >= 0; --q) {
    const size_t i = (size_t)q * bs.hist_ld + b * K + s;
    o[q] = bs.hist_tok[i];
    s = bs.hist_par[i];
  }
}
void launch_beam_finish(const BeamState& bs, int B, int K, int max_len, int pad, int32_t* out_ids, int32_t* out_len, float* out_score,
                        hipStream_t st) {
  hipLaunchKernelGGL(beam_finish_kernel, dim3((B + 63) / 64), dim3(64), 0, st, bs, B, K, max_len, pad, out_ids, out_len, out_score);
}

}  // namespace cmt

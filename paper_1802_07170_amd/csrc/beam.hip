// Beam search bookkeeping on the device (hyperparameter table: beam size 10, length penalty 0.6;
// the Settings section names the length normalisation of Wu et al. 2016).  The decoder runs on
// R = B * K rows, row r = b * K + s holding live hypothesis s of sentence b.  Per step:
//   beam_logits_kernel  the logits of all rows, and the maximum and sum of exponentials of every group of them;
//   beam_pick_kernel    one workgroup per sentence: log-sum-exp of its rows, and the K best one-token extensions over all live
//                       hypotheses (equal scores: the lower (slot, token) pair first), finished
//                       hypotheses split off, history written;
//   beam_reorder_kernel the surviving hypotheses' decoder states and H_o move to their new rows, and
//                       the embeddings of their tokens become the next step's input.
// After the last step beam_finish_kernel walks the back-pointers of each sentence's best finished
// hypothesis.  Nothing returns to the host inside the loop.
#include <type_traits>

#include "gemm_core.h"
#include "kernels.h"

namespace cmt {

// dst[r, 0:cols] = src[r / K, 0:cols] for r < R, zero rows for r in [R, Rp).
// Row pitches in elements; cols * sizeof(T) is a multiple of 16.
template <typename T>
__global__ __launch_bounds__(128) void beam_expand_kernel(const T* __restrict__ src, int ld_src, T* __restrict__ dst, int ld_dst, int R,
                                                          int K, int cols) {
  const int r = blockIdx.x;
  constexpr int VE = 16 / sizeof(T);
  const T* s = r < R ? src + (size_t)(r / K) * ld_src : nullptr;
  T* d = dst + (size_t)r * ld_dst;
  for (int c = threadIdx.x * VE; c < cols; c += 128 * VE)
    *reinterpret_cast<uint4*>(d + c) = s ? *reinterpret_cast<const uint4*>(s + c) : make_uint4(0, 0, 0, 0);
}
void launch_beam_expand(int elem_bytes, const void* src, int ld_src, void* dst, int ld_dst, int R, int Rp, int K, int cols, hipStream_t st) {
  if (elem_bytes == 2)
    hipLaunchKernelGGL(beam_expand_kernel<bf16_t>, dim3(Rp), dim3(128), 0, st, (const bf16_t*)src, ld_src, (bf16_t*)dst, ld_dst, R, K, cols);
  else
    hipLaunchKernelGGL(beam_expand_kernel<float>, dim3(Rp), dim3(128), 0, st, (const float*)src, ld_src, (float*)dst, ld_dst, R, K, cols);
}

// start of a search: one live hypothesis per sentence (slot 0, score 0, previous token bos)
__global__ __launch_bounds__(256) void beam_init_kernel(BeamState bs, int B, int Rp, int K, int bos) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < Rp) {
    const int b = r / K, s = r - b * K;
    const bool real = b < B;
    bs.cum[r] = real && s == 0 ? 0.f : -INFINITY;
    bs.tok[r] = bos;
    bs.mask[r] = real && s == 0 ? 1.f : 0.f;
  }
  if (r < B) { bs.nlive[r] = 1; bs.fin_score[r] = -INFINITY; bs.fin_step[r] = -1; bs.fin_par[r] = 0; bs.fin_tok[r] = 0; }
}
void launch_beam_init(const BeamState& bs, int B, int Rp, int K, int bos, hipStream_t st) {
  hipLaunchKernelGGL(beam_init_kernel, dim3((Rp + 255) / 256), dim3(256), 0, st, bs, B, Rp, K, bos);
}

constexpr int BEAM_MAX = 16;

// Pairs (value, index), the larger value first, then the lower index, as one number: of two keys the larger is the better pair.  (Two comparisons and a branch per pair, with an LDS read
// in it, made the counting below take 4.7 us for 56 entries; this 0.6.)
__device__ __forceinline__ unsigned beam_sortable(float v) {
  const unsigned u = __float_as_uint(v);
  return u ^ ((int)u < 0 ? 0xffffffffu : 0x80000000u);
}
__device__ __forceinline__ float beam_unsortable(unsigned u) { return __uint_as_float((int)u < 0 ? u ^ 0x80000000u : ~u); }
__device__ __forceinline__ uint64_t beam_key(float v, int f) { return (uint64_t)beam_sortable(v + 0.f) << 32 | (unsigned)~f; }   // (-0 is 0)
__device__ __forceinline__ float beam_key_value(uint64_t k) { return beam_unsortable((unsigned)(k >> 32)); }
__device__ __forceinline__ int beam_key_index(uint64_t k) { return (int)~(unsigned)k; }
// how many of n keys in LDS are better
__device__ __forceinline__ int beam_place(const uint64_t* keys, int n, uint64_t key) {
  int place = 0;
#pragma unroll 8
  for (int k = 0; k < n; ++k) place += keys[k] > key;
  return place;
}
// Appends the values of the lanes with `take` to a list in LDS of at most cap entries: one atomic per wavefront.
__device__ __forceinline__ void beam_append(bool take, uint64_t key, uint64_t* list, int* n, int cap) {
  const unsigned long long at = __ballot(take);
  if (at == 0) return;
  const int lane = threadIdx.x & 63;
  int base = 0;
  if (lane == 0) base = atomicAdd(n, __popcll(at));
  const int pos = __builtin_amdgcn_readfirstlane(base) + __popcll(at & ((1ull << lane) - 1));
  if (take && pos < cap) list[pos] = key;
}

// Largest value of a wavefront, in every lane, by DPP moves: about a tenth of the time of six shuffles through LDS.
__device__ __forceinline__ float beam_wave_max(float v) {
#define STEP(ctrl, rows) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, rows, 0xf, false)))
  STEP(0x111, 0xf); STEP(0x112, 0xf); STEP(0x114, 0xf); STEP(0x118, 0xf);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16
  STEP(0x142, 0xa);                                                        // row_bcast15 into rows 1, 3
  STEP(0x143, 0xc);                                                        // row_bcast31 into rows 2, 3
#undef STEP
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// z^T = W_o Ho^T + B_o, [V, pitch] fp32 with the R rows of the search side by side, and per group of 32 TA vocabulary entries
// (gmax, gsum: [rows, groups]) each row's largest logit and its sum of exp(logit - that).  The tile is computed as in the output
// layer's forward kernel, vocabulary entries on the matrix cores' row side, so that a lane holds 32 TA / 2 entries of one row.
// With the groups' statistics the choice of the K best reads 40 KB per sentence and the K best groups instead of every logit.
// The row tile is as wide as makes the rounds of workgroups over the chip come out (beam_logits_plan): what a workgroup takes in is
// its rows and its weights, 49 GB/s per CU.  640 rows x 32000, k 1024: 256 x 320 tiles, one round of 250: 80 -> 52 us.  (That tile has 160
// accumulators a lane and spills two registers.)
// fp32: the large tile keeps all products in one sum, as the output layer's does and for its reasons (ce.hip); 3.64 ms a search of 320 rows,
// 3.67 with two.
template <typename T, int WM, int WN, int TA, int TB>
__global__ __launch_bounds__(64 * WM * WN) void beam_logits_kernel(const T* __restrict__ Ho, int ldho, const T* __restrict__ Wo,
                                                                   const float* __restrict__ Bo, int R, int V, int H, float* __restrict__ zT,
                                                                   int pitch, float* __restrict__ gmax, float* __restrict__ gsum) {
  using G = GemmTile<T, WM, WN, TA, TB>;
  constexpr bool FAST = sizeof(T) == 2;
  __shared__ __align__(16) char smem[FAST ? 2 * (G::BM + G::BN) * 128 : G::SMEM_BYTES];
  int v0, r0;
  if (!gemm_tile_of_block((V + G::BM - 1) / G::BM, (R + G::BN - 1) / G::BN, G::BM, G::BN, v0, r0)) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ng = (V + 32 * TA - 1) / (32 * TA);
  const int wm = w / WN, wn = w % WN, vw = v0 + wm * 32 * TA;
  v16f acc[TA][TB];
  gemm_mainloop<T, WM, WN, TA, TB, TA * TB == 1 ? GEMM_F32_SPLIT : GEMM_F32_ONE_SUM>(Wo, H, Ho, ldho, V, R, H, v0, r0, acc, smem, [&](v16f (&acc)[TA][TB]) {
#pragma unroll
    for (int mt = 0; mt < TA; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int v = vw + mt * 32 + acc32_row(lane, i);
        const float bv = v < V ? Bo[v] : 0.f;
#pragma unroll
        for (int nt = 0; nt < TB; ++nt) acc[mt][nt][i] = bv;
      }
  });
  if (vw >= V) return;                                     // (no barrier behind this)
  const int g = vw / (32 * TA), q = lane >> 5;
  if (vw + 32 * TA > V) {                                  // the group that reaches past the vocabulary
#pragma unroll
    for (int mt = 0; mt < TA; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (vw + mt * 32 + acc32_row(lane, i) >= V) {
#pragma unroll
          for (int nt = 0; nt < TB; ++nt) acc[mt][nt][i] = -INFINITY;
        }
  }
  const bool whole = vw + 32 * TA <= V;
#pragma unroll
  for (int nt = 0; nt < TB; ++nt) {
    const int r = r0 + wn * 32 * TB + nt * 32 + (lane & 31);
    float mx = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < TA; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[mt][nt][i]);   // (a NaN is never the best)
    if (r < R) {                                           // row of entry i: a uniform one plus the lane's 4 q
      const unsigned off = (unsigned)(4 * q * pitch + r);
#pragma unroll
      for (int mt = 0; mt < TA; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int v = vw + mt * 32 + 8 * (i >> 2) + (i & 3);
          if (whole || v + 4 * q < V) (zT + (size_t)v * pitch)[off] = acc[mt][nt][i];
        }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float ms = mx > -INFINITY ? mx : 0.f;
    float e = 0.f;
#pragma unroll
    for (int mt = 0; mt < TA; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) e += FAST ? __expf(acc[mt][nt][i] - ms) : expf(acc[mt][nt][i] - ms);
    e += __shfl_xor(e, 32, 64);
    if (lane < 32 && r < R) { gmax[(size_t)r * ng + g] = mx; gsum[(size_t)r * ng + g] = e; }
    __builtin_amdgcn_sched_barrier(0);                     // (one column tile at a time: registers)
  }
}

// One workgroup per sentence.  A group's largest extension, (score - lse) + gmax, is one of its extensions.  With groups in the order of
// (that value, slot, place in the vocabulary) the K best groups hold the K best extensions: an extension of another group is worse than
// the largest one of each of them, by the value or, where it is equal, by the slot or the token.
//   lse of the live rows from the groups' statistics;
//   the K best groups: the K-th best of a row's 64 threads' best is a bound that K threads of a row at most pass; their groups that
//   pass are listed in LDS and each counts how many are better;
//   the entries of those groups that reach the K-th one's value are listed, and each counts how many are better: that is its place.
// Equal logits in any number stay within the lists (all extensions of 640 rows equal: 10.7 ms a search, 10.4 else).  More than BEAM_PICK_CAP groups can pass only
// where a few threads own nearly all the best groups of a long vocabulary: then K rounds of a workgroup-wide maximum over the groups (64
// rows x 40000, eight steps: 0.96 ms where the best groups are spread 0.43; rounds over all extensions took 34).
// What bounds it is the chain of these steps, each a trip to memory or a barrier.  640 rows, V = 32000: 9.2 us in the place of 29
// for the rows' K best (a pass over 82 MB) and 11 for their merge.
constexpr int BEAM_PICK_NT = 1024, BEAM_PICK_CAP = 1024, BEAM_TOKEN_BITS = 27;   // (slot, token) in one ordered word
constexpr int BEAM_PICK_ENTRIES = BEAM_MAX << 6;        // (groups of 32 or 64 entries)
__global__ __launch_bounds__(BEAM_PICK_NT) void beam_pick_kernel(const float* __restrict__ zT, int pitch, const float* __restrict__ gmax,
                                                                 const float* __restrict__ gsum, int gbits, int V, BeamState bs, int K, int j,
                                                                 int max_len, int eos, float alpha) {
  constexpr int NW = BEAM_PICK_NT / 64;
  __shared__ float s_base[BEAM_MAX];
  __shared__ uint64_t s_g[BEAM_PICK_CAP], s_c[BEAM_PICK_ENTRIES];   // keys of (bound, slot and group) and of (value, slot and token)
  __shared__ uint64_t s_bound[NW];
  __shared__ int s_top[BEAM_MAX];
  __shared__ float s_winv[BEAM_MAX], s_least;
  __shared__ int s_winf[BEAM_MAX];
  __shared__ int s_ng, s_n, s_ntop;
  // (the pointers that the tail needs are fetched now, not one after the other behind the last barrier)
  CMT_PIN_UNIFORM_PTR(bs.parent); CMT_PIN_UNIFORM_PTR(bs.new_cum); CMT_PIN_UNIFORM_PTR(bs.new_tok); CMT_PIN_UNIFORM_PTR(bs.hist_tok);
  CMT_PIN_UNIFORM_PTR(bs.hist_par); CMT_PIN_UNIFORM_PTR(bs.nlive); CMT_PIN_UNIFORM_PTR(bs.fin_score); CMT_PIN_UNIFORM_PTR(bs.fin_step);
  CMT_PIN_UNIFORM_PTR(bs.fin_par); CMT_PIN_UNIFORM_PTR(bs.fin_tok); CMT_PIN_UNIFORM_PTR(bs.cum);
  constexpr int NQ = 16;                                 // a row's first 64 NQ groups stay in its wavefront's registers
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int row0 = b * K, ng = (V + (1 << gbits) - 1) >> gbits;
  // wavefront s takes row s; everything is requested at once, before it is known which rows live
  const size_t r = row0 + min(w, K - 1);
  float m[NQ], x[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const bool in = lane + 64 * q < ng;
    m[q] = in ? gmax[r * ng + lane + 64 * q] : -INFINITY;
    x[q] = in ? gsum[r * ng + lane + 64 * q] : 0.f;
  }
  const int nl = bs.nlive[b];
  const float fin_score = bs.fin_score[b], cum = bs.cum[r];
  if (nl == 0) {                                         // the sentence is done (uniform over the workgroup)
    if (t < K) { bs.parent[row0 + t] = -1; bs.new_cum[row0 + t] = -INFINITY; }
    return;
  }
  if (t == 0) { s_ng = 0; s_n = 0; s_ntop = 0; s_least = -INFINITY; }
  if (t < BEAM_MAX) { s_winv[t] = -INFINITY; s_winf[t] = 0; }
  float base = 0.f;
  uint64_t tau = 0;
  if (w < nl) {                                          // (uniform over the wavefront)
    float tv = -INFINITY;
#pragma unroll
    for (int q = 0; q < NQ; ++q) tv = fmaxf(tv, m[q]);
    for (int g = lane + 64 * NQ; g < ng; g += 64) tv = fmaxf(tv, gmax[r * ng + g]);
    const float mx = beam_wave_max(tv);
    float e = 0.f;
#pragma unroll
    for (int q = 0; q < NQ; ++q) e += m[q] > -INFINITY ? x[q] * expf(m[q] - mx) : x[q];   // (a group of -inf alone has the sum 0, one with NaN a NaN)
    for (int g = lane + 64 * NQ; g < ng; g += 64) {
      const float mg = gmax[r * ng + g], xg = gsum[r * ng + g];
      e += mg > -INFINITY ? xg * expf(mg - mx) : xg;
    }
    base = cum - (mx + logf(wave_sum(e)));
    if (lane == 0) s_base[w] = base;
    // ---- the K best groups ---------------------------------------------------------------------------------
    tv += base;
    if (!(tv > -INFINITY)) tv = -INFINITY;               // (nor NaN)
    // (the largest number that K lanes reach, to the last bit: scores of -500 whose logits lie within 0.5 of each other differ in the
    // lower half alone, and a bound from the upper one let every group pass, 1300 us a step; where K do not hold a group, -inf)
    // Where more than K lanes reach it, the K of them with the first groups: equal logits must not overflow the list.)
    const unsigned key = beam_sortable(tv + 0.f);
    unsigned least = 0;
#pragma unroll
    for (int bit = 31; bit >= 0; --bit)
      if (__popcll(__ballot(key >= (least | 1u << bit))) >= K) least |= 1u << bit;
    if (least >= 0x00800000u) {
      unsigned first = 0;
      if (__popcll(__ballot(key >= least)) > K) {
        int at = 0;                                      // the first of the lane's groups that has its largest value
        for (int g = lane + 64 * ((ng - 1) / 64); g >= 0; g -= 64)
          if (g < ng && base + gmax[r * ng + g] == tv) at = g;
        const unsigned lo = (unsigned)~(w << BEAM_TOKEN_BITS | at);
        first = (unsigned)~(w << BEAM_TOKEN_BITS | ((1 << BEAM_TOKEN_BITS) - 1));
#pragma unroll 1
        for (int bit = BEAM_TOKEN_BITS - 1; bit >= 0; --bit)
          if (__popcll(__ballot(key > least || (key == least && lo >= (first | 1u << bit)))) >= K) first |= 1u << bit;
      }
      tau = (uint64_t)least << 32 | first;
    }
  }
  if (lane == 0) s_bound[w] = tau;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) tau = max(tau, s_bound[i]);
  if (w < nl) {
    const float value = tau ? beam_key_value(tau) : -INFINITY;
    auto list = [&](bool in, float bound, int g) {
      if (__ballot(in && bound >= value) == 0) return;
      const uint64_t key = beam_key(bound, w << BEAM_TOKEN_BITS | g);
      beam_append(in && bound > -INFINITY && key >= tau, key, s_g, &s_ng, BEAM_PICK_CAP);
    };
#pragma unroll
    for (int q = 0; q < NQ; ++q) list(lane + 64 * q < ng, base + m[q], lane + 64 * q);
    for (int g0 = 64 * NQ; g0 < ng; g0 += 64) list(g0 + lane < ng, base + gmax[r * ng + min(g0 + lane, ng - 1)], g0 + lane);
  }
  __syncthreads();
  if (s_ng <= BEAM_PICK_CAP) {
    const int n = s_ng;
    for (int i = t; i < n; i += BEAM_PICK_NT) {
      const int place = beam_place(s_g, n, s_g[i]);
      if (place == K - 1) s_least = beam_key_value(s_g[i]);   // (fewer than K groups: every entry passes)
      if (place < K) s_top[atomicAdd(&s_ntop, 1)] = beam_key_index(s_g[i]);
    }
  } else {                                               // K rounds, each for the best of those behind the one before
    uint64_t last = ~0ull;                               // (short code: what is seldom run is fetched all the same)
#pragma unroll 1
    for (int round = 0; round < K; ++round) {
      uint64_t best = 0;
#pragma unroll 1
      for (int g = w < nl ? lane : ng; g < ng; g += 64) {
        const float bound = base + gmax[r * ng + g];
        const uint64_t key = beam_key(bound, w << BEAM_TOKEN_BITS | g);
        if (bound > -INFINITY && key < last) best = max(best, key);
      }
#pragma unroll 1
      for (int o = 32; o > 0; o >>= 1) best = max(best, (uint64_t)__shfl_xor((unsigned long long)best, o, 64));
      if (lane == 0) s_bound[w] = best;
      __syncthreads();
#pragma unroll 1
      for (int i = 0; i < NW; ++i) best = max(best, s_bound[i]);
      if (t == 0) { s_top[round] = beam_key_index(best); s_least = beam_key_value(best); s_ntop = round + 1; }
      last = best;                                       // (the list's capacity and more are there: never 0)
      __syncthreads();
    }
  }
  __syncthreads();
  {
    // ---- their entries -------------------------------------------------------------------------------------
    const float least = s_least;
    const int entries = s_ntop << gbits;
    for (int i0 = 0; i0 < entries; i0 += BEAM_PICK_NT) {
      const int i = min(i0 + t, entries - 1), id = s_top[i >> gbits], s = id >> BEAM_TOKEN_BITS;
      const int v = ((id & ((1 << BEAM_TOKEN_BITS) - 1)) << gbits) + (i & ((1 << gbits) - 1));
      const bool in = i0 + t < entries && v < V;
      const float x = in ? s_base[s] + zT[(size_t)v * pitch + row0 + s] : -INFINITY;
      beam_append(x >= least && x > -INFINITY, beam_key(x, s << BEAM_TOKEN_BITS | v), s_c, &s_n, BEAM_PICK_ENTRIES);   // (neither NaN nor impossible)
    }
    __syncthreads();
    const int n = s_n;
    for (int i = t; i < n; i += BEAM_PICK_NT) {
      const int place = beam_place(s_c, n, s_c[i]);
      if (place < K) { s_winv[place] = beam_key_value(s_c[i]); s_winf[place] = beam_key_index(s_c[i]); }
    }
  }
  __syncthreads();
  if (t >= 64) return;
  // ---- split the winners into finished and live hypotheses ---------------------------------------------
  const float v = t < K ? s_winv[t] : -INFINITY;
  const int f = t < K ? s_winf[t] : 0;
  const int s = f >> BEAM_TOKEN_BITS, tk = f & ((1 << BEAM_TOKEN_BITS) - 1);
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

// 0: 64 x 64 tiles (groups of 32 entries); 1 .. 5: 256 x (64 n) tiles (groups of 64).  Few rows or a short vocabulary leave the big tiles
// short of workgroups; else rounds over the chip's CUs times what a workgroup takes in decides.
static int beam_logits_plan(int prec, int R, int V) {
  const long tv = (V + 255) / 256;
  if (R <= 64 || tv * ((R + 127) / 128) < 96) return 0;
  if (!prec) return 2;
  int best = 0; long cost = 0;
  for (int n = 1; n <= 5; ++n) {
    const long c = (tv * ((R + 64 * n - 1) / (64 * n)) + 255) / 256 * (256 + 64 * n);
    if (best == 0 || c <= cost) { best = n; cost = c; }
  }
  return best;
}
void launch_beam_select(int prec, const void* Ho, int ldho, const void* Wo, const float* Bo, int Rp, int V, int H, float* zT, float* gmax,
                        float* gsum, const BeamState& bs, int B, int K, int j, int max_len, int eos, float alpha, hipStream_t st) {
  const int R = B * K, plan = beam_logits_plan(prec, R, V);
  auto go = [&](auto type, auto wm, auto ta, auto tb) {
    using T = decltype(type);
    using G = GemmTile<T, decltype(wm)::value, 2, decltype(ta)::value, decltype(tb)::value>;
    const int grid = ((V + G::BM - 1) / G::BM * ((R + G::BN - 1) / G::BN) + 7) / 8 * 8;
    hipLaunchKernelGGL((beam_logits_kernel<T, G::WM, G::WN, G::TA, G::TB>), dim3(grid), dim3(G::NT), 0, st, (const T*)Ho, ldho, (const T*)Wo, Bo,
                       R, V, H, zT, Rp, gmax, gsum);
  };
  using std::integral_constant;
  const integral_constant<int, 1> one; const integral_constant<int, 2> two; const integral_constant<int, 3> three;
  const integral_constant<int, 4> four; const integral_constant<int, 5> five;
  if (!prec) { if (plan) go(float{}, four, two, two); else go(float{}, two, one, one); }
  else if (plan == 0) go(bf16_t{}, two, one, one);
  else if (plan == 1) go(bf16_t{}, four, two, one);
  else if (plan == 2) go(bf16_t{}, four, two, two);
  else if (plan == 3) go(bf16_t{}, four, two, three);
  else if (plan == 4) go(bf16_t{}, four, two, four);
  else go(bf16_t{}, four, two, five);
  hipLaunchKernelGGL(beam_pick_kernel, dim3(B), dim3(BEAM_PICK_NT), 0, st, zT, Rp, gmax, gsum, plan ? 6 : 5, V, bs, K, j, max_len, eos, alpha);
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
  // dst_fm: 8 elements of one k chunk at a time; the kernels that read it read no rows (but a dead row's state, which is anything)
  auto copy = [&](const T* src, T* dst, T* dst_fm, int n, int k0, int nsteps) {
    for (int c = t * VE; c < n; c += 256 * VE) {
      const uint4 v = *reinterpret_cast<const uint4*>(src + c);
      if (sizeof(T) == 2 && dst_fm) *reinterpret_cast<uint4*>(dst_fm + fm_offset(r, k0 + c, nsteps)) = v;
      else *reinterpret_cast<uint4*>(dst + c) = v;
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

// One workgroup per sentence walks the back-pointers of its best finished hypothesis: they are brought to LDS together, a step at a time
// from memory they took 1 us each (50 steps 47 us); the tokens of the path then come together as well.  (FINISH_SLOTS bytes: a
// longer history is walked in memory.)
constexpr int FINISH_SLOTS = 16384;
__global__ __launch_bounds__(256) void beam_finish_kernel(BeamState bs, int B, int K, int max_len, int pad, int32_t* __restrict__ out_ids,
                                                          int32_t* __restrict__ out_len, float* __restrict__ out_score) {
  __shared__ uint8_t s_par[FINISH_SLOTS];
  __shared__ uint8_t s_path[FINISH_SLOTS];
  const int b = blockIdx.x, t = threadIdx.x;
  const int j = bs.fin_step[b];                          // -1: nothing finished
  int32_t* o = out_ids + (size_t)b * max_len;
  const bool staged = j * K <= FINISH_SLOTS;             // (K >= 1: the path fits as well)
  const auto at = [&](int q, int s) { return (size_t)q * bs.hist_ld + b * K + s; };
  if (staged)
    for (int i = t; i < j * K; i += 256) s_par[i] = (uint8_t)bs.hist_par[at(i / K, i % K)];
  for (int q = t; q < max_len; q += 256)
    if (q >= j) o[q] = q == j && j >= 0 ? bs.fin_tok[b] : pad;
  __syncthreads();
  if (t == 0) {
    out_len[b] = j + 1;
    out_score[b] = bs.fin_score[b];
    int s = j < 0 ? 0 : bs.fin_par[b];
    for (int q = j - 1; q >= 0; --q) {
      if (staged) { s_path[q] = (uint8_t)s; s = s_par[q * K + s]; }
      else { o[q] = bs.hist_tok[at(q, s)]; s = bs.hist_par[at(q, s)]; }
    }
  }
  __syncthreads();
  if (staged)
    for (int q = t; q < j; q += 256) o[q] = bs.hist_tok[at(q, s_path[q])];
}
void launch_beam_finish(const BeamState& bs, int B, int K, int max_len, int pad, int32_t* out_ids, int32_t* out_len, float* out_score,
                        hipStream_t st) {
  hipLaunchKernelGGL(beam_finish_kernel, dim3(B), dim3(256), 0, st, bs, B, K, max_len, pad, out_ids, out_len, out_score);
}

}  // namespace cmt

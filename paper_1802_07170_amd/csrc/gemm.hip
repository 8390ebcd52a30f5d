// Batched-over-time GEMMs of the training step (the paper's LinearLayer forward / backward /
// calculateGradient, Fig. "Codes of Performing Actual Computation"), all in the single
// "A * B^T, both k-contiguous" form, plus the tiled transpose that brings the backward and
// weight-gradient operands into that form.
#include "gemm_core.h"
#include "kernels.h"
#include <algorithm>
#include <cstdlib>
#include <type_traits>
#include <vector>

namespace cmt {

// Dispatch thresholds, from measurements on MI355X, us (256 x 256 | 128 x 128 | 64 x 64).
// bf16: 160 big tiles (10240 x 1024, k 1024) 30 | 43 | 38, 104 (3200 x 2048, k 1024) 29 | 26 | 27: big from 144 up.  Below
// that the medium tile only with a round of workgroups and a k to spread its prologue and store over: 200 medium tiles
// 25.8 | 27.3 (k 1024; 1472 x 2048, k 512: 16.5 | 9.9), 100 (3200 x 1024, k 1024) 21.5 | 15.3, (1472 x 1024, k 512) 16.1 | 7.6,
// one or two tiles 11 | 5; rows or columns that fit a small tile (16 x 32000, k 1024) 17.5 | 12.3.
// fp32 (256 x 128 | 64 x 64, bound by the matrix cores): 208 big tiles (3200 x 2048, k 512) 51 | 62, 104 (3200 x 1024) 46 | 38; 128 x 128 in
// between 38, and 54 against 32 at 1000 x 1000, k 1000: no such tile.
static int env_int(const char* name, int dflt) {
  const char* e = getenv(name);
  return e && *e ? atoi(e) : dflt;
}
static const int GEMM_BIG_MIN_TILES = env_int("CMT_GEMM_BIG_MIN_TILES", 144);
static const int GEMM_SPLIT_BELOW = env_int("CMT_GEMM_SPLIT_BELOW", 257);       // small tiles
// Workgroups of the 64 x 64 tile that a CU's LDS holds: four, of fp32 products in parts three (the 256 bytes: their vote).  A split of k aims at
// one round of them over the chip: fp32 training steps with 768 instead of 1024 workgroups wanted: width 512, 64 sentences, vocabulary 16000 4.44 -> 4.38
// ms, 6400 2.76 -> 2.72; width 256, vocabulary 2000 1.60 -> 1.59; widths 64 - 128 and 768 - 1024 0 - 0.5 %.
template <typename T> constexpr int gemm_small_per_cu(bool chain) {
  return 160 * 1024 / ((chain ? GemmSmall<T>::CHAIN_BYTES : GemmSmall<T>::SMEM_BYTES) + 256);
}
static_assert(gemm_small_per_cu<bf16_t>(false) == 4 && gemm_small_per_cu<float>(true) == 4 && gemm_small_per_cu<float>(false) == 3,
              "what the rules below were measured with");
// Medium tiles of which there is at most one per CU take four k tiles of LDS, three of them on their way, instead of two for two
// workgroups per CU, us (two | four): 200 tiles, k 4096 56 | 50, k 2048 35 | 31; 234 tiles, k 1096 29 | 26; 400 tiles, k 1024 28 | 40.
static const int GEMM_DEEP_MAX_TILES = env_int("CMT_GEMM_DEEP_MAX_TILES", 256);
static const int GEMM_SPLIT_MAX = env_int("CMT_GEMM_SPLIT_MAX", 16);
static const int GEMM_BIGSPLIT_MIN_K = env_int("CMT_GEMM_BIGSPLIT_MIN_K", 8192);
// beyond this many big tiles (by the host's row count) the small tile without a split measured faster (large
// workload: 160 tiles, 3.15 against 3.57 ms for the output layer)
static const int GEMM_BIGSPLIT_MAX_TILES = env_int("CMT_GEMM_BIGSPLIT_MAX_TILES", 96);

// the 64 x 64 tile instead of the 128 x 128 one, of which there would be `tiles`
static bool gemm_small_tile(int prec, long tiles, int M, int N, int K) {
  if (!prec) return true;
  return tiles < 192 || K < 1024 || M <= GemmSmall<bf16_t>::BM || N <= GemmSmall<bf16_t>::BN;
}

// Number of k splits when the row count is known to the device alone: as many as make one round of workgroups
// (fp32, whose tiles are half as large: two) over the chip's 256 CUs out of the tiles that exist, at most the launched number.  The kernel and the plane
// sum both derive it from the same count.
#define GEMM_DYN_ROUNDS(prec) ((prec) ? 1 : 2)
__host__ __device__ inline int gemm_dyn_splits(int tiles, int launched, int rounds) {
  const int ns = 256 * rounds / (tiles > 0 ? tiles : 1);
  return ns < 1 ? 1 : (ns > launched ? launched : ns);
}

// One output tile (the one of virtual workgroup id vb) of C (+)= A B^T (+ bias): main loop and store.
template <typename T, int WM, int WN, int TA, int TB, bool CHAIN, int STAGES>
__device__ __forceinline__ void gemm_nt_tile(const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb, int M, int N, int K,
                                             float* __restrict__ Cf0, T* __restrict__ Ct, int ldc, const float* __restrict__ bias,
                                             int accumulate, int ntn, int kchunk, size_t plane_stride, int dyn_split, int vb,
                                             char* smem) {
  using G = GemmTile<T, WM, WN, TA, TB>;
  int m0, n0;
  if (!gemm_tile_of_block((M + G::BM - 1) / G::BM, ntn, G::BM, G::BN, m0, n0, vb)) return;
  if (dyn_split) {                                 // the number of k splits follows the tiles that exist: one round of workgroups
    const int ns = gemm_dyn_splits((M + G::BM - 1) / G::BM * ntn, gridDim.y, GEMM_DYN_ROUNDS(sizeof(T) == 2));
    if ((int)blockIdx.y >= ns) return;
    kchunk = ((K + ns - 1) / ns + 63) / 64 * 64;
  }
  const int k0 = blockIdx.y * kchunk;
  const int klen = min(kchunk, K - k0);
  if (klen <= 0 && gridDim.y == 1) return;
  v16f acc[TA][TB];
  gemm_mainloop<T, WM, WN, TA, TB, CHAIN ? GEMM_F32_CHAIN : GEMM_F32_SPLIT, STAGES>(A + k0, lda, B + k0, ldb, M, N, klen, m0, n0, acc, smem, GemmZero{});
  float* const Cf = gridDim.y > 1 ? Cf0 + blockIdx.y * plane_stride : Cf0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wm = w / WN, wn = w % WN;
#pragma unroll
  for (int nt = 0; nt < TB; ++nt) {
    const int col = n0 + wn * 32 * TB + nt * 32 + (lane & 31);
    if (col >= N) continue;
    const float bv = bias ? bias[col] : 0.f;
#pragma unroll
    for (int mt = 0; mt < TA; ++mt) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = m0 + wm * 32 * TA + mt * 32 + acc32_row(lane, i);
        if (row >= M) continue;
        const size_t o = (size_t)row * ldc + col;
        float v = acc[mt][nt][i] + bv;
        if (accumulate) v += Cf[o];
        if (Cf) Cf[o] = v;
        if (Ct) Ct[o] = from_f<T>(v);
      }
    }
  }
}

// blockIdx.y = k split index: each split contracts kchunk elements of k and, when there is more
// than one, writes its own fp32 plane Cf + split * plane_stride (summed afterwards, fixed order).
// WALK: the launch has fewer workgroups than tiles (it is to leave part of the chip to other streams) and every
// workgroup walks the tiles of the virtual ids blockIdx.x, blockIdx.x + grid, ...  It is a variant of its own because
// the loop costs the one-tile-per-workgroup kernel a spilled register (fp32 in parts on the large tile, which walks under a cap alone: six).
template <typename T, int WM, int WN, int TA, int TB, bool WALK = false, bool CHAIN = false, int STAGES = 2>
__global__ __launch_bounds__(64 * WM * WN) void gemm_nt_kernel(const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
                                                               int M, int N, int K, float* __restrict__ Cf0, T* __restrict__ Ct,
                                                               int ldc, const float* __restrict__ bias, int accumulate, int ntn,
                                                               int kchunk, size_t plane_stride, RowLimit lim, int lim_kind,
                                                               int dyn_split) {
  using G = GemmTile<T, WM, WN, TA, TB>;
  __shared__ __align__(16) char smem[STAGES > 2 ? STAGES * (G::BM + G::BN) * 128 : CHAIN ? G::CHAIN_BYTES : G::SMEM_BYTES];
  if (lim.n) {                                     // a bound that only the device knows (uniform over the grid)
    const int e = max(*lim.n - lim.base, 0);
    if (lim_kind == 1) M = min(M, e);
    else K = min(K, (e + 63) / 64 * 64);
    if (M <= 0 || K <= 0) return;
  }
  if constexpr (WALK) {
    const int ntiles8 = (((M + G::BM - 1) / G::BM * ntn + 7) >> 3) << 3;
    for (int vb = blockIdx.x; vb < ntiles8; vb += gridDim.x) {
      gemm_nt_tile<T, WM, WN, TA, TB, CHAIN, STAGES>(A, lda, B, ldb, M, N, K, Cf0, Ct, ldc, bias, accumulate, ntn, kchunk, plane_stride, dyn_split,
                                          vb, smem);
      __syncthreads();                             // (the next tile refills the LDS)
    }
  } else {
    gemm_nt_tile<T, WM, WN, TA, TB, CHAIN, STAGES>(A, lda, B, ldb, M, N, K, Cf0, Ct, ldc, bias, accumulate, ntn, kchunk, plane_stride, dyn_split,
                                        (int)blockIdx.x, smem);
  }
}

// out = sum of planes (+ bias per column) (+ previous out).  VEC = 4: four consecutive columns per thread as one
// 16-byte access per plane (N, ldc and the plane stride multiples of 4, all bases 16-byte aligned).
template <int VEC>
__global__ __launch_bounds__(256) void gemm_planes_sum_kernel(const float* __restrict__ planes, int np, size_t stride,
                                                              float* __restrict__ out, int M, int N, int ldc,
                                                              const float* __restrict__ bias, int accumulate, RowLimit lim,
                                                              int dyn_bm, int dyn_ntn, int dyn_rounds) {
  if (lim.n) M = min(M, max(*lim.n - lim.base, 0));
  if (dyn_bm) np = gemm_dyn_splits((M + dyn_bm - 1) / dyn_bm * dyn_ntn, np, dyn_rounds);   // the planes the GEMM wrote
  const unsigned nq = (unsigned)N / VEC;                  // column groups per row
  const size_t n = (size_t)M * nq;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const unsigned r = (unsigned)(i / nq), c = ((unsigned)i - r * nq) * VEC;
    const float* src = planes + (size_t)r * N + c;
    float* o = out + (size_t)r * ldc + c;
    if (VEC == 4) {
      float4 v = bias ? *reinterpret_cast<const float4*>(bias + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      for (int p = 0; p < np; ++p) {
        const float4 a = *reinterpret_cast<const float4*>(src + (size_t)p * stride);
        v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
      }
      if (accumulate) {
        const float4 a = *reinterpret_cast<const float4*>(o);
        v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
      }
      *reinterpret_cast<float4*>(o) = v;
    } else {
      float v = bias ? bias[c] : 0.f;
      for (int p = 0; p < np; ++p) v += src[(size_t)p * stride];
      *o = accumulate ? *o + v : v;
    }
  }
}

static void launch_planes_sum(const float* planes, int nks, size_t pstride, float* Cf, int M, int N, int ldc, const float* bias,
                              int accumulate, RowLimit rl, hipStream_t st, int dyn_bm = 0, int dyn_ntn = 0, int dyn_rounds = 0) {
  const bool vec = N % 4 == 0 && ldc % 4 == 0 && pstride % 4 == 0 && ((size_t)Cf | (size_t)planes | (size_t)bias) % 16 == 0;
  size_t g = (pstride / (vec ? 4 : 1) + 255) / 256;
  if (g > 4096) g = 4096;
  if (vec)
    hipLaunchKernelGGL(gemm_planes_sum_kernel<4>, dim3((unsigned)g), dim3(256), 0, st, planes, nks, pstride, Cf, M, N, ldc, bias,
                       accumulate, rl, dyn_bm, dyn_ntn, dyn_rounds);
  else
    hipLaunchKernelGGL(gemm_planes_sum_kernel<1>, dim3((unsigned)g), dim3(256), 0, st, planes, nks, pstride, Cf, M, N, ldc, bias,
                       accumulate, rl, dyn_bm, dyn_ntn, dyn_rounds);
}

template <typename T, int WM, int WN, int TA, int TB, int STAGES = 2>
static void gemm_go(dim3 grid, hipStream_t st, const void* A, int lda, const void* B, int ldb, int M, int N, int K, float* out,
                    void* Ct, int ldc, const float* bias, int acc, int ntn, int kchunk, size_t pstride, RowLimit lim, int lim_kind,
                    int dyn_split = 0, int wg_cap = 0, int chain = 0) {
  const bool walk = wg_cap > 0 && (int)grid.x > (wg_cap + 7) / 8 * 8;
  if (walk) grid.x = (wg_cap + 7) / 8 * 8;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WM * WN), 0, st, (const T*)A, lda, (const T*)B, ldb, M, N, K, out, (T*)Ct, ldc, bias, acc, ntn,
                       kchunk, pstride, lim, lim_kind, dyn_split);
  };
  if constexpr (sizeof(T) == 4)
    if (chain) {
      if (walk) go(gemm_nt_kernel<T, WM, WN, TA, TB, true, true>);
      else go(gemm_nt_kernel<T, WM, WN, TA, TB, false, true>);
      return;
    }
  if (walk) go(gemm_nt_kernel<T, WM, WN, TA, TB, true>);
  else go(gemm_nt_kernel<T, WM, WN, TA, TB, false, false, STAGES>);
}

void launch_gemm_nt(int prec, const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                    float* Cf, void* Ct, int ldc, const float* bias, int accumulate, hipStream_t st,
                    float* split_scratch, size_t split_scratch_floats, RowLimit lim, int lim_kind, int wg_cap, int chain) {
  if (M <= 0 || N <= 0) return;
  // enough 256 x 256 tiles to fill the chip: the big tile (half the L2 traffic per flop)
  const int bn_b = prec ? GemmBig<bf16_t>::BN : GemmBig<float>::BN;
  const int ntm_b = (M + GemmBig<bf16_t>::BM - 1) / GemmBig<bf16_t>::BM, ntn_b = (N + bn_b - 1) / bn_b;
  // (of rows that only the device counts, the valid target positions, some 60 - 75 % exist)
  const bool counted = lim.n && lim_kind == 1;
  if (ntm_b * ntn_b >= (counted ? GEMM_BIG_MIN_TILES * 5 / 3 : GEMM_BIG_MIN_TILES)) {
    const int grid = ((ntm_b * ntn_b + 7) / 8) * 8;
    if (prec) gemm_go<bf16_t, 4, 4, 2, 2>(dim3(grid, 1), st, A, lda, B, ldb, M, N, K, Cf, Ct, ldc, bias, accumulate, ntn_b, K, 0, lim, lim_kind, 0, wg_cap);
    else gemm_go<float, 4, 2, 2, 2>(dim3(grid, 1), st, A, lda, B, ldb, M, N, K, Cf, Ct, ldc, bias, accumulate, ntn_b, K, 0, lim, lim_kind, 0, wg_cap, chain);
    return;
  }
  // a long contraction over few output tiles (dH_o = dz W_o: k = the vocabulary): big tiles with k split into
  // planes.  With a device-side row limit the kernel picks the number of splits itself (gemm_dyn_splits) out of
  // the launched maximum; otherwise the host aims at about one and a half rounds of workgroups.
  if (split_scratch && Cf && !Ct && K >= GEMM_BIGSPLIT_MIN_K && ntm_b * ntn_b <= GEMM_BIGSPLIT_MAX_TILES) {
    const bool dyn = counted;
    int ks = dyn ? GEMM_SPLIT_MAX : (384 + ntm_b * ntn_b - 1) / (ntm_b * ntn_b);
    if (ks > GEMM_SPLIT_MAX) ks = GEMM_SPLIT_MAX;
    while (ks > 1 && ((size_t)ks * M * N > split_scratch_floats || K / ks < 2048)) --ks;
    if (ks > 1 && (dyn || ks * ntm_b * ntn_b >= GEMM_BIG_MIN_TILES)) {     // else the small tile fills the chip better
      const int kchunk = ((K + ks - 1) / ks + 63) / 64 * 64;
      const int nks = dyn ? ks : (K + kchunk - 1) / kchunk;
      const size_t pstride = (size_t)M * N;
      const int grid = ((ntm_b * ntn_b + 7) / 8) * 8;
      if (prec) gemm_go<bf16_t, 4, 4, 2, 2>(dim3(grid, nks), st, A, lda, B, ldb, M, N, K, split_scratch, nullptr, N, nullptr, 0, ntn_b, kchunk, pstride, lim, lim_kind, dyn, wg_cap, chain);
      else gemm_go<float, 4, 2, 2, 2>(dim3(grid, nks), st, A, lda, B, ldb, M, N, K, split_scratch, nullptr, N, nullptr, 0, ntn_b, kchunk, pstride, lim, lim_kind, dyn, wg_cap, chain);
      launch_planes_sum(split_scratch, nks, pstride, Cf, M, N, ldc, bias, accumulate, lim_kind == 1 ? lim : RowLimit{}, st,
                        dyn ? GemmBig<bf16_t>::BM : 0, ntn_b, GEMM_DYN_ROUNDS(prec));
      return;
    }
  }
  const auto medium = [&](int d) { return (d + GemmMedium<bf16_t>::BM - 1) / GemmMedium<bf16_t>::BM; };
  const bool small = gemm_small_tile(prec, (long)medium(M) * medium(N), M, N, K);
  const int bm = small ? GemmSmall<bf16_t>::BM : GemmMedium<bf16_t>::BM;
  const int ntm = (M + bm - 1) / bm, ntn = (N + bm - 1) / bm;
  const int nb = ntm * ntn;
  const int grid = ((nb + 7) / 8) * 8;
  const int esz = prec ? 2 : 4;
  const int bk = 128 / esz;
  // few output tiles but a long contraction: split k over workgroups, one round of them over the chip
  const int per_cu = prec ? gemm_small_per_cu<bf16_t>(false) : gemm_small_per_cu<float>(chain);
  int ks = 1;
  if (split_scratch && Cf && !Ct && small && nb < GEMM_SPLIT_BELOW && K >= 16 * bk) {
    ks = (256 * per_cu + nb - 1) / nb;
    if (ks > GEMM_SPLIT_MAX) ks = GEMM_SPLIT_MAX;
    while (ks > 1 && ((size_t)ks * M * N > split_scratch_floats || K / ks < 4 * bk)) --ks;
  }
  int kchunk = K;
  if (ks > 1) kchunk = ((K + ks - 1) / ks + bk - 1) / bk * bk;
  const int nks = (K + kchunk - 1) / kchunk;
  const size_t pstride = (size_t)M * N;
  float* out = nks > 1 ? split_scratch : Cf;
  const int oldc = nks > 1 ? N : ldc;
  const float* obias = nks > 1 ? nullptr : bias;
  const int oacc = nks > 1 ? 0 : accumulate;
  const int cap = small ? per_cu * wg_cap : wg_cap;
  auto go = [&](auto type, auto shape) {
    using T = decltype(type);
    if constexpr (decltype(shape)::value == 1)
      gemm_go<T, 2, 2, 1, 1>(dim3(grid, nks), st, A, lda, B, ldb, M, N, K, out, Ct, oldc, obias, oacc, ntn, kchunk, pstride, lim, lim_kind, 0, cap, chain);
    else
      (nb <= GEMM_DEEP_MAX_TILES ? gemm_go<T, 2, 2, 2, 2, 4> : gemm_go<T, 2, 2, 2, 2, 2>)(dim3(grid, nks), st, A, lda, B, ldb, M, N, K, out, Ct, oldc, obias, oacc, ntn, kchunk, pstride, lim, lim_kind, 0, cap, chain);
  };
  using One = std::integral_constant<int, 1>;
  using Two = std::integral_constant<int, 2>;
  if (prec) { if (small) go(bf16_t{}, One{}); else go(bf16_t{}, Two{}); }
  else go(float{}, One{});
  if (nks > 1) launch_planes_sum(split_scratch, nks, pstride, Cf, M, N, ldc, bias, accumulate, lim_kind == 1 ? lim : RowLimit{}, st);
}

constexpr int GEMM_GROUP_MAX = 16;
struct GemmGroupArgs { int n; int tile_start[GEMM_GROUP_MAX + 1]; GemmProb p[GEMM_GROUP_MAX]; };

template <typename T, int WM, int WN, int TA, int TB, int STAGES>
__global__ __launch_bounds__(64 * WM * WN) void gemm_nt_group_kernel(GemmGroupArgs g) {
  using G = GemmTile<T, WM, WN, TA, TB>;
  __shared__ __align__(16) char smem[STAGES > 2 ? STAGES * (G::BM + G::BN) * 128 : G::SMEM_BYTES];
  // the workgroups walk the tile queue: workgroup v takes the tiles of the virtual ids v, v + grid, v + 2 grid, ...
  // (the grid is a multiple of 8, so a workgroup stays with the tile range of its XCD); a grid as large as the
  // queue is the plain one-tile-per-workgroup launch
  const int nt_all = g.tile_start[g.n], per = (nt_all + 7) >> 3;
  for (int vb = blockIdx.x; (vb >> 3) < per; vb += gridDim.x) {
  const int id = (vb & 7) * per + (vb >> 3);
  if (id >= nt_all) continue;
  int q = 0;
  while (q + 1 < g.n && id >= g.tile_start[q + 1]) ++q;   // uniform over the workgroup
  const GemmProb& pr = g.p[q];
  const int M = pr.M, N = pr.N, ldc = pr.ldc;
  int m0, n0;
  gemm_tile_from_index(id - g.tile_start[q], (M + G::BM - 1) / G::BM, (N + G::BN - 1) / G::BN, G::BM, G::BN, m0, n0);
  v16f acc[TA][TB];
  GemmZero{}(acc);
  for (int part = 0; part < (pr.A2 ? 2 : 1); ++part)
    gemm_mainloop<T, WM, WN, TA, TB, 0, STAGES>((const T*)(part ? pr.A2 : pr.A), part ? pr.lda2 : pr.lda, (const T*)(part ? pr.B2 : pr.B),
                                                part ? pr.ldb2 : pr.ldb, M, N, part ? pr.K2 : pr.K, m0, n0, acc, smem, [](v16f (&)[TA][TB]) {});
  __syncthreads();                                        // (the next tile of a walking workgroup refills the LDS)
  float* __restrict__ C = pr.C;
  T* __restrict__ Ct = (T*)pr.Ct;
  const int accumulate = pr.accumulate;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wm = w / WN, wn = w % WN;
#pragma unroll
  for (int nt = 0; nt < TB; ++nt) {
    const int col = n0 + wn * 32 * TB + nt * 32 + (lane & 31);
    if (col >= N) continue;
    const float bv = pr.bias ? pr.bias[col] : 0.f;
#pragma unroll
    for (int mt = 0; mt < TA; ++mt) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = m0 + wm * 32 * TA + mt * 32 + acc32_row(lane, i);
        if (row >= M) continue;
        const size_t o = (size_t)row * ldc + col;
        float v = acc[mt][nt][i] + bv;
        if (accumulate) v += C[o];
        if (C) C[o] = v;
        if (Ct) Ct[o] = from_f<T>(v);
      }
    }
  }
  }
}

template <typename T, int WM, int WN, int TA, int TB, int STAGES = 2>
static void gemm_group_go(const GemmProb* probs, int n, hipStream_t st, int wg_cap) {
  using G = GemmTile<T, WM, WN, TA, TB>;
  for (int c0 = 0; c0 < n; c0 += GEMM_GROUP_MAX) {
    GemmGroupArgs g{};
    g.n = std::min(GEMM_GROUP_MAX, n - c0);
    int nt = 0;
    for (int i = 0; i < g.n; ++i) {
      g.p[i] = probs[c0 + i];
      g.tile_start[i] = nt;
      nt += ((g.p[i].M + G::BM - 1) / G::BM) * ((g.p[i].N + G::BN - 1) / G::BN);
    }
    g.tile_start[g.n] = nt;
    if (nt == 0) continue;
    int grid = ((nt + 7) / 8) * 8;
    if (wg_cap > 0 && grid > (wg_cap + 7) / 8 * 8) grid = (wg_cap + 7) / 8 * 8;
    hipLaunchKernelGGL((gemm_nt_group_kernel<T, WM, WN, TA, TB, STAGES>), dim3(grid), dim3(64 * WM * WN), 0, st, g);
  }
}

void launch_gemm_nt_group(int prec, const GemmProb* probs, int n, hipStream_t st, float* split_scratch, size_t split_scratch_floats,
                          int wg_cap, int big_cap) {
  if (!prec) {
    // fp32 operands: one launch per problem, k split over workgroups where there are few tiles.  These GEMMs are
    // matrix-core bound either way, and the shorter workgroups of the split form leave the CUs sooner to the
    // recurrences' kernels running beside them (small workload: 11.2 against 11.4 ms per step).
    for (int i = 0; i < n; ++i) {
      const GemmProb& q = probs[i];
      launch_gemm_nt(prec, q.A, q.lda, q.B, q.ldb, q.M, q.N, q.K, q.C, q.Ct, q.ldc, q.bias, q.accumulate, st, split_scratch,
                     split_scratch_floats, RowLimit{}, 0, wg_cap);
      if (q.A2)
        launch_gemm_nt(prec, q.A2, q.lda2, q.B2, q.ldb2, q.M, q.N, q.K2, q.C, nullptr, q.ldc, nullptr, 1, st, split_scratch, split_scratch_floats,
                       RowLimit{}, 0, wg_cap);
    }
    return;
  }
  std::vector<GemmProb> live;
  long big = 0, medium = 0;
  for (int i = 0; i < n; ++i) {
    if (probs[i].M <= 0 || probs[i].N <= 0) continue;
    live.push_back(probs[i]);
    big += (long)((probs[i].M + GemmBig<bf16_t>::BM - 1) / GemmBig<bf16_t>::BM) * ((probs[i].N + GemmBig<bf16_t>::BN - 1) / GemmBig<bf16_t>::BN);
    medium += (long)((probs[i].M + GemmMedium<bf16_t>::BM - 1) / GemmMedium<bf16_t>::BM) * ((probs[i].N + GemmMedium<bf16_t>::BN - 1) / GemmMedium<bf16_t>::BN);
  }
  if (live.empty()) return;
  // the tile by the number of them over the whole group (k is the batch's positions: long)
  if (big >= GEMM_BIG_MIN_TILES) gemm_group_go<bf16_t, 4, 4, 2, 2>(live.data(), (int)live.size(), st, wg_cap ? wg_cap : big_cap);
  else if (medium >= 192 && medium <= GEMM_DEEP_MAX_TILES) gemm_group_go<bf16_t, 2, 2, 2, 2, 4>(live.data(), (int)live.size(), st, wg_cap);
  else if (medium >= 192) gemm_group_go<bf16_t, 2, 2, 2, 2>(live.data(), (int)live.size(), st, wg_cap);
  else gemm_group_go<bf16_t, 2, 2, 1, 1>(live.data(), (int)live.size(), st, gemm_small_per_cu<bf16_t>(false) * wg_cap);
}

// Measurement aid: nothing but matrix-core instructions (4 independent 32x32x16 bf16 accumulator chains per
// wavefront, operands in registers), to read the rate the matrix cores reach on this chip beside the
// nominal peak.  out receives one value per lane so that the loop cannot be dropped.
__global__ __launch_bounds__(256) void mfma_rate_kernel(float* __restrict__ out, int iters) {
  Frag<bf16_t> a, b;
  a.v = make_uint4(0x3f803f80u + threadIdx.x, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  b.v = make_uint4(0x3f803f80u, 0x3f803f80u + blockIdx.x, 0x3f803f80u, 0x3f803f80u);
  v16f acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[q][i] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int q = 0; q < 4; ++q) mma32(acc[q], a, b);
  }
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 16; ++i) s += acc[q][i];
  out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}
double launch_mfma_rate(float* out, int blocks, int iters, hipStream_t st) {
  hipLaunchKernelGGL(mfma_rate_kernel, dim3(blocks), dim3(256), 0, st, out, iters);
  return (double)blocks * 4 /*wavefronts*/ * iters * 4.0 * (2.0 * 32 * 32 * 16);
}

// Several transposes in one launch.  A lane takes a block of 8 x 8 16-bit (4 x 4 32-bit) elements: it reads 16 bytes of each of its
// rows, turns the block over in registers and writes 16 bytes of each column, so that 8 neighbouring lanes read 128
// contiguous bytes and 8 others write such, with no LDS in between.  A wavefront takes 8 x 8 such blocks.  With `parts` the
// column sums come along (a bias' gradient: the matrix is read once instead of twice): the rows go in TRANSPOSE_SPLITS shares, each
// with its partial sums.  Memory-bound: four [3200, 4096] bf16 matrices with
// their sums and a [3200, 1024] one 52 us (4.3 TB/s) + 5; one element per lane through LDS, a pass of its own for the sums and a
// launch for each took 230 us.
struct TransposeJobD { const void* in; void* out; float* parts; int ldin, ldout, R, C, nx, blocks, tpb; };
struct TransposeJobs { TransposeJobD j[TRANSPOSE_MAX_JOBS]; };
template <typename T>
__global__ __launch_bounds__(256) void transpose_multi_kernel(TransposeJobs jobs) {
  constexpr int NB = 16 / sizeof(T);                      // elements per side of a lane's block
  constexpr int TILE = 8 * NB;
  __shared__ float s_sum[4][TILE];
  int blk = blockIdx.x, k = 0;
  while (blk >= jobs.j[k].blocks) blk -= jobs.j[k++].blocks;
  const TransposeJobD& job = jobs.j[k];
  const int by = blk / job.nx, bx = blk - by * job.nx;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, rb = lane >> 3, cb = lane & 7;
  const int c = bx * TILE + cb * NB;
  const T* const in = (const T*)job.in;
  T* const out = (T*)job.out;
  float sum[NB];
#pragma unroll
  for (int e = 0; e < NB; ++e) sum[e] = 0.f;
  for (int t = w; t < job.tpb; t += 4) {
    const int r = (by * job.tpb + t) * TILE + rb * NB;
    if (r >= job.R || c >= job.C) continue;               // (both are multiples of NB)
    uint4 v[NB], o[NB];
#pragma unroll
    for (int e = 0; e < NB; ++e) v[e] = *reinterpret_cast<const uint4*>(in + (size_t)(r + e) * job.ldin + c);
    if constexpr (NB == 8) {
#pragma unroll
      for (int q = 0; q < 4; ++q)                         // words of the rows: columns 2q, 2q + 1
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const uint32_t a = (&v[2 * m].x)[q], b = (&v[2 * m + 1].x)[q];
          (&o[2 * q].x)[m] = __builtin_amdgcn_perm(b, a, 0x05040100u);
          (&o[2 * q + 1].x)[m] = __builtin_amdgcn_perm(b, a, 0x07060302u);
        }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = make_uint4((&v[0].x)[q], (&v[1].x)[q], (&v[2].x)[q], (&v[3].x)[q]);
    }
#pragma unroll
    for (int e = 0; e < NB; ++e) *reinterpret_cast<uint4*>(out + (size_t)(c + e) * job.ldout + r) = o[e];
    if (job.parts) {
#pragma unroll
      for (int e = 0; e < NB; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t x = (&o[e].x)[q];
          if constexpr (NB == 8) sum[e] += __uint_as_float(x << 16) + __uint_as_float(x & 0xffff0000u);
          else sum[e] += __uint_as_float(x);
        }
    }
  }
  if (!job.parts) return;
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    float x = sum[e];
#pragma unroll
    for (int d = 8; d < 64; d <<= 1) x += __shfl_xor(x, d, 64);
    if (rb == 0) s_sum[w][cb * NB + e] = x;
  }
  __syncthreads();
  if (threadIdx.x < TILE && bx * TILE + (int)threadIdx.x < job.C)
    job.parts[(size_t)by * job.C + bx * TILE + threadIdx.x] = (s_sum[0][threadIdx.x] + s_sum[1][threadIdx.x]) +
                                                              (s_sum[2][threadIdx.x] + s_sum[3][threadIdx.x]);
}

// 64x64 tiles through LDS: sizes, pitches or addresses that 16-byte pieces do not fit.
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ in, int ldin, T* __restrict__ out, int ldout,
                                                        int R, int C) {
  __shared__ T tile[64][64 + 4 / sizeof(T)];             // row pitch of an odd number of 32-bit words: no bank conflicts in either pass
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = r0 + ty + 4 * i, c = c0 + tx;
    if (r < R && c < C) tile[ty + 4 * i][tx] = in[(size_t)r * ldin + c];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = c0 + ty + 4 * i, r = r0 + tx;
    if (r < R && c < C) out[(size_t)c * ldout + r] = tile[tx][ty + 4 * i];
  }
}

static void transpose_one(int prec, const TransposeJob& j, hipStream_t st) {
  const dim3 grid((j.C + 63) / 64, (j.R + 63) / 64);
  if (prec)
    hipLaunchKernelGGL(transpose_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)j.in, j.ldin, (bf16_t*)j.out, j.ldout, j.R, j.C);
  else
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, st, (const float*)j.in, j.ldin, (float*)j.out, j.ldout, j.R, j.C);
}
void launch_transpose_multi(int prec, const TransposeJob* jobs, int n, hipStream_t st) {
  const int nb = prec ? 8 : 4, tile = 8 * nb;
  TransposeJobs a;
  int m = 0, blocks = 0;
  auto go = [&]() {
    if (m == 0) return;
    for (int k = m; k < TRANSPOSE_MAX_JOBS; ++k) a.j[k] = TransposeJobD{nullptr, nullptr, nullptr, 0, 0, 0, 0, 1, 0, 0};
    if (prec) hipLaunchKernelGGL(transpose_multi_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(transpose_multi_kernel<float>, dim3(blocks), dim3(256), 0, st, a);
    m = 0; blocks = 0;
  };
  for (int k = 0; k < n; ++k) {
    const TransposeJob& j = jobs[k];
    if (j.R <= 0 || j.C <= 0) continue;
    const bool pieces = ((uintptr_t)j.in | (uintptr_t)j.out) % 16 == 0 && (j.ldin | j.ldout | j.R | j.C) % nb == 0;
    if (!pieces) {
      transpose_one(prec, j, st);
      if (j.parts) launch_colsum_parts(prec, j.in, j.ldin, j.R, j.C, j.parts, st);
      continue;
    }
    const int tiles = (j.R + tile - 1) / tile, tpb = j.parts ? (tiles + TRANSPOSE_SPLITS - 1) / TRANSPOSE_SPLITS : 4;
    const int nx = (j.C + tile - 1) / tile, ny = j.parts ? TRANSPOSE_SPLITS : (tiles + tpb - 1) / tpb;
    a.j[m++] = TransposeJobD{j.in, j.out, j.parts, j.ldin, j.ldout, j.R, j.C, nx, nx * ny, tpb};
    blocks += nx * ny;
    if (m == TRANSPOSE_MAX_JOBS) go();
  }
  go();
}

}  // namespace cmt

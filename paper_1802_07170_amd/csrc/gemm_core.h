// LDS-tiled matrix-core main loop for C = A * B^T with both operands k-contiguous (the paper's
// LinearLayer forward GEMM form; every batched-over-time contraction of the step is brought to
// this form).  WM x WN wavefronts; each wavefront owns TA x TB MFMA 32x32 tiles, so the workgroup
// tile is (32 TA WM) x (32 TB WN).  Three shapes are used:
//   * 2x2 wavefronts, one tile each: 64 x 64, 256 threads, 36 KB of LDS, four workgroups per CU (fp32 in parts 48 KB, three): for the many
//     products of a small network or batch that are a few dozen tiles of the next size, where what a launch takes is
//     the chain prologue - contraction - store of one workgroup (16 stores a lane instead of 64).
//   * 2x2 wavefronts, 2x2 tiles each: 128 x 128, 256 threads, 72 KB of LDS, two workgroups per CU
//     hiding each other's barriers (128 KB, four k tiles, where there is one per CU at most).  Needs 32 KB from L2 per 2 x 128 x 128 x 64 flops.
//   * 4x4 wavefronts, 2x2 tiles each: 256 x 256, 1024 threads, 144 KB of LDS, one workgroup per CU.
//     Half the L2 traffic per flop (64 KB per k tile): 1.3 PFLOP/s on large problems, and faster than the
//     others from about 150 tiles up.
// (fp32: the first, and 256 x 128 on 512 threads.)
// What bounds both is the rate at which a CU takes data from L2: about 49 GB/s per CU measured with the main
// loop's loads alone (12.6 TB/s over the chip), i.e. at most 1.6 PFLOP/s for the big tile and 0.8 for the small.
// Tiles of k are double-buffered in LDS (or four deep); the next tile's global loads are in
// flight while the current one feeds the matrix cores.  16-bit operands go from global memory straight
// into LDS (global_load_lds_dwordx4, no staging registers): rows of 128 bytes without padding, the
// 16-byte chunks of a row XOR-swizzled by the row number so that fragment reads stay free of bank
// conflicts (gemm_swz).  32-bit operands are staged through registers, where each becomes three bf16 numbers whose
// sum it is (gemm_mainloop_f32).
#pragma once
#include "common.h"

namespace cmt {

// T's tile shape: WM x WN wavefronts of TA x TB tiles of 32 x 32.
template <typename T, int WM_, int WN_, int TA_, int TB_> struct GemmTile {
  static constexpr int WM = WM_, WN = WN_, TA = TA_, TB = TB_;
  static constexpr int NT = 64 * WM * WN;                  // threads
  static constexpr int BM = 32 * TA * WM, BN = 32 * TB * WN;
  static constexpr int BK = 128 / (int)sizeof(T);          // k per stage
  static constexpr int ROWB = BK * (int)sizeof(T) + 16;    // row pitch of the padded LDS image
  static constexpr int STAGE_BYTES = (BM + BN) * ROWB;
  static constexpr int SPLIT_BYTES = (BM + BN) * BK * 6;   // a stage of three bf16 planes
  static constexpr int CHAIN_BYTES = 2 * STAGE_BYTES;      // of a kernel that makes fp32 products on the fp32 instructions alone
  static constexpr int SMEM_BYTES = 2 * (sizeof(T) == 4 && SPLIT_BYTES > STAGE_BYTES ? SPLIT_BYTES : STAGE_BYTES);
};
template <typename T> using GemmSmall = GemmTile<T, 2, 2, 1, 1>;                     // 64 x 64, 256 threads
template <typename T> using GemmMedium = GemmTile<T, 2, 2, 2, 2>;                    // 128 x 128, 256 threads
// 256 x 256, 1024 threads; fp32, whose three planes are one and a half times the LDS: 256 x 128, 512 threads
template <typename T> using GemmBig = GemmTile<T, 4, sizeof(T) == 2 ? 4 : 2, 2, 2>;

// Workgroup id -> output tile.  Consecutive workgroup ids go round-robin to the 8 XCDs (each with
// its own L2), so XCD x is given the contiguous range of tile numbers [x * per, (x + 1) * per); tile
// numbers run down groups of GROUP_M tile rows column by column, so that the ~32 tiles an XCD works
// on at a time form a block of GROUP_M x 8 tiles that share their A and B panels in that L2 (a strip
// of 1 x 32 tiles would pull 33 panels through L2 instead of 12).  Returns false for padding ids.  The
// launched grid must hold at least 8 * ceil(ntm * ntn / 8) workgroups.
constexpr int GEMM_GROUP_M = 4;
// tile number (in the grouped order described above) -> first row and column of the tile
__device__ __forceinline__ void gemm_tile_from_index(int id, int ntm, int ntn, int bm, int bn, int& m0, int& n0) {
  const int gsz = GEMM_GROUP_M * ntn;
  const int grp = id / gsz, rem = id - grp * gsz;
  const int first = grp * GEMM_GROUP_M;
  const int gm = min(GEMM_GROUP_M, ntm - first);
  m0 = (first + rem % gm) * bm;
  n0 = (rem / gm) * bn;
}
// workgroup id -> tile number for a launch of at least 8 * ceil(nt / 8) workgroups over nt tiles; -1 for padding ids.
// `per` comes from the tiles that exist, not from the launched grid: a launch sized for more rows than the
// device-side count leaves (ids beyond the last tile exit) still spreads its tiles evenly over the XCDs.
// `vb` = the (virtual) workgroup id: blockIdx.x, or blockIdx.x + a multiple of the grid for a workgroup that walks
// several tiles (the grid is a multiple of 8, so it stays with the tile range of its XCD).
__device__ __forceinline__ int gemm_tile_index(int nt, int vb) {
  const int per = (nt + 7) >> 3, j = vb >> 3;
  const int id = (vb & 7) * per + j;
  return (j >= per || id >= nt) ? -1 : id;
}
__device__ __forceinline__ int gemm_tile_index(int nt) { return gemm_tile_index(nt, (int)blockIdx.x); }
__device__ __forceinline__ bool gemm_tile_of_block(int ntm, int ntn, int bm, int bn, int& m0, int& n0, int vb = -1) {
  const int id = gemm_tile_index(ntm * ntn, vb < 0 ? (int)blockIdx.x : vb);
  if (id < 0) return false;
  gemm_tile_from_index(id, ntm, ntn, bm, bn, m0, n0);
  return true;
}

// Global -> register half of a tile copy.  The rows a thread fetches do not change from one k tile to the next, so
// their offsets from the tile's first element (32-bit, element units; rows beyond `rows` are clamped to the last
// one — they are never stored) are computed once (gemm_tile_offsets) and every load is "uniform base + 32-bit
// thread offset": no 64-bit per-thread addresses are kept across the main loop.
template <typename T, int NT, int ROWS, int KB>
__device__ __forceinline__ void gemm_tile_offsets(int ld, int rows, int r0, unsigned (&off)[ROWS * KB / 16 / NT]) {
  constexpr int EPC = 16 / sizeof(T);                     // elements per 16-byte chunk
  constexpr int CPR = KB / 16;                            // chunks per row
  constexpr int RPP = NT / CPR;                           // rows per pass
  const int t = threadIdx.x;
#pragma unroll
  for (int p = 0; p < ROWS / RPP; ++p) {
    int r = r0 + (t / CPR) + RPP * p;
    r = r < rows ? r : rows - 1;
    off[p] = (unsigned)(r - r0) * (unsigned)ld + (unsigned)((t % CPR) * EPC);
  }
}
// base = first element of the tile row r0 at the k tile's first column (uniform); kleft = K - k0.
template <typename T, int NT, int ROWS, int KB>
__device__ __forceinline__ void gemm_load_tile(const T* __restrict__ base, const unsigned (&off)[ROWS * KB / 16 / NT], int kleft,
                                               uint4 (&regs)[ROWS * KB / 16 / NT]) {
  constexpr int EPC = 16 / sizeof(T);
  constexpr int CPR = KB / 16;
  const bool in = (int)((threadIdx.x % CPR) * EPC) < kleft;
#pragma unroll
  for (int p = 0; p < ROWS * KB / 16 / NT; ++p) {
    if (in) regs[p] = *reinterpret_cast<const uint4*>(base + off[p]);
    else regs[p] = make_uint4(0, 0, 0, 0);
  }
}
template <int NT, int ROWS, int KB>
__device__ __forceinline__ void gemm_store_tile(char* tile, const uint4 (&regs)[ROWS * KB / 16 / NT]) {
  constexpr int CPR = KB / 16, RPP = NT / CPR;
  const int t = threadIdx.x;
#pragma unroll
  for (int p = 0; p < ROWS / RPP; ++p)
    *reinterpret_cast<uint4*>(tile + ((t / CPR) + RPP * p) * (KB + 16) + (t % CPR) * 16) = regs[p];
}

// ---- 16-bit operands: global -> LDS without staging registers ----
// LDS image of a tile: row r (128 bytes = 64 elements of k) at r * 128; the 16-byte chunk c of the row sits at
// position c ^ gemm_swz(r).  A load instruction of wavefront w writes 64 consecutive 16-byte slots (the hardware
// adds lane * 16 to the base in M0), so slot (p * NT + thread) holds row slot / 8, position slot % 8, and the
// thread fetches the chunk that belongs there.
__device__ __forceinline__ int gemm_swz(int r) { return (r ^ (r >> 3)) & 7; }

// byte offsets from the tile's first row at the k tile's first column; rows beyond `rows` clamped (never stored)
template <int NT, int ROWS>
__device__ __forceinline__ void gemm_dl_offsets(int ld, int rows, int r0, unsigned (&off)[ROWS * 8 / NT]) {
  static_assert((ROWS * 8) % NT == 0, "tile rows must fill whole passes of the workgroup");
#pragma unroll
  for (int p = 0; p < ROWS * 8 / NT; ++p) {
    const int slot = p * NT + threadIdx.x, r = slot >> 3, c = (slot & 7) ^ gemm_swz(r);
    const int row = min(r0 + r, rows - 1) - r0;
    off[p] = ((unsigned)row * (unsigned)ld + (unsigned)(c * 8)) * 2u;
  }
}
__device__ __forceinline__ unsigned gemm_lds_address(const char* p) {
  return (unsigned)(size_t)(__attribute__((address_space(3))) const char*)p;
}
// Asynchronous: completion is awaited with gemm_dl_wait() before the barrier that publishes the stage.
// The instruction is written out because the compiler, when it knows a load writes LDS, waits for every
// outstanding one before the next LDS read of any address — which would serialise the two stages.  M0 (the LDS
// base of the transfer) is a register the compiler reserves and loads directly before each use of its own, so
// setting it here disturbs nothing (it cannot be named as a clobber).
template <int NT, int ROWS>
__device__ __forceinline__ void gemm_dl_issue(const bf16_t* __restrict__ base, const unsigned (&off)[ROWS * 8 / NT], char* tile, int w) {
#pragma unroll
  for (int p = 0; p < ROWS * 8 / NT; ++p) {
    const unsigned dst = gemm_lds_address(tile) + (unsigned)((p * NT + w * 64) * 16);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off[p]), "s"(base) : "memory");
  }
}
__device__ __forceinline__ void gemm_dl_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// A k tile with fewer than 64 valid columns (the last one of a K that is no multiple of 64): through registers,
// chunks beyond K as zeros, into the same LDS image.
template <int NT, int ROWS>
__device__ __forceinline__ void gemm_dl_fill_tail(const bf16_t* __restrict__ base, const unsigned (&off)[ROWS * 8 / NT], int kleft, char* tile) {
#pragma unroll
  for (int p = 0; p < ROWS * 8 / NT; ++p) {
    const int slot = p * NT + threadIdx.x, r = slot >> 3, c = (slot & 7) ^ gemm_swz(r);
    uint4 v = make_uint4(0, 0, 0, 0);
    if (c * 8 < kleft) v = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(base) + off[p]);
    *reinterpret_cast<uint4*>(tile + slot * 16) = v;
  }
}

// At most n transfers of this wavefront are still on their way (a stage makes PER of them).
template <int PER> __device__ __forceinline__ void gemm_dl_wait_but(int stages) {
  if (stages >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
  else if (stages == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
  else gemm_dl_wait();
}
// STAGES k tiles in LDS, STAGES - 1 of them on their way while one feeds the matrix cores.
template <int WM, int WN, int TA, int TB, int STAGES>
__device__ __forceinline__ void gemm_mainloop_dl(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                                 int M, int N, int K, int m0, int n0, v16f (&acc)[TA][TB], char* smem) {
  constexpr int NT = 64 * WM * WN, BM = 32 * TA * WM, BN = 32 * TB * WN;
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128, PER = (BM + BN) * 8 / NT;
  static_assert(STAGES >= 2 && STAGES <= 4, "the waits count up to two later stages");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w / WN, wn = w % WN;
  unsigned oa[BM * 8 / NT], ob[BN * 8 / NT];
  gemm_dl_offsets<NT, BM>(lda, M, m0, oa);
  gemm_dl_offsets<NT, BN>(ldb, N, n0, ob);
  const bf16_t* __restrict__ pa = A + (size_t)m0 * lda;    // uniform: first row of the tile
  const bf16_t* __restrict__ pb = B + (size_t)n0 * ldb;
  auto fill = [&](char* stage, int k0) {
    if (K - k0 >= 64) {
      gemm_dl_issue<NT, BM>(pa + k0, oa, stage, w);
      gemm_dl_issue<NT, BN>(pb + k0, ob, stage + A_BYTES, w);
    } else {
      gemm_dl_fill_tail<NT, BM>(pa + k0, oa, K - k0, stage);
      gemm_dl_fill_tail<NT, BN>(pb + k0, ob, K - k0, stage + A_BYTES);
    }
  };
  // fragment of row r at k step ks: chunk 2 ks + lane / 32, at position chunk ^ gemm_swz(r)
  int fa_row[TA], fa_s[TA], fb_row[TB], fb_s[TB];
#pragma unroll
  for (int x = 0; x < TA; ++x) { const int r = (wm * TA + x) * 32 + (lane & 31); fa_row[x] = r * 128; fa_s[x] = gemm_swz(r) ^ (lane >> 5); }
#pragma unroll
  for (int x = 0; x < TB; ++x) { const int r = (wn * TB + x) * 32 + (lane & 31); fb_row[x] = A_BYTES + r * 128; fb_s[x] = gemm_swz(r) ^ (lane >> 5); }
  auto products = [&](const char* cur) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      Frag<bf16_t> fa[TA], fb[TB];
#pragma unroll
      for (int x = 0; x < TA; ++x) fa[x].load(reinterpret_cast<const bf16_t*>(cur + fa_row[x] + ((fa_s[x] ^ (2 * ks)) << 4)));
#pragma unroll
      for (int x = 0; x < TB; ++x) fb[x].load(reinterpret_cast<const bf16_t*>(cur + fb_row[x] + ((fb_s[x] ^ (2 * ks)) << 4)));
#pragma unroll
      for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) mma32(acc[a][b], fa[a], fb[b]);
    }
  };
  const int nk = (K + 63) / 64;
  if constexpr (STAGES == 2) {
    fill(smem, 0);
    gemm_dl_wait();
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      if (kt + 1 < nk) fill(smem + ((kt + 1) & 1) * STAGE, (kt + 1) * 64);
      products(smem + (kt & 1) * STAGE);
      gemm_dl_wait();
      __syncthreads();
    }
  } else {
    const int whole = K / 64;                              // (a last part of a k tile goes through registers: nothing of it is on its way)
    int in = 0, out = 0;                                   // stage buffers
#pragma unroll
    for (int i = 0; i < STAGES - 1; ++i)
      if (i < nk) fill(smem + i * STAGE, i * 64);
    in = STAGES - 1;
    for (int kt = 0; kt < nk; ++kt) {
      gemm_dl_wait_but<PER>(min(STAGES - 2, whole - 1 - kt));
      __syncthreads();                                     // every wavefront's share is there, and the last stage read is free
      if (kt + STAGES - 1 < nk) fill(smem + in * STAGE, (kt + STAGES - 1) * 64);
      products(smem + out * STAGE);
      in = in + 1 == STAGES ? 0 : in + 1;
      out = out + 1 == STAGES ? 0 : out + 1;
    }
    __syncthreads();
  }
}

// ---- 32-bit operands ----
// fp32 products on the bf16 matrix cores, which are 16 times as fast: x = h + m + l with h = bf16(x), m = bf16(x - h), l = x - h - m,
// all three bf16 and (round to nearest, 3 x 8 significant bits and their signs) without a remainder, so that
// a b = ha hb + (ha mb + ma hb) + (ha lb + la hb + ma mb) + what is below 2^-25 of |a b| and of either sign.  Six products of bf16
// instead of one of fp32: 2.7 times the rate.  Error against 64 bits, relative (fp32 instructions | split): 3200 x 2048, k 512 4.0e-7 |
// 1.1e-7; k 3200 4.6e-7 | 1.9e-7; gradients of 32 shapes of training steps 0.40 - 1.00 times as far off as they were.  REST: the five small
// products go into a sum of their own.  In one sum with ha hb they are lost where that has grown large - and together, as what is
// lost is much the same for every row of a coherent operand (bias gradients up to 2.6 times as far off).
// Range: operands are split at 2^16 times their size, where the last bit that any of them can have, 2^-149, is the least bf16, 2^-133
// (conversions and products keep subnormal numbers; at their own size parts were cut off below 2^-110).  From 0x1.ffp111 up h is infinite, and sums
// from 2^96 up can be: a tile with a sum that is infinite or NaN is made again on the fp32 instructions.  That costs nothing: the factor
// goes into what blanks out k beyond the last, and the sums are looked at once (small_step 5.17 -> 5.14 ms; the operands' magnitudes were looked at before).
// It is bound by power as much as by instructions: 8192 x 8192, k 4096 128 TFLOP/s with fp32 instructions, 206 with the split
// (1.24 PFLOP/s of bf16) at 1.8 GHz with the matrix cores busy 70 % of the time; k 512, 3200 x 2048 82 | 51 us.
//
// LDS image of a stage, per operand and plane: blocks of 32 rows x 16 k as the matrix cores take them, 1 KB [k half][row][8], rows
// permuted by the k chunk so that neither the 8-byte stores (a quad of k of one row) nor the fragment reads meet bank conflicts.
template <int BK> __device__ __forceinline__ int gemm_split_at(int r, int c /* chunk of 8 k */) {
  return ((r >> 5) * (BK / 16) + (c >> 1)) * 1024 + (c & 1) * 512 + ((r & 31) ^ (c * (64 / BK))) * 16;
}
constexpr float GEMM_SPLIT_SCALE = 0x1p16f;
struct GemmSplit2 { uint32_t h, m, l; };
__device__ __forceinline__ GemmSplit2 gemm_split2(float x, float y) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  GemmSplit2 s;
  s.h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
  x -= __uint_as_float(s.h << 16); y -= __uint_as_float(s.h & 0xffff0000u);
  s.m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
  x -= __uint_as_float(s.m << 16); y -= __uint_as_float(s.m & 0xffff0000u);
  s.l = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
  return s;
}
// A quad of k of row r, chunk half c (4 k each) -> the three planes of a tile of ROWS rows.
template <int ROWS, int BK>
__device__ __forceinline__ void gemm_split_store(char* tile, int r, int c, const float4& x) {
  constexpr int PLANE = ROWS * BK * 2;
  const GemmSplit2 a = gemm_split2(x.x, x.y), b = gemm_split2(x.z, x.w);
  char* const at = tile + gemm_split_at<BK>(r, c >> 1) + (c & 1) * 8;
  *reinterpret_cast<uint2*>(at) = make_uint2(a.h, b.h);
  *reinterpret_cast<uint2*>(at + PLANE) = make_uint2(a.m, b.m);
  *reinterpret_cast<uint2*>(at + 2 * PLANE) = make_uint2(a.l, b.l);
}
// A thread's pieces of a stage (16 bytes of one row each, first A's, then B's) are asked for two stages ahead and split one stage
// ahead, piece by piece between the matrix instructions: those take 32 clocks each, the splitting of a piece some 27 others.
// false: the sums are to be made by gemm_mainloop_regs.
template <int WM, int WN, int TA, int TB, bool REST>
__device__ __forceinline__ bool gemm_mainloop_f32(const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
                                                  int M, int N, int K, int m0, int n0, v16f (&acc)[TA][TB], char* smem) {
  using G = GemmTile<float, WM, WN, TA, TB>;
  constexpr int NT = G::NT, BK = G::BK, CPR = BK / 4, RPP = NT / CPR, NA = G::BM / RPP, NP = NA + G::BN / RPP;
  constexpr int A_PLANE = G::BM * BK * 2, B_PLANE = G::BN * BK * 2, STEPS = BK / 16 * 6;
  if (K <= 0) return true;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wm = w / WN, wn = w % WN, pr = threadIdx.x / CPR, pc = threadIdx.x % CPR;
  unsigned off[NP];                                        // of the pieces' rows (rows beyond the last: the last, never stored)
#pragma unroll
  for (int p = 0; p < NP; ++p)
    off[p] = p < NA ? (unsigned)(min(m0 + pr + RPP * p, M - 1) - m0) * (unsigned)lda : (unsigned)(min(n0 + pr + RPP * (p - NA), N - 1) - n0) * (unsigned)ldb;
  const float* __restrict__ pa = A + (size_t)m0 * lda;
  const float* __restrict__ pb = B + (size_t)n0 * ldb;
  float4 x[NP];
  auto load = [&](int p, int kt) {                         // (k beyond the last: the last, made zero when it is split)
    const unsigned k = (unsigned)min(kt * BK + 4 * pc, K - 4);
    x[p] = *reinterpret_cast<const float4*>((p < NA ? pa : pb) + (off[p] + k));
  };
  v16f rest[TA][TB];
  constexpr float SCALE2 = GEMM_SPLIT_SCALE * GEMM_SPLIT_SCALE;
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) { acc[a][b][i] *= SCALE2; rest[a][b][i] = 0.f; }   // (REST)
  auto store = [&](char* stage, int p, int kt) {
    const float s = kt * BK + 4 * pc < K ? GEMM_SPLIT_SCALE : 0.f;
    const float4 v = make_float4(s * x[p].x, s * x[p].y, s * x[p].z, s * x[p].w);
    if (p < NA) gemm_split_store<G::BM, BK>(stage, pr + RPP * p, pc, v);
    else gemm_split_store<G::BN, BK>(stage + 3 * A_PLANE, pr + RPP * (p - NA), pc, v);
  };
#pragma unroll
  for (int p = 0; p < NP; ++p) load(p, 0);
#pragma unroll
  for (int p = 0; p < NP; ++p) { store(smem, p, 0); load(p, 1); }
  __syncthreads();
  const int nk = (K + BK - 1) / BK;
  for (int kt = 0; kt < nk; ++kt) {
    const char* cur = smem + (kt & 1) * G::SPLIT_BYTES;
    char* nxt = smem + ((kt + 1) & 1) * G::SPLIT_BYTES;
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      Frag<bf16_t> fa[TA][3], fb[TB][3];
      const int at = gemm_split_at<BK>(lane & 31, 2 * ks + (lane >> 5));
#pragma unroll
      for (int p = 2; p >= 0; --p) {
#pragma unroll
        for (int a = 0; a < TA; ++a) fa[a][p].load(reinterpret_cast<const bf16_t*>(cur + p * A_PLANE + (wm * TA + a) * (BK / 16) * 1024 + at));
#pragma unroll
        for (int b = 0; b < TB; ++b) fb[b][p].load(reinterpret_cast<const bf16_t*>(cur + 3 * A_PLANE + p * B_PLANE + (wn * TB + b) * (BK / 16) * 1024 + at));
      }
      // the small products first
      constexpr int PA[6] = {0, 1, 2, 0, 1, 0}, PB[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
          for (int b = 0; b < TB; ++b) mma32(q == 5 || !REST ? acc[a][b] : rest[a][b], fa[a][PA[q]], fb[b][PB[q]]);
        // the pieces of this part of the stage
#pragma unroll
        for (int p = NP * (ks * 6 + q) / STEPS; p < NP * (ks * 6 + q + 1) / STEPS; ++p) {
          store(nxt, p, kt + 1);
          load(p, kt + 2);
        }
      }
      __builtin_amdgcn_sched_barrier(0x108);               // (fragment reads and matrix instructions may cross)
    }
    __syncthreads();
  }
  float zero = 0.f;                                        // (NaN as soon as one of the sums is not finite)
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (REST) acc[a][b][i] += rest[a][b][i];
        zero = fmaf(acc[a][b][i], 0.f, zero);
        acc[a][b][i] *= 1.f / SCALE2;
      }
  return !__syncthreads_or(!(zero == 0.f));
}

// fp32 on the fp32 matrix cores.
template <int WM, int WN, int TA, int TB>
__device__ __forceinline__ void gemm_mainloop_regs(const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
                                                   int M, int N, int K, int m0, int n0, v16f (&acc)[TA][TB], char* smem) {
  typedef float T;
  using G = GemmTile<T, WM, WN, TA, TB>;
  constexpr int NT = G::NT, BK = G::BK, KB = 4 * BK, GEMM_ROWB = G::ROWB, A_BYTES = G::BM * G::ROWB;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wm = w / WN, wn = w % WN;
  uint4 ra[G::BM * KB / 16 / NT], rb[G::BN * KB / 16 / NT];
  unsigned oa[G::BM * KB / 16 / NT], ob[G::BN * KB / 16 / NT];
  gemm_tile_offsets<T, NT, G::BM, KB>(lda, M, m0, oa);
  gemm_tile_offsets<T, NT, G::BN, KB>(ldb, N, n0, ob);
  const T* __restrict__ pa = A + (size_t)m0 * lda;        // uniform: first row of the tile
  const T* __restrict__ pb = B + (size_t)n0 * ldb;
  gemm_load_tile<T, NT, G::BM, KB>(pa, oa, K, ra);
  gemm_load_tile<T, NT, G::BN, KB>(pb, ob, K, rb);
  gemm_store_tile<NT, G::BM, KB>(smem, ra);
  gemm_store_tile<NT, G::BN, KB>(smem + A_BYTES, rb);
  __syncthreads();
  const int nk = (K + BK - 1) / BK;
  for (int kt = 0; kt < nk; ++kt) {
    char* cur = smem + (kt & 1) * G::STAGE_BYTES;
    char* nxt = smem + ((kt + 1) & 1) * G::STAGE_BYTES;
    const bool more = kt + 1 < nk;
    if (more) {
      gemm_load_tile<T, NT, G::BM, KB>(pa + (kt + 1) * BK, oa, K - (kt + 1) * BK, ra);
      gemm_load_tile<T, NT, G::BN, KB>(pb + (kt + 1) * BK, ob, K - (kt + 1) * BK, rb);
    }
    const char* ta = cur + (wm * 32 * TA + (lane & 31)) * GEMM_ROWB + (lane >> 5) * 8 * sizeof(T);
    const char* tb = cur + A_BYTES + (wn * 32 * TB + (lane & 31)) * GEMM_ROWB + (lane >> 5) * 8 * sizeof(T);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      Frag<T> fa[TA], fb[TB];
#pragma unroll
      for (int x = 0; x < TA; ++x) fa[x].load(reinterpret_cast<const T*>(ta + x * 32 * GEMM_ROWB + ks * 16 * sizeof(T)));
#pragma unroll
      for (int x = 0; x < TB; ++x) fb[x].load(reinterpret_cast<const T*>(tb + x * 32 * GEMM_ROWB + ks * 16 * sizeof(T)));
#pragma unroll
      for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) mma32(acc[a][b], fa[a], fb[b]);
    }
    if (more) {
      gemm_store_tile<NT, G::BM, KB>(nxt, ra);
      gemm_store_tile<NT, G::BN, KB>(nxt + A_BYTES, rb);
    }
    __syncthreads();
  }
}

// With w = wavefront index, wm = w / WN, wn = w % WN:
// acc[a][b]: rows m0 + (wm*TA + a)*32 + acc32_row(lane,i), cols n0 + (wn*TB + b)*32 + lane%32
// init(acc) sets what the products are added to (zeros, or e.g. a bias).  
// FORM, of fp32: split with the small products in a sum of their own; all products in one sum; fp32 instructions.
enum { GEMM_F32_SPLIT = 0, GEMM_F32_ONE_SUM = 1, GEMM_F32_CHAIN = 2 };
template <typename T, int WM, int WN, int TA, int TB, int FORM = 0, int STAGES = 2, typename Init>
__device__ __forceinline__ void gemm_mainloop(const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
                                              int M, int N, int K, int m0, int n0, v16f (&acc)[TA][TB], char* smem, Init init) {
  init(acc);
  if constexpr (sizeof(T) == 2) gemm_mainloop_dl<WM, WN, TA, TB, STAGES>(A, lda, B, ldb, M, N, K, m0, n0, acc, smem);
  else if constexpr (FORM == GEMM_F32_CHAIN) gemm_mainloop_regs<WM, WN, TA, TB>(A, lda, B, ldb, M, N, K, m0, n0, acc, smem);
  else if (!gemm_mainloop_f32<WM, WN, TA, TB, FORM != GEMM_F32_ONE_SUM>(A, lda, B, ldb, M, N, K, m0, n0, acc, smem)) {
    init(acc);
    gemm_mainloop_regs<WM, WN, TA, TB>(A, lda, B, ldb, M, N, K, m0, n0, acc, smem);
  }
}
struct GemmZero {
  template <int TA, int TB> __device__ __forceinline__ void operator()(v16f (&acc)[TA][TB]) const {
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
  }
};

}  // namespace cmt

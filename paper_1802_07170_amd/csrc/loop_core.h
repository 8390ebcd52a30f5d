// What the two directions of the decoder's whole loop share (loop.hip).
#pragma once
#include "kernels.h"
#include "recur_core.h"
#include "recur_plan.h"

namespace cmt {

constexpr int LOOP_WAVES = 8;                          // wavefronts of a workgroup: the k slices of its contractions
constexpr int LOOP_QT = 16;                            // source positions per thread in the mix: 8 threads and more per sentence

// Fragments at x + off(i) bytes (x uniform; each lane has its own 16 or 32 bytes there), in two steps: loop_issue requests them
// through the caches; loop_settle waits for them and, while a piece is still empty, reads it again from memory - only what
// is still empty: a wavefront takes up to 16 KB per phase here, and reading all of it because one piece is late would make
// the others late.
template <typename T, int N, typename Off>
__device__ __forceinline__ void loop_issue(const T* x, Off off, Frag<T> (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) f[i].load(reinterpret_cast<const T*>(reinterpret_cast<const char*>(x) + off(i, 0u)));
}
template <typename T, int N, typename Off>
__device__ __forceinline__ void loop_settle(const T* x, Off off, Frag<T> (&f)[N], bool& dead, int* gave_up, int wait_ticks) {
  unsigned top = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) top = max(top, recur_top(f[i]));
  if (dead || !__any(top == RECUR_EMPTY)) return;
  long long t_end = 0;
  for (int spin = 0;; ++spin) {
    unsigned zero = 0;
    asm volatile("" : "+v"(zero));                     // (the addresses are worked out again: not kept for this path)
    bool again = false;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (__any(recur_top(f[i]) == RECUR_EMPTY)) {
        unsigned t = 0;
        recur_load(reinterpret_cast<const T*>(reinterpret_cast<const char*>(x) + off(i, zero)), f[i], t);
        again = true;
      }
    if (!again) return;
    if ((spin & 15) == 15) {
      const long long now = wall_clock64();
      if (t_end == 0) t_end = now + wait_ticks;
      else if (now > t_end || __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        dead = true;
        if ((threadIdx.x & 63) == 0) atomicOr(gave_up, 1);
        return;
      }
    }
  }
}
// Where the fragments of tiles t0 .. t0 + BT - 1 of a slot lie, k steps w, w + 8, ... (tiles `tile` bytes apart, ns steps long);
// what is beyond the last step or tile repeats it: the weights are zero there, and those tiles' sums are not used.
template <typename T, int BT>
__device__ __forceinline__ unsigned loop_frag_at(int i, unsigned zero, unsigned tile, int ns, int H, int w, int t0, int nbt, int lane) {
  const int q = i / BT, t = i - q * BT, s = min(w + LOOP_WAVES * q, ns - 1);
  unsigned at = (unsigned)lane * (8u * sizeof(T)) + zero;
  // the upper half of the last step of a width that is no multiple of 32 is never written: those lanes read what the lower
  // ones do
  if ((H & 31) != 0 && s == ns - 1) at &= 32u * 8u * sizeof(T) - 1u;
  return at + (unsigned)min(t0 + t, nbt - 1) * tile + (unsigned)s * (512u * sizeof(T));
}
// A barrier for what goes through LDS alone (__syncthreads would wait for every store to memory).
__device__ __forceinline__ void loop_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Words of a slot, one per lane and item q, at p + q * stride + off bytes (p and stride uniform) where first + q * step < n, in
// the same two steps.  cached: through the caches at first.
template <int N>
__device__ __forceinline__ void loop_words_issue(const float* p, unsigned stride, unsigned off, int first, int step, int n, float (&v)[N], bool cached) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const char* at = (const char*)p + (size_t)(i * stride);
    v[i] = 0.f;
    if (first + i * step < n)
      v[i] = cached ? *(const float*)(at + off) : __hip_atomic_load((const float*)(at + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
template <int N>
__device__ __forceinline__ void loop_words_settle(const float* p, unsigned stride, unsigned off, float (&v)[N], bool& dead, int* gave_up, int wait_ticks) {
  unsigned top = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) top = max(top, __float_as_uint(v[i]));
  if (dead || !__any(top == RECUR_EMPTY)) return;
  long long t_end = 0;
  for (int spin = 0;; ++spin) {
    top = 0;
    asm volatile("" : "+v"(off));                      // (the addresses are worked out again: not kept for this path)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (__float_as_uint(v[i]) == RECUR_EMPTY)
        v[i] = __hip_atomic_load((const float*)((const char*)p + (size_t)(i * stride) + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < N; ++i) top = max(top, __float_as_uint(v[i]));
    if (!__any(top == RECUR_EMPTY)) return;
    if ((spin & 15) == 15) {
      const long long now = wall_clock64();
      if (t_end == 0) t_end = now + wait_ticks;
      else if (now > t_end || __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        dead = true;
        if ((threadIdx.x & 63) == 0) atomicOr(gave_up, 1);
        return;
      }
    }
  }
}
// what goes into a slot is never the empty pattern
__device__ __forceinline__ float loop_word(float v) { return v != v ? __uint_as_float(0x7fc00000u) : v; }
__device__ __forceinline__ void loop_put(float* p, float v) { __hip_atomic_store(p, loop_word(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The four values of a quad of lanes (units u .. u + 3 of one sentence, one per lane) to a slot at element `at` of the first,
// and to a row-major copy (may be null).
__device__ __forceinline__ void loop_quad_put(bf16_t* slot, size_t at, bf16_t* row, size_t row_at, float v, int lane, bool send) {
  const bf16_t h = f2bf(loop_word(v));
  const unsigned p = quad_pair(h), p2 = __builtin_amdgcn_mov_dpp(p, 0x4e, 0xf, 0xf, true);
  if ((lane & 3) == 0) {
    const uint64_t w = (uint64_t)p | ((uint64_t)p2 << 32);
    if (send) __hip_atomic_store(reinterpret_cast<uint64_t*>(slot + at), w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (row) *reinterpret_cast<uint64_t*>(row + row_at) = w;
  }
}
__device__ __forceinline__ void loop_quad_put(float* slot, size_t at, float* row, size_t row_at, float v, int lane, bool send) {
  const float h = loop_word(v);
  if (send) __hip_atomic_store(slot + at + (lane & 3), h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (row) row[row_at + (lane & 3)] = h;
}

// Reductions over groups of 8, 16 or 32 neighbouring lanes, the result in all of them.
template <int CTRL> __device__ __forceinline__ float loop_dpp(float v) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <typename Op> __device__ __forceinline__ float loop_group(float v, int lanes, Op op) {
  v = op(v, loop_dpp<0xb1>(v));
  v = op(v, loop_dpp<0x4e>(v));
  v = op(v, loop_dpp<0x141>(v));                       // (mirrored: the quads hold one value each by now)
  if (lanes > 8) v = op(v, loop_dpp<0x140>(v));
  if (lanes > 16) v = op(v, __shfl_xor(v, 16, 64));
  return v;
}

// the sum over the wavefront, in all lanes
__device__ __forceinline__ float loop_wave_sum(float v) {
  v += loop_dpp<0xb1>(v);
  v += loop_dpp<0x4e>(v);
  v += loop_dpp<0x141>(v);
  v += loop_dpp<0x140>(v);
  const int i = (int)__float_as_uint(v);
  return (__uint_as_float(__builtin_amdgcn_readlane(i, 0)) + __uint_as_float(__builtin_amdgcn_readlane(i, 16))) +
         (__uint_as_float(__builtin_amdgcn_readlane(i, 32)) + __uint_as_float(__builtin_amdgcn_readlane(i, 48)));
}

// A pointer that came out of the kernel's arguments, known to be global memory.
template <typename P> __device__ __forceinline__ P* loop_global(P* p) { return (P*)(__attribute__((address_space(1))) P*)p; }
// The kernel's first argument, read again from where it is used: the loop's description does not fit the scalar registers.
template <typename A> __device__ __forceinline__ const __attribute__((address_space(4))) A* loop_args() {
  auto p = (const __attribute__((address_space(4))) A*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}
// (per-lane addresses are worked out where they are used, too: kept from one position to the next they would take the
// registers that the weights need)
#define LOOP_FRESH(x) asm volatile("" : "+v"(x))
// (a phase's exchanged operands are asked for behind everything before them: mixed by the compiler with the rows that were to be
// under way first, an evaluation of 64 sentences, 4 layers of 1024, takes 2020 instead of 2010 us)
#define LOOP_PHASE() __builtin_amdgcn_sched_barrier(0)

// Where a lane's partial sums of (sentence, rows 4 q .. 4 q + 3 of a tile) lie, in units of 16 bytes: written with 16
// sentences, read with 4 rows groups in neighbouring lanes, both without bank conflicts.
__device__ __forceinline__ int loop_pos(int sentence, int q) { return q * 16 + (sentence ^ (4 * q)); }

// Place of a workgroup: its group of sentences and its four units within the group.  The hardware deals workgroups round
// robin to the 8 XCDs: the workgroups of a group go to as few of them as hold it, and neighbouring units to one XCD, so that
// what they store next to each other in memory meets in one L2.
struct LoopPlace { int group, pos; };
__device__ __forceinline__ LoopPlace loop_place(int blk, int ngroups, int nwg) {
  LoopPlace p;
  if ((ngroups & (ngroups - 1)) == 0) { p.group = blk & (ngroups - 1); p.pos = blk >> __builtin_ctz(ngroups); }
  else { p.group = blk / nwg; p.pos = blk - p.group * nwg; }
  const int xcds = ngroups == 1 ? 8 : ngroups == 2 ? 4 : ngroups == 4 ? 2 : 1;
  if (xcds > 1 && nwg % xcds == 0) p.pos = (p.pos & (xcds - 1)) * (nwg / xcds) + p.pos / xcds;
  return p;
}

}  // namespace cmt

// What the kernels that run a whole recurrence in one launch share (recur.hip, loop.hip): the reads of the slots their
// workgroups exchange states through, and the cells.
#pragma once
#include "cell.h"
#include "common.h"

namespace cmt {

constexpr unsigned RECUR_EMPTY = 0xffffffffu;          // a word of a slot that nobody has written
constexpr int RECUR_WAIT_TICKS = 5000000;              // 50 ms of the 100 MHz wall clock, then a wait is given up

// one 16-byte (32-byte for float) fragment of a slot; `top` becomes RECUR_EMPTY if any of its pieces is still empty
__device__ __forceinline__ void recur_load(const bf16_t* p, Frag<bf16_t>& f, unsigned& top) {
  const uint64_t a = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t b = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  f.v = make_uint4((unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32));
  top = max(top, max(f.v.x, f.v.z));                   // pieces of 8 bytes are written whole
}
__device__ __forceinline__ void recur_load(const float* p, Frag<float>& f, unsigned& top) {
  uint64_t v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  unsigned w[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) { w[2 * i] = (unsigned)v[i]; w[2 * i + 1] = (unsigned)(v[i] >> 32); }
#pragma unroll
  for (int i = 0; i < 8; ++i) top = max(top, w[i]);    // pieces of 4 bytes
  f.lo = make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), __uint_as_float(w[3]));
  f.hi = make_float4(__uint_as_float(w[4]), __uint_as_float(w[5]), __uint_as_float(w[6]), __uint_as_float(w[7]));
}

// this lane's 16-bit value and its neighbour's (lane ^ 1), the even lane's in the lower half of the even lane's result
__device__ __forceinline__ unsigned quad_pair(bf16_t v) {
  return (unsigned)v | ((unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true) << 16);
}


__device__ __forceinline__ unsigned recur_top(const Frag<bf16_t>& f) { return max(f.v.x, f.v.z); }
__device__ __forceinline__ unsigned recur_top(const Frag<float>& f) {
  unsigned t = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) t = max(t, __float_as_uint(f.get(i)));
  return t;
}
// N fragments of a slot, each at a uniform base p[i] plus this lane's offset; in[i]: whether this lane has a part in it
// (else zero).  First through the caches, which usually finds everything there (the wavefront has slept for about the
// time that a store takes to be visible); while any piece is still empty, again from memory.  `dead`: this workgroup or
// another one of the launch has given up (*gave_up), take what there is.
template <typename T, int N>
__device__ __forceinline__ void recur_issue(const T* const (&p)[N], const bool (&in)[N], unsigned off, Frag<T> (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    f[i].zero();
    if (in[i]) f[i].load(p[i] + off);
  }
}
template <typename T, int N>
__device__ __forceinline__ void recur_settle(const T* const (&p)[N], const bool (&in)[N], unsigned off, Frag<T> (&f)[N], bool& dead,
                                             int* gave_up, int wait_ticks) {
  unsigned top = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) top = max(top, recur_top(f[i]));
  if (dead || !__any(top == RECUR_EMPTY)) return;
  long long t_end = 0;
  for (int spin = 0;; ++spin) {
    top = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (in[i]) recur_load(p[i] + off, f[i], top);
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
// For the launch behind one whose waits may have been given up (null: behind none): whether there is anything to do, and if so it
// is counted.
__device__ __forceinline__ bool recur_again(const int* gave_up, int* again) {
  if (!gave_up) return true;
  if (*gave_up == 0) return false;
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(again, 1);
  return true;
}
// about n * 64 clocks
__device__ __forceinline__ void recur_nap(int n) { for (int z = 0; z < n; ++z) __builtin_amdgcn_s_sleep(1); }


// 4 x 4 transpose of 16-bit values over the lanes of a quad: lane j of the quad brings gates 0..3 of its unit and receives
// gate j of the quad's four units.
__device__ __forceinline__ uint64_t quad_transpose(bf16_t g0, bf16_t g1, bf16_t g2, bf16_t g3, int lane) {
  const unsigned a = (unsigned)g0 | ((unsigned)g1 << 16), b = (unsigned)g2 | ((unsigned)g3 << 16);
  const unsigned ax = __builtin_amdgcn_mov_dpp((int)a, 0xb1, 0xf, 0xf, true), bx = __builtin_amdgcn_mov_dpp((int)b, 0xb1, 0xf, 0xf, true);
  // after the exchange with lane ^ 1: an even lane holds gates 0 and 2 of the pair's two units, an odd one gates 1 and 3
  const bool odd = lane & 1;
  const unsigned p = odd ? (ax >> 16) | (a & 0xffff0000u) : (a & 0xffffu) | (ax << 16);
  const unsigned q = odd ? (bx >> 16) | (b & 0xffff0000u) : (b & 0xffffu) | (bx << 16);
  // after the exchange with lane ^ 2: lanes 0, 1 of the quad hold gates 0, 1 of all four units, lanes 2, 3 gates 2, 3
  const bool high = lane & 2;
  const unsigned px = __builtin_amdgcn_mov_dpp((int)p, 0x4e, 0xf, 0xf, true), qx = __builtin_amdgcn_mov_dpp((int)q, 0x4e, 0xf, 0xf, true);
  return high ? (uint64_t)qx | ((uint64_t)q << 32) : (uint64_t)p | ((uint64_t)px << 32);
}


// The cell of one sentence and unit: recurrent part `pre` and input part `gx` of its four gates, cell state c (in and out), h
// = the stored state that a masked step carries on.  Returns the new state as computed, NaN in its canonical form.
template <bool FAST>
__device__ __forceinline__ float seq_cell(const v4f& pre, const float (&gx)[4], float mask, float h, float& c, float (&g)[4]) {
  g[0] = sigm_of<FAST>(pre[0] + gx[0]);
  g[1] = sigm_of<FAST>(pre[1] + gx[1]);
  g[2] = tanh_of<FAST>(pre[2] + gx[2]);
  g[3] = sigm_of<FAST>(pre[3] + gx[3]);
  const float cn = g[1] * c + g[0] * g[2];
  const float hn = g[3] * tanh_of<FAST>(cn);
  if (!(mask > 0.f)) return h;
  c = cn;
  return hn != hn ? __uint_as_float(0x7fc00000u) : hn;
}
// Its backward: gate activations g, the cell state before (cp) and the tanh of the one after (tc), the gradient dy at its
// output and the recurrent part rec; dh, dc = the state's gradients that pass by (in and out), o = the gate gradients.
__device__ __forceinline__ void seq_cell_bwd(const float (&g)[4], float cp, float tc, float dy, float rec, float mask, float& dh, float& dc,
                                             float (&o)[4]) {
  const bool valid = mask > 0.f;
  const float ig = g[0], fg = g[1], gg = g[2], og = g[3];
  const float state = dh + rec;
  const float dht = state + dy;
  const float dct = dc + dht * og * (1.f - tc * tc);
  o[0] = dct * gg * ig * (1.f - ig);
  o[1] = dct * cp * fg * (1.f - fg);
  o[2] = dct * ig * (1.f - gg * gg);
  o[3] = dht * tc * og * (1.f - og);
  dh = valid ? 0.f : state;                                        // masked: the state's gradient passes through
  dc = valid ? dct * fg : dc;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    o[q] = valid ? o[q] : 0.f;
    if (o[q] != o[q]) o[q] = __uint_as_float(0x7fc00000u);
  }
}

}  // namespace cmt

// Whole recurrences in one launch: the time loop of an LSTM layer whose input part is batched over time (both
// directions of the bottom encoder layer, the upper encoder layers), run by workgroups that stay on the chip for all
// positions and keep their share of the recurrent weights in registers.
//
// Sentences do not interact, so a launch is a set of independent groups: one group = one (layer, direction) on 16 BT
// sentences, its hidden units spread over the group's workgroups.  What a position must exchange is the new state (backward:
// the gate gradients) of the group's sentences: every workgroup needs all units of the previous position.  It travels
// through device memory, in the fragment-major layout the matrix cores take, one slot per position:
//   * a slot is filled with 0xff bytes before the launch and written once, by 8-byte (fp32: 4-byte) agent-scope stores,
//     which go to memory; the data never contains that bit pattern (NaNs are made canonical), so a reader that finds it
//     reads again.  The data is its own flag: one store and one load per position, no fence, barrier or counter;
//   * a reader first loads through its caches (a line that another workgroup of the same L2 has fetched complete is
//     complete for good: nothing in a slot is written twice) and, where it finds something empty, again from memory
//     with agent-scope loads.  It sleeps for about the time that a store takes to be visible before it looks: looking
//     earlier costs more than it gains, since the reads then stand in the way of the stores they wait for.
// Roles are taken from a ticket counter, in order of arrival, so that the workgroups on the chip always form complete
// groups and at most one incomplete one per launch.  Groups have at most 64 workgroups (recur_plan.h), so the four launches
// that a process's hardware queues can run at once leave a CU free, nearly always for one of them to complete its group.  Nothing rests on
// that but speed: more queues, other processes or a stream confined to a few CUs may stop a group from forming as well.  Every wait
// is bounded, a workgroup that gives up says so and finishes without waiting, the others of the launch follow, and a second
// launch (2 - 4 us of a step where there is nothing to do) makes the recurrence again without waits, one workgroup per 16 sentences:
// 0.4 ms a position at width 1024.  That form also serves devices too small for the groups.
//
// What a position costs within a training step (bf16, us; a launch per position cost 8.5 - 9, upper layers forward 5.6 of a
// shared one).  Forward: width 256 x two directions, 32 sentences 1.2; 512, 32 sentences 1.4; 512 x two directions, 64 and 128
// sentences 1.6 and 3.4; 1024, 64 and 128 sentences 2.1 and 4.7.  Backward, beside the second stream's GEMMs: 256 x two
// directions, 32 sentences 2.0; 512, 32 sentences 2.5; 512 x two directions, 64 and 128 sentences 3.6 and 4.0; 1024, 64
// sentences 3.6 - 5.3 (median 3.7), 128 sentences 4.0 - 12 (median 4.7; the first of a step's layers, which runs beside the decoder's
// weight gradients, takes longest).  About 0.5 of it is the store on its way to memory, 0.5 the load, the rest contraction,
// reduction and cell; at 128 sentences also the volume.
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "cell.h"
#include "common.h"
#include "kernels.h"
#include "recur_core.h"
#include "recur_plan.h"

namespace cmt {

// s_sleep units (64 clocks) before a workgroup looks for its neighbours' results.  They come the later the more bytes of state
// a workgroup has to read and multiply, and a look that comes too early fetches lines that it has to fetch again.  Whole passes
// over 150 positions x 3 layers, us, with 16 | 20 | 24 | 28 | 36 units forward (evaluation; bf16, 64 sentences): hidden size 64
// 581 | 624 | 658 | 715 | 800, 128 654 | 663 | 711 | 764 | 855, 512 1208 | 1041 | 963 | 996 | 1087, 1024 1871 | 1814 | 1745 | 1595 | 1492; fp32, 64
// (8 sentences) 1023 | 909 | 889 | 918 | 1013, 512 3054 | 2988 | 2739 | 2493 | 2541; two tiles of sentences (128), 512 1565 | 1409 | 1316 | 1261 | 1292,
// 1024 3870 | 3510 | 3373 | 3393 | 2933.  24 | 36 | 42 | 50 units backward (training step): 64 1475 | 1598 | 1675 | 1786, 256 (32
// sentences) 1925 | 1762 | 1822 | 1923, 512 3285 | 3039 | 2901 | 2913, 1024 5439 | 5054 | 4869 | 4847.  The lines below follow these minima.
static int recur_nap_fwd(int elem, int bt, int Hh) { return elem * bt == 2 ? 16 + std::min(Hh, 1024) * 20 / 1024 : 20 + std::min(Hh, 1024) * 16 / 1024; }
static int recur_nap_bwd(int Hh) { return 24 + std::min(Hh, 512) * 24 / 512; }

// Where the four gate sums of (sentence, unit 4 rt + q of the workgroup) lie in a 16-byte-grained tile of partial
// sums: written sentence by sentence, read unit by unit, both free of bank conflicts.
__device__ __forceinline__ int recur_pos(int sentence, int q, int rt) { return q * 16 + (sentence ^ ((q + 4 * rt) & 15)); }
// The same for the backward kernel's tiles: the sums of units 4 q .. 4 q + 3 of row tile rt for a sentence.
__device__ __forceinline__ int recur_pos_bwd(int sentence, int q, int rt) { return q * 16 + (sentence ^ (4 * q + 2 * (rt & 1))); }
// The role of this workgroup (its number in order of arrival), and whether the launch has given up already; ticket as in
// SeqFwdArgs.  With wait_ticks = 0 every wait is given up beforehand.
__device__ __forceinline__ int recur_role(int* ticket, int wait_ticks, int (&s_role)[2], bool& dead) {
  if (threadIdx.x == 0) {
    if (wait_ticks == 0) atomicOr(ticket + 1, 1);
    s_role[1] = __hip_atomic_load(ticket + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_role[0] = atomicAdd(ticket, 1);
  }
  __syncthreads();
  dead = s_role[1] != 0;
  return s_role[0];
}

template <typename T, int KS, int NK, int LK, int RT, int BT, int NE>
__global__ __launch_bounds__(64 * (KS + NE)) void lstm_seq_fwd_kernel(SeqFwdArgs args, int L, int Bp, int Hh, int ndir, int nap) {
  __shared__ __align__(16) float red[2][KS * RT * BT * 256];
  __shared__ Frag<T> wlds[LK ? KS * LK * RT * 64 : 1];           // the last LK k steps' weights, read by the wavefront that put them there
  __shared__ int s_role[2];
  bool dead;
  const int id = recur_role(args.ticket, args.wait_ticks, s_role, dead);
  const int nwg = (Hh + 4 * RT - 1) / (4 * RT);                  // workgroups per group
  const int grp = id / nwg, u0 = (id - grp * nwg) * 4 * RT;
  const SeqFwdDir d = args.d[grp % ndir];
  const int bt0 = (grp / ndir) * BT;
  const int nbt = min(BT, (Bp >> 4) - bt0);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nsteps = (Hh + 31) >> 5;
  const size_t slot = (size_t)(Bp >> 4) * nsteps * 512;          // elements per slot of the exchange buffer
  const int rev = d.reverse;
  if (w < KS) {
    // ---- contraction: wavefront w takes the k steps w, w + KS, ...; its weights stay in registers (and LDS) ---------
    Frag<T> wf[NK - LK][RT];
    Frag<T>* const wl = wlds + w * LK * RT * 64 + lane;
    bool kin[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      const int k = 32 * (w + KS * q) + 8 * (lane >> 4);
      kin[q] = k < Hh;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int m = lane & 15, u = min(u0 + 4 * rt + (m >> 2), Hh - 1);
        Frag<T> f;
        if (kin[q]) f.load((const T*)d.W + (size_t)((m & 3) * Hh + u) * d.ldw + d.wh_off + k);
        else f.zero();
        if (q < NK - LK) wf[q][rt] = f;
        else wl[((q - (NK - LK)) * RT + rt) * 64] = f;
      }
    }
    for (int i = 0; i < L; ++i) {
      if (i > 0) {
        const T* x = (const T*)d.X + (size_t)(rev ? L - i : i) * slot + (size_t)bt0 * nsteps * 512;
        Frag<T> fx[NK * BT];
        const T* px[NK * BT];
        bool in[NK * BT];
#pragma unroll
        for (int q = 0; q < NK; ++q)
#pragma unroll
          for (int b = 0; b < BT; ++b) {
            px[q * BT + b] = x + ((size_t)b * nsteps + w + KS * q) * 512;
            in[q * BT + b] = kin[q] && b < nbt;
          }
        recur_nap(nap);
        recur_issue<T, NK * BT>(px, in, lane * 8, fx);
        recur_settle<T, NK * BT>(px, in, lane * 8, fx, dead, args.ticket + 1, args.wait_ticks);
        v4f acc[RT][BT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int b = 0; b < BT; ++b) acc[rt][b] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NK; ++q)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const Frag<T> f = q < NK - LK ? wf[q < NK - LK ? q : 0][rt] : wl[((q - (NK - LK)) * RT + rt) * 64];
#pragma unroll
            for (int b = 0; b < BT; ++b) mma16(acc[rt][b], f, fx[q * BT + b]);
          }
        float* r = red[i & 1];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int b = 0; b < BT; ++b) 
            *reinterpret_cast<v4f*>(r + (((w * RT + rt) * BT + b) * 64 + recur_pos(lane & 15, lane >> 4, rt)) * 4) = acc[rt][b];
      }
      __syncthreads();
    }
    return;
  }
  // ---- cells: one per lane and pass; cell and hidden state stay in registers ---------------------------------------
  // A wavefront takes all units of its workgroup for 64 / UW sentences, so that what it reads and writes per sentence is
  // one contiguous piece (with the accumulator's own mapping, 4 units x 16 sentences, the same data is 4 times as many
  // cache requests, and those were what a position waited for).  Addresses are a uniform base per position plus a
  // 32-bit lane offset that never changes: the instructions of this path are on every position's critical path.
  constexpr int UW = 4 * RT;
  const int e = w - KS, passes = nbt * RT;
  auto cells = [&](auto count) {
    constexpr int NA = decltype(count)::value;
    constexpr bool FAST = sizeof(T) == 2;
    const int u = min(u0 + lane % UW, Hh - 1), uw = u - u0;        // (surplus lanes repeat the last unit)
    const bool sender = !FAST || (lane % 4 == 0 && u0 + lane % UW < Hh);
    float c[NA], hcar[NA];
    unsigned off_r[NA], off_u[NA], off_g[NA], off_m[NA], off_x[NA], off_h[NA], off_y[NA];
    int row[NA];
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      c[n] = 0.f; hcar[n] = 0.f;
      const int b = 16 * bt0 + lane / UW + (e + NE * n) * (64 / UW), bt = (b >> 4) - bt0;
      row[n] = b;
      off_r[n] = (unsigned)(((uw >> 2) * BT + bt) * 1024 + recur_pos(b & 15, uw & 3, uw >> 2) * 16);
      off_u[n] = (unsigned)(b * Hh + u) * 4u;
      off_g[n] = (unsigned)(b * 4 * Hh + u) * 4u;
      off_m[n] = (unsigned)b * 4u;
      off_x[n] = (unsigned)(fm_offset(b, u, nsteps) * sizeof(T));
      off_h[n] = (unsigned)((b * d.ldh + u) * sizeof(T));
      off_y[n] = (unsigned)((b * d.ldy + d.y_col0 + u) * sizeof(T));
    }
    struct In { float g[NA][4]; float mask[NA]; };
    auto fetch = [&](In& in, int i) {
      const int t = rev ? L - 1 - i : i;
      const char* g = (const char*)(d.gx + (size_t)t * Bp * 4 * Hh);
      const char* m = (const char*)(d.mask + (size_t)t * Bp);
#pragma unroll
      for (int n = 0; n < NA; ++n) {
#pragma unroll
        for (int q = 0; q < 4; ++q) in.g[n][q] = *(const float*)(g + (size_t)q * Hh * 4 + off_g[n]);
        in.mask[n] = *(const float*)(m + off_m[n]);
      }
    };
    // The inputs of the next position are requested before this one's results are stored: loads and stores complete in
    // order, so the other way round every position would wait until its predecessor's stores have reached memory.
    auto step = [&](const In& in, In& next, int i) {
      const int t = rev ? L - 1 - i : i, sn = rev ? t : t + 1;
      char* const xs = (char*)d.X + (size_t)sn * slot * sizeof(T);
      char* const hs = (char*)d.H + (size_t)sn * Bp * d.ldh * sizeof(T);
      char* const cs = (char*)(d.C + (size_t)sn * Bp * Hh);
      char* const gs = (char*)(d.G + (size_t)t * Bp * 4 * Hh);
      char* const ys = (char*)d.Y + (size_t)t * Bp * d.ldy * sizeof(T);
      const DropSpec drop = seq_drop(d.drop, d.drop_step, t);
      const bool has_y = d.Y != nullptr;
      __syncthreads();
      fetch(next, min(i + 1, L - 1));
      asm volatile("" ::: "memory");
      const char* r = (const char*)red[i & 1];
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        v4f pre = v4f{0.f, 0.f, 0.f, 0.f};
        if (i > 0) {
#pragma unroll
          for (int k = 0; k < KS; ++k) pre += *reinterpret_cast<const v4f*>(r + off_r[n] + k * RT * BT * 1024);
        }
        float g[4];
        const float state = seq_cell<FAST>(pre, in.g[n], in.mask[n], hcar[n], c[n], g);
        T hv;
        if constexpr (FAST) {
          hv = f2bf(state);
          hcar[n] = bf2f(hv);
          const unsigned p = quad_pair(hv), p2 = __builtin_amdgcn_mov_dpp(p, 0x4e, 0xf, 0xf, true);      // lanes ^ 2
          if (sender)
            __hip_atomic_store(reinterpret_cast<uint64_t*>(xs + off_x[n]), (uint64_t)p | ((uint64_t)p2 << 32), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        } else {
          hv = hcar[n] = state;
          __hip_atomic_store(reinterpret_cast<unsigned*>(xs + off_x[n]), __float_as_uint(hv), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("" ::: "memory");                             // (the state first: the other workgroups wait for it)
        *(T*)(hs + off_h[n]) = hv;
        *(float*)(cs + off_u[n]) = c[n];
#pragma unroll
        for (int q = 0; q < 4; ++q) *(float*)(gs + (size_t)q * Hh * 4 + off_g[n]) = g[q];
        // (the copy after dropout is rounded once, from the state as computed)
        if (has_y) *(T*)(ys + off_y[n]) = from_f<T>(state * drop_factor(drop, row[n], d.y_col0 + u));
      }
    };
    In in0, in1;
    fetch(in0, 0);
    for (int i = 0; i < L; i += 2) {                              // two positions per round: no copies between the input sets
      step(in0, in1, i);
      if (i + 1 < L) step(in1, in0, i + 1);
    }
  };
  constexpr int NT = (RT * BT + NE - 1) / NE;                     // passes per wavefront
  if (e >= passes) { for (int i = 0; i < L; ++i) __syncthreads(); }
  else if (NT == 1 || e + NE >= passes) cells(std::integral_constant<int, 1>{});
  else cells(std::integral_constant<int, NT>{});
}

// ------------------------------------------------------------------------------------------------
// backward
// ------------------------------------------------------------------------------------------------
// The recurrent part of the state gradient, dG(next position) W_h, has the 4 Hh gate gradients as its contraction
// length: a workgroup owns 16 RT units (rows of W^T), its KS wavefronts split the gate rows and keep their share of W^T
// in registers, and what the group exchanges per position is its gate gradients.  The fragments of a position arrive CH at
// a time, the next ones in flight while the matrix cores take the current ones.
template <typename T, int KS, int NK, int RT, int NE>
__global__ __launch_bounds__(64 * (KS + NE)) void lstm_seq_bwd_kernel(SeqBwdArgs args, int L, int Bp, int Hh, int ndir, int nap) {
  constexpr int CH = NK * RT * (int)sizeof(Frag<T>) >= 512 ? (sizeof(T) == 2 ? 2 : 1) : NK < 4 ? NK : 4;   // (registers: weights and two chunks)
  __shared__ __align__(16) float red[2][KS * RT * 256];
  __shared__ int s_role[2];
  bool dead;
  const int id = recur_role(args.ticket, args.wait_ticks, s_role, dead);
  const int nwg = (Hh + 16 * RT - 1) / (16 * RT);
  const int grp = id / nwg, u0 = (id - grp * nwg) * 16 * RT;
  const SeqBwdDir d = args.d[grp % ndir];
  const int bt = grp / ndir;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nsteps = Hh >> 3;                                    // k steps of 32 gate rows
  const size_t slot = (size_t)Bp * 4 * Hh;                       // elements per slot
  const int rev = d.reverse;                                     // of the forward pass: positions run upwards here
  if (w < KS) {
    Frag<T> wf[NK][RT];
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int s = w + KS * q, u = min(u0 + 16 * rt + (lane & 15), Hh - 1);
        if (s < nsteps) wf[q][rt].load((const T*)d.Wt + (size_t)u * d.ldw + 32 * s + 8 * (lane >> 4));
        else wf[q][rt].zero();
      }
    for (int i = 0; i < L; ++i) {
      if (i > 0) {
        const T* x = (const T*)d.X + (size_t)(rev ? i - 1 : L - i) * slot + (size_t)bt * nsteps * 512;
        v4f acc[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = v4f{0.f, 0.f, 0.f, 0.f};
        recur_nap(nap);
        Frag<T> fx[2][CH];
        const T* p[2][CH];
        bool in[2][CH];
        auto issue = [&](int c) {
#pragma unroll
          for (int q = 0; q < CH; ++q) {
            const int s = w + KS * (c * CH + q);
            p[c & 1][q] = x + (size_t)s * 512;
            in[c & 1][q] = s < nsteps;
          }
          recur_issue<T, CH>(p[c & 1], in[c & 1], lane * 8, fx[c & 1]);
        };
        issue(0);
#pragma unroll
        for (int c = 0; c < NK / CH; ++c) {
          asm volatile("" ::: "memory");                         // (no more than two chunks in flight: registers)
          if (c + 1 < NK / CH) issue(c + 1);
          recur_settle<T, CH>(p[c & 1], in[c & 1], lane * 8, fx[c & 1], dead, args.ticket + 1, args.wait_ticks);
#pragma unroll
          for (int q = 0; q < CH; ++q)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) mma16(acc[rt], wf[c * CH + q][rt], fx[c & 1][q]);
        }
        float* r = red[i & 1];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          *reinterpret_cast<v4f*>(r + ((w * RT + rt) * 64 + recur_pos_bwd(lane & 15, lane >> 4, rt)) * 4) = acc[rt];
      }
      __syncthreads();
    }
    return;
  }
  constexpr int UW = 16 * RT, NT = (4 * RT + NE - 1) / NE;
  static_assert(4 * RT % NE == 0, "every cell wavefront has the same number of passes");
  constexpr bool FAST = sizeof(T) == 2;
  const int e = w - KS;
  const int u = min(u0 + lane % UW, Hh - 1), uw = u - u0;          // (surplus lanes repeat the last unit)
  const bool real = u0 + lane % UW < Hh;
  const int gate = lane & 3, u4 = u & ~3;                        // 16-bit types: the lane stores this gate of units u4 .. u4 + 3
  float cn[NT], dh[NT], dc[NT];
  unsigned off_r[NT], off_u[NT], off_g[NT], off_m[NT], off_x[NT], off_d[NT], off_y[NT];
  int row[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int sb = lane / UW + (e + NE * n) * (64 / UW), b = 16 * bt + sb;
    row[n] = b;
    off_r[n] = (unsigned)((uw >> 4) * 1024 + recur_pos_bwd(sb, (uw >> 2) & 3, uw >> 4) * 16 + (uw & 3) * 4);
    off_u[n] = (unsigned)(b * Hh + u) * 4u;
    off_g[n] = (unsigned)(b * 4 * Hh + u) * 4u;
    off_m[n] = (unsigned)b * 4u;
    off_y[n] = (unsigned)(b * d.lddy + d.dy_col + u) * 4u;
    if constexpr (FAST) {
      off_x[n] = (unsigned)(fm_offset(b, gate * Hh + u4, nsteps) * sizeof(T));
      off_d[n] = (unsigned)((b * d.lddg + gate * Hh + u4) * sizeof(T));
    } else {
      off_x[n] = 0;                                                // (the four gates' places are worked out where they are stored)
      off_d[n] = (unsigned)((b * d.lddg + u) * sizeof(T));
    }
    cn[n] = *(const float*)((const char*)(d.C + (size_t)(rev ? 0 : L) * Bp * Hh) + off_u[n]);
    dh[n] = d.dh0[(size_t)b * d.ldd0 + u];
    dc[n] = d.dc0[(size_t)b * d.ldd0 + u];
  }
  struct In { float g[NT][4]; float cp[NT], dy[NT], mask[NT]; };
  auto fetch = [&](In& in, int i) {
    const int t = rev ? i : L - 1 - i;
    const char* g = (const char*)(d.G + (size_t)t * Bp * 4 * Hh);
    const char* c = (const char*)(d.C + (size_t)(rev ? t + 1 : t) * Bp * Hh);
    const char* y = (const char*)(d.dY + (size_t)t * Bp * d.lddy);
    const char* m = (const char*)(d.mask + (size_t)t * Bp);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
#pragma unroll
      for (int q = 0; q < 4; ++q) in.g[n][q] = *(const float*)(g + (size_t)q * Hh * 4 + off_g[n]);
      in.cp[n] = *(const float*)(c + off_u[n]);
      in.dy[n] = *(const float*)(y + off_y[n]);
      in.mask[n] = *(const float*)(m + off_m[n]);
    }
  };
  auto step = [&](const In& in, In& next, int i) {
    const int t = rev ? i : L - 1 - i;
    char* const xs = (char*)d.X + (size_t)t * slot * sizeof(T);
    char* const ds = (char*)d.dG + (size_t)t * Bp * d.lddg * sizeof(T);
    const DropSpec drop = seq_drop(d.drop, d.drop_step, t);
    // what does not wait for the recurrent part: dy's share and the factors of the cell backward
    float dyf[NT], tc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      dyf[n] = in.dy[n] * drop_factor(drop, row[n], d.dy_col + u);
      tc[n] = tanh_of<FAST>(cn[n]);
    }
    __syncthreads();
    fetch(next, min(i + 1, L - 1));
    asm volatile("" ::: "memory");
    const char* r = (const char*)red[i & 1];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      float rec = 0.f;
      if (i > 0) {
#pragma unroll
        for (int k = 0; k < KS; ++k) rec += *reinterpret_cast<const float*>(r + off_r[n] + k * RT * 1024);
      }
      float o[4];
      seq_cell_bwd(in.g[n], in.cp[n], tc[n], dyf[n], rec, in.mask[n], dh[n], dc[n], o);
      cn[n] = in.cp[n];
      if constexpr (FAST) {
        const uint64_t v = quad_transpose(f2bf(o[0]), f2bf(o[1]), f2bf(o[2]), f2bf(o[3]), lane);
        if (real) {
          __hip_atomic_store(reinterpret_cast<uint64_t*>(xs + off_x[n]), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          *reinterpret_cast<uint64_t*>(ds + off_d[n]) = v;
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const size_t xo = fm_offset(row[n], q * Hh + u, nsteps) * sizeof(T);
          __hip_atomic_store(reinterpret_cast<unsigned*>(xs + xo), __float_as_uint(o[q]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) *(float*)(ds + (size_t)q * Hh * 4 + off_d[n]) = o[q];
      }
    }
  };
  In in0, in1;
  fetch(in0, 0);
  for (int i = 0; i < L; i += 2) {
    step(in0, in1, i);
    if (i + 1 < L) step(in1, in0, i + 1);
  }
}

// ------------------------------------------------------------------------------------------------
// without waits
// ------------------------------------------------------------------------------------------------
// The same recurrences by one workgroup per (direction, 16 sentences), which needs no other: it reads the recurrent weights
// at every position, and that (from L2, at some 50 GB/s per CU) is what a position costs.  gave_up (may be null): nothing is
// to be done while it is zero.  States and gate gradients are read back through memory, written by the same workgroup before
// a barrier; everything else of a (sentence, unit) stays with one lane.  Few registers and half the wavefronts that fit: a
// launch with nothing to do is to start and end beside other kernels' workgroups.
constexpr int SOLO_WAVES = 8;

template <typename T>
__global__ __launch_bounds__(64 * SOLO_WAVES) void lstm_seq_fwd_solo_kernel(const int* gave_up, int L, int Bp, int Hh, int ndir,
                                                                             SeqFwdArgs args) {
  if (!recur_again(gave_up, args.again)) return;
  constexpr bool FAST = sizeof(T) == 2;
  const SeqFwdDir d = args.d[blockIdx.x % ndir];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int sentence = 16 * (blockIdx.x / ndir) + (lane & 15);
  for (int i = 0; i < L; ++i) {
    const int t = d.reverse ? L - 1 - i : i, sp = d.reverse ? t + 1 : t, sn = d.reverse ? t : t + 1;
    const T* hp = (const T*)d.H + ((size_t)sp * Bp + sentence) * d.ldh;
    const float mask = d.mask[(size_t)t * Bp + sentence];
    const DropSpec drop = seq_drop(d.drop, d.drop_step, t);
    for (int rt = w; rt < Hh >> 2; rt += SOLO_WAVES) {             // tiles of 4 units x 4 gates
      v4f pre = v4f{0.f, 0.f, 0.f, 0.f};
      if (i > 0) {
        const int m = lane & 15;
        const T* wr = (const T*)d.W + (size_t)((m & 3) * Hh + 4 * rt + (m >> 2)) * d.ldw + d.wh_off;
        for (int k0 = 0; k0 < Hh; k0 += 32) {
          const int k = k0 + 8 * (lane >> 4);
          Frag<T> fw, fx;
          fw.zero(); fx.zero();
          if (k < Hh) { fw.load(wr + k); fx.load(hp + k); }
          mma16(pre, fw, fx);
        }
      }
      const int u = 4 * rt + (lane >> 4);
      const size_t at = (size_t)t * Bp + sentence, next = (size_t)sn * Bp + sentence;
      float gx[4], g[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) gx[q] = d.gx[at * 4 * Hh + (size_t)q * Hh + u];
      float c = i > 0 ? d.C[((size_t)sp * Bp + sentence) * Hh + u] : 0.f;
      const float state = seq_cell<FAST>(pre, gx, mask, i > 0 ? to_f<T>(hp[u]) : 0.f, c, g);
      ((T*)d.H)[next * d.ldh + u] = from_f<T>(state);
      d.C[next * Hh + u] = c;
#pragma unroll
      for (int q = 0; q < 4; ++q) d.G[at * 4 * Hh + (size_t)q * Hh + u] = g[q];
      if (d.Y) ((T*)d.Y)[at * d.ldy + d.y_col0 + u] = from_f<T>(state * drop_factor(drop, sentence, d.y_col0 + u));
    }
    __syncthreads();
  }
}

template <typename T>
__global__ __launch_bounds__(64 * SOLO_WAVES) void lstm_seq_bwd_solo_kernel(const int* gave_up, int L, int Bp, int Hh, int ndir,
                                                                             SeqBwdArgs args) {
  if (!recur_again(gave_up, args.again)) return;
  constexpr bool FAST = sizeof(T) == 2;
  const SeqBwdDir d = args.d[blockIdx.x % ndir];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int sentence = 16 * (blockIdx.x / ndir) + (lane & 15);
  // the gradients that pass by are kept in the exchange buffer, which nobody else uses now: [2, Bp, Hh] floats
  float* const keep = (float*)d.X + (size_t)sentence * Hh;
  const size_t plane = (size_t)Bp * Hh;
  for (int i = 0; i < L; ++i) {
    const int t = d.reverse ? i : L - 1 - i, sp = d.reverse ? t + 1 : t, sn = d.reverse ? t : t + 1;   // slots before and after the position
    const T* gp = (const T*)d.dG + ((size_t)(d.reverse ? t - 1 : t + 1) * Bp + sentence) * d.lddg;     // (of the position that came before here)
    const float mask = d.mask[(size_t)t * Bp + sentence];
    const DropSpec drop = seq_drop(d.drop, d.drop_step, t);
    const size_t at = (size_t)t * Bp + sentence;
    for (int u16 = 16 * w; u16 < Hh; u16 += 16 * SOLO_WAVES) {
      v4f rec = v4f{0.f, 0.f, 0.f, 0.f};
      if (i > 0) {
        const T* wr = (const T*)d.Wt + (size_t)min(u16 + (lane & 15), Hh - 1) * d.ldw;
        for (int k = 8 * (lane >> 4); k < 4 * Hh; k += 32) {       // (4 Hh is a multiple of 32)
          Frag<T> fw, fx;
          fw.load(wr + k); fx.load(gp + k);
          mma16(rec, fw, fx);
        }
      }
      for (int k = 0; k < 4; ++k) {
        const int u = u16 + 4 * (lane >> 4) + k;
        if (u >= Hh) break;
        const float r = k == 0 ? rec[0] : k == 1 ? rec[1] : k == 2 ? rec[2] : rec[3];
        float dh = i > 0 ? keep[u] : d.dh0[(size_t)sentence * d.ldd0 + u], dc = i > 0 ? keep[plane + u] : d.dc0[(size_t)sentence * d.ldd0 + u];
        float g[4], o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = d.G[at * 4 * Hh + (size_t)q * Hh + u];
        const float cp = d.C[((size_t)sp * Bp + sentence) * Hh + u], cn = d.C[((size_t)sn * Bp + sentence) * Hh + u];
        const float dy = d.dY[at * d.lddy + d.dy_col + u] * drop_factor(drop, sentence, d.dy_col + u);
        seq_cell_bwd(g, cp, tanh_of<FAST>(cn), dy, r, mask, dh, dc, o);
        keep[u] = dh; keep[plane + u] = dc;
#pragma unroll
        for (int q = 0; q < 4; ++q) ((T*)d.dG)[at * d.lddg + (size_t)q * Hh + u] = from_f<T>(o[q]);
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------------
// launches
// ------------------------------------------------------------------------------------------------
// Groups that wait only where as many launches as a process runs at once fit the device (recur_plan.h).
static bool seq_together(const SeqPlan& p, const SeqRun& run) { return run.mode != SEQ_RUN_ALONE && SEQ_QUEUES * (p.group - 1) < run.cus; }
static int seq_wait(const SeqRun& run) { return run.mode == SEQ_RUN_GIVE_UP ? 0 : RECUR_WAIT_TICKS; }

template <typename T, int KS, int NK, int RT, int NE>
static void seq_bwd_go(const SeqPlan& p, const SeqBwdArgs& a, int ndir, int L, int Bp, int Hh, hipStream_t st) {
  hipLaunchKernelGGL((lstm_seq_bwd_kernel<T, KS, NK, RT, NE>), dim3(p.groups * p.group), dim3(64 * (KS + NE)), 0, st, a, L, Bp, Hh, ndir,
                     recur_nap_bwd(Hh));
}
void launch_lstm_seq_bwd(int prec, const SeqBwdArgs& args, int ndir, int L, int Bp, int Hh, const SeqRun& run, hipStream_t st) {
  const SeqPlan p = seq_bwd_plan(prec, ndir, Bp, Hh);
  const bool together = seq_together(p, run);
  SeqBwdArgs a = args;
  a.wait_ticks = seq_wait(run);
#define GO(KS, NK)                                                                                   \
  do {                                                                                               \
    if (!prec) seq_bwd_go<float, KS, NK, 1, 4>(p, a, ndir, L, Bp, Hh, st);                           \
    else if (p.rt == 1) seq_bwd_go<bf16_t, KS, NK, 1, 4>(p, a, ndir, L, Bp, Hh, st);                 \
    else seq_bwd_go<bf16_t, KS, NK, 2, (NK > 8 ? 4 : 8)>(p, a, ndir, L, Bp, Hh, st);                 \
  } while (0)
  if (!together) {}
  else if (p.ks == 2) GO(2, 2);
  else if (p.nk == 2) GO(8, 2);
  else if (p.nk == 4) GO(8, 4);
  else if (p.nk == 8) GO(8, 8);
  else GO(8, 16);
#undef GO
  if (together && L == 1) return;                    // (nothing to wait for)
  const int* gave_up = together ? a.ticket + 1 : nullptr;
  const dim3 grid(ndir * (Bp >> 4)), block(64 * SOLO_WAVES);
  if (prec) hipLaunchKernelGGL(lstm_seq_bwd_solo_kernel<bf16_t>, grid, block, 0, st, gave_up, L, Bp, Hh, ndir, a);
  else hipLaunchKernelGGL(lstm_seq_bwd_solo_kernel<float>, grid, block, 0, st, gave_up, L, Bp, Hh, ndir, a);
}

template <typename T, int KS, int NK, int LK, int BT, int NE>
static void seq_fwd_go(const SeqPlan& p, const SeqFwdArgs& a, int ndir, int L, int Bp, int Hh, hipStream_t st) {
  hipLaunchKernelGGL((lstm_seq_fwd_kernel<T, KS, NK, LK, 4, BT, NE>), dim3(p.groups * p.group), dim3(64 * (KS + NE)), 0, st, a, L, Bp, Hh,
                     ndir, recur_nap_fwd(sizeof(T), BT, Hh));
}
void launch_lstm_seq_fwd(int prec, const SeqFwdArgs& args, int ndir, int L, int Bp, int Hh, const SeqRun& run, hipStream_t st) {
  const SeqPlan p = seq_fwd_plan(prec, ndir, Bp, Hh);
  const bool together = seq_together(p, run);
  SeqFwdArgs a = args;
  a.wait_ticks = seq_wait(run);
#define GO(KS, NK, NE2)                                                                              \
  do {                                                                                               \
    if (prec && p.bt == 1) seq_fwd_go<bf16_t, KS, NK, 0, 1, 4>(p, a, ndir, L, Bp, Hh, st);           \
    else if (prec) seq_fwd_go<bf16_t, KS, NK, 0, 2, NE2>(p, a, ndir, L, Bp, Hh, st);                 \
    else if (p.bt == 1) seq_fwd_go<float, KS, NK, NK == 4, 1, 4>(p, a, ndir, L, Bp, Hh, st);         \
    else if constexpr (NK < 4) seq_fwd_go<float, KS, NK, 0, 2, 4>(p, a, ndir, L, Bp, Hh, st);        \
  } while (0)
  if (!together) {}
  else if (p.ks == 2 && p.nk == 1) GO(2, 1, 4);
  else if (p.ks == 2) GO(2, 2, 4);
  else if (p.nk == 1) GO(8, 1, 8);
  else if (p.nk == 2) GO(8, 2, 8);
  else GO(8, 4, 4);
#undef GO
  if (together && L == 1) return;                    // (nothing to wait for)
  const int* gave_up = together ? a.ticket + 1 : nullptr;
  const dim3 grid(ndir * (Bp >> 4)), block(64 * SOLO_WAVES);
  if (prec) hipLaunchKernelGGL(lstm_seq_fwd_solo_kernel<bf16_t>, grid, block, 0, st, gave_up, L, Bp, Hh, ndir, a);
  else hipLaunchKernelGGL(lstm_seq_fwd_solo_kernel<float>, grid, block, 0, st, gave_up, L, Bp, Hh, ndir, a);
}

}  // namespace cmt

// The forward loop's kernels and their launch, training (loop.hip) and greedy decoding (loop_dec.hip).
#pragma once
#include <algorithm>
#include <type_traits>

#include "loop_core.h"

namespace cmt {

// DEC: greedy decoding (LoopTokens).  Every workgroup takes each H / 4-th tile of 16 vocabulary entries, W_o's rows streaming in from
// memory (they do not fit the chip) while H_o's fragments stay in registers between the bottom layer's product and this one; the best
// of its entries per sentence go to the wavefront that owns the sentence, which sends the token to all.
template <typename T, int NK, int BT, int NCH, bool DEC, int LM = LOOP_MAX_LAYERS>
__global__ __launch_bounds__(64 * LOOP_WAVES) void loop_fwd_kernel(LoopFwdArgs args_, int L, int Tn, int Bp, int H, int S, LoopPlan plan,
                                                                   int nap) {
  constexpr bool FAST = sizeof(T) == 2;
  constexpr int LREG = NK * sizeof(T) >= 8 ? 2 : LM;               // layers whose recurrent weights are in registers, not LDS
  constexpr int LLDS = LM - LREG;
  // decoding: tiles of W_o on their way, as many as the registers hold, and most of W_c2 in LDS where that makes room
  constexpr int PD = NK * sizeof(T) * BT * LM >= 128 ? 1 : LM == 2 && NK * sizeof(T) * BT < 32 ? 4 : 2;
  constexpr int CL = DEC && LLDS ? NK - 1 : 0;
  constexpr int NQ = (NK * 32 * LOOP_WAVES + 511) / 512;           // 8-element pieces of a row per lane
  __shared__ __align__(16) float red_[2][LOOP_WAVES * BT * 256];
  __shared__ Frag<T> wlds[LLDS ? (LLDS * NK + CL) * LOOP_WAVES * 64 : 1];
  __shared__ __align__(16) float s_bias[LM][4][4];   // [layer][unit][gate]
  __shared__ float s_u[LOOP_MAX_BATCH][4];
  __shared__ int s_len[LOOP_MAX_BATCH];
  __shared__ int s_dead;
  const LoopPlace place = loop_place(blockIdx.x, plan.groups, plan.nwg);
  if (place.group >= plan.groups || place.pos >= plan.nwg) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u0 = 4 * place.pos, bt0 = place.group * plan.tiles, nbt = min(plan.tiles, (Bp >> 4) - bt0), NB = 16 * nbt;
  const int ns = (H + 31) >> 5;
  const size_t slot = (size_t)Bp * ns * 32;
  const auto A = [] { return loop_args<LoopFwdArgs>(); };
  int* const gave_up = loop_global(A()->ticket) + 1;
  const int ticks = A()->wait_ticks;
  if (threadIdx.x == 0) {
    if (ticks == 0) atomicOr(gave_up, 1);
    s_dead = __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int i = threadIdx.x; i < NB; i += 64 * LOOP_WAVES) s_len[i] = min(loop_global(A()->len)[16 * bt0 + i], S);
  // ---- weights: wavefront w takes the k steps w, w + 8, ... of every product -------------------------------------------
  bool kin[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q) kin[q] = 32 * (w + LOOP_WAVES * q) + 8 * (lane >> 4) < H;
  Frag<T> wx[LM][NK], wh[LREG][NK], wc[NK - CL];
  Frag<T>* const wl = wlds + (size_t)w * 64 + lane;                // + ((layer - LREG) * NK + q) * LOOP_WAVES * 64
  const int m = lane & 15;
#pragma unroll
  for (int l = 0; l < LM; ++l)
    if (l < L) {
      const auto a = A();
      const int xo = a->l[l].wx_off, ho = a->l[l].wh_off;
      const T* row = loop_global((const T*)a->l[l].W) + (size_t)((m & 3) * H + u0 + (m >> 2)) * a->l[l].ldw;
#pragma unroll
      for (int q = 0; q < NK; ++q) {
        const int k = 32 * (w + LOOP_WAVES * q) + 8 * (lane >> 4);
        Frag<T> f;
        f.zero(); wx[l][q].zero();
        if (kin[q]) { wx[l][q].load(row + xo + k); f.load(row + ho + k); }
        if (l < LREG) wh[l < LREG ? l : 0][q] = f;
        else wl[((l - LREG) * NK + q) * LOOP_WAVES * 64] = f;
      }
      if ((l > 0 || DEC) && threadIdx.x < 16)
        s_bias[l][threadIdx.x >> 2][threadIdx.x & 3] = loop_global(a->l[l].bias)[(threadIdx.x & 3) * H + u0 + (threadIdx.x >> 2)];
    }
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const auto a = A();
    Frag<T> f;
    f.zero();                                                      // (four columns of W_c2; the tile's other rows repeat them)
    if (kin[q]) f.load(loop_global((const T*)a->Wc) + (size_t)(u0 + (m & 3)) * a->ldwc + 32 * (w + LOOP_WAVES * q) + 8 * (lane >> 4));
    if (q < CL) wl[(LLDS * NK + q) * LOOP_WAVES * 64] = f;
    else wc[q < CL ? 0 : q - CL] = f;
  }
  // ---- cells: wavefront w finishes tile w, a lane one unit of one sentence ----------------------------------------------
  const bool mine = w < nbt;
  const int btw = bt0 + min(w, nbt - 1);
  float c[LM], hcar[LM];
#pragma unroll
  for (int l = 0; l < LM; ++l)
    if (l < L) {
      const auto a = A();
      const int b = 16 * btw + (lane >> 2), u = u0 + (lane & 3);
      c[l] = loop_global(a->l[l].C)[(size_t)b * H + u];
      hcar[l] = to_f<T>(loop_global((const T*)a->l[l].H)[(size_t)b * a->l[l].ldh + u]);
      if (mine) loop_quad_put(loop_global((T*)a->l[l].X), fm_offset(b, u0, ns), (T*)nullptr, 0, hcar[l], lane, true);
    }
  float gx[4], mask;
  auto fetch = [&](int j) {
    if constexpr (DEC) { mask = 16 * btw + (lane >> 2) < A()->t.B ? 1.f : 0.f; return; }
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const int b = 16 * btw + (ln >> 2);
    const char* g = (const char*)(loop_global(a->gx) + (size_t)j * Bp * 4 * H);
    const unsigned off = (unsigned)(b * 4 * H + u0 + (ln & 3)) * 4u;
#pragma unroll
    for (int q = 0; q < 4; ++q) gx[q] = *(const float*)(g + (size_t)q * H * 4 + off);
    mask = loop_global(a->mask)[(size_t)j * Bp + b];
  };
  fetch(0);
  // ---- attention: a wavefront's rows of the scores; a thread's share of the mix ----------------------------------------
  const int np = max(1, plan.nwg * LOOP_WAVES / NB);               // wavefronts per sentence
  const int spw = nbt > 2 ? 8 : 2 * nbt, tps = 64 / spw;           // mix: sentences per wavefront, threads per sentence
  __syncthreads();
  bool dead = s_dead != 0;
  float* red = red_[0];                                            // (the two take turns)
  const unsigned tile = (unsigned)ns * 512u * (unsigned)sizeof(T);
  const size_t group = (size_t)bt0 * ns * 512;
  Frag<T> fx[NK * BT];                                             // the fragments in flight
  v4f acc[NCH][BT];
  auto issue = [&](const T* x, int ch) {
    int ln = lane;
    LOOP_FRESH(ln);
    loop_issue<T, NK * BT>(x + group, [&](int i, unsigned z) { return loop_frag_at<T, BT>(i, z, tile, ns, H, w, ch * BT, nbt, ln); }, fx);
  };
  auto settle = [&](const T* x, int ch) {
    loop_settle<T, NK * BT>(x + group, [&](int i, unsigned z) { return loop_frag_at<T, BT>(i, z, tile, ns, H, w, ch * BT, nbt, lane); }, fx, dead,
                            gave_up, ticks);
  };
  auto multiply = [&](const Frag<T> (&wf)[NK], int ch) {
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
      for (int t = 0; t < BT; ++t) mma16(acc[ch][t], wf[q], fx[q * BT + t]);
  };
  auto clear = [&]() {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
      for (int t = 0; t < BT; ++t) acc[ch][t] = v4f{0.f, 0.f, 0.f, 0.f};
  };
  auto spread = [&](int ch) {
#pragma unroll
    for (int t = 0; t < BT; ++t) *reinterpret_cast<v4f*>(red + ((w * BT + t) * 64 + loop_pos(lane & 15, lane >> 4)) * 4) = acc[ch][t];
  };
  auto from_lds = [&](int n, Frag<T> (&f)[NK]) {
#pragma unroll
    for (int q = 0; q < NK; ++q) f[q] = wl[(n * NK + q) * LOOP_WAVES * 64];
  };
  // the pointers of layer l, read where they are used
  auto states = [&](int l, int j) {
    const auto a = A();
    return loop_global((const T*)(l == 0 ? a->l[0].X : l == 1 ? a->l[1].X : l == 2 ? a->l[2].X : a->l[3].X)) + (size_t)j * slot;
  };

  // ---- greedy decoding ---------------------------------------------------------------------------------------------------
  // rows of W_o of a tile of 16 vocabulary entries (beyond the last: the last)
  // and their biases (as loads return in order, those would wait for all rows on their way if they were asked for where they are used)
  struct VocabRows { Frag<T> w[NK]; v4f bias; };
  auto vocab_rows = [&](int tl, VocabRows& wo) {
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const int V = a->t.V, tiles = (V + 15) >> 4;
    const T* const Wo = loop_global((const T*)a->t.Wo);
    tl = min(tl, tiles - 1);
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      const int s = min(w + LOOP_WAVES * q, ns - 1);
      if (a->t.fm) wo.w[q].load(Wo + ((size_t)tl * ns + s) * 512 + (unsigned)(ln * 8));
      else {
        const unsigned row = (unsigned)min(16 * tl + (ln & 15), V - 1), kk = (unsigned)min(32 * s + 8 * (ln >> 4), H - 8);
        wo.w[q].load(Wo + (size_t)row * H + kk);
      }
    }
    wo.bias = *reinterpret_cast<const v4f*>(loop_global(a->t.Bo) + (unsigned)min(16 * tl + 4 * (ln >> 4), V - 4));   // (V is a multiple of 8)
  };
  int fin = 0;                                                     // the sentence that this wavefront owns has ended
  // The best token of step j, whose H_o fragments are in fx; wo: the rows of this workgroup's first tile.
  auto first_rows = [&](VocabRows (&wo)[PD]) {
#pragma unroll
    for (int d = 0; d < PD; ++d) vocab_rows(place.pos + d * plan.nwg, wo[d]);
  };
  auto best_tokens = [&](int j, VocabRows (&rows)[PD]) {
    const int V = A()->t.V, tiles = (V + 15) >> 4;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    auto take = [&](int tl, VocabRows& wo) {
      v4f lg[BT];
#pragma unroll
      for (int t = 0; t < BT; ++t) lg[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < NK; ++q) {
        // (steps beyond the last, and the half step of an odd width, repeat something: not to be counted)
        Frag<T> f = wo.w[q];
        if (!kin[q]) f.zero();
#pragma unroll
        for (int t = 0; t < BT; ++t) mma16(lg[t], f, fx[q * BT + t]);
      }
      const v4f bias = wo.bias;
      if (tl + PD * plan.nwg < tiles) vocab_rows(tl + PD * plan.nwg, wo);
#pragma unroll
      for (int t = 0; t < BT; ++t) *reinterpret_cast<v4f*>(red + ((w * BT + t) * 64 + loop_pos(lane & 15, lane >> 4)) * 4) = lg[t];
      loop_barrier();
      const float* r = red;
      red = red == red_[0] ? red_[1] : red_[0];
      if (mine && w < BT) {
        int ln = lane;
        LOOP_FRESH(ln);
        v4f z = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < LOOP_WAVES; ++k) z += *reinterpret_cast<const v4f*>(r + ((k * BT + w) * 64 + loop_pos(ln & 15, ln >> 4)) * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 16 * tl + 4 * (ln >> 4) + i;               // (ascending: the first of equal values stays)
          if (v < V) {
            const float x = z[i] + bias[i];
            if (x > bv) { bv = x; bi = v; }
          }
        }
      }
    };
    for (int tl = place.pos; tl < tiles; tl += PD * plan.nwg) {
#pragma unroll
      for (int d = 0; d < PD; ++d)
        if (tl + d * plan.nwg < tiles) take(tl + d * plan.nwg, rows[d]);
    }
    if (mine && w < BT) {
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
      if (lane < 16) {
        uint64_t* const p = loop_global(A()->t.part) + ((size_t)(j & 1) * plan.nwg + place.pos) * Bp + 16 * btw + lane;
        __hip_atomic_store(p, (uint64_t)__float_as_uint(bv) | ((uint64_t)(unsigned)bi << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    // the wavefront that owns a sentence
    const int own = w * plan.nwg + place.pos, b = 16 * bt0 + own;
    if (own < NB && b < A()->t.B) {
      const auto a = A();
      uint64_t* const p = loop_global(a->t.part) + (size_t)(j & 1) * plan.nwg * Bp + b;
      uint64_t v[4];
      long long t_end = 0;
      for (int spin = 0;; ++spin) {
        bool some = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int g = lane + 64 * i;
          v[i] = g < plan.nwg ? __hip_atomic_load(p + (size_t)g * Bp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (uint64_t)0x7fffffffff800000ull;
          some = some || (unsigned)(v[i] >> 32) == RECUR_EMPTY;
        }
        if (dead || !__any(some)) break;
        if ((spin & 15) == 15) {
          const long long now = wall_clock64();
          if (t_end == 0) t_end = now + ticks;
          else if (now > t_end || __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            dead = true;
            if (lane == 0) atomicOr(gave_up, 1);
          }
        }
      }
      float x = -INFINITY;
      int y = 0x7fffffff;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float ov = __uint_as_float((unsigned)v[i]);
        const int oi = (int)(unsigned)(v[i] >> 32);
        if (ov > x || (ov == x && oi < y)) { x = ov; y = oi; }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(x, o, 64);
        const int oi = __shfl_xor(y, o, 64);
        if (ov > x || (ov == x && oi < y)) { x = ov; y = oi; }
      }
      const int token = (unsigned)y < (unsigned)V ? y : 0;         // (a row of NaNs: keep the token in range)
      // (what was put back a step ago is in place before the token that lets its slots' writers go on)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) {
        int* const tk = loop_global(a->t.tok);
        __hip_atomic_store(tk + (size_t)((j + 1) & 3) * Bp + b, token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(tk + (size_t)((j + 3) & 3) * Bp + b, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!fin) {
          loop_global(a->t.out_ids)[(size_t)b * Tn + j] = token;
          if (token == a->t.eos || j == Tn - 1) loop_global(a->t.out_len)[b] = j + 1;
        }
      }
      if (token == a->t.eos) fin = 1;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (lane + 64 * i < plan.nwg) __hip_atomic_store(p + (size_t)(lane + 64 * i) * Bp, ~(uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  // The bottom layer's product with the embeddings of position j's tokens.
  auto embedding = [&](int j) {
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const int E = a->t.emb, ne = (E + 31) >> 5, V = a->t.V;
    const T* const table = loop_global((const T*)a->t.table);
    const T* const row = loop_global((const T*)a->l[0].W) + (size_t)((ln & 3) * H + u0 + ((ln & 15) >> 2)) * a->l[0].ldw;
    int tk[BT];
#pragma unroll
    for (int t = 0; t < BT; ++t) tk[t] = a->t.bos;
    for (int e0 = 0; e0 < ne; e0 += LOOP_WAVES * NK) {
      Frag<T> we[NK];
#pragma unroll
      for (int q = 0; q < NK; ++q) {
        const int kk = 32 * (e0 + w + LOOP_WAVES * q) + 8 * (ln >> 4);
        we[q].zero();
        if (kk < E) we[q].load(row + kk);
      }
      if (e0 == 0 && j > 0) {
        const int* const tok = loop_global(a->t.tok) + (size_t)(j & 3) * Bp;
        long long t_end = 0;
        for (int spin = 0;; ++spin) {
          bool some = false;
#pragma unroll
          for (int t = 0; t < BT; ++t) {
            const int b = 16 * (bt0 + min(t, nbt - 1)) + (ln & 15);
            tk[t] = b < a->t.B ? __hip_atomic_load(tok + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            some = some || tk[t] == -1;
          }
          if (dead || !__any(some)) break;
          if ((spin & 15) == 15) {
            const long long now = wall_clock64();
            if (t_end == 0) t_end = now + ticks;
            else if (now > t_end || __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
              dead = true;
              if (lane == 0) atomicOr(gave_up, 1);
            }
          }
        }
      }
#pragma unroll
      for (int q = 0; q < NK; ++q) {
        const int kk = 32 * (e0 + w + LOOP_WAVES * q) + 8 * (ln >> 4);
#pragma unroll
        for (int t = 0; t < BT; ++t) {
          fx[q * BT + t].zero();                                   // (a wait given up: any token in range)
          if (kk < E) fx[q * BT + t].load(table + (size_t)((unsigned)tk[t] < (unsigned)V ? tk[t] : 0) * E + kk);
        }
      }
#pragma unroll
      for (int q = 0; q < NK; ++q)
#pragma unroll
        for (int t = 0; t < BT; ++t) mma16(acc[0][t], we[q], fx[q * BT + t]);
    }
  };

  // One layer of one position: the recurrent half first, whose state was sent a position ago, while the input is on its way.
  auto layer = [&](auto lc, int j) {
    constexpr int l = decltype(lc)::value, lo = l > 0 ? l - 1 : 0;
    if constexpr (DEC && l == 0) {
      if (j > 0) {
        const T* x = loop_global((const T*)A()->XO) + (size_t)j * slot;
        VocabRows wo[PD];
        first_rows(wo);
        LOOP_PHASE();
        issue(x, 0);
        settle(x, 0);
        best_tokens(j - 1, wo);
        clear();
        multiply(wx[0], 0);
      } else clear();
    } else clear();
    {
      Frag<T> f[NK];
      if (l >= LREG) from_lds(l - LREG, f);
      const T* h = states(l, j);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        issue(h, ch);
        settle(h, ch);
        if (l < LREG) multiply(wh[l < LREG ? l : 0], ch);
        else multiply(f, ch);
      }
    }
    if constexpr (DEC && l == 0) embedding(j);
    const T* x = nullptr;
    if constexpr (!(DEC && l == 0)) {
      const auto a = A();
      x = l == 0 ? loop_global((const T*)a->XO) + (size_t)j * slot
                 : a->l[lo].XY ? loop_global((const T*)a->l[lo].XY) + (size_t)j * slot : loop_global((const T*)a->l[lo].X) + (size_t)(j + 1) * slot;
    }
    if constexpr (!(DEC && l == 0)) {
      if (l > 0) recur_nap(nap);
      else LOOP_PHASE();
      issue(x, 0);
    }
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      if constexpr (!(DEC && l == 0)) {
        settle(x, ch);
        multiply(wx[l], ch);
      }
      spread(ch);
      const auto a = A();
      T* const ys = loop_global((T*)a->l[l].XY), * const yr = loop_global((T*)a->l[l].Y), * const xs = loop_global((T*)a->l[l].X);
      T* const hr = loop_global((T*)a->l[l].H);
      const int ldh = a->l[l].ldh;
      float* const cs = loop_global(a->l[l].C), * const gs = loop_global(a->l[l].G);
      loop_barrier();
      const float* r = red;
      red = red == red_[0] ? red_[1] : red_[0];
      if (ch + 1 < NCH) issue(x, ch + 1);
      if (mine && w >= ch * BT && w < ch * BT + BT) {
        int ln = lane;
        LOOP_FRESH(ln);
        const int uw = ln & 3, sl = ln >> 2, b = 16 * btw + sl;
        v4f pre = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < LOOP_WAVES; ++k)
          pre += *reinterpret_cast<const v4f*>(r + ((k * BT + w - ch * BT) * 64 + loop_pos(sl, uw)) * 4);
        float add[4], g[4];
        if (l == 0 && !DEC) {
#pragma unroll
          for (int q = 0; q < 4; ++q) add[q] = gx[q];
        } else {
          const v4f bv = *reinterpret_cast<const v4f*>(&s_bias[l][uw][0]);
#pragma unroll
          for (int q = 0; q < 4; ++q) add[q] = bv[q];
        }
        const float state = seq_cell<FAST>(pre, add, mask, hcar[l], c[l], g);
        hcar[l] = FAST ? bf2f(f2bf(state)) : state;
        const unsigned off_x = (unsigned)fm_offset(b, u0, ns), off_h = (unsigned)(b * ldh + u0);
        if (!DEC && yr) {
          const DropSpec drop = seq_drop(DropSpec{a->l[l].drop.key0, a->l[l].drop.thresh, a->l[l].drop.scale, a->l[l].drop.width, 1},
                                         a->drop_step, j);
          loop_quad_put(ys + (size_t)j * slot, off_x, yr + (size_t)j * Bp * ldh, off_h, state * drop_factor(drop, b, u0 + uw), ln, true);
        }
        loop_quad_put(xs + (size_t)(j + 1) * slot, off_x, DEC ? (T*)nullptr : hr + (size_t)(j + 1) * Bp * ldh, off_h, state, ln, true);
        if (DEC) continue;
        asm volatile("" ::: "memory");                             // (the state first: the other workgroups wait for it)
        *(float*)((char*)(cs + (size_t)(j + 1) * Bp * H) + (unsigned)(b * H + u0 + uw) * 4u) = c[l];
        char* const gj = (char*)(gs + (size_t)j * Bp * 4 * H);
#pragma unroll
        for (int q = 0; q < 4; ++q) *(float*)(gj + (size_t)q * H * 4 + (unsigned)(b * 4 * H + u0 + uw) * 4u) = g[q];
      }
    }
  };

  // A wavefront's rows of the scores: task t = sentence t % NB, rows t / NB, + np, ...; the keys of the first four are requested
  // ahead of the top layer's cells.
  Frag<T> kr[4][NQ];
  auto key_rows = [&](int t, int i0, int n) {
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const T* const K = loop_global((const T*)a->K) + (size_t)(16 * bt0 + t % NB) * H;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        kr[r][q].zero();
        if (i0 + np * r < n && 8 * ln + 512 * q < H) kr[r][q].load(K + (size_t)(i0 + np * r) * Bp * H + 512 * q + (unsigned)(8 * ln));
      }
  };

  // Softmax over at most tps * QT source positions, mix, tanh -> H_o.  The rows of the first positions are requested before the
  // workgroup's sums W_c2 H_t meet.
  auto mix = [&](auto qc, int j) {
    constexpr int QT = decltype(qc)::value, PF = QT < 8 ? QT : 8;
    typedef typename std::conditional<FAST, uint2, float4>::type P4;
    P4 pr[PF];
    auto rows = [&](int s0, int q0) {
      int ln = lane;
      LOOP_FRESH(ln);
      const int sr = ln & (tps - 1), bs = s0 + w * spw + ln / tps, bc = min(bs, NB - 1), n = bs < NB ? s_len[bc] : 0;
      const unsigned off = (unsigned)((16 * bt0 + bc) * S + sr);
      const char* const pg = (const char*)loop_global(A()->Pg) + (size_t)place.pos * Bp * S * sizeof(P4);
#pragma unroll
      for (int q = 0; q < PF; ++q)
        if (sr + tps * (q0 + q) < n) pr[q] = *(const P4*)(pg + (size_t)((q0 + q) * tps * (int)sizeof(P4)) + off * (unsigned)sizeof(P4));
    };
    rows(0, 0);
    loop_barrier();                                                // (s_u is there)
    for (int s0 = 0; s0 < NB; s0 += LOOP_WAVES * spw) {
      const auto a = A();
      int ln = lane;
      LOOP_FRESH(ln);
      const int sr = ln & (tps - 1), bs = s0 + w * spw + ln / tps, bc = min(bs, NB - 1), bg = 16 * bt0 + bc, n = bs < NB ? s_len[bc] : 0;
      const unsigned off = (unsigned)(bg * S + sr);
      if (s0 > 0) rows(s0, 0);
      LOOP_PHASE();
      float sv[QT];
      loop_words_issue<QT>(loop_global(a->scores) + (size_t)j * Bp * S, 4 * tps, 4 * off, sr, tps, n, sv, true);
      loop_words_settle<QT>(loop_global(a->scores) + (size_t)j * Bp * S, 4 * tps, 4 * off, sv, dead, gave_up, ticks);
      float mx = -INFINITY;
#pragma unroll
      for (int q = 0; q < QT; ++q) mx = sr + tps * q < n ? fmaxf(mx, sv[q]) : mx;
      mx = loop_group(mx, tps, [](float x, float y) { return fmaxf(x, y); });
      const auto plus = [](float x, float y) { return x + y; };
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        sv[q] = sr + tps * q < n ? expf(sv[q] - mx) : 0.f;
        sum += sv[q];
        if (QT > 8) __builtin_amdgcn_sched_barrier(0);             // (one at a time: registers)
      }
      sum = loop_group(sum, tps, plus);
      const float inv = n > 0 ? 1.f / sum : 0.f;
      float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q0 = 0; q0 < QT; q0 += PF) {
        if (q0 > 0) rows(s0, q0);
#pragma unroll
        for (int q = 0; q < PF; ++q) {
          sv[q0 + q] *= inv;
          if (!(sr + tps * (q0 + q) < n)) continue;
          float pv[4];
          if constexpr (FAST) {
            pv[0] = __uint_as_float(pr[q].x << 16); pv[1] = __uint_as_float(pr[q].x & 0xffff0000u);
            pv[2] = __uint_as_float(pr[q].y << 16); pv[3] = __uint_as_float(pr[q].y & 0xffff0000u);
          } else {
            pv[0] = pr[q].x; pv[1] = pr[q].y; pv[2] = pr[q].z; pv[3] = pr[q].w;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] += sv[q0 + q] * pv[e];
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = loop_group(o[e], tps, plus);
      const float pre = ((ln & 2) ? ((ln & 1) ? o[3] : o[2]) : ((ln & 1) ? o[1] : o[0])) + s_u[bc][ln & 3];
      const float hv = tanh_of<FAST>(pre);
      if (bs < NB && sr < 4) {
        const unsigned at = (unsigned)(bg * a->ldho + u0), xat = (unsigned)fm_offset(bg, u0, ns);
        T* const xo = loop_global((T*)a->XO) + (size_t)(j + 1) * slot;
        const size_t jrow = (size_t)(j + 1) * Bp * a->ldho;
        T* const ho = loop_global((T*)a->Ho) + jrow;
        if (!DEC && a->HoD) {
          const DropSpec drop = seq_drop(DropSpec{a->drop_o.key0, a->drop_o.thresh, a->drop_o.scale, a->drop_o.width, 1}, a->drop_step, j);
          loop_quad_put(xo, xat, loop_global((T*)a->HoD) + jrow, at, hv * drop_factor(drop, bg, u0 + (ln & 3)), ln, true);
          loop_quad_put(xo, xat, ho, at, hv, ln, false);
        } else loop_quad_put(xo, xat, DEC ? (T*)nullptr : ho, at, hv, ln, true);
        asm volatile("" ::: "memory");
      }
      if (!DEC && bs < NB && bs % plan.nwg == place.pos) {         // the weights of this sentence: one workgroup stores them
        char* const aj = (char*)(loop_global(a->a) + (size_t)j * Bp * S);
#pragma unroll
        for (int q = 0; q < QT; ++q)
          if (sr + tps * q < S) *(float*)(aj + (size_t)(4 * q * tps) + 4 * off) = sv[q];
      }
    }
  };

  const int task0 = place.pos * LOOP_WAVES + w, tasks = NB * np;
  for (int j = 0; j < Tn; ++j) {
    layer(std::integral_constant<int, 0>{}, j);
    if (L > 1) layer(std::integral_constant<int, 1>{}, j);
    if constexpr (LM > 2) {
      if (L > 2) layer(std::integral_constant<int, 2>{}, j);
      if (L > 3) layer(std::integral_constant<int, 3>{}, j);
    }
    const T* ht = states(L - 1, j + 1);
    // ---- scores: K_i . H_t, a wavefront per row ----------------------------------------------------------------------
    for (int t = task0; t < tasks; t += plan.nwg * LOOP_WAVES) {
      const auto a = A();
      int ln = lane;
      LOOP_FRESH(ln);
      const int part = t / NB, bs = t - part * NB, n = __builtin_amdgcn_readfirstlane(s_len[bs]), bg = 16 * bt0 + bs;
      float* const sc = loop_global(a->scores) + ((size_t)j * Bp + bg) * S;
      Frag<T> hv[NQ];
      key_rows(t, part, n);
      LOOP_PHASE();
      const T* hrow = ht + (size_t)(bg >> 4) * ns * 512 + (bg & 15) * 8;
      auto piece = [&](int q, unsigned zero) {                     // (a lane beyond the row's end repeats the first)
        const int p = (8 * ln + 512 * q < H ? ln + 64 * q : 0) + (int)zero;
        return (unsigned)((p >> 2) * 512 + (p & 3) * 128) * (unsigned)sizeof(T);
      };
      loop_issue<T, NQ>(hrow, piece, hv);
      loop_settle<T, NQ>(hrow, piece, hv, dead, gave_up, ticks);
      for (int i0 = part; i0 < n; i0 += 4 * np) {
        if (i0 != part) key_rows(t, i0, n);
        float s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[r] = 0.f;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[r] += kr[r][q].get(e) * hv[q].get(e);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = loop_wave_sum(s[r]);
        const float sv = ln == 0 ? s[0] : ln == 1 ? s[1] : ln == 2 ? s[2] : s[3];
        if (ln < 4 && i0 + np * ln < n) loop_put(sc + (unsigned)(i0 + np * ln), sv);
      }
    }
    // ---- W_c2 H_t for this workgroup's four columns -------------------------------------------------------------------
    clear();
    issue(ht, 0);
    {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        settle(ht, ch);
        if constexpr (CL > 0) {
          Frag<T> f[NK];
#pragma unroll
          for (int q = 0; q < NK; ++q) f[q] = q < CL ? wl[(LLDS * NK + (q < CL ? q : 0)) * LOOP_WAVES * 64] : wc[q < CL ? 0 : q - CL];
          multiply(f, ch);
        } else multiply(wc, ch);
        spread(ch);
        if (ch + 1 < NCH) issue(ht, ch + 1);
        else if (j + 1 < Tn) fetch(j + 1);
        loop_barrier();
        const float* r = red;
        red = red == red_[0] ? red_[1] : red_[0];
        if (mine && w >= ch * BT && w < ch * BT + BT) {
          float v = 0.f;
#pragma unroll
          for (int k = 0; k < LOOP_WAVES; ++k) v += r[((k * BT + w - ch * BT) * 64 + loop_pos(lane >> 2, 0)) * 4 + (lane & 3)];
          s_u[16 * w + (lane >> 2)][lane & 3] = v;
        }
      }
    }
    if (S <= 4 * tps) mix(std::integral_constant<int, 4>{}, j);
    else if (S <= 8 * tps) mix(std::integral_constant<int, 8>{}, j);
    else mix(std::integral_constant<int, LOOP_QT>{}, j);
  }
  if constexpr (DEC) {                                             // the last step's token
    VocabRows wo[PD];
    first_rows(wo);
    const T* x = loop_global((const T*)A()->XO) + (size_t)Tn * slot;
    issue(x, 0);
    settle(x, 0);
    best_tokens(Tn - 1, wo);
  }
}

// The same loop by one workgroup per 16 sentences that waits for no other: it reads every weight at every position.  For a
// launch above that gave up a wait, and nothing to do otherwise.
template <typename T, bool DEC>
__global__ __launch_bounds__(64 * LOOP_WAVES) void loop_fwd_solo_kernel(const int* gave_up, int L, int Tn, int Bp, int H, int S, LoopFwdArgs args) {
  if (!recur_again(gave_up, args.again)) return;
  constexpr bool FAST = sizeof(T) == 2;
  __shared__ float s_a[16][LOOP_MAX_SRC];
  __shared__ float s_bv[LOOP_WAVES][16];
  __shared__ int s_bi[LOOP_WAVES][16], s_tok[16], s_fin[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, b0 = 16 * blockIdx.x, b = b0 + (lane & 15), kl = 8 * (lane >> 4);
  const bool drop = !DEC && args.HoD != nullptr;
  if (DEC) {
    if (threadIdx.x < 16) { s_tok[threadIdx.x] = args.t.bos; s_fin[threadIdx.x] = 0; }
    for (int i = threadIdx.x; i < 16 * Tn; i += 64 * LOOP_WAVES)
      if (b0 + i / Tn < args.t.B) args.t.out_ids[(size_t)b0 * Tn + i] = args.t.pad;
    __syncthreads();
  }
  for (int j = 0; j < Tn; ++j) {
    const float mask = DEC ? (b < args.t.B ? 1.f : 0.f) : args.mask[(size_t)j * Bp + b];
    for (int l = 0; l < L; ++l) {
      const LoopFwdLayer d = args.l[l];
      const T* hp = (const T*)d.H + ((size_t)j * Bp + b) * d.ldh;
      const T* x = l == 0 ? (const T*)(drop ? args.HoD : args.Ho) + ((size_t)j * Bp + b) * args.ldho
                          : args.l[l - 1].Y ? (const T*)args.l[l - 1].Y + ((size_t)j * Bp + b) * d.ldh
                                            : (const T*)args.l[l - 1].H + ((size_t)(j + 1) * Bp + b) * d.ldh;
      for (int rt = w; rt < H >> 2; rt += LOOP_WAVES) {            // tiles of 4 units x 4 gates
        v4f pre = v4f{0.f, 0.f, 0.f, 0.f};
        const int m = lane & 15;
        const T* wr = (const T*)d.W + (size_t)((m & 3) * H + 4 * rt + (m >> 2)) * d.ldw;
        for (int k0 = 0; k0 < H; k0 += 32) {
          const int k = k0 + kl;
          Frag<T> fw, fx, gw, gh;
          fw.zero(); fx.zero(); gw.zero(); gh.zero();
          if (k < H) { fw.load(wr + d.wx_off + k); fx.load(x + k); gw.load(wr + d.wh_off + k); gh.load(hp + k); }
          mma16(pre, fw, fx);
          mma16(pre, gw, gh);
        }
        if (DEC && l == 0) {
          const T* xe = (const T*)args.t.table + (size_t)s_tok[lane & 15] * args.t.emb;
          for (int k0 = 0; k0 < args.t.emb; k0 += 32) {
            const int k = k0 + kl;
            Frag<T> fw, fx;
            fw.zero(); fx.zero();
            if (k < args.t.emb) { fw.load(wr + k); fx.load(xe + k); }
            mma16(pre, fw, fx);
          }
        }
        const int u = 4 * rt + (lane >> 4);
        const size_t at = (size_t)j * Bp + b, next = at + Bp;
        float add[4], g[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) add[q] = l == 0 && !DEC ? args.gx[at * 4 * H + (size_t)q * H + u] : d.bias[q * H + u];
        float c = d.C[at * H + u];
        const float state = seq_cell<FAST>(pre, add, mask, to_f<T>(hp[u]), c, g);
        ((T*)d.H)[next * d.ldh + u] = from_f<T>(state);
        d.C[next * H + u] = c;
        if (DEC) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) d.G[at * 4 * H + (size_t)q * H + u] = g[q];
        if (d.Y) ((T*)d.Y)[at * d.ldh + u] = from_f<T>(state * drop_factor(seq_drop(d.drop, args.drop_step, j), b, u));
      }
      __syncthreads();
    }
    const T* ht = (const T*)args.l[L - 1].H + (size_t)(j + 1) * Bp * args.l[L - 1].ldh;
    const int ldh = args.l[L - 1].ldh;
    for (int s = w; s < 16; s += LOOP_WAVES) {                     // scores and softmax, a wavefront per sentence
      const int bg = b0 + s, n = min(args.len[bg], S);
      float* const sc = args.scores + ((size_t)j * Bp + bg) * S;
      for (int i = 0; i < n; ++i) {
        const T* kr = (const T*)args.K + ((size_t)i * Bp + bg) * H;
        float v = 0.f;
        for (int k = lane; k < H; k += 64) v += to_f<T>(kr[k]) * to_f<T>(ht[(size_t)bg * ldh + k]);
        v = wave_sum(v);
        if (lane == (i & 63)) { s_a[s][i] = v; sc[i] = v; }
      }
      // (lane i % 64 wrote position i and reads it)
      float mx = -INFINITY, sum = 0.f;
      for (int i = lane; i < n; i += 64) mx = fmaxf(mx, s_a[s][i]);
      mx = wave_max(mx);
      for (int i = lane; i < n; i += 64) { const float e = expf(s_a[s][i] - mx); s_a[s][i] = e; sum += e; }
      sum = wave_sum(sum);
      const float inv = n > 0 ? 1.f / sum : 0.f;
      for (int i = lane; i < S; i += 64) {
        const float a = i < n ? s_a[s][i] * inv : 0.f;
        s_a[s][i] = a;
        if (!DEC) args.a[((size_t)j * Bp + bg) * S + i] = a;
      }
    }
    __syncthreads();
    const int n = min(args.len[b], S);
    for (int ct = w; ct < H >> 4; ct += LOOP_WAVES) {              // tiles of 16 columns of H_o
      v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
      for (int k0 = 0; k0 < H; k0 += 32) {
        const int k = k0 + kl;
        Frag<T> fw, fx;
        fw.zero(); fx.zero();
        if (k < H) { fw.load((const T*)args.Wc + (size_t)(16 * ct + (lane & 15)) * args.ldwc + k); fx.load(ht + (size_t)b * ldh + k); }
        mma16(acc, fw, fx);
      }
      const int u = 16 * ct + 4 * (lane >> 4);
      for (int i = 0; i < n; ++i) {
        const float a = s_a[lane & 15][i];
        const T* pr = (const T*)args.P + ((size_t)i * Bp + b) * H + u;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += a * to_f<T>(pr[e]);
      }
      const size_t at = ((size_t)(j + 1) * Bp + b) * args.ldho + u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float hv = tanh_of<FAST>(acc[e]);
        ((T*)args.Ho)[at + e] = from_f<T>(hv);
        if (drop) ((T*)args.HoD)[at + e] = from_f<T>(hv * drop_factor(seq_drop(args.drop_o, args.drop_step, j), b, u + e));
      }
    }
    __syncthreads();
    if (DEC) {                                                     // the best token: 16 vocabulary entries at a time
      const LoopTokens& t = args.t;
      const T* ho = (const T*)args.Ho + ((size_t)(j + 1) * Bp + b) * args.ldho;
      float bv = -INFINITY;
      int bi = 0x7fffffff;
      for (int tl = w; tl < (t.V + 15) >> 4; tl += LOOP_WAVES) {
        v4f z = v4f{0.f, 0.f, 0.f, 0.f};
        const int row = min(16 * tl + (lane & 15), t.V - 1);
        for (int k0 = 0; k0 < H; k0 += 32) {
          const int k = k0 + kl;
          Frag<T> fw, fx;
          fw.zero(); fx.zero();
          if (k < H) {
            fw.load((const T*)t.Wo + (t.fm ? ((size_t)tl * ((H + 31) >> 5) + (k0 >> 5)) * 512 + lane * 8 : (size_t)row * H + k));
            fx.load(ho + k);
          }
          mma16(z, fw, fx);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 16 * tl + 4 * (lane >> 4) + i;
          if (v < t.V) {
            const float x = z[i] + t.Bo[v];
            if (x > bv) { bv = x; bi = v; }
          }
        }
      }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
      if (lane < 16) { s_bv[w][lane] = bv; s_bi[w][lane] = bi; }
      __syncthreads();
      if (threadIdx.x < 16) {
        const int s = threadIdx.x;
        bv = s_bv[0][s]; bi = s_bi[0][s];
        for (int q = 1; q < LOOP_WAVES; ++q)
          if (s_bv[q][s] > bv || (s_bv[q][s] == bv && s_bi[q][s] < bi)) { bv = s_bv[q][s]; bi = s_bi[q][s]; }
        const int token = (unsigned)bi < (unsigned)t.V ? bi : 0;
        s_tok[s] = token;
        if (b0 + s < t.B && !s_fin[s]) {
          t.out_ids[(size_t)(b0 + s) * Tn + j] = token;
          if (token == t.eos || j == Tn - 1) { t.out_len[b0 + s] = j + 1; s_fin[s] = 1; }
        }
      }
      __syncthreads();
    }
  }
}

template <bool DEC>
static void loop_fwd_go(int prec, const LoopFwdArgs& args, int L, int T, int Bp, int H, int S, const SeqRun& run, hipStream_t st) {
  const LoopPlan p = loop_plan(prec, L, Bp, H, S, std::min(run.cus, 256));
  LoopFwdArgs a = args;
  a.wait_ticks = run.mode == SEQ_RUN_GIVE_UP ? 0 : RECUR_WAIT_TICKS;
  // s_sleep units before the input of a layer above the bottom one is looked for, where the reading of its recurrent half does not take
  // as long as the exchange: whole evaluations with 0 | 16 units, us: attn 1874 | 1770, paper_512x2 846 | 809, 336 units x 3 layers
  // 714 | 669, medium 2216 | 2268.
  const int nap = p.nk * p.bt < 16 ? 16 : 0;
  const dim3 grid(p.groups * p.nwg), block(64 * LOOP_WAVES);
  // (decoding networks of one or two layers: the registers that more would take hold tiles of W_o on their way)
#define GO(TT, NK, BT)                                                                                                             \
  do {                                                                                                                             \
    if (DEC && L <= 2) hipLaunchKernelGGL((loop_fwd_kernel<TT, NK, BT, 1, DEC, DEC ? 2 : 4>), grid, block, 0, st, a, L, T, Bp, H, S, p, nap); \
    else hipLaunchKernelGGL((loop_fwd_kernel<TT, NK, BT, 1, DEC, 4>), grid, block, 0, st, a, L, T, Bp, H, S, p, nap);               \
  } while (0)
  if (prec) {
    if (p.nk == 1) { if (p.bt == 1) GO(bf16_t, 1, 1); else GO(bf16_t, 1, 2); }
    else if (p.nk == 2) { if (p.bt == 1) GO(bf16_t, 2, 1); else if (p.bt == 2) GO(bf16_t, 2, 2); else GO(bf16_t, 2, 4); }
    else if (p.nch > 1) { if constexpr (!DEC) hipLaunchKernelGGL((loop_fwd_kernel<bf16_t, 4, 2, 4, false, 4>), grid, block, 0, st, a, L, T, Bp, H, S, p, nap); }
    else { if (p.bt == 1) GO(bf16_t, 4, 1); else if (p.bt == 2) GO(bf16_t, 4, 2); else GO(bf16_t, 4, 4); }
  } else {
    if (p.nk == 1) { if (p.bt == 1) GO(float, 1, 1); else GO(float, 1, 2); }
    else { if (p.bt == 1) GO(float, 2, 1); else if (p.bt == 2) GO(float, 2, 2); else GO(float, 2, 4); }
  }
#undef GO
  if (prec) hipLaunchKernelGGL((loop_fwd_solo_kernel<bf16_t, DEC>), dim3(Bp >> 4), block, 0, st, a.ticket + 1, L, T, Bp, H, S, a);
  else hipLaunchKernelGGL((loop_fwd_solo_kernel<float, DEC>), dim3(Bp >> 4), block, 0, st, a.ticket + 1, L, T, Bp, H, S, a);
}

}  // namespace cmt

// The decoder's time loop in one launch: all layers, the attention and the attentional layer of every target position, forward
// and backward, by workgroups that stay on the chip and keep their share of all layers' weights in registers and LDS.
//
// A launch per layer and position reads the layer's weights again at every position and pays a launch (2.4 us) and the head and
// tail of a kernel for each of the L + 2 dependent steps of a position: 7 - 9 us a step at width 1024, 64 sentences.  Here a step
// costs an exchange instead: what a workgroup has computed goes out in write-once slots of memory that are their own flags
// (recur.hip), and the others read it.  Sentences do not interact, so a group of workgroups serves up to 128 of them (loop_plan):
// H / 4 workgroups own four units of every layer each, i.e. 16 gate rows x all of k.  All weights of four layers of width 1024 are 66 MB
// of the 172 MB of registers and LDS of 256 CUs; the 8 wavefronts of a workgroup split k and meet in LDS.
//
// What bounds a position.  Forward at width 1024, 4 layers, 64 sentences 20.8 us (a launch per step 44), of which a layer takes
// 3.7: its state and its input are 128 KB each that every CU reads through its L1 at no more than 64 bytes a clock (1.0 - 1.6 us each
// measured, 0.85 at that rate), then 0.65 until the sums have met, 0.5 the cells, 0.7 until a store can be seen.  So the recurrent
// half is read while the layer below is still being exchanged.  Narrow layers are bound by the exchange alone: width 512, 2 layers,
// 32 sentences 9 us a position (21).  Backward 36 us (54) and 15 us (24): a layer is two exchanges there.
// Counted (64 | 128 sentences, width 1024): a CU's L1 takes 1.38 | 2.85 MB a position from L2 forward, 9 of 20.8 | 19 of 51 us at 64 bytes
// a clock, and 1.00 | 2.03 MB backward, 6.5 of 36 | 13 of 59 us: volume is less than half of either, the rest are the exchanges.
// Whole steps with everything else alike, launch per step | one launch, ms: medium 8.33 | 6.45, attn 7.68 | 5.10, small (fp32)
// 8.99 | 6.45, 336 units x 3 layers, 23 sentences 2.99 | 1.92, large 21.9 | 20.3; forward-only evaluation of medium 3.17 | 2.20.
//
// The waits are bounded, and a launch behind each loop makes it again without waits where one was given up, as the encoder's
// recurrences have it; loops of several streams are kept apart (section_gate.h).
#include <algorithm>
#include <type_traits>

#include "loop_fwd.h"

namespace cmt {

// ------------------------------------------------------------------------------------------------
// backward
// ------------------------------------------------------------------------------------------------
// Per position dpre, its scores with the projected rows, the gradient of H_t and the top layer's cells, then per layer the
// product of the gate gradients with the layer's weights.  That one's contraction is over 4H gate rows: four workgroups, one
// per gate, take the same 16 columns (input and recurrent ones: two full tiles), so that a workgroup reads H gate gradients
// of every sentence instead of 4H - what a phase takes is the time its loads take to pass a CU's L1 - and send each other
// partial sums for their four units.  Those go through a few slots that are used again every other position: the reader puts
// the empty pattern back, a position before the slot's next writer could come (it needs gate gradients that the reader sends
// afterwards).
// s_sleep units before a workgroup looks for a layer's gate gradients, and for its partial sums
struct LoopNaps { int gates, sums; };
template <typename T, int NK, int BT>
__global__ __launch_bounds__(64 * LOOP_WAVES) void loop_bwd_kernel(LoopBwdArgs args_, int L, int Tn, int Bp, int H, int S, LoopPlan plan, LoopNaps nap) {
  constexpr bool FAST = sizeof(T) == 2;
  constexpr int LREG = NK * sizeof(T) >= 8 ? 1 : 4;                // layers whose recurrent columns are in registers, not LDS
  constexpr int CL = LREG < LOOP_MAX_LAYERS ? NK - 1 : 0;          // fragments of W_c2 in LDS beside them
  constexpr int NL = (LOOP_MAX_LAYERS - LREG) * NK + CL;
  constexpr int NQ = (NK * 32 * LOOP_WAVES + 511) / 512;           // 8-element pieces of a row per lane
  constexpr int RW = NQ > 1 || !FAST ? 2 : 4;                               // rows of scores that a wavefront has in flight
  __shared__ __align__(16) float red[LOOP_WAVES * BT * 256];
  __shared__ Frag<T> wlds[NL ? NL * LOOP_WAVES * 64 : 1];
  __shared__ float s_u[LOOP_MAX_BATCH][4];
  __shared__ int s_len[LOOP_MAX_BATCH];
  __shared__ int s_dead;
  const LoopPlace place = loop_place(blockIdx.x, plan.groups, plan.nwg);
  if (place.group >= plan.groups || place.pos >= plan.nwg) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u0 = 4 * place.pos, cg = place.pos >> 2, gate = place.pos & 3;
  const int bt0 = place.group * plan.tiles, nbt = min(plan.tiles, (Bp >> 4) - bt0), NB = 16 * nbt;
  const int ns = (H + 31) >> 5;
  const size_t slot = (size_t)Bp * ns * 32;
  const auto A = [] { return loop_args<LoopBwdArgs>(); };
  int* const gave_up = loop_global(A()->ticket) + 1;
  const int ticks = A()->wait_ticks;
  if (threadIdx.x == 0) {
    if (ticks == 0) atomicOr(gave_up, 1);
    s_dead = __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int i = threadIdx.x; i < NB; i += 64 * LOOP_WAVES) s_len[i] = min(loop_global(A()->len)[16 * bt0 + i], S);
  // ---- weights ----------------------------------------------------------------------------------------------------------
  bool kin[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q) kin[q] = 32 * (w + LOOP_WAVES * q) + 8 * (lane >> 4) < H;
  Frag<T> wx[LOOP_MAX_LAYERS][NK], wh[LREG][NK], wc[NK - CL];
  Frag<T>* const wl = wlds + (size_t)w * 64 + lane;                // + ((layer - LREG) * NK + q) * LOOP_WAVES * 64
#pragma unroll
  for (int l = 0; l < LOOP_MAX_LAYERS; ++l)
    if (l < L) {
      const auto a = A();
      const int ld = a->l[l].ldw;
      const T* wt = loop_global((const T*)a->l[l].Wt) + (size_t)(16 * cg + (lane & 15)) * ld + (size_t)gate * H;
      const T* xr = wt + (size_t)a->l[l].x_row * ld, * hr = wt + (size_t)a->l[l].h_row * ld;
#pragma unroll
      for (int q = 0; q < NK; ++q) {
        const int k = 32 * (w + LOOP_WAVES * q) + 8 * (lane >> 4);
        Frag<T> f;
        f.zero(); wx[l][q].zero();
        if (kin[q]) { wx[l][q].load(xr + k); f.load(hr + k); }
        if (l < LREG) wh[l < LREG ? l : 0][q] = f;
        else wl[((l - LREG) * NK + q) * LOOP_WAVES * 64] = f;
      }
    }
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const auto a = A();
    Frag<T> f;
    f.zero();
    if (kin[q]) f.load(loop_global((const T*)a->Wct) + (size_t)(u0 + (lane & 3)) * H + 32 * (w + LOOP_WAVES * q) + 8 * (lane >> 4));
    if (q < CL) wl[(NL - CL + q) * LOOP_WAVES * 64] = f;
    else wc[q < CL ? 0 : q - CL] = f;
  }
  // ---- cells: a wavefront takes 2 nbt sentences, a lane one unit of one of them (surplus lanes repeat the last) -----------
  const int per = 2 * nbt;
  const bool real = lane < 4 * per;
  float dc[LOOP_MAX_LAYERS], dh[LOOP_MAX_LAYERS], cn[LOOP_MAX_LAYERS];
#pragma unroll
  for (int l = 0; l < LOOP_MAX_LAYERS; ++l)
    if (l < L) {
      const int b = 16 * bt0 + w * per + min(lane >> 2, per - 1);
      dc[l] = 0.f; dh[l] = 0.f;
      cn[l] = loop_global(A()->l[l].C)[((size_t)Tn * Bp + b) * H + u0 + (lane & 3)];
    }
  const int np = max(1, plan.nwg * LOOP_WAVES / NB);               // wavefronts per sentence of the scores
  int spw = nbt > 2 ? 8 : 2 * nbt;                                 // mix: sentences per wavefront and pass, threads per sentence
  if (S > 8 * (64 / spw)) spw >>= 1;
  const int tps = 64 / spw;
  __syncthreads();
  bool dead = s_dead != 0;
  const unsigned tile = (unsigned)ns * 512u * (unsigned)sizeof(T);
  Frag<T> fx[NK * BT];
  // tiles of a slot: `step` bytes apart
  auto issue = [&](const T* x, unsigned step, int ch) {
    int ln = lane;
    LOOP_FRESH(ln);
    loop_issue<T, NK * BT>(x, [&](int i, unsigned z) { return loop_frag_at<T, BT>(i, z, step, ns, H, w, ch * BT, nbt, ln); }, fx);
  };
  auto settle = [&](const T* x, unsigned step, int ch) {
    loop_settle<T, NK * BT>(x, [&](int i, unsigned z) { return loop_frag_at<T, BT>(i, z, step, ns, H, w, ch * BT, nbt, lane); }, fx, dead, gave_up,
                            ticks);
  };
  auto multiply = [&](const Frag<T> (&wf)[NK], v4f (&acc)[BT]) {
#pragma unroll
    for (int t = 0; t < BT; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
      for (int t = 0; t < BT; ++t) mma16(acc[t], wf[q], fx[q * BT + t]);
  };
  auto spread = [&](const v4f (&acc)[BT]) {
    int ln = lane;
    LOOP_FRESH(ln);
#pragma unroll
    for (int t = 0; t < BT; ++t) *reinterpret_cast<v4f*>(red + ((w * BT + t) * 64 + loop_pos(ln & 15, ln >> 4)) * 4) = acc[t];
  };
  // (weights at fragment n of the LDS, the last ones in `more`)
  auto multiply_lds = [&](int n, auto count, const auto& more, v4f (&acc)[BT]) {
    constexpr int QL = decltype(count)::value;
#pragma unroll
    for (int t = 0; t < BT; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      const Frag<T> f = q < QL ? wl[(n + (q < QL ? q : 0)) * LOOP_WAVES * 64] : more[q < QL ? 0 : q - QL];
#pragma unroll
      for (int t = 0; t < BT; ++t) mma16(acc[t], f, fx[q * BT + t]);
      __builtin_amdgcn_sched_barrier(0);                           // (one fragment of weights at a time: registers)
    }
  };
  // partial sums: [position & 1][input, recurrent][unit / 4][gate][sentence][4]
  const size_t pplane = (size_t)H * Bp * 4;
  auto fresh = [&]() { int ln = lane; LOOP_FRESH(ln); return ln; };
  auto part_at = [&](float* p, int j, int kind, int quad) { return p + ((size_t)(j & 1) * 2 + kind) * pplane + (size_t)quad * 16 * Bp; };
  // this workgroup's sums of one tile, for the four workgroups that own its columns
  auto send = [&](float* part, int j, int kind, int t, int ch) {
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
    int ln = lane;
    LOOP_FRESH(ln);
#pragma unroll
    for (int k = 0; k < LOOP_WAVES; ++k) v += *reinterpret_cast<const v4f*>(red + ((k * BT + t) * 64 + loop_pos(ln & 15, ln >> 4)) * 4);
    if (ch * BT + t >= nbt) return;
    const int b = 16 * (bt0 + ch * BT + t) + (ln & 15);
    uint64_t* d = reinterpret_cast<uint64_t*>(part_at(part, j, kind, 4 * cg) + (unsigned)((ln >> 4) * 16 * Bp + (gate * Bp + b) * 4));
    const uint64_t lo = (uint64_t)__float_as_uint(loop_word(v[0])) | ((uint64_t)__float_as_uint(loop_word(v[1])) << 32);
    const uint64_t hi = (uint64_t)__float_as_uint(loop_word(v[2])) | ((uint64_t)__float_as_uint(loop_word(v[3])) << 32);
    __hip_atomic_store(d, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(d + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // the sums for this lane's unit: ask, then take and put the empty pattern back
  auto ask = [&](const float* part, int b, float (&v)[4]) {
    loop_words_issue<4>(part, 16u * (unsigned)Bp, (unsigned)(b * 4 + (fresh() & 3)) * 4u, 0, 0, 1, v, false);
  };
  auto take = [&](float* part, int b, float (&v)[4]) {
    const unsigned off = (unsigned)(b * 4 + (fresh() & 3)) * 4u;
    loop_words_settle<4>(part, 16u * (unsigned)Bp, off, v, dead, gave_up, ticks);
    if (real) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        __hip_atomic_store((unsigned*)((char*)part + (size_t)(q * 16 * Bp) + off), RECUR_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return (v[0] + v[1]) + (v[2] + v[3]);
  };
  struct CellIn { float g[4], cp, mask, rec[4]; };
  auto cell_fetch = [&](int l, int j, CellIn& in) {
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const int b = 16 * bt0 + w * per + min(ln >> 2, per - 1), u = u0 + (ln & 3);
    const char* g = (const char*)(loop_global(a->l[l].G) + (size_t)j * Bp * 4 * H);
#pragma unroll
    for (int q = 0; q < 4; ++q) in.g[q] = *(const float*)(g + (size_t)q * H * 4 + (unsigned)(b * 4 * H + u) * 4u);
    in.cp = loop_global(a->l[l].C)[(size_t)j * Bp * H + (unsigned)(b * H + u)];
    in.mask = loop_global(a->mask)[(size_t)j * Bp + (unsigned)b];
#pragma unroll
    for (int q = 0; q < 4; ++q) in.rec[q] = 0.f;
    if (j + 1 < Tn) ask(part_at(loop_global(a->l[l].part), j + 1, 1, place.pos), b, in.rec);
  };
  // cell backward of layer l: its gate gradients to their slot and rows
  auto cell = [&](int l, int j, CellIn& in, float dy, float& c_next, float& d_h, float& d_c) {
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const int b = 16 * bt0 + w * per + min(ln >> 2, per - 1);
    float rec = 0.f;
    if (j + 1 < Tn) rec = take(part_at(loop_global(a->l[l].part), j + 1, 1, place.pos), b, in.rec);
    float o[4];
    seq_cell_bwd(in.g, in.cp, tanh_of<FAST>(c_next), dy, rec, in.mask, d_h, d_c, o);
    c_next = in.cp;
    T* const xs = loop_global((T*)a->l[l].X) + (size_t)j * 4 * slot + (size_t)(b >> 4) * 4 * ns * 512;
    T* const rows = loop_global((T*)a->l[l].dG) + (size_t)j * Bp * a->l[l].lddg;
    const unsigned lddg = (unsigned)a->l[l].lddg, at = (unsigned)fm_offset(b & 15, u0, ns);
    if constexpr (FAST) {
      const uint64_t v = quad_transpose(f2bf(o[0]), f2bf(o[1]), f2bf(o[2]), f2bf(o[3]), ln);   // gate ln & 3 of the quad's units
      if (real) {
        __hip_atomic_store(reinterpret_cast<uint64_t*>(xs + (unsigned)((ln & 3) * ns * 512) + at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *reinterpret_cast<uint64_t*>(rows + (unsigned)b * lddg + (unsigned)((ln & 3) * H + u0)) = v;
      }
    } else if (real) {
#pragma unroll
      for (int q = 0; q < 4; ++q) loop_put((float*)xs + (unsigned)(q * ns * 512) + at + (ln & 3), o[q]);
#pragma unroll
      for (int q = 0; q < 4; ++q) ((float*)rows)[(unsigned)b * lddg + (unsigned)(q * H + u0 + (ln & 3))] = o[q];
    }
  };

  // what dpre of position j needs besides the feed
  float p_ce = 0.f, p_ho = 0.f;
  int p_row = -1;
  auto dpre_row = [&](int j) {
    int ln = lane;
    LOOP_FRESH(ln);
    p_row = loop_global(A()->pos)[(size_t)j * Bp + (unsigned)(16 * bt0 + w * per + min(ln >> 2, per - 1))];
  };
  auto dpre_fetch = [&](int j) {
    const auto a = A();
    int ln = lane;
    LOOP_FRESH(ln);
    const int b = 16 * bt0 + w * per + min(ln >> 2, per - 1), u = u0 + (ln & 3);
    p_ce = 0.f;
    if (p_row >= 0) p_ce = loop_global(a->dce)[(size_t)p_row * H + u];
    p_ho = to_f<T>((loop_global((const T*)a->Ho) + (size_t)(j + 1) * Bp * a->ldho)[(unsigned)(b * a->ldho + u)]);
  };

  // The recurrent columns' sums of the last chunk go out after the cells (their readers are a position away), in the shadow of
  // what the cells have sent.
  v4f rest[BT];
  auto send_rest = [&](int l, int j) {
    const auto a = A();
    float* const part = loop_global(l == 0 ? a->l[0].part : l == 1 ? a->l[1].part : l == 2 ? a->l[2].part : a->l[3].part);
    loop_barrier();                                                // (`red` has been read)
    spread(rest);
    loop_barrier();
    if (w >= LOOP_WAVES - BT) send(part, j, 1, w - (LOOP_WAVES - BT), (nbt - 1) / BT);
  };
  // One layer's products and the cells of the layer below; `in`: that layer's, on their way.
  auto layer = [&](auto lc, int j) {
    constexpr int l = decltype(lc)::value, lo = l > 0 ? l - 1 : 0;
    const bool dx = l > 0 || j > 0;                                // (H_o before the first position is a constant)
    float* part;
    const T* x;
    {
      const auto a = A();
      part = loop_global(a->l[l].part);
      x = loop_global((const T*)a->l[l].X) + (size_t)j * 4 * slot + ((size_t)bt0 * 4 + gate) * ns * 512;
    }
    CellIn in;
    // (not before every wavefront's gate gradients are on their way: the loads would stand in front of those stores; and
    // `red` has been read)
    loop_barrier();
    recur_nap(nap.gates);
    issue(x, 4 * tile, 0);
    if (l > 0) cell_fetch(lo, j, in);
    else if (j > 0) dpre_fetch(j - 1);
    for (int ch = 0; ch * BT < nbt; ++ch) {
      if (ch > 0) loop_barrier();                                  // (`red` has been read)
      settle(x, 4 * tile, ch);
      if (dx) {
        v4f acc[BT];
        multiply(wx[l], acc);
        spread(acc);
      }
      loop_barrier();
      if (dx && w < BT) send(part, j, 0, w, ch);
      if constexpr (l < LREG) multiply(wh[l < LREG ? l : 0], rest);
      else {
        multiply_lds((l - LREG) * NK, std::integral_constant<int, NK>{}, wc, rest);
      }
      if ((ch + 1) * BT < nbt) {
        issue(x, 4 * tile, ch + 1);
        loop_barrier();
        spread(rest);
        loop_barrier();
        if (w >= LOOP_WAVES - BT) send(part, j, 1, w - (LOOP_WAVES - BT), ch);
      }
    }
    if (l > 0) {
      const auto a = A();
      const int ln = fresh(), b = 16 * bt0 + w * per + min(ln >> 2, per - 1);
      float v[4];
      float* const mine = part_at(part, j, 0, place.pos);
      recur_nap(nap.sums);
      ask(mine, b, v);
      float dy = take(mine, b, v);
      if (a->l[lo].drop.on) {
        const DropSpec drop = seq_drop(DropSpec{a->l[lo].drop.key0, a->l[lo].drop.thresh, a->l[lo].drop.scale, a->l[lo].drop.width, 1},
                                       a->drop_step, j);
        dy *= drop_factor(drop, b, u0 + (ln & 3));
      }
      cell(lo, j, in, dy, cn[lo], dh[lo], dc[lo]);
      send_rest(l, j);
    }
  };

  // The scores' gradients (softmax backward), and with them the keys' part of dH_t; returns it for this lane's cell.  What the first
  // pass needs is requested before the workgroup's sums dpre W_c2 meet.
  auto mix = [&](int j) {
    constexpr int QT = LOOP_QT / 2;                                // (8 tps >= S)
    typedef typename std::conditional<FAST, uint2, float4>::type P4;
    float res = 0.f;
    for (int s0 = 0; s0 < per; s0 += spw) {
      const auto a = A();
      const int ln = fresh();
      const int sr = ln & (tps - 1), so = s0 + ln / tps, bs = w * per + min(so, per - 1), bg = 16 * bt0 + bs, n = so < per ? s_len[bs] : 0;
      const unsigned off = (unsigned)(bg * S + sr);
      P4 pr[QT];
      float av[QT], dv[QT];
      const char* const kg = (const char*)loop_global(a->Kg) + (size_t)place.pos * Bp * S * sizeof(P4);
      const char* const aj = (const char*)(loop_global(a->a) + (size_t)j * Bp * S);
      float* const da = loop_global(a->da) + (size_t)j * Bp * S;
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        av[q] = 0.f;
        if (sr + tps * q < n) {
          av[q] = *(const float*)(aj + (size_t)(4 * q * tps) + 4 * off);
          pr[q] = *(const P4*)(kg + (size_t)(q * tps * (int)sizeof(P4)) + off * (unsigned)sizeof(P4));
        }
      }
      loop_words_issue<QT>(da, 4 * tps, 4 * off, sr, tps, n, dv, true);
      if (s0 == 0) loop_barrier();                                 // (s_u is there)
      loop_words_settle<QT>(da, 4 * tps, 4 * off, dv, dead, gave_up, ticks);
      const auto plus = [](float x, float y) { return x + y; };
      float dot = 0.f;
#pragma unroll
      for (int q = 0; q < QT; ++q) dot += av[q] * dv[q];
      dot = loop_group(dot, tps, plus);
      float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        dv[q] = av[q] * (dv[q] - dot);
        if (!(sr + tps * q < n)) { dv[q] = 0.f; continue; }
        float kv[4];
        if constexpr (FAST) {
          kv[0] = __uint_as_float(pr[q].x << 16); kv[1] = __uint_as_float(pr[q].x & 0xffff0000u);
          kv[2] = __uint_as_float(pr[q].y << 16); kv[3] = __uint_as_float(pr[q].y & 0xffff0000u);
        } else {
          kv[0] = pr[q].x; kv[1] = pr[q].y; kv[2] = pr[q].z; kv[3] = pr[q].w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] += dv[q] * kv[e];
      }
      if (so < per && bs % plan.nwg == place.pos) {
        char* const dsj = (char*)(loop_global(a->ds) + (size_t)j * Bp * S);
#pragma unroll
        for (int q = 0; q < QT; ++q)
          if (sr + tps * q < S) *(float*)(dsj + (size_t)(4 * q * tps) + 4 * off) = dv[q];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = loop_group(o[e], tps, plus);
      const float mine = (ln & 2) ? ((ln & 1) ? o[3] : o[2]) : ((ln & 1) ? o[1] : o[0]);
      // to the lane that has this unit of the sentence in the cells: lane 4 s + unit
      const int cs = min(ln >> 2, per - 1) - s0;
      const float got = __shfl(mine, (max(cs, 0) * tps + (ln & 3)) & 63, 64);
      if (cs >= 0 && cs < spw) res = got;
    }
    return res;
  };

  const int task0 = place.pos * LOOP_WAVES + w, tasks = NB * np;
  dpre_row(Tn - 1);
  dpre_fetch(Tn - 1);
  for (int j = Tn - 1; j >= 0; --j) {
    // ---- dpre = (output layer's gradient + what the bottom layer's next step sent back) tanh' -------------------------------
    {
      const auto a = A();
      const int ln = fresh(), b = 16 * bt0 + w * per + min(ln >> 2, per - 1), u = u0 + (ln & 3);
      float feed = 0.f;
      if (j + 1 < Tn) {
        float v[4];
        float* const mine = part_at(loop_global(a->l[0].part), j + 1, 0, place.pos);
        ask(mine, b, v);
        feed = take(mine, b, v);
      }
      // (once per position every store of this wavefront is known to be done: the empty patterns that it put back are in place
      // before it sends the gate gradients that their slots' next writers wait for)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      float f = 1.f;
      if (a->drop_o.on) {
        const DropSpec drop = seq_drop(DropSpec{a->drop_o.key0, a->drop_o.thresh, a->drop_o.scale, a->drop_o.width, 1}, a->drop_step, j);
        f = drop_factor(drop, b, u);
      }
      const float v = (p_ce + feed) * f * (1.f - p_ho * p_ho);
      if (real)
        loop_quad_put(loop_global((T*)a->XP) + (size_t)j * slot, fm_offset(b, u0, ns), loop_global((T*)a->dPre) + (size_t)j * Bp * a->ldp,
                      (unsigned)(b * a->ldp + u0), v, ln, true);
    }
    if (j + 1 < Tn) send_rest(0, j + 1);
    const T* xp = loop_global((const T*)A()->XP) + (size_t)j * slot;
    const T* xg = xp + (size_t)bt0 * ns * 512;
    // ---- dpre . P_i, a wavefront per row ------------------------------------------------------------------------------------
    Frag<float> kr[RW][NQ];
    auto rows = [&](int t, int i0, int n) {
      const int ln = fresh();
      const float* const P = loop_global(A()->P) + (size_t)(16 * bt0 + t % NB) * H;
#pragma unroll
      for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          kr[r][q].zero();
          if (i0 + np * r < n && 8 * ln + 512 * q < H) kr[r][q].load(P + (size_t)(i0 + np * r) * Bp * H + 512 * q + (unsigned)(8 * ln));
        }
    };
    for (int t = task0; t < tasks || t == task0; t += plan.nwg * LOOP_WAVES) {
      const int ln = fresh();
      const bool some = t < tasks;
      const int p0 = t / NB, bs = t - p0 * NB, n = some ? __builtin_amdgcn_readfirstlane(s_len[bs]) : 0, bg = 16 * bt0 + bs;
      float* const da = loop_global(A()->da) + ((size_t)j * Bp + bg) * S;
      Frag<T> hv[NQ];
      if (some) rows(t, p0, n);
      const T* hrow = xp + (size_t)(bg >> 4) * ns * 512 + (bg & 15) * 8;
      auto piece = [&](int q, unsigned zero) {                     // (a lane beyond the row's end repeats the first)
        const int p = (8 * ln + 512 * q < H ? ln + 64 * q : 0) + (int)zero;
        return (unsigned)((p >> 2) * 512 + (p & 3) * 128) * (unsigned)sizeof(T);
      };
      if (t == task0) loop_barrier();                              // (every wavefront's dpre is on its way)
      if (some) loop_issue<T, NQ>(hrow, piece, hv);
      if (!some) break;
      loop_settle<T, NQ>(hrow, piece, hv, dead, gave_up, ticks);
      for (int i0 = p0; i0 < n; i0 += RW * np) {
        if (i0 != p0) rows(t, i0, n);
        float s[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
          s[r] = 0.f;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[r] += kr[r][q].get(e) * hv[q].get(e);
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) s[r] = loop_wave_sum(s[r]);
        float sv = s[0];
#pragma unroll
        for (int r = 1; r < RW; ++r) sv = ln == r ? s[r] : sv;
        if (ln < RW && i0 + np * ln < n) loop_put(da + (unsigned)(i0 + np * ln), sv);
      }
    }
    // ---- dpre W_c2 for this workgroup's four columns, then the keys' part, then the top layer's cells ------------------------
    issue(xg, tile, 0);
    CellIn in;
    cell_fetch(L - 1, j, in);
    if (j > 0) dpre_row(j - 1);
    for (int ch = 0; ch * BT < nbt; ++ch) {
      if (ch > 0) loop_barrier();
      settle(xg, tile, ch);
      v4f acc[BT];
      multiply_lds(NL - CL, std::integral_constant<int, CL>{}, wc, acc);
      spread(acc);
      if ((ch + 1) * BT < nbt) issue(xg, tile, ch + 1);
      loop_barrier();
      if (w < BT) {
        const int ln = fresh();
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < LOOP_WAVES; ++k) v += red[((k * BT + w) * 64 + loop_pos(ln >> 2, 0)) * 4 + (ln & 3)];
        s_u[(16 * (ch * BT + w) + (ln >> 2)) & (LOOP_MAX_BATCH - 1)][ln & 3] = v;
      }
    }
    float dy = mix(j);
    {
      const int ln = fresh();
      dy += s_u[w * per + min(ln >> 2, per - 1)][ln & 3];
    }
    {   // (the top layer's state, whichever that is)
      float t0 = cn[0], t1 = dh[0], t2 = dc[0];
#pragma unroll
      for (int l = 1; l < LOOP_MAX_LAYERS; ++l)
        if (l == L - 1) { t0 = cn[l]; t1 = dh[l]; t2 = dc[l]; }
      cell(L - 1, j, in, dy, t0, t1, t2);
#pragma unroll
      for (int l = 0; l < LOOP_MAX_LAYERS; ++l)
        if (l == L - 1) { cn[l] = t0; dh[l] = t1; dc[l] = t2; }
    }
    if (L > 3) layer(std::integral_constant<int, 3>{}, j);
    if (L > 2) layer(std::integral_constant<int, 2>{}, j);
    if (L > 1) layer(std::integral_constant<int, 1>{}, j);
    layer(std::integral_constant<int, 0>{}, j);
  }
  send_rest(0, 0);
  // ---- the initial states' gradients: what passed by, and the first position's recurrent part -------------------------------
#pragma unroll
  for (int l = 0; l < LOOP_MAX_LAYERS; ++l)
    if (l < L) {
      const auto a = A();
      const int b = 16 * bt0 + w * per + min(lane >> 2, per - 1);
      float v[4];
      float* const mine = part_at(loop_global(a->l[l].part), 0, 1, place.pos);
      ask(mine, b, v);
      const float rec = take(mine, b, v);
      if (real) {
        loop_global(a->l[l].dh)[(size_t)b * H + u0 + (lane & 3)] = dh[l] + rec;
        loop_global(a->l[l].dc)[(size_t)b * H + u0 + (lane & 3)] = dc[l];
      }
    }
}

// The same without waits, as loop_fwd_solo_kernel.  The states' gradients that pass from position to position and the feed are
// kept where the other form has its partial sums: per layer [dh | dc | recurrent part | feed] of [Bp, H].
template <typename T>
__global__ __launch_bounds__(64 * LOOP_WAVES) void loop_bwd_solo_kernel(const int* gave_up, int L, int Tn, int Bp, int H, int S, LoopBwdArgs args) {
  if (!recur_again(gave_up, args.again)) return;
  constexpr bool FAST = sizeof(T) == 2;
  __shared__ float s_d[16][LOOP_MAX_SRC];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, b0 = 16 * blockIdx.x, b = b0 + (lane & 15), kl = 8 * (lane >> 4);
  const size_t plane = (size_t)Bp * H, own = (size_t)b * H;
  // the cell backward of layer l for units u .. u + 3 of sentence b
  auto cells = [&](int l, int j, int u, const float (&dy)[4]) {
    const LoopBwdLayer& d = args.l[l];
    const size_t at = (size_t)j * Bp + b;
    const float mask = args.mask[at];
    float* const keep = d.part + own;
    for (int e = 0; e < 4; ++e) {
      float g[4], o[4], dh = 0.f, dc = 0.f, rec = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) g[q] = d.G[at * 4 * H + (size_t)q * H + u + e];
      if (j + 1 < Tn) { dh = keep[u + e]; dc = keep[plane + u + e]; rec = keep[2 * plane + u + e]; }
      const float x = e == 0 ? dy[0] : e == 1 ? dy[1] : e == 2 ? dy[2] : dy[3];
      seq_cell_bwd(g, d.C[at * H + u + e], tanh_of<FAST>(d.C[(at + Bp) * H + u + e]), x, rec, mask, dh, dc, o);
      keep[u + e] = dh; keep[plane + u + e] = dc;
#pragma unroll
      for (int q = 0; q < 4; ++q) ((T*)d.dG)[at * d.lddg + (size_t)q * H + u + e] = from_f<T>(o[q]);
    }
  };
  for (int j = Tn - 1; j >= 0; --j) {
    const size_t at = (size_t)j * Bp + b;
    for (int u = 4 * (w * 4 + (lane >> 4)); u < H; u += 16 * LOOP_WAVES) {
      const int r = args.pos[at];
      for (int e = 0; e < 4; ++e) {
        const float ho = to_f<T>(((const T*)args.Ho)[(at + Bp) * args.ldho + u + e]);
        const float feed = j + 1 < Tn ? args.l[0].part[3 * plane + own + u + e] : 0.f;
        const float f = args.drop_o.on ? drop_factor(seq_drop(args.drop_o, args.drop_step, j), b, u + e) : 1.f;
        ((T*)args.dPre)[at * args.ldp + u + e] = from_f<T>(((r >= 0 ? args.dce[(size_t)r * H + u + e] : 0.f) + feed) * f * (1.f - ho * ho));
      }
    }
    __syncthreads();
    for (int s = w; s < 16; s += LOOP_WAVES) {
      const int bg = b0 + s, n = min(args.len[bg], S);
      const T* dp = (const T*)args.dPre + ((size_t)j * Bp + bg) * args.ldp;
      const size_t row = ((size_t)j * Bp + bg) * S;
      for (int i = 0; i < n; ++i) {
        const float* pr = args.P + ((size_t)i * Bp + bg) * H;
        float v = 0.f;
        for (int k = lane; k < H; k += 64) v += pr[k] * to_f<T>(dp[k]);
        v = wave_sum(v);
        if (lane == (i & 63)) s_d[s][i] = v;
      }
      float dot = 0.f;                                             // (lane i % 64 wrote position i and reads it)
      for (int i = lane; i < n; i += 64) dot += args.a[row + i] * s_d[s][i];
      dot = wave_sum(dot);
      for (int i = lane; i < S; i += 64) {
        const float v = i < n ? args.a[row + i] * (s_d[s][i] - dot) : 0.f;
        s_d[s][i] = v;
        args.ds[row + i] = v;
      }
    }
    __syncthreads();
    const int n = min(args.len[b], S);
    for (int ct = w; ct < H >> 4; ct += LOOP_WAVES) {              // dH_t, 16 columns at a time, and the top layer's cells
      v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
      for (int k0 = 0; k0 < H; k0 += 32) {
        const int k = k0 + kl;
        Frag<T> fw, fx;
        fw.zero(); fx.zero();
        if (k < H) { fw.load((const T*)args.Wct + (size_t)(16 * ct + (lane & 15)) * H + k); fx.load((const T*)args.dPre + at * args.ldp + k); }
        mma16(acc, fw, fx);
      }
      const int u = 16 * ct + 4 * (lane >> 4);
      for (int i = 0; i < n; ++i) {
        const float d = s_d[lane & 15][i];
        const T* kr = (const T*)args.K + ((size_t)i * Bp + b) * H + u;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += d * to_f<T>(kr[e]);
      }
      const float dy[4] = {acc[0], acc[1], acc[2], acc[3]};
      cells(L - 1, j, u, dy);
    }
    __syncthreads();
    for (int l = L - 1; l >= 0; --l) {
      const LoopBwdLayer& d = args.l[l];
      for (int ct = w; ct < H >> 3; ct += LOOP_WAVES) {            // 16 columns: first the input's, then the recurrent ones
        const bool in = ct < (H >> 4);
        const int c0 = in ? ct : ct - (H >> 4);
        if (in && l == 0 && j == 0) continue;
        v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
        const T* wr = (const T*)d.Wt + (size_t)((in ? d.x_row : d.h_row) + 16 * c0 + (lane & 15)) * d.ldw;
        const T* gr = (const T*)d.dG + at * d.lddg;
        for (int k = kl; k < 4 * H; k += 32) {                     // (4H is a multiple of 32)
          Frag<T> fw, fx;
          fw.load(wr + k); fx.load(gr + k);
          mma16(acc, fw, fx);
        }
        const int u = 16 * c0 + 4 * (lane >> 4);
        if (!in) {
#pragma unroll
          for (int e = 0; e < 4; ++e) d.part[2 * plane + own + u + e] = acc[e];
        } else if (l > 0) {
          float dy[4] = {acc[0], acc[1], acc[2], acc[3]};
          const DropSpec& dr = args.l[l - 1].drop;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (dr.on) dy[e] *= drop_factor(seq_drop(dr, args.drop_step, j), b, u + e);
          cells(l - 1, j, u, dy);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) d.part[3 * plane + own + u + e] = acc[e];
        }
      }
      __syncthreads();
    }
  }
  for (int l = 0; l < L; ++l)
    for (int u = 4 * (w * 4 + (lane >> 4)); u < H; u += 16 * LOOP_WAVES)
      for (int e = 0; e < 4; ++e) {
        const float* keep = args.l[l].part + own + u + e;
        args.l[l].dh[own + u + e] = keep[0] + keep[2 * plane];
        args.l[l].dc[own + u + e] = keep[plane];
      }
}

// A wavefront: 64 positions of one sentence, 32 columns.
template <typename T>
__global__ __launch_bounds__(64) void loop_columns_kernel(const T* __restrict__ src, T* __restrict__ dst, int S, int Bp, int H) {
  typedef typename std::conditional<sizeof(T) == 2, uint2, float4>::type V4;
  const int i = blockIdx.z * 64 + threadIdx.x, b = blockIdx.y;
  if (i >= S) return;
  const V4* s = (const V4*)(src + ((size_t)i * Bp + b) * H) + blockIdx.x * 8;
#pragma unroll
  for (int c = 0; c < 8; ++c)
    if ((int)blockIdx.x * 8 + c < H >> 2) ((V4*)dst)[((size_t)(blockIdx.x * 8 + c) * Bp + b) * S + i] = s[c];
}
void launch_loop_columns(int prec, const void* src, void* dst, int S, int Bp, int H, hipStream_t st) {
  const dim3 grid((H + 31) / 32, Bp, (S + 63) / 64);
  if (prec) hipLaunchKernelGGL(loop_columns_kernel<bf16_t>, grid, dim3(64), 0, st, (const bf16_t*)src, (bf16_t*)dst, S, Bp, H);
  else hipLaunchKernelGGL(loop_columns_kernel<float>, grid, dim3(64), 0, st, (const float*)src, (float*)dst, S, Bp, H);
}

LoopFit loop_fits(int prec, int L, int Bp, int H, int S, int T, const SeqRun& run) {
  const LoopPlan p = loop_plan(prec, L, Bp, H, S, std::min(run.cus, 256));
  const bool fits = run.mode != SEQ_RUN_ALONE && p.ok;
  return LoopFit{fits, fits && loop_pays(p, L, T), loop_runs_alone(p)};
}

void launch_loop_fwd(int prec, const LoopFwdArgs& args, int L, int T, int Bp, int H, int S, const SeqRun& run, hipStream_t st) {
  loop_fwd_go<false>(prec, args, L, T, Bp, H, S, run, st);
}
void launch_loop_bwd(int prec, const LoopBwdArgs& args, int L, int T, int Bp, int H, int S, const SeqRun& run, hipStream_t st) {
  const LoopPlan p = loop_plan(prec, L, Bp, H, S, std::min(run.cus, 256));
  LoopBwdArgs a = args;
  a.wait_ticks = run.mode == SEQ_RUN_GIVE_UP ? 0 : RECUR_WAIT_TICKS;
  const LoopNaps nap{16, p.nk * std::min(p.tiles, 4) < 16 ? 0 : 16};
  const dim3 grid(p.groups * p.nwg), block(64 * LOOP_WAVES);
#define GO(TT, NK, BT) hipLaunchKernelGGL((loop_bwd_kernel<TT, NK, BT>), grid, block, 0, st, a, L, T, Bp, H, S, p, nap)
  if (prec) {
    if (p.nk == 1) { if (p.tiles == 1) GO(bf16_t, 1, 1); else GO(bf16_t, 1, 2); }
    else if (p.nk == 2) { if (p.tiles == 1) GO(bf16_t, 2, 1); else if (p.tiles == 2) GO(bf16_t, 2, 2); else GO(bf16_t, 2, 4); }
    else { if (p.tiles == 1) GO(bf16_t, 4, 1); else if (p.tiles == 2) GO(bf16_t, 4, 2); else GO(bf16_t, 4, 4); }
  } else {
    if (p.nk == 1) { if (p.tiles == 1) GO(float, 1, 1); else GO(float, 1, 2); }
    else { if (p.tiles == 1) GO(float, 2, 1); else if (p.tiles == 2) GO(float, 2, 2); else GO(float, 2, 4); }
  }
#undef GO
  if (prec) hipLaunchKernelGGL(loop_bwd_solo_kernel<bf16_t>, dim3(Bp >> 4), block, 0, st, a.ticket + 1, L, T, Bp, H, S, a);
  else hipLaunchKernelGGL(loop_bwd_solo_kernel<float>, dim3(Bp >> 4), block, 0, st, a.ticket + 1, L, T, Bp, H, S, a);
}

}  // namespace cmt

// Shapes of the whole-recurrence kernels (recur.hip): which workgroups form a group that waits for one another.  No
// device code, so that the rules can be checked with a host compiler.
#pragma once

namespace cmt {

// A launch starts its workgroups group by group, so of its groups at most one is incomplete.  SEQ_QUEUES such launches run at
// once in a process (its hardware queues).  With one workgroup per CU they can all be stuck only if their incomplete groups,
// one workgroup short each, take every CU: not while SEQ_QUEUES * (group - 1) < CUs, i.e. 4 x 63 < 256.  That is as good as always and no
// proof: workgroups are dealt to the chip's eight parts (XCDs) in turn, and the CUs that stay free may be in a part for which no incomplete
// group has a workgroup left.  Four handles with groups of 64 on streams of their own, fp32, width 1024: waits given up in a step of 100 to 250.
constexpr int SEQ_QUEUES = 4, SEQ_MAX_GROUP = 64;

// ks wavefronts split the contraction, nk k steps of 32 each, of which the weights of lk stay in LDS and the others in
// registers; rt row tiles (forward 4 units x 4 gates, backward 16 units) x bt tiles of 16 sentences per workgroup; ne
// wavefronts for the cells.
struct SeqPlan { int ks, nk, lk, rt, bt, ne, group, groups; };

inline SeqPlan seq_fwd_plan(int prec, int ndir, int Bp, int Hh) {
  const int nsteps = (Hh + 31) / 32;
  SeqPlan p{};
  p.ks = nsteps <= 4 ? 2 : 8;
  p.nk = nsteps <= 2 ? 1 : nsteps <= 4 ? 2 : nsteps <= 8 ? 1 : nsteps <= 16 ? 2 : 4;
  p.rt = 4;
  p.group = (Hh + 4 * p.rt - 1) / (4 * p.rt);
  // Long fp32 rows: 16 units are 256 KB of weights.  A quarter of them in LDS leaves room for one tile of sentences in the
  // registers.  (8 units per workgroup fit the registers alone, but in groups of up to 128, too many to wait for one
  // another; the times agree within 1 %, e.g. a step of 2 layers of 1024 units, 64 sentences 8.80 | 8.74 ms.)
  p.lk = !prec && p.nk == 4 ? 1 : 0;
  // one tile of sentences per group while that is one round of workgroups over the chip, else two
  p.bt = p.lk || ndir * (Bp >> 4) * p.group <= 256 ? 1 : 2;
  // (registers: twice as many cell wavefronts for two tiles of sentences where 128 per lane are enough)
  p.ne = prec && p.bt == 2 && (nsteps > 4 && nsteps <= 16) ? 8 : 4;
  p.groups = ndir * (((Bp >> 4) + p.bt - 1) / p.bt);
  return p;
}

inline SeqPlan seq_bwd_plan(int prec, int ndir, int Bp, int Hh) {
  const int nsteps = Hh / 8;                           // k steps of 32 gate rows
  SeqPlan p{};
  p.ks = nsteps <= 4 ? 2 : 8;
  p.nk = nsteps <= 16 ? 2 : nsteps <= 32 ? 4 : nsteps <= 64 ? 8 : 16;
  p.bt = 1;
  p.groups = ndir * (Bp >> 4);
  p.rt = prec && p.groups * ((Hh + 15) / 16) > 128 ? 2 : 1;
  p.ne = p.rt == 2 && p.nk <= 8 ? 8 : 4;
  p.group = (Hh + 16 * p.rt - 1) / (16 * p.rt);
  return p;
}

// The decoder's whole loop: a group = up to 128 sentences, its H / 4 workgroups own four units of every layer.  All layers'
// weights stay on the chip, so a group is as large as the widest network needs (256 workgroups at width 1024) and a launch
// may take every CU there is.  One of at most SEQ_MAX_GROUP workgroups counts as a group of the recurrences above (its workgroups
// start in any order, so at worst all but one of the whole launch wait); a larger one has nothing beside it on the chip that
// waits, in this process (section_gate.h).  Nothing keeps it apart from another process, or from the recurrences of a graph that
// is replayed on another stream: waits may be given up there, and what was given up is made again without them.
// nk k steps per wavefront; bt tiles of 16 sentences at a time, nch times; tiles = the most a group has; rows = source rows that a
// wavefront scores per position
struct LoopPlan { bool ok; int nk, nwg, bt, nch, groups, tiles, rows; };
inline LoopPlan loop_plan(int prec, int L, int Bp, int H, int S, int cus) {
  LoopPlan p{};
  const int nt = Bp / 16, nsteps = (H + 31) / 32;
  p.nwg = H / 4;
  p.nk = nsteps <= 8 ? 1 : nsteps <= 16 ? 2 : 4;
  // (fp32 wider than 512: the weights of four layers are more than a CU's registers and LDS hold, and there is no form for fewer)
  if (L > 4 || nt > 8 || S > 128 || p.nwg > cus || nsteps > 32 || (!prec && p.nk > 2)) return p;
  p.groups = nt < cus / p.nwg ? nt : cus / p.nwg;
  p.tiles = (nt + p.groups - 1) / p.groups;
  p.groups = (nt + p.tiles - 1) / p.tiles;
  // a chunk's fragments are in flight at once: 4 tiles of them, or 2 where twice 4 tiles' sums take the registers (3 run as 4)
  p.bt = p.tiles < 3 || p.tiles > 4 ? (p.tiles < 2 ? 1 : 2) : 4;
  p.nch = p.tiles > 4 ? 4 : 1;
  if ((p.nch > 1 && !(prec && p.nk == 4)) || (p.nk == 1 && p.bt > 2)) return p;
  const int waves = 8 * p.nwg, sentences = 16 * p.tiles, share = waves > sentences ? waves / sentences : 1;   // wavefronts per sentence
  p.rows = (sentences * share + waves - 1) / waves * ((S + share - 1) / share);
  p.ok = true;
  return p;
}

// Whether the loops of a step or an evaluation, where they fit, are faster than launches.  Not for narrow layers with long sources,
// whose rows H / 4 workgroups score: evaluations of 40 positions, bf16, one layer, one group of sentences are so many times as fast with
// the loop at 20 | 32 | 64 rows per wavefront: width 16 1.11 | 0.87 | 0.67; at 16 | 24 | 32, width 32 1.08 | 0.99 | 0.90.  Two layers, 32 | 48
// rows 1.00 | 0.89, three, 48 rows 0.96.  Groups of sentences run side by side: with 8, one layer, 32 | 48 rows 1.06 | 0.93, two, 48 | 64
// 1.09 | 0.99.  Nor for one position (0.94 - 1.03 over widths 64 - 1024, 1 to 4 layers) or two of one layer (0.96 - 1.07): the clears
// and copies around a loop.
inline bool loop_pays(const LoopPlan& p, int L, int T) { return T > 1 && T * L > 2 && p.rows <= 10 + 12 * L + 3 * (p.groups - 1); }

// The same for greedy decoding, whose logits, 16 vocabulary entries at a time (0.6 us each, W_o streaming in), are shared among the
// group's H / 4 workgroups where the launches spread them over the chip: `tiles` = such tiles per workgroup, each as long as three
// rows.  So many times as fast with the loop, translations of 30 tokens, one group, 2 - 10 rows, 12 | 18 | 24 tiles:
//              bf16 width 16        128                  fp32 width 16        128
//   1 layer    1.08 | 0.93 | 0.82   1.15 | 1.00 | 0.89   1.01 | 0.85 | 0.76   1.09 | 0.95 | 0.83
//   2 layers   1.15 | 1.00 | 0.90   1.22 | 1.07 | 0.96   1.08 | 0.95 | 0.82   1.17 | 1.03 | 0.91
//   4 layers   1.22 | 1.08 | 1.00   1.28 | 1.16 | 1.06   1.22 | 1.08 | 0.96   1.27 | 1.14 | 1.03
// and with 50 rows (bf16, width 16, 2 layers) 0.89 | 0.82 | 0.75.  A wide layer's launches take longer (1 layer, 24 tiles, widths 256 | 512: bf16
// 0.93 | 1.16, fp32 1.17 | 1.65), and so do those of several groups of sentences (bf16, 128, 1 layer, 24 tiles, 1 | 4 | 8 groups 0.90 | 0.96 | 0.98).
constexpr int LOOP_DECODE_TILES = 24;      // (the most that was measured)
inline bool loop_decode_pays(const LoopPlan& p, int prec, int L, int H, int V) {
  const int tiles = ((V + 15) / 16 + p.nwg - 1) / p.nwg, launches = prec ? 44 + H * H / 8192 : 34 + H * H / 2048;
  return tiles <= LOOP_DECODE_TILES && 3 * tiles + p.rows <= launches + 10 * L + 3 * (p.groups - 1);
}

inline bool loop_runs_alone(const LoopPlan& p) { return p.groups * p.nwg > SEQ_MAX_GROUP; }

}  // namespace cmt

// Greedy decoding as one launch: the forward loop (loop_fwd.h) with the embedding, the logits and the choice of the tokens in it.
#include "loop_fwd.h"

namespace cmt {

// The logits are shared among the workgroups of a group, H / 4 of them, 16 vocabulary entries at a time (0.6 us each, W_o streaming in),
// where the launches spread them over the chip: few workgroups with many entries lose.  Whole translations of 20 tokens, 2 bf16
// layers, one sentence, launches | loop, us: 16 tiles per workgroup (width 128, vocabulary 8000) 626 | 577, 18 (512, 37000) 876 | 722, 31 (64,
// 8000) 604 | 738, 36 (256, 37000) 762 | 838, 72 (128, 37000) 707 | 1228.  50 tokens of 64 sentences, 4 layers of 1024 (8 tiles) 3853 |
// 3041; 25 tokens of one sentence, 2 fp32 layers of 512 (16 tiles) 2123 | 1292.
constexpr int LOOP_DECODE_TILES = 24;
bool loop_decode_fits(int prec, int L, int Bp, int H, int S, int V, const SeqRun& run) {
  const LoopPlan p = loop_plan(prec, L, Bp, H, S, std::min(run.cus, 256));
  return loop_fits(prec, L, Bp, H, S, run) && p.nch == 1 && (V + 15) / 16 <= LOOP_DECODE_TILES * p.nwg;
}

void launch_loop_decode(int prec, const LoopFwdArgs& args, int L, int T, int Bp, int H, int S, const SeqRun& run, hipStream_t st) {
  loop_fwd_go<true>(prec, args, L, T, Bp, H, S, run, st);
}

}  // namespace cmt

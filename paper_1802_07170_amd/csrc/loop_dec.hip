// Greedy decoding as one launch: the forward loop (loop_fwd.h) with the embedding, the logits and the choice of the tokens in it.
#include "loop_fwd.h"

namespace cmt {

LoopFit loop_decode_fits(int prec, int L, int Bp, int H, int S, int V, const SeqRun& run) {
  const LoopPlan p = loop_plan(prec, L, Bp, H, S, std::min(run.cus, 256));
  const bool fits = run.mode != SEQ_RUN_ALONE && p.ok && p.nch == 1;
  return LoopFit{fits, fits && loop_decode_pays(p, prec, L, H, V), loop_runs_alone(p)};
}

void launch_loop_decode(int prec, const LoopFwdArgs& args, int L, int T, int Bp, int H, int S, const SeqRun& run, hipStream_t st) {
  loop_fwd_go<true>(prec, args, L, T, Bp, H, S, run, st);
}

}  // namespace cmt

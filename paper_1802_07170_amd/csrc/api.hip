// Host side of the C ABI (include/cytonmt_hip.h): argument validation, the workspace layout, and
// the kernel schedules of a training step, of greedy decoding and of beam search.  No arithmetic of
// the method happens here.
//
// Schedule of one training step:
//   gathers -> encoder layers (per layer the input GEMM batched over all source positions, then the whole
//   recurrence as one launch, the bottom layer's two directions together) -> attention-key hoist K = H_s W_a -> decoder time loop (per step: one
//   fused LSTM kernel per layer, attention, attentional tanh layer) -> output layer in slabs of
//   target positions (projection + log-sum-exp partials, e -> dz rescale, dH_o and dW_o GEMMs) ->
//   decoder loop backwards -> deferred attention gradients -> encoder loops backwards.  Everything
//   that does not feed a recurrence — transposes, weight gradients as GEMMs batched over all time
//   steps (the paper's calculateGradient accumulation becomes the k = B*T contraction), dW_o, the
//   deterministic embedding scatters — runs on the library's second stream and is joined before the
//   step ends on the caller's stream.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <chrono>
#include <string>
#include <vector>

#include "../../include/cytonmt_hip.h"
#include "kernels.h"
#include "recur_plan.h"
#include "row_pitch.h"
#include "section_gate.h"

using namespace cmt;

namespace {

// Which of the decoder's whole loops a workspace has slots for: none, the forward one without dropout (an evaluation), all.
enum { LOOP_SLOTS_NONE = 0, LOOP_SLOTS_EVAL = 1, LOOP_SLOTS_ALL = 2 };
enum { LOOP_RAN_FWD = 1, LOOP_RAN_BWD = 2 };

struct ParamInfo { std::string name; int64_t rows, cols; size_t off; };

// one LSTM (layer, direction)
struct LD {
  int Kin = 0, Hh = 0;
  int ph = 0, pg = 0;                // row pitches (elements) of Hst and dG: Hh, 4Hh + padding (see row_pitch.h)
  size_t w_off = 0, b_off = 0;       // element offsets in the flat parameter vector
  char* W = nullptr;                 // T [4Hh, Kin+Hh]
  char* Wt = nullptr;                // T [Kin+Hh, 4Hh]
  char* Hst = nullptr;               // T [(Lmax+1), Bp, Hh]
  float* Cst = nullptr;              // [(Lmax+1), Bp, Hh]
  float* Gs = nullptr;               // [Lmax, Bp, 4Hh] gate activations
  float* Gx = nullptr;               // [Lmax, Bp, 4Hh] batched input pre-activations (may be null)
  char* dG = nullptr;                // T [Lmax, Bp, 4Hh]
  char* dGT = nullptr;               // T [4Hh, Lmax*Bp]
  char* HstT = nullptr;              // T [Hh, (Lmax+1)*Bp]
  char* Yd = nullptr;                // T [Lmax, Bp, Hh] the layer's output after dropout (row pitch ph) ...
  char* YdT = nullptr;               // ... and its transpose [Hh, L*Bp]; used only while dropout is on
  float* dh = nullptr; float* dc = nullptr;   // decoder: [Bp, Hh]
  float* bwdp = nullptr;             // decoder: [8][Bp][2Hh] backward step-GEMM planes
  // decoder: fragment-major copies read by the per-step kernels (bf16 path, Hh a multiple of 32; see fm_offset)
  int Kstep = 0;                     // width of the per-step input segment: the x columns [Kin - Kstep, Kin) of W
  char* Wfm = nullptr;               // gate rows of W, columns [Kin - Kstep, Kin + Hh)
  char* HstF = nullptr;              // [(Lmax+1)] slots of [Bp, Hh]
  char* YdF = nullptr;               // [Lmax] slots of [Bp, Hh] (the layer's output after dropout)
  char* XH = nullptr; char* XY = nullptr; char* XD = nullptr;   // decoder: the whole loop's slots (states, after dropout, gate
                                     // gradients): the copies above and dGF where there are such
  bool fm = false;
  // encoder: exchange slots of the whole-recurrence kernels, for the states and for the gate gradients (recur.hip); they
  // share the memory of dGT and Gx
  char* X = nullptr; char* XG = nullptr;
  char* WtF = nullptr;               // W^T [Kin+Hh, 4Hh] (backward step GEMMs; needs Kin a multiple of 16)
  char* dGF = nullptr;               // [Lmax] slots of [Bp, 4Hh]
  bool fmb = false;
};

// Row capacity of an output-layer slab: CE_SLAB_MAX_ROWS unless CMT_CE_SLAB_ROWS asks for less (a multiple of 256
// from 256 up; read whenever a handle or a size query is set up, so both see the same value).
static int ce_cap_env() {
  const char* e = getenv("CMT_CE_SLAB_ROWS");
  const int v = e ? atoi(e) / 256 * 256 : 0;
  return v >= 256 ? std::min(CE_SLAB_MAX_ROWS, v) : CE_SLAB_MAX_ROWS;
}

struct Bump {
  char* base; size_t off = 0;
  explicit Bump(char* b) : base(b) {}
  char* take(size_t bytes) {
    off = (off + 255) & ~(size_t)255;
    char* p = base ? base + off : nullptr;
    off += bytes;
    return p;
  }
};

// how the gate that keeps sections of several streams apart talks to the device
struct GateRt {
  using Event = hipEvent_t;
  using Stream = hipStream_t;
  static bool record(Event e, Stream st) { return hipEventRecord(e, st) == hipSuccess; }
  static void wait(Stream st, Event e) { (void)hipStreamWaitEvent(st, e, 0); }
  static void finish(Event e) { if (e) (void)hipEventSynchronize(e); }
};
using Gate = SectionGate<GateRt>;
constexpr int GATES = 64;
Gate g_gates[GATES];                    // by device

}  // namespace

struct cmt_handle {
  cmt_config cfg;
  int prec = 0; size_t esz = 4;
  hipStream_t st = nullptr;
  float* params = nullptr; float* grads = nullptr; char* ws = nullptr;
  size_t nparams = 0;
  std::vector<ParamInfo> table;
  std::string err;
  int Bpm = 0;                          // padded max batch
  int PH = 0;                           // row pitch of HoBuf, Cs, dPre: H + padding (see row_pitch.h)
  int ldWoT = 0;                        // row pitch of WoT
  bool pad_lines = true;                // (not in the static array: what fits there does not depend on it)
  // last-step shape
  int B = 0, Bp = 0, S = 0, T = 0;
  bool have_step = false;
  // pinned host
  float* h_loss = nullptr; int* h_flags = nullptr;

  // parameter working copies
  char* Pc = nullptr;                   // T copy of the flat parameter vector (bf16 path) or the master itself
  std::vector<LD> enc, dec;             // enc: [l0 fwd, l0 bwd, l1, ...]; dec: [l0, l1, ...]
  size_t off_Esrc = 0, off_Etgt = 0, off_Wa = 0, off_Wc = 0, off_Wo = 0, off_Bo = 0;
  char *WaT = nullptr, *WcT = nullptr, *WoT = nullptr;

  // source side
  char* Xs = nullptr; float* mask_s = nullptr; int32_t* tok_s = nullptr; int32_t* len_s = nullptr;
  char* Y0 = nullptr; char* Y0T = nullptr; char* Kmat = nullptr;
  float* Pmat = nullptr; char* PmatT = nullptr;   // the source states through the context half of W_c, [S * Bp, H] in fp32 and in
                                        // the operand type (Eq. 7 regrouped)
  int att_proj = 1;                     // attention on the projected source rows (see enqueue_step): 1 both decoder loops,
                                        // 2 the forward loop alone, 0 neither
  float* dHs = nullptr; char* dK = nullptr; char* dKT = nullptr;
  float* dYa = nullptr; float* dXs = nullptr; char* XsT = nullptr;
  // target side
  char* Xt = nullptr; float* mask_t = nullptr; int32_t* tok_t = nullptr; int32_t* labels = nullptr; int32_t* len_t = nullptr;
  char* HoBuf = nullptr; char* HoBufT = nullptr; char* Cs = nullptr; char* CsT = nullptr;
  float* att_a = nullptr; float* att_ds = nullptr; float* dCs = nullptr; float* dots = nullptr;
  float* att_s = nullptr;               // [Tmax, Bp, Smax] attention scores of every step of the last training step
  char* dPre = nullptr; char* dPreT = nullptr;
  float* dHoCE = nullptr;
  float* dHt = nullptr; float* wcp = nullptr;
  float* dXt = nullptr; char* XtT = nullptr;
  float *pmax = nullptr, *psum = nullptr, *zy = nullptr, *lse = nullptr, *nll = nullptr, *rowscale = nullptr;
  // the output layer works on the valid target positions only, numbered densely on the device
  int32_t *ce_pos = nullptr, *ce_row = nullptr, *ce_nvalid = nullptr, *labels_c = nullptr;
  char* Hoc = nullptr; char* HocT = nullptr;   // H_o (as the output layer sees it) of the valid positions, and its transpose
  float* loss = nullptr; int* flags = nullptr; float* colscr = nullptr;
  int* tickets = nullptr;               // SEQ_TICKETS words, two per recurrence launch of a pass (layers <= 8)
  SeqRun seq{};                         // how the recurrences run (env CMT_RECUR)
  int loop = 1;                         // the decoder's loops as one launch each: 0 never, 1 where that is faster, 2 where it
                                        // fits (env CMT_DEC_LOOP); its slots, where the layers have no fragment-major copies
                                        // that can serve (LD::HstF, YdF, dGF)
  char* HoFeedX = nullptr; char* dPreX = nullptr;
  int loop_slots = LOOP_SLOTS_ALL;      // what the layout holds for them
  int* again = nullptr;                 // launches made again after a wait that was given up, counted on the device
  int64_t n_loops = 0;                  // decoder loops enqueued as one launch
  int ran_loops = 0;                    // those of the last step
  bool capturing = false;               // the pass being enqueued is captured into a graph
  Gate* gate = nullptr; Gate::Client* section = nullptr;   // the device's gate, and this handle's place in it
  char* dzs = nullptr; char* dzTs = nullptr; float* dbo_parts = nullptr;
  std::vector<GemmProb> dw_group;       // weight-gradient GEMMs collected for one grouped launch (flush_dw_group), the transposes
  std::vector<TransposeJob> dw_tr;      // of their operands and the sums for the biases that come with those
  std::vector<SumPartsJob> dw_sums;
  int ce_rows = 0, ce_pitch = 0;        // row capacity of an output-layer slab and the row pitch of its buffers
  int ce_cap = ce_cap_env();            // upper bound of ce_rows
  float* gsplit = nullptr; size_t gsplit_floats = 0;   // split-k planes of dH_o = dz W_o (also the probes' scratch)
  float* gsplit2 = nullptr; size_t gsplit2_floats = 0; // split-k planes of the second stream's GEMMs (fp32 path)
  hipStream_t side = nullptr;           // library-owned second stream for work off the recurrences' critical path
  std::vector<hipEvent_t> ev; size_t ev_next = 0;
  int use_side = 1;
  char* dzs2 = nullptr; char* dzTs2 = nullptr;
  char* WcF = nullptr; char* WcTF = nullptr;  // fragment-major W_c [H, 2H] and W_c^T [2H, H]
  char* WoF = nullptr;                        // fragment-major W_o [V, H] (greedy decoding's logits; V a multiple of 16)
  char* CsF = nullptr; char* dPreF = nullptr; // fragment-major copies of the contexts and of dpre, [Tmax] slots of [Bp, H]
  char* HoFeedF = nullptr;              // fragment-major copy of the H_o rows fed to the decoder's bottom layer, [(Tmax+1)] slots of [Bp, H]
  // decoding (greedy, beam): the bottom decoder layer contracts [embedding; H_o; h] in one step, so it needs the gate
  // rows of all E + 2H columns of its weights and its input [Bp, E + H] in fragment-major form
  char* Wdec0F = nullptr; char* xcatF = nullptr;
  int kb_wc = 0;                        // caps on the k blocks of the decoder's k-split step GEMMs (0 = default): dpre W_c, and
  int kb_bwd_dec = 0;                   // the layers' backward GEMMs
  // Workgroup caps of the second stream's GEMMs (weight gradients; dW_o), 0 = none (env CMT_SIDE_WGS, CMT_SIDE_WGS_WO).  A cap leaves
  // part of the chip to the kernels of the caller's stream, which paid while the decoder's loops were chains of short launches
  // beside them; a loop that takes the whole chip waits for them instead.  Step time with a cap of 128 / without, ms: medium 6.01 /
  // 6.04, attn 5.02 / 4.92, small (fp32) 6.43 / 6.39; at 128 sentences (large) 19.6 / 19.0; with the update paper_512x2 2.64 / 2.58,
  // paper_1024x2 4.38 / 4.24.
  int side_wgs = 0, side_wgs_wo = 0;
  int wc_whole_k = 1;                   // fused decoder loop: dpre W_c with the whole k range per workgroup (env CMT_WC_WHOLE_K)
  // decoder's backward loop with the whole-k step GEMM and the consumer in its epilogue (env CMT_BWD_FUSED, bit 1), up
  // to 128 sentences: 8.1 against 8.7 ms for the large workload's loop; wider batches keep the k-split GEMM +
  // pointwise pair
  int bwd_fused = 1;
  // phase timing of a step on the caller's stream (measurement aid, env CMT_PHASE_TIMING=1)
  int phase_timing = 0;
  std::vector<hipEvent_t> phase_ev; std::vector<const char*> phase_name; size_t phase_n = 0;
  std::vector<double> phase_host;       // host clock (ms) when each mark was enqueued
  // regularisation of the next steps (cmt_set_regularization)
  float drop_p = 0.f, drop_scale = 1.f, ls_eps = 0.f;
  unsigned drop_thresh = 0; unsigned long long drop_seed = 0;
  // greedy decoding
  char* xcat = nullptr; int ldxcat = 0; // decoder bottom-layer input [emb(y_{j-1}) ; H_o^{<j-1>}] of the current step
  int32_t* dec_tok = nullptr; int32_t* dec_done = nullptr; float* dec_mask = nullptr; float* logits = nullptr;
  // beam search: the search's state
  BeamState beam{};
  char* HoDrop = nullptr;               // H_o after dropout: what the output layer and the input feed read
  float* psz = nullptr;                 // per-group sums of logits (label smoothing)
  size_t ws_bytes = 0;

  const char* Pw(size_t off) const { return Pc + off * esz; }
};

namespace {

int round_up(int v, int m) { return (v + m - 1) / m * m; }

// jobs for launch_fill_multi / launch_copy2d_multi (units of 32-bit words; esz = bytes per T element)
void add_fill(std::vector<FillJob>& v, void* p, size_t elems, size_t esz) { v.push_back(FillJob{p, elems * esz / 4}); }
void add_empty(std::vector<FillJob>& v, void* p, size_t elems, size_t esz) { v.push_back(FillJob{p, elems * esz / 4, 0xffffffffu}); }
void add_copy(std::vector<CopyJob>& v, const void* s, int lds, void* d, int ldd, int rows, int cols, size_t esz) {
  const int f = (int)(4 / esz);                    // elements per word: row pitches and widths are multiples of it
  v.push_back(CopyJob{s, lds / f, d, ldd / f, rows, cols / f});
}

bool config_ok(const cmt_config* c, std::string* why) {
  auto bad = [&](const char* m) { if (why) *why = m; return false; };
  if (!c) return bad("null config");
  if (c->src_vocab < 8 || c->tgt_vocab < 8 || c->src_vocab % 8 || c->tgt_vocab % 8) return bad("vocabulary sizes must be positive multiples of 8");
  if (c->emb_dim < 8 || c->emb_dim % 8 || c->emb_dim > 2048) return bad("emb_dim must be a multiple of 8 in [8, 2048]");
  if (c->hidden < 16 || c->hidden % 16 || c->hidden > 1024) return bad("hidden must be a multiple of 16 in [16, 1024]");
  if (c->layers < 1 || c->layers > 8) return bad("layers must be in [1, 8]");
  if (c->max_batch < 1 || c->max_batch > 4096) return bad("max_batch must be in [1, 4096]");
  if (c->max_src_len < 1 || c->max_src_len > 512) return bad("max_src_len must be in [1, 512]");
  if (c->max_tgt_len < 1 || c->max_tgt_len > 4096) return bad("max_tgt_len must be in [1, 4096]");
  if (c->precision != 0 && c->precision != 1) return bad("precision must be 0 (fp32) or 1 (bf16)");
  if (c->bos_id < 0 || c->bos_id >= c->tgt_vocab) return bad("bos_id outside the target vocabulary");
  if (c->pad_id < 0 || c->pad_id >= c->tgt_vocab || c->pad_id >= c->src_vocab) return bad("pad_id outside a vocabulary");
  return true;
}

void build_table(const cmt_config& c, std::vector<ParamInfo>& t, size_t& total) {
  const int64_t Vs = c.src_vocab, Vt = c.tgt_vocab, E = c.emb_dim, H = c.hidden, Hd = H / 2;
  size_t off = 0;
  auto add = [&](const std::string& n, int64_t r, int64_t cc) { t.push_back({n, r, cc, off}); off += (size_t)(r * cc); };
  add("E_src", Vs, E); add("E_tgt", Vt, E);
  add("enc.l0.fwd.W", 4 * Hd, E + Hd); add("enc.l0.fwd.b", 4 * Hd, 1);
  add("enc.l0.bwd.W", 4 * Hd, E + Hd); add("enc.l0.bwd.b", 4 * Hd, 1);
  for (int l = 1; l < c.layers; ++l) {
    add("enc.l" + std::to_string(l) + ".W", 4 * H, 2 * H); add("enc.l" + std::to_string(l) + ".b", 4 * H, 1);
  }
  add("dec.l0.W", 4 * H, E + 2 * H); add("dec.l0.b", 4 * H, 1);
  for (int l = 1; l < c.layers; ++l) {
    add("dec.l" + std::to_string(l) + ".W", 4 * H, 2 * H); add("dec.l" + std::to_string(l) + ".b", 4 * H, 1);
  }
  add("W_a", H, H); add("W_c", H, 2 * H); add("W_o", Vt, H); add("B_o", Vt, 1);
  total = off;
}

size_t find_off(const std::vector<ParamInfo>& t, const std::string& n) {
  for (auto& p : t) if (p.name == n) return p.off;
  return 0;
}

// Carves the workspace.  With base == nullptr only the size is computed.
size_t layout(cmt_handle* h, char* base) {
  const cmt_config& c = h->cfg;
  const size_t esz = h->esz;
  const int E = c.emb_dim, H = c.hidden, Hd = H / 2, L = c.layers;
  const int Bp = h->Bpm, Sm = c.max_src_len, Tm = c.max_tgt_len;
  const size_t Ms = (size_t)Sm * Bp, Mt = (size_t)Tm * Bp;
  Bump a(base);
  const RowPitch pad = row_pitch(c.precision, E, H, h->pad_lines);
  h->PH = H + pad.states;
  const size_t PH = h->PH;
  h->Pc = c.precision ? a.take(h->nparams * esz) : (char*)h->params;
  // (The whole loops take batches up to LOOP_MAX_BATCH; Bl: the rows of their slots.  The slots are there whether or not
  // CMT_DEC_LOOP asks for the loops: the size that a caller was told holds for every handle.)
  const bool loops = h->loop_slots != LOOP_SLOTS_NONE && L <= LOOP_MAX_LAYERS;
  const bool loop_all = loops && h->loop_slots == LOOP_SLOTS_ALL;
  const size_t Bl = std::min(Bp, LOOP_MAX_BATCH);
  auto ld_alloc = [&](LD& d, int Kin, int Hh, int Lm, bool gx, int Kstep, bool encoder) {
    d.Kin = Kin; d.Hh = Hh; d.ph = Hh + pad.states; d.pg = 4 * Hh + (&d == &h->dec[0] ? pad.gates_bottom : pad.gates);
    const size_t M = (size_t)Lm * Bp;
    d.Kstep = Kstep;
    d.fm = !encoder && c.precision && Hh % 32 == 0 && Kstep % 32 == 0;
    if (d.fm) {
      d.Wfm = a.take((size_t)4 * Hh * (Kstep + Hh) * esz);
      d.HstF = a.take((M + Bp) * Hh * esz);
      d.YdF = a.take(M * Hh * esz);
    }
    d.fmb = !encoder && c.precision && Hh % 32 == 0 && Kin % 16 == 0;
    if (d.fmb) {
      d.WtF = a.take((size_t)(Kin + Hh) * 4 * Hh * esz);
      d.dGF = a.take(M * 4 * Hh * esz);
    }
    d.Wt = a.take((size_t)(Kin + Hh) * 4 * Hh * esz);
    d.Hst = a.take((M + Bp) * d.ph * esz);
    d.Cst = (float*)a.take((M + Bp) * Hh * 4);
    d.Gs = (float*)a.take(M * 4 * Hh * 4);
    d.Gx = gx ? (float*)a.take(M * 4 * Hh * 4) : nullptr;
    d.dG = a.take(M * d.pg * esz);
    // The recurrences' exchange slots are filled afresh by every pass and take no memory of their own: the states' lie
    // where the gate gradients are transposed to after the backward pass, the gate gradients' where the forward pass had
    // its input parts.
    // (The decoder's whole loops likewise, where there are no fragment-major copies that can serve.  An evaluation's has no use
    // for the second half, and the bottom layer's takes the fed H_o.)
    const size_t row = loop_slot_elems(1, Hh), Ml = (size_t)Lm * Bl;
    const bool eval_feed = !loop_all && &d == &h->dec[0];
    const size_t fwd_slots = d.fm ? 0 : loop_all ? (2 * Ml + Bl) * row : (eval_feed ? 2 : 1) * (Ml + Bl) * row;
    const size_t slots = encoder ? seq_exchange_elems(Lm + 1, Bp, Hh) : !loops ? 0 : std::max(fwd_slots, d.fmb || !loop_all ? 0 : Ml * 4 * row);
    d.dGT = a.take(std::max(M * 4 * Hh, slots) * esz);
    if (encoder) { d.X = d.dGT; d.XG = (char*)d.Gx; }
    else if (loops) {
      char* const second = d.dGT + (base ? (Ml + Bl) * row * esz : 0);
      d.XH = d.fm ? d.HstF : d.dGT;
      if (loop_all) {
        d.XY = d.fm ? d.YdF : second;
        d.XD = d.fmb ? d.dGF : d.dGT;
      } else if (eval_feed) h->HoFeedX = second;
    }
    d.HstT = a.take((M + Bp) * Hh * esz);
    if (!encoder) {
      d.dh = (float*)a.take((size_t)Bp * Hh * 4);
      d.dc = (float*)a.take((size_t)Bp * Hh * 4);
      d.bwdp = (float*)a.take((size_t)8 * Bp * 2 * Hh * 4);
    }
    d.Yd = a.take(M * d.ph * esz);                 // the layer's output after dropout, and its transpose
    d.YdT = a.take(M * Hh * esz);
  };
  h->enc.assign(L + 1, LD());
  h->dec.assign(L, LD());
  // the encoder's input parts are batched over time; per-step input segment of the decoder: the fed H_o for the bottom
  // layer, the layer below's state for the others
  ld_alloc(h->enc[0], E, Hd, Sm, true, 0, true);
  ld_alloc(h->enc[1], E, Hd, Sm, true, 0, true);
  for (int l = 1; l < L; ++l) ld_alloc(h->enc[l + 1], H, H, Sm, true, 0, true);
  ld_alloc(h->dec[0], E + H, H, Tm, true, H, false);
  for (int l = 1; l < L; ++l) ld_alloc(h->dec[l], H, H, Tm, false, H, false);
  if (c.precision && H % 32 == 0) {
    h->HoFeedF = a.take((Mt + Bp) * H * esz);
    h->WcF = a.take((size_t)2 * H * H * esz); h->WcTF = a.take((size_t)2 * H * H * esz);
    h->CsF = a.take(Mt * H * esz); h->dPreF = a.take(Mt * H * esz);
    if (c.tgt_vocab % 16 == 0) h->WoF = a.take((size_t)c.tgt_vocab * H * esz);
    if (E % 32 == 0) { h->Wdec0F = a.take((size_t)4 * H * (E + 2 * H) * esz); h->xcatF = a.take((size_t)Bp * (E + H) * esz); }
  }
  h->WaT = a.take((size_t)H * H * esz);
  h->WcT = a.take((size_t)2 * H * H * esz);
  h->ldWoT = h->pad_lines ? round_up(c.tgt_vocab, 128 / (int)esz) : c.tgt_vocab;   // (rows of whole cache lines, as dz)
  h->WoT = a.take((size_t)H * h->ldWoT * esz);
  // source side
  h->Xs = a.take(Ms * E * esz); h->XsT = a.take(Ms * E * esz);
  h->mask_s = (float*)a.take(Ms * 4); h->tok_s = (int32_t*)a.take(Ms * 4); h->len_s = (int32_t*)a.take((size_t)Bp * 4);
  h->Y0 = a.take(Ms * H * esz); h->Y0T = a.take(Ms * H * esz); h->Kmat = a.take(Ms * H * esz);
  h->Pmat = (float*)a.take(Ms * H * 4); h->PmatT = a.take(Ms * H * esz);
  h->dHs = (float*)a.take(Ms * H * 4); h->dK = a.take(Ms * H * esz); h->dKT = a.take(Ms * H * esz);
  // (until the encoder's backward pass the decoder's backward loop exchanges its scores there, in dYa and on into dXs)
  const size_t loop_scores = loop_all ? (size_t)Tm * Bl * std::min(Sm, LOOP_MAX_SRC) : 0;
  h->dYa = (float*)a.take(std::max(Ms * H, loop_scores > Ms * E ? loop_scores - Ms * E : 0) * 4);
  h->dXs = (float*)a.take(Ms * E * 4);
  // target side
  h->Xt = a.take(Mt * E * esz); h->XtT = a.take(Mt * E * esz);
  h->mask_t = (float*)a.take(Mt * 4); h->tok_t = (int32_t*)a.take(Mt * 4); h->labels = (int32_t*)a.take(Mt * 4);
  h->len_t = (int32_t*)a.take((size_t)Bp * 4);
  const size_t loop_row = loop_all ? loop_slot_elems(1, H) * esz : 0;  // bytes of a row in a loop's slots
  h->HoBuf = a.take((Mt + Bp) * PH * esz); h->HoBufT = a.take(std::max((Mt + Bp) * H * esz, ((size_t)Tm + 1) * Bl * loop_row));
  if (!loops) h->HoFeedX = nullptr;
  else if (h->HoFeedF) h->HoFeedX = h->HoFeedF;
  else if (loop_all) h->HoFeedX = h->HoBufT;                             // (transposed after the forward loop)
  h->HoDrop = a.take((Mt + Bp) * PH * esz);
  h->ldxcat = E + H + pad.states;
  h->xcat = a.take((size_t)Bp * h->ldxcat * esz);
  h->dec_tok = (int32_t*)a.take((size_t)Bp * 4); h->dec_done = (int32_t*)a.take((size_t)Bp * 4);
  h->dec_mask = (float*)a.take((size_t)Bp * 4);
  h->logits = (float*)a.take((size_t)Bp * c.tgt_vocab * 4);
  {
    BeamState& bs = h->beam;
    bs.cum = (float*)a.take((size_t)Bp * 4); bs.new_cum = (float*)a.take((size_t)Bp * 4); bs.mask = (float*)a.take((size_t)Bp * 4);
    bs.tok = (int32_t*)a.take((size_t)Bp * 4); bs.new_tok = (int32_t*)a.take((size_t)Bp * 4);
    bs.parent = (int32_t*)a.take((size_t)Bp * 4); bs.nlive = (int32_t*)a.take((size_t)Bp * 4);
    bs.fin_score = (float*)a.take((size_t)Bp * 4); bs.fin_step = (int32_t*)a.take((size_t)Bp * 4);
    bs.fin_par = (int32_t*)a.take((size_t)Bp * 4); bs.fin_tok = (int32_t*)a.take((size_t)Bp * 4);
    bs.hist_tok = (int32_t*)a.take(Mt * 4); bs.hist_par = (int32_t*)a.take(Mt * 4);
    bs.hist_ld = Bp;
  }
  h->Cs = a.take(Mt * PH * esz); h->CsT = a.take(Mt * H * esz);
  h->att_a = (float*)a.take(Mt * Sm * 4); h->att_ds = (float*)a.take(Mt * Sm * 4);
  h->dCs = (float*)a.take(std::max(Mt * H * 4, (size_t)Tm * Bl * loop_row));
  h->dPreX = !loop_all ? nullptr : h->dPreF ? h->dPreF : (char*)h->dCs;  // (dC_s is made after the backward loop)
  h->dots = (float*)a.take((size_t)Bp * Sm * 4);
  h->att_s = (float*)a.take(Mt * Sm * 4);
  h->dPre = a.take(Mt * PH * esz); h->dPreT = a.take(Mt * H * esz);
  h->dHoCE = (float*)a.take(Mt * H * 4);
  h->dHt = (float*)a.take((size_t)Bp * H * 4);
  h->wcp = (float*)a.take((size_t)8 * Bp * 2 * H * 4);
  h->dXt = (float*)a.take(Mt * E * 4);
  const int np = ce_num_partials(c.tgt_vocab);
  // output-layer slabs: one slab for the whole batch up to the cap, else full slabs of the cap and a remainder
  h->ce_rows = (int)std::min<size_t>((size_t)h->ce_cap, (Mt + 255) / 256 * 256);
  h->ce_pitch = ce_slab_pitch(h->ce_rows);
  const size_t ce_slabs = (Mt + h->ce_rows - 1) / h->ce_rows;
  const size_t slab_elems = (size_t)h->ce_pitch * c.tgt_vocab;      // elements of a slab buffer (e / dz, and dz^T)
  {   // per slab a [np, pitch] block of partials (slab sl starts at sl * np * pitch)
    const size_t bytes = ce_slabs * h->ce_pitch * np * 4;
    h->pmax = (float*)a.take(bytes); h->psum = (float*)a.take(bytes); h->psz = (float*)a.take(bytes);
  }
  h->zy = (float*)a.take(Mt * 4); h->lse = (float*)a.take(Mt * 4); h->nll = (float*)a.take(Mt * 4);
  h->rowscale = (float*)a.take(Mt * 4);
  h->ce_pos = (int32_t*)a.take(Mt * 4); h->ce_row = (int32_t*)a.take(Mt * 4); h->labels_c = (int32_t*)a.take(Mt * 4);
  h->ce_nvalid = (int32_t*)a.take(256);
  h->Hoc = a.take(Mt * PH * esz); h->HocT = a.take(Mt * H * esz);
  h->loss = (float*)a.take(256); h->flags = (int*)a.take(256); h->tickets = (int*)a.take(SEQ_TICKETS * 4);
  h->colscr = (float*)a.take((size_t)16 * 4 * H * 4);
  h->dzs = a.take(slab_elems * esz); h->dzTs = a.take(slab_elems * esz);
  h->dbo_parts = (float*)a.take((Mt / 64 + Mt / 256 + 4) * c.tgt_vocab * 4);
  {   // split-k planes of dH_o = dz W_o of a slab (k = the vocabulary): 16 planes, at most 256 MB, at least 1 MB
    const size_t slab_rows = std::min<size_t>(Mt, (size_t)h->ce_rows);
    h->gsplit_floats = std::max((size_t)1 << 18, std::min((size_t)64 << 20, 16 * slab_rows * H));
  }
  h->gsplit = (float*)a.take(h->gsplit_floats * 4);
  h->gsplit2_floats = c.precision ? 0 : std::min((size_t)8 << 20, (size_t)16 * 4 * H * std::max(E, H));
  h->gsplit2 = (float*)a.take(h->gsplit2_floats * 4);
  if (ce_slabs > 1) {                             // a second pair, so that slab s + 1 starts while dW_o of slab s still runs
    h->dzs2 = a.take(slab_elems * esz); h->dzTs2 = a.take(slab_elems * esz);
  } else {
    h->dzs2 = h->dzs; h->dzTs2 = h->dzTs;
  }
  return (a.off + 255) & ~(size_t)255;
}

void bind_params(cmt_handle* h) {
  const cmt_config& c = h->cfg;
  auto& t = h->table;
  h->off_Esrc = find_off(t, "E_src"); h->off_Etgt = find_off(t, "E_tgt");
  h->off_Wa = find_off(t, "W_a"); h->off_Wc = find_off(t, "W_c");
  h->off_Wo = find_off(t, "W_o"); h->off_Bo = find_off(t, "B_o");
  auto bind = [&](LD& d, const std::string& n) {
    d.w_off = find_off(t, n + ".W"); d.b_off = find_off(t, n + ".b");
    d.W = h->Pc + d.w_off * h->esz;
  };
  bind(h->enc[0], "enc.l0.fwd"); bind(h->enc[1], "enc.l0.bwd");
  for (int l = 1; l < c.layers; ++l) bind(h->enc[l + 1], "enc.l" + std::to_string(l));
  for (int l = 0; l < c.layers; ++l) bind(h->dec[l], "dec.l" + std::to_string(l));
}

// refresh the kernels' working copies of the parameters: operand-type cast, transposes
void refresh_params(cmt_handle* h, bool cast = true) {
  const cmt_config& c = h->cfg;
  const int H = c.hidden, p = h->prec;
  hipStream_t st = h->st;
  if (p && cast) launch_cast(1, h->params, h->Pc, h->nparams, st);
  std::vector<TransposeJob> t;
  for (auto* v : {&h->enc, &h->dec})
    for (auto& d : *v) t.push_back({d.W, d.Kin + d.Hh, d.Wt, 4 * d.Hh, 4 * d.Hh, d.Kin + d.Hh});
  t.push_back({h->Pw(h->off_Wa), H, h->WaT, H, H, H});
  t.push_back({h->Pw(h->off_Wc), 2 * H, h->WcT, H, H, 2 * H});
  t.push_back({h->Pw(h->off_Wo), H, h->WoT, h->ldWoT, c.tgt_vocab, H});
  launch_transpose_multi(p, t.data(), (int)t.size(), st);
  auto tr = [&](LD& d) {
    if (d.fm) launch_fm_pack_lstm_weights(d.W, d.Kin + d.Hh, d.Kin - d.Kstep, d.Kstep + d.Hh, d.Hh, d.Wfm, st);
    if (d.fmb) launch_fm_pack(d.Wt, 4 * d.Hh, d.Kin + d.Hh, 4 * d.Hh, d.WtF, st);
  };
  for (auto& d : h->enc) tr(d);
  for (auto& d : h->dec) tr(d);
  if (h->WcF) {
    launch_fm_pack(h->Pw(h->off_Wc), 2 * H, H, 2 * H, h->WcF, st);
    launch_fm_pack(h->WcT, H, 2 * H, H, h->WcTF, st);
    if (h->WoF) launch_fm_pack(h->Pw(h->off_Wo), H, c.tgt_vocab, H, h->WoF, st);
    if (h->Wdec0F) launch_fm_pack_lstm_weights(h->dec[0].W, c.emb_dim + 2 * H, 0, c.emb_dim + 2 * H, H, h->Wdec0F, st);
  }
}

int fail(cmt_handle* h, int code, const std::string& msg) {
  if (h) h->err = msg;
  return code;
}
int hip_fail(cmt_handle* h, hipError_t e, const char* what) {
  return fail(h, CMT_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

// ------------------------------------------------------------------------------------------------
// the schedule
// ------------------------------------------------------------------------------------------------
// make stream `to` wait for everything enqueued so far on stream `from`
void stream_after(cmt_handle* h, hipStream_t to, hipStream_t from) {
  if (to == from) return;
  hipEvent_t e = h->ev[h->ev_next++ % h->ev.size()];
  (void)hipEventRecord(e, from);
  (void)hipStreamWaitEvent(to, e, 0);
}

void weight_grads(cmt_handle* h, LD& d, int Lsteps, const std::vector<std::pair<const char*, int>>& segs /* (XT ptr, ld) */,
                  const std::vector<int>& seg_k, hipStream_t st) {
  // dW[:, segment] = dG^T * X_segment as one GEMM with k = Lsteps * Bp; db = column sums of dG
  const int Bp = h->Bp, Hh = d.Hh;
  const int M = Lsteps * Bp;
  // (the partial sums' places: the backward loop's partial sums of some decoder layer are used up)
  const size_t k = h->dw_sums.size();
  float* const parts = k == 0 ? h->colscr : (int)k < h->cfg.layers ? h->dec[k].bwdp : h->wcp;
  h->dw_tr.push_back({d.dG, d.pg, d.dGT, M, M, 4 * Hh, parts});
  h->dw_sums.push_back({parts, (size_t)4 * Hh, h->grads + d.b_off});
  float* dW = h->grads + d.w_off;
  int col = 0;
  for (size_t i = 0; i < segs.size(); ++i) {
    h->dw_group.push_back(GemmProb{d.dGT, segs[i].first, dW + col, M, segs[i].second, d.Kin + Hh, 4 * Hh, seg_k[i], M, 0});
    col += seg_k[i];
  }
}
// launches what weight_grads (and the callers that add W_c / W_a problems) have collected, as one queue of tiles
// big_cap: see launch_gemm_nt_group.
void flush_dw_group(cmt_handle* h, hipStream_t st, int big_cap = 0) {
  launch_transpose_multi(h->prec, h->dw_tr.data(), (int)h->dw_tr.size(), st);
  launch_sum_parts_multi(h->dw_sums.data(), (int)h->dw_sums.size(), TRANSPOSE_SPLITS, st);
  h->dw_tr.clear(); h->dw_sums.clear();
  launch_gemm_nt_group(h->prec, h->dw_group.data(), (int)h->dw_group.size(), st, h->gsplit2, h->gsplit2_floats,
                       st != h->st ? h->side_wgs : 0, st != h->st ? big_cap : 0);
  h->dw_group.clear();
}

// marks the start of a phase of the step on the caller's stream (only when phase timing is on)
void phase_mark(cmt_handle* h, const char* name) {
  if (!h->phase_timing) return;
  if (h->phase_n >= h->phase_ev.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return;
    h->phase_ev.push_back(e); h->phase_name.push_back(name);
  }
  h->phase_name[h->phase_n] = name;
  if (h->phase_host.size() <= h->phase_n) h->phase_host.resize(h->phase_n + 1);
  h->phase_host[h->phase_n] = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
  (void)hipEventRecord(h->phase_ev[h->phase_n++], h->st);
}

// The output layer's slabs: full slabs of the handle's slab capacity and one remainder (a single slab whenever
// the batch fits).  Returns the rows of all slabs but the last.
int ce_slab_plan(const cmt_handle* h, int Mt, int* nslab_out) {
  *nslab_out = (Mt + h->ce_rows - 1) / h->ce_rows;
  return h->ce_rows;
}

// dropout sites (the oracle and the tests use the same numbering): encoder layer l output, decoder
// layer l output, H_o
constexpr int DROP_SITE_ENC = 0, DROP_SITE_DEC = 16, DROP_SITE_HO = 32;
DropSpec drop_spec(const cmt_handle* h, int site, int t) {
  DropSpec d;
  if (h->drop_p > 0.f) {
    const unsigned long long H = (unsigned long long)h->cfg.hidden;
    d.on = 1; d.thresh = h->drop_thresh; d.scale = h->drop_scale; d.width = h->cfg.hidden;
    d.key0 = h->drop_seed + ((unsigned long long)site << 48) + (unsigned long long)t * (unsigned long long)h->B * H;
  }
  return d;
}

// the cell backward of decoder layer l at step j; dy / dhrec are filled in by the caller
LstmBwdPoint dec_cell(cmt_handle* h, int l, int j) {
  const int H = h->cfg.hidden, Bp = h->Bp;
  const size_t BH = (size_t)Bp * H;
  LD& e = h->dec[l];
  LstmBwdPoint q;
  q.dy = Planes{nullptr, 0, 0, 0}; q.dy_col = 0; q.dhrec = Planes{nullptr, 0, 0, 0}; q.dhrec_col = 0;
  q.dh = e.dh; q.dc = e.dc;
  q.gsave = e.Gs + (size_t)j * Bp * 4 * H;
  q.cprev = e.Cst + j * BH; q.cnext = e.Cst + (j + 1) * BH;
  q.mask = h->mask_t + (size_t)j * Bp;
  q.dg = e.dG + (size_t)j * Bp * e.pg * h->esz; q.lddg = e.pg;
  if (e.fmb) q.dg_fm = e.dGF + (size_t)j * Bp * 4 * H * h->esz;
  return q;
}

// Backward step GEMM of decoder layer l at step j in its fused form: [dx; dh_prev] = dgates [W_x; W_h] with the
// whole contraction inside the workgroup.  The dx half feeds the cell backward of the layer below in the
// epilogue (bottom layer: the tanh backward of the previous step's H_o, which received it through the input
// feed); the dh_prev half is stored (one fp32 matrix per layer, the first Bp * H floats of bwdp) for that
// layer's next step.
StepBwd dec_bwd_gemm(cmt_handle* h, int l, int j) {
  const cmt_config& c = h->cfg;
  const int E = c.emb_dim, H = c.hidden, Bp = h->Bp, PH = h->PH;
  const size_t esz = h->esz, BP = (size_t)Bp * PH;
  const bool last = j == h->T - 1;
  LD& e = h->dec[l];
  StepBwd g{};
  g.dg = e.dG + (size_t)j * Bp * e.pg * esz; g.lddg = e.pg; g.K = 4 * H; g.ldw = 4 * H;
  BwdEpi store{};
  store.kind = BWD_EPI_STORE; store.ncols = H; store.hh = H; store.out = e.bwdp; store.ldout = H;
  if (l > 0) {
    g.Wt = e.Wt;
    BwdEpi& c0 = g.part[0];
    c0.kind = BWD_EPI_CELL_DY; c0.ncols = H; c0.hh = H;
    c0.cell = dec_cell(h, l - 1, j);
    c0.cell.drop_dy = drop_spec(h, DROP_SITE_DEC + l - 1, j);
    c0.cell.dhrec = Planes{h->dec[l - 1].bwdp, H, last ? 0 : 1, 0};
    g.part[1] = store;
  } else if (j > 0) {
    g.Wt = e.Wt + (size_t)E * 4 * H * esz;                       // rows [feed; h] of the bottom layer's W^T
    BwdEpi& t0 = g.part[0];
    t0.kind = BWD_EPI_TANH; t0.ncols = H; t0.hh = H;
    t0.dce = h->dHoCE; t0.pos = h->ce_pos + (size_t)(j - 1) * Bp; t0.Ho = h->HoBuf + j * BP * esz; t0.ldho = PH;
    t0.dpre = h->dPre + (j - 1) * BP * esz; t0.ldp = PH; t0.drop = drop_spec(h, DROP_SITE_HO, j - 1);
    if (h->dPreF) t0.dpre_fm = h->dPreF + (size_t)(j - 1) * Bp * H * esz;
    g.part[1] = store;
  } else {
    g.Wt = e.Wt + (size_t)(E + H) * 4 * H * esz;                 // H_o^{<-1>} is a constant: only dh_prev
    g.part[0] = store;
  }
  if (e.fmb) {                                                   // the same operands in fragment-major form
    g.dg_fm = e.dGF + (size_t)j * Bp * 4 * H * esz; g.Wt_fm = e.WtF;
    g.wt_tile0 = (l > 0 ? 0 : j > 0 ? E : E + H) / 16;
  }
  return g;
}

// forward step j of decoder layer l (layer 0 takes [H_o^{<j-1>}; h] per step, its embedding part is pre-batched)
void dec_lstm_fwd(cmt_handle* h, int l, int j) {
  const cmt_config& c = h->cfg;
  const int E = c.emb_dim, H = c.hidden, Bp = h->Bp;
  const size_t esz = h->esz, BH = (size_t)Bp * H, BP = (size_t)Bp * h->PH;
  LD& e = h->dec[l];
  LstmFwdDir d;
  const bool drop = h->drop_p > 0.f;
  if (l == 0) {
    d.x = (drop ? h->HoDrop : h->HoBuf) + j * BP * esz; d.ldx = h->PH; d.Kx = H; d.wx_off = E; d.wh_off = E + H;
    d.gx = e.Gx + (size_t)j * Bp * 4 * H; d.ldgx = 4 * H; d.bias = nullptr; d.ldw = E + 2 * H;
  } else {
    d.x = drop ? h->dec[l - 1].Yd + j * BP * esz : h->dec[l - 1].Hst + (j + 1) * BP * esz;
    d.ldx = e.ph; d.Kx = H; d.wx_off = 0; d.wh_off = H;
    d.gx = nullptr; d.ldgx = 0; d.bias = h->params + e.b_off; d.ldw = 2 * H;
  }
  d.hprev = e.Hst + j * BP * esz; d.ldh = e.ph; d.W = e.W;
  d.cprev = e.Cst + j * BH; d.mask = h->mask_t + (size_t)j * Bp;
  d.hnext = e.Hst + (j + 1) * BP * esz; d.ldhn = e.ph; d.cnext = e.Cst + (j + 1) * BH;
  d.gsave = e.Gs + (size_t)j * Bp * 4 * H; d.ycat = nullptr; d.ldy = 0;
  if (drop && l + 1 < c.layers) {                  // what the layer above reads
    d.ycat = e.Yd + j * BP * esz; d.ldy = e.ph; d.drop = drop_spec(h, DROP_SITE_DEC + l, j); d.drop_col0 = 0;
  }
  if (e.fm) {                                      // the contraction's operands in fragment-major form
    d.W_fm = e.Wfm;
    d.x_fm = l == 0 ? h->HoFeedF + j * BH * esz
                    : (drop ? h->dec[l - 1].YdF + j * BH * esz : h->dec[l - 1].HstF + (j + 1) * BH * esz);
    d.hprev_fm = e.HstF + j * BH * esz; d.hnext_fm = e.HstF + (j + 1) * BH * esz;
    if (d.ycat) d.ycat_fm = e.YdF + j * BH * esz;
  }
  launch_lstm_fwd(h->prec, d, Bp, H, h->st);
}

// Attention and attentional layer of decoder step j on the projected source rows P_i = W_c1 H_s^i (Eq. 3-7
// regrouped: W_c [C_s; H_t] = sum_i a_i P_i + W_c2 H_t), two dependent launches: the scores together with the sums
// W_c2 H_t (both wait for the top layer's state alone), then softmax, mix, tanh -> H_o and its copies.
void dec_att_fwd_proj(cmt_handle* h, int j, int S, float* scores) {
  const int p = h->prec, H = h->cfg.hidden, L = h->cfg.layers, Bp = h->Bp, PH = h->PH;
  const size_t esz = h->esz, BH = (size_t)Bp * H, BP = (size_t)Bp * PH;
  const char* Ht = h->dec[L - 1].Hst + (j + 1) * BP * esz;
  StepGemm g{};
  g.a0 = nullptr; g.lda0 = PH; g.K0 = H; g.w0_off = 0; g.skip0 = 1;
  g.a1 = Ht; g.lda1 = PH; g.K1 = H; g.w1_off = H;
  g.W = h->Pw(h->off_Wc); g.ldw = 2 * H; g.N = H; g.mode = 3;
  g.out = h->wcp; g.ldout = H; g.plane_stride = BH;
  if (h->HoFeedF) { g.W_fm = h->WcF; g.a1_fm = h->dec[L - 1].HstF + (j + 1) * BH * esz; g.a0_fm = g.a1_fm; }
  AttOut o{};
  o.outT = h->HoBuf + (j + 1) * BP * esz; o.ldo = PH;
  if (h->drop_p > 0.f) { o.outD = h->HoDrop + (j + 1) * BP * esz; o.ldod = PH; o.drop = drop_spec(h, DROP_SITE_HO, j); }
  if (h->HoFeedF) o.outF = h->HoFeedF + (j + 1) * BH * esz;
  launch_att_fwd_proj(p, h->Kmat, H, h->PmatT, H, Ht, PH, g, o, h->len_s, S, Bp, H, scores, h->att_a + (size_t)j * Bp * S, h->st);
}
// The backward of the same on the projected rows, two dependent launches: the score gradients da_i = dC_s . H_s^i
// are dpre . P_i (fp32 rows), so they need dpre alone and ride in the launch of [dC_s ; dH_t] = dpre W_c, whose halves
// go where their readers want them (dC_s to its slot for the deferred gradients, the dH_t half beside it); then
// the softmax Jacobian, the gradient sent to the top layer's output and that layer's cell backward.
void dec_att_bwd_proj(cmt_handle* h, int j, int S, bool last) {
  const int p = h->prec, H = h->cfg.hidden, L = h->cfg.layers, Bp = h->Bp, PH = h->PH;
  const size_t esz = h->esz, BH = (size_t)Bp * H, BP = (size_t)Bp * PH;
  char* dpre = h->dPre + j * BP * esz;
  char* dpreF = h->dPreF ? h->dPreF + j * BH * esz : nullptr;
  StepBwd g{};
  g.dg = dpre; g.lddg = PH; g.K = H; g.Wt = h->WcT; g.ldw = H;
  g.part[0].kind = BWD_EPI_STORE; g.part[0].ncols = H; g.part[0].out = h->dCs + j * BH; g.part[0].ldout = H;
  g.part[1].kind = BWD_EPI_STORE; g.part[1].ncols = H; g.part[1].out = h->wcp; g.part[1].ldout = H;
  g.dg_fm = dpreF; g.Wt_fm = dpreF ? h->WcTF : nullptr; g.wt_tile0 = 0;
  const AttScores sc{h->Pmat, H, dpre, PH, h->len_s, S, H, h->dots, 1};
  launch_step_bwd_fused(p, g, Bp, h->st, &sc);
  LstmBwdPoint top = dec_cell(h, L - 1, j);
  top.dhrec = Planes{h->dec[L - 1].bwdp, H, last ? 0 : 1, 0};
  launch_att_bwd_mix(p, h->Kmat, H, Planes{h->wcp, H, 1, 0}, 0, h->att_a + (size_t)j * Bp * S, h->len_s, S, Bp, H, h->dots,
                     h->att_ds + (size_t)j * Bp * S, h->dHt, h->st, &top);
}

// Encoder forward for the batch whose source embeddings, masks and lengths are in the workspace (gather done by the
// caller): per layer one GEMM for the input part of all positions and one launch for the whole recurrence (bottom layer:
// both directions), then the attention keys and the decoder's initial states.  Returns H_s (top-layer states) and its
// row pitch.
// states_fm: the decoder's per-position kernels read the initial states (its loops make copies of their own).  proj: the projected
// source rows P_i = W_c1 H_s^i are wanted (operand type; and fp32 to Pmat if that is set).  z: fills that go along.
void enqueue_encoder(cmt_handle* h, int S, const char** Hs_out, int* ldHs_out, bool states_fm, bool proj, float* Pmat,
                     std::vector<FillJob> z = {}) {
  const cmt_config& c = h->cfg;
  const int p = h->prec, E = c.emb_dim, H = c.hidden, Hd = H / 2, L = c.layers, Bp = h->Bp;
  const size_t esz = h->esz;
  hipStream_t st = h->st;
  const int Ms = S * Bp;
  const size_t BH = (size_t)Bp * H;
  const int PH = h->PH;
  const bool drop = h->drop_p > 0.f;
  const size_t BP = (size_t)Bp * PH;
  float* P = h->params;
  LD& ef = h->enc[0]; LD& eb = h->enc[1];
  const size_t BHd = (size_t)Bp * Hd, BPd = (size_t)Bp * ef.ph;
  const unsigned long long drop_step = (unsigned long long)h->B * H;
  {   // initial states of every encoder LSTM (zero), and the exchange slots and tickets of the recurrences: one launch
    add_fill(z, ef.Hst, BPd, esz); add_fill(z, ef.Cst, BHd, 4);
    add_fill(z, eb.Hst + (size_t)S * BPd * esz, BPd, esz); add_fill(z, eb.Cst + (size_t)S * BHd, BHd, 4);
    for (int l = 1; l < L; ++l) { add_fill(z, h->enc[l + 1].Hst, BP, esz); add_fill(z, h->enc[l + 1].Cst, BH, 4); }
    for (int l = 0; l <= L; ++l) add_empty(z, h->enc[l].X, seq_exchange_elems(S + 1, Bp, h->enc[l].Hh), esz);
    add_fill(z, h->tickets, SEQ_TICKETS, 4);
    launch_fill_multi(z.data(), (int)z.size(), st);
  }
  {   // the input parts of both directions: one launch
    GemmProb g[2];
    for (int i = 0; i < 2; ++i) {
      LD& d = i ? eb : ef;
      g[i] = GemmProb{h->Xs, d.W, d.Gx, E, E + Hd, 4 * Hd, Ms, 4 * Hd, E, 0, P + d.b_off};
    }
    launch_gemm_nt_group(p, g, 2, st, nullptr, 0);
  }
  auto seq_dir = [&](LD& e) {
    SeqFwdDir d{};
    d.W = e.W; d.ldw = e.Kin + e.Hh; d.wh_off = e.Kin; d.gx = e.Gx; d.mask = h->mask_s; d.X = e.X;
    d.H = e.Hst; d.ldh = e.ph; d.C = e.Cst; d.G = e.Gs;
    return d;
  };
  SeqFwdArgs sa{};
  sa.ticket = h->tickets; sa.again = h->again;
  for (int i = 0; i < 2; ++i) {
    SeqFwdDir& d = sa.d[i];
    d = seq_dir(i ? eb : ef);
    d.Y = h->Y0; d.ldy = H; d.y_col0 = i ? Hd : 0; d.reverse = i;
    if (L > 1) { d.drop = drop_spec(h, DROP_SITE_ENC + 0, 0); d.drop_step = drop_step; }
  }
  launch_lstm_seq_fwd(p, sa, 2, S, Bp, Hd, h->seq, st);
  phase_mark(h, "encoder upper layers");
  const char* Yprev = h->Y0;                       // [S*Bp, H] what the next layer (or the attention) reads
  int ldY = H;
  for (int l = 1; l < L; ++l) {
    LD& e = h->enc[l + 1];
    launch_gemm_nt(p, Yprev, ldY, e.W, 2 * H, Ms, 4 * H, H, e.Gx, nullptr, 4 * H, P + e.b_off, 0, st);
    sa.ticket = h->tickets + 2 * l;
    sa.d[0] = seq_dir(e);
    const bool dropped = drop && l + 1 < L;
    if (dropped) {
      sa.d[0].Y = e.Yd; sa.d[0].ldy = PH;
      sa.d[0].drop = drop_spec(h, DROP_SITE_ENC + l, 0); sa.d[0].drop_step = drop_step;
    }
    launch_lstm_seq_fwd(p, sa, 1, S, Bp, H, h->seq, st);
    Yprev = dropped ? e.Yd : e.Hst + BP * esz; ldY = PH;
  }
  const char* Hs = Yprev;
  const int ldHs = ldY;                          // source-side top-layer states [S, Bp, H]
  *Hs_out = Hs; *ldHs_out = ldHs;
  // attention keys K_i = W_a^T H_s^i for all i at once (Eq. 4 regrouped)
  // and the projected rows: one launch (3200 positions, width 1024: 22 + 23 -> 33 us)
  {
    GemmProb g[2];
    g[0] = GemmProb{Hs, h->WaT, nullptr, ldHs, H, H, Ms, H, H, 0}; g[0].Ct = h->Kmat;
    g[1] = GemmProb{Hs, h->Pw(h->off_Wc), Pmat, ldHs, 2 * H, H, Ms, H, H, 0}; g[1].Ct = h->PmatT;
    launch_gemm_nt_group(p, g, proj ? 2 : 1, st, nullptr, 0);
  }

  phase_mark(h, "keys, decoder init, decoder input GEMM");
  // ---- decoder initial state = encoder final state of the same depth ------------------------------
  {
    LD& d0 = h->dec[0];
    std::vector<CopyJob> cp;
    add_copy(cp, ef.Hst + (size_t)S * BPd * esz, ef.ph, d0.Hst, d0.ph, Bp, Hd, esz);
    add_copy(cp, eb.Hst, eb.ph, d0.Hst + (size_t)Hd * esz, d0.ph, Bp, Hd, esz);
    add_copy(cp, ef.Cst + (size_t)S * BHd, Hd, d0.Cst, H, Bp, Hd, 4);
    add_copy(cp, eb.Cst, Hd, d0.Cst + Hd, H, Bp, Hd, 4);
    for (int l = 1; l < L; ++l) {
      LD& e = h->enc[l + 1]; LD& d = h->dec[l];
      add_copy(cp, e.Hst + (size_t)S * BP * esz, e.ph, d.Hst, d.ph, Bp, H, esz);
      add_copy(cp, e.Cst + (size_t)S * BH, H, d.Cst, H, Bp, H, 4);
    }
    launch_copy2d_multi(cp.data(), (int)cp.size(), st);
    for (int l = 0; states_fm && l < L; ++l)        // fragment-major copies of the initial states
      if (h->dec[l].fm) launch_fm_pack(h->dec[l].Hst, h->dec[l].ph, Bp, H, h->dec[l].HstF, st);
  }
}

// The parts of a pass whose workgroups wait for one another, the encoder's recurrences and the decoder's loops, as sections of
// the device's gate (section_gate.h): a loop may take every CU there is, and if parts of two such launches were on the chip
// at once, neither might get on until its waits are given up.  Nothing of the kind under capture, where an event from outside
// must not be waited for; loops are not captured.
// A loop that runs alone shares its section with the encoder's recurrences beside it while no handle of the device has another stream
// (each section's end costs an event, 5 us of a step), and has one of its own otherwise: steps of three handles on their streams, 512
// units, 32 sentences 3.88 | 3.68 ms a round, 256 units, 64 sentences 3.50 | 3.23.
class Section {
 public:
  explicit Section(cmt_handle* h) : h_(h) {}
  ~Section() { close(); }
  Section(const Section&) = delete;
  Section& operator=(const Section&) = delete;
  void open(bool alone) {
    if (open_ || h_->capturing || h_->seq.mode == SEQ_RUN_ALONE) return;
    alone_ = alone;
    h_->gate->enter(*h_->section, h_->st, alone_);
    open_ = true;
  }
  void close() {
    if (open_) h_->gate->leave(*h_->section, h_->st, alone_);
    open_ = false;
  }
 private:
  cmt_handle* h_;
  bool open_ = false, alone_ = false;
};
void note_capture(cmt_handle* h) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  h->capturing = hipStreamIsCapturing(h->st, &s) == hipSuccess && s != hipStreamCaptureStatusNone;
}

// Whether the decoder's loops run as one launch each, given what the plan of their workgroups says.
bool dec_loop(const cmt_handle* h, const LoopFit& f) {
  return h->loop && !h->capturing && h->att_proj == 1 && h->HoFeedX && f.fits && (f.pays || h->loop == 2);
}
// All target positions of the forward pass, on the projected source rows.
void enqueue_dec_loop_fwd(cmt_handle* h, int S, int T) {
  const cmt_config& c = h->cfg;
  const int p = h->prec, E = c.emb_dim, H = c.hidden, L = c.layers, Bp = h->Bp;
  const size_t esz = h->esz, slot = loop_slot_elems(Bp, H);
  const bool drop = h->drop_p > 0.f;
  hipStream_t st = h->st;
  LoopFwdArgs a{};
  std::vector<FillJob> z;
  for (int l = 0; l < L; ++l) {
    LD& e = h->dec[l];
    LoopFwdLayer& d = a.l[l];
    d.W = e.W; d.ldw = e.Kin + H; d.wx_off = l == 0 ? E : 0; d.wh_off = e.Kin; d.bias = l > 0 ? h->params + e.b_off : nullptr;
    d.H = e.Hst; d.ldh = e.ph; d.C = e.Cst; d.G = e.Gs; d.X = e.XH;
    if (drop && l + 1 < L) { d.Y = e.Yd; d.XY = e.XY; d.drop = drop_spec(h, DROP_SITE_DEC + l, 0); add_empty(z, e.XY, T * slot, esz); }
    add_empty(z, e.XH, (T + 1) * slot, esz);
  }
  a.gx = h->dec[0].Gx; a.mask = h->mask_t; a.len = h->len_s;
  a.Wc = h->Pw(h->off_Wc) + (size_t)H * esz; a.ldwc = 2 * H;
  a.K = h->Kmat; a.P = h->PmatT; a.Pg = h->dK;     // (dK is made after the backward loop)
  a.scores = h->att_s; a.a = h->att_a;
  a.Ho = h->HoBuf; a.HoD = drop ? h->HoDrop : nullptr; a.ldho = h->PH; a.XO = h->HoFeedX;
  if (drop) a.drop_o = drop_spec(h, DROP_SITE_HO, 0);
  a.drop_step = (unsigned long long)h->B * H;
  a.ticket = h->tickets + LOOP_TICKET_FWD; a.again = h->again;
  add_empty(z, h->HoFeedX + slot * esz, T * slot, esz);
  add_empty(z, h->att_s, (size_t)T * Bp * S, 4);
  // (slot 0 of the bottom layer's input, H_o^{<-1>} = 0)
  add_fill(z, h->HoFeedX, slot, esz);
  launch_fill_multi(z.data(), (int)z.size(), st);
  launch_loop_columns(p, h->PmatT, h->dK, S, Bp, H, st);
  launch_loop_fwd(p, a, L, T, Bp, H, S, h->seq, st);
}

// All steps of greedy decoding, on the projected source rows.
void enqueue_greedy_loop(cmt_handle* h, int B, int S, int T, int eos, int32_t* out_ids, int32_t* out_len) {
  const cmt_config& c = h->cfg;
  const int p = h->prec, E = c.emb_dim, H = c.hidden, L = c.layers, Bp = h->Bp;
  const size_t esz = h->esz, slot = loop_slot_elems(Bp, H);
  hipStream_t st = h->st;
  LoopFwdArgs a{};
  std::vector<FillJob> z;
  for (int l = 0; l < L; ++l) {
    LD& e = h->dec[l];
    LoopFwdLayer& d = a.l[l];
    d.W = e.W; d.ldw = e.Kin + H; d.wx_off = l == 0 ? E : 0; d.wh_off = e.Kin; d.bias = h->params + e.b_off;
    d.H = e.Hst; d.ldh = e.ph; d.C = e.Cst; d.X = e.XH;
    add_empty(z, e.XH, (T + 1) * slot, esz);
  }
  a.len = h->len_s; a.Wc = h->Pw(h->off_Wc) + (size_t)H * esz; a.ldwc = 2 * H;
  a.K = h->Kmat; a.P = h->PmatT; a.Pg = h->dK; a.scores = h->att_s;
  a.Ho = h->HoBuf; a.ldho = h->PH; a.XO = h->HoFeedX;
  a.ticket = h->tickets + LOOP_TICKET_FWD; a.again = h->again;
  h->n_loops++;
  LoopTokens& t = a.t;
  t.table = h->Pw(h->off_Etgt); t.emb = E; t.fm = h->WoF ? 1 : 0; t.Wo = h->WoF ? h->WoF : h->Pw(h->off_Wo);
  t.Bo = h->params + h->off_Bo; t.V = c.tgt_vocab;
  t.part = (uint64_t*)h->wcp; t.tok = (int*)((char*)h->wcp + (size_t)4 * H * Bp);   // (of 64 H Bp bytes)
  t.B = B; t.bos = c.bos_id; t.eos = eos; t.pad = c.pad_id; t.out_ids = out_ids; t.out_len = out_len;
  add_empty(z, h->HoFeedX + slot * esz, T * slot, esz);
  add_empty(z, h->att_s, (size_t)T * Bp * S, 4);
  add_empty(z, h->wcp, (size_t)H * Bp + 4 * Bp, 4);
  add_fill(z, h->HoBuf, (size_t)Bp * h->PH, esz);              // (H_o before the first step, for the form without waits)
  launch_fill_multi(z.data(), (int)z.size(), st);
  launch_loop_columns(p, h->PmatT, h->dK, S, Bp, H, st);
  launch_loop_decode(p, a, L, T, Bp, H, S, h->seq, st);
}

// All target positions of the backward pass.
void enqueue_dec_loop_bwd(cmt_handle* h, int S, int T) {
  const cmt_config& c = h->cfg;
  const int p = h->prec, E = c.emb_dim, H = c.hidden, L = c.layers, Bp = h->Bp;
  const size_t esz = h->esz, slot = loop_slot_elems(Bp, H);
  const bool drop = h->drop_p > 0.f;
  hipStream_t st = h->st;
  LoopBwdArgs a{};
  std::vector<FillJob> z;
  for (int l = 0; l < L; ++l) {
    LD& e = h->dec[l];
    LoopBwdLayer& d = a.l[l];
    d.Wt = e.Wt; d.ldw = 4 * H; d.x_row = l == 0 ? E : 0; d.h_row = e.Kin;
    d.C = e.Cst; d.G = e.Gs; d.dG = e.dG; d.lddg = e.pg; d.X = e.XD; d.part = e.bwdp; d.dh = e.dh; d.dc = e.dc;
    if (drop && l + 1 < L) d.drop = drop_spec(h, DROP_SITE_DEC + l, 0);
    add_empty(z, e.XD, T * 4 * slot, esz);
    add_empty(z, e.bwdp, (size_t)16 * Bp * H, 4);
  }
  a.mask = h->mask_t; a.len = h->len_s; a.Wct = h->WcT + (size_t)H * H * esz;
  a.K = h->Kmat; a.Kg = h->dKT; a.P = h->Pmat;     // (dKT is made after the loop)
  a.a = h->att_a; a.da = h->dYa; a.ds = h->att_ds;
  a.dce = h->dHoCE; a.pos = h->ce_pos; a.Ho = h->HoBuf; a.ldho = h->PH;
  a.dPre = h->dPre; a.ldp = h->PH; a.XP = h->dPreX;
  if (drop) a.drop_o = drop_spec(h, DROP_SITE_HO, 0);
  a.drop_step = (unsigned long long)h->B * H;
  a.ticket = h->tickets + LOOP_TICKET_BWD; a.again = h->again;
  add_empty(z, h->dPreX, T * slot, esz);
  add_empty(z, h->dYa, (size_t)T * Bp * S, 4);
  launch_fill_multi(z.data(), (int)z.size(), st);
  launch_loop_columns(p, h->Kmat, h->dKT, S, Bp, H, st);
  launch_loop_bwd(p, a, L, T, Bp, H, S, h->seq, st);
}
// dC_s of all positions (the deferred gradients read it): dpre W_c1
void enqueue_dec_contexts_bwd(cmt_handle* h, int T) {
  const int p = h->prec, H = h->cfg.hidden, Bp = h->Bp;
  const size_t esz = h->esz;
  // (fp32: a quarter of k at a time.  Summed up in one go it made the encoder's gradients 10 - 30 % worse against 64 bits than the launch per
  // position, whose wavefronts share k, did: 512 units, 2 layers, error of the upper encoder layer's dW 5.0e-7 instead of 3.9e-7, 3.8e-7 so)
  for (int k = 0, kc = p ? H : std::max(round_up(H, 64) / 4, 32); k < H; k += kc)
    launch_gemm_nt(p, (const char*)h->dPre + k * esz, h->PH, (const char*)h->WcT + k * esz, H, T * Bp, H, std::min(kc, H - k), h->dCs, nullptr, H,
                   nullptr, k > 0, h->st);
}

int enqueue_step(cmt_handle* h, const int32_t* src_ids, const int32_t* src_len, const int32_t* tgt_ids,
                 const int32_t* tgt_len, int B, int S, int T, bool forward_only) {
  const cmt_config& c = h->cfg;
  if (!src_ids || !src_len || !tgt_ids || !tgt_len) return fail(h, CMT_EINVAL, "null input pointer");
  if (B < 1 || B > c.max_batch || S < 1 || S > c.max_src_len || T < 1 || T > c.max_tgt_len)
    return fail(h, CMT_EINVAL, "B, S or T outside [1, configured maximum]");
  const int p = h->prec, E = c.emb_dim, H = c.hidden, Hd = H / 2, L = c.layers, V = c.tgt_vocab;
  const int Bp = round_up(B, 16);
  const size_t esz = h->esz;
  hipStream_t st = h->st;
  h->B = B; h->Bp = Bp; h->S = S; h->T = T;
  const int Ms = S * Bp, Mt = T * Bp;
  const size_t BH = (size_t)Bp * H;
  const int PH = h->PH;                            // row pitch of the H-wide per-step operands
  const bool drop = h->drop_p > 0.f;
  char* HoFeed = drop ? h->HoDrop : h->HoBuf;      // H_o as its consumers (output layer, input feed) see it
  const size_t BP = (size_t)Bp * PH;
  float* G = h->grads;
  float* P = h->params;

  h->phase_n = 0;
  phase_mark(h, "gathers + encoder bottom layer");
  // H_o^{<-1>} = 0, and the decoder's state gradients at the end of time = 0: with the encoder's fills.  (The error flags
  // are not cleared here: they accumulate over the steps enqueued since the last read-back.)
  std::vector<FillJob> z0;
  add_fill(z0, h->HoBuf, BP, esz);
  if (drop) add_fill(z0, h->HoDrop, BP, esz);
  if (h->HoFeedF) add_fill(z0, h->HoFeedF, BH, esz);
  for (int l = 0; l < L; ++l) { add_fill(z0, h->dec[l].dh, BH, 4); add_fill(z0, h->dec[l].dc, BH, 4); }
  // ---- embeddings, masks ------------------------------------------------------------------------
  const GatherSide sides[2] = {
      {h->Pw(h->off_Esrc), c.src_vocab, src_ids, src_len, S, 0, 0, h->Xs, h->mask_s, h->tok_s, nullptr, h->len_s},
      {h->Pw(h->off_Etgt), c.tgt_vocab, tgt_ids, tgt_len, T, 1, c.bos_id, h->Xt, h->mask_t, h->tok_t, h->labels, h->len_t}};
  launch_gather(p, sides, 2, E, B, Bp, h->flags, st);
  // valid target positions numbered densely, n_tok, 1 / n_tok: the lengths give them
  launch_ce_compact(h->mask_t, h->labels, Mt, h->ce_pos, h->ce_row, h->labels_c, h->rowscale, h->ce_nvalid, h->loss, st);

  const char* Hs; int ldHs;                        // source-side top-layer states [S, Bp, H] and their row pitch
  note_capture(h);
  const LoopFit fit = loop_fits(p, L, Bp, H, S, T, h->seq);
  const bool loop = dec_loop(h, fit), alone = loop && fit.alone;   // the whole decoder loop as one launch
  h->ran_loops = loop ? LOOP_RAN_FWD : 0;
  const bool split = alone && h->gate->crowded(*h->section);
  Section sec(h);
  sec.open(alone && !split);
  const bool proj = h->att_proj && Bp < 256;
  enqueue_encoder(h, S, &Hs, &ldHs, !loop, proj, h->Pmat, std::move(z0));
  if (!loop || split) sec.close();
  LD& ef = h->enc[0]; LD& eb = h->enc[1];
  // ---- decoder time loop --------------------------------------------------------------------------
  // The attentional layer's pre-activation W_c [C_s; H_t] (Eq. 7) is sum_i a_i (W_c1 H_s^i) + W_c2 H_t: with the rows
  // W_c1 H_s^i made once per batch, a step needs no context before its H_o, and the W_c2 H_t sums share a launch
  // with the scores (both wait for the top layer's state alone) — two dependent launches per step instead of three.
  // The contexts themselves (the weight gradient of W_c needs them) are made for all steps at once afterwards.
  {
    LD& d0 = h->dec[0];
    launch_gemm_nt(p, h->Xt, E, d0.W, E + 2 * H, Mt, 4 * H, E, d0.Gx, nullptr, 4 * H, P + d0.b_off, 0, st);
    phase_mark(h, "decoder forward loop");
    if (loop) {
      sec.open(alone);
      enqueue_dec_loop_fwd(h, S, T);
      sec.close();
      h->n_loops++;
    }
    for (int j = loop ? T : 0; j < T; ++j) {
      for (int l = 0; l < L; ++l) dec_lstm_fwd(h, l, j);
      const char* Ht = h->dec[L - 1].Hst + (j + 1) * BP * esz;
      if (proj) { dec_att_fwd_proj(h, j, S, h->att_s + (size_t)j * Bp * S); continue; }
      StepGemm g{};
      g.a0 = h->Cs + j * BP * esz; g.lda0 = PH; g.K0 = H; g.w0_off = 0;
      g.a1 = Ht; g.lda1 = PH; g.K1 = H; g.w1_off = H;
      g.W = h->Pw(h->off_Wc); g.ldw = 2 * H; g.N = H; g.mode = 0;
      g.out = h->wcp; g.ldout = H; g.plane_stride = BH;
      launch_att_fwd(p, h->Kmat, H, Hs, ldHs, Ht, PH, h->len_s, S, Bp, H, h->att_s + (size_t)j * Bp * S,
                     h->att_a + (size_t)j * Bp * S, h->Cs + j * BP * esz, PH, st, h->CsF ? h->CsF + j * BH * esz : nullptr);
      g.outT = h->HoBuf + (j + 1) * BP * esz; g.ldo = PH;
      if (drop) { g.outD = h->HoDrop + (j + 1) * BP * esz; g.ldod = PH; g.drop = drop_spec(h, DROP_SITE_HO, j); }
      if (h->HoFeedF) {
        g.outF = h->HoFeedF + (j + 1) * BH * esz;
        g.W_fm = h->WcF; g.a0_fm = h->CsF + j * BH * esz; g.a1_fm = h->dec[L - 1].HstF + (j + 1) * BH * esz;
      }
      launch_step_gemm(p, g, Bp, st);
    }
  }
  phase_mark(h, "output layer forward + backward");
  // =================================== output layer (Eq. 1) and backward ==============================
  // The recurrences' backward loops are chains of short dependent kernels that leave most of the
  // chip idle; everything that does not feed them (transposes, weight gradients, dW_o, embedding
  // scatters) runs on the library's second stream and joins at the end of the step.
  const char* Ho = HoFeed + BP * esz;              // [T*Bp, H], row pitch PH
  const int np = ce_num_partials(V);
  // The output layer sees the valid target positions only: their H_o rows are gathered into a dense
  // matrix (the count is known to the device alone, so launches are sized for all T * Bp rows and the
  // kernels stop at the count).
  launch_ce_gather_rows(p, Ho, PH, h->ce_row, h->ce_nvalid, Mt, h->Hoc, PH, H, st);
  if (forward_only) {                              // Eq. 1 and the loss only: logits slab by slab, no gradient
    if (proj) launch_att_context(p, Hs, ldHs, h->att_a, h->len_s, S, T, Bp, H, h->Cs, PH, st);   // (for the read-back by name)
    int nslab;
    const int rows = ce_slab_plan(h, Mt, &nslab);
    int sl = 0;
    for (int m0 = 0; m0 < Mt; ++sl) {
      const int Mc = (sl == nslab - 1 || Mt - m0 < rows) ? Mt - m0 : rows;
      const RowLimit lim{h->ce_nvalid, m0};
      const size_t po = (size_t)sl * np * h->ce_pitch;       // this slab's block of partials
      launch_ce_fwd(p, h->Hoc + (size_t)m0 * PH * esz, PH, h->Pw(h->off_Wo), P + h->off_Bo, h->labels_c + m0, Mc, V, H, h->dzTs,
                    h->ce_pitch, h->pmax + po, h->psum + po, h->ls_eps > 0.f ? h->psz + po : nullptr, h->zy + m0, st, lim);
      launch_ce_rows(h->pmax + po, h->psum + po, h->psz + po, h->zy + m0, nullptr, Mc, np, h->ce_pitch, h->ls_eps, V,
                     h->lse + m0, h->nll + m0, st, lim);
      m0 += Mc;
    }
    launch_ce_loss(h->nll, Mt, h->loss, h->flags, h->h_loss, st, RowLimit{h->ce_nvalid, 0});
    phase_mark(h, "end");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "enqueue");
    h->have_step = true;
    return CMT_OK;
  }
  hipStream_t sd = h->use_side ? h->side : st;
  const int ldHoT = Mt + Bp;
  stream_after(h, sd, st);
  // the dense embedding gradients start from zero: cleared now, while the second stream has little to do
  launch_fill_f32(G + h->off_Esrc, (size_t)c.src_vocab * E, 0.f, sd);
  launch_fill_f32(G + h->off_Etgt, (size_t)c.tgt_vocab * E, 0.f, sd);
  hipEvent_t esrc_cleared = nullptr;               // the source table's scatter runs on the caller's stream at the end
  if (sd != st) {
    esrc_cleared = h->ev[h->ev_next++ % h->ev.size()];
    (void)hipEventRecord(esrc_cleared, sd);
  }
  {
    std::vector<TransposeJob> t;
    t.push_back({h->Hoc, PH, h->HocT, Mt, Mt, H});                   // dense H_o rows, for dW_o
    t.push_back({HoFeed, PH, h->HoBufT, ldHoT, Mt + Bp, H});
    for (auto& d : h->enc) t.push_back({d.Hst, d.ph, d.HstT, (S + 1) * Bp, (S + 1) * Bp, d.Hh});
    for (auto& d : h->dec) t.push_back({d.Hst, d.ph, d.HstT, (T + 1) * Bp, (T + 1) * Bp, d.Hh});
    if (drop) {                                    // inputs of the layers above, as they saw them
      for (int l = 1; l + 1 < L; ++l) t.push_back({h->enc[l + 1].Yd, PH, h->enc[l + 1].YdT, Ms, Ms, H});
      for (int l = 0; l + 1 < L; ++l) t.push_back({h->dec[l].Yd, PH, h->dec[l].YdT, Mt, Mt, H});
    }
    t.push_back({h->Y0, H, h->Y0T, Ms, Ms, H});
    t.push_back({h->Xs, E, h->XsT, Ms, Ms, E});
    t.push_back({h->Xt, E, h->XtT, Mt, Mt, E});
    launch_transpose_multi(p, t.data(), (int)t.size(), sd);
  }
  if (proj) launch_att_context(p, Hs, ldHs, h->att_a, h->len_s, S, T, Bp, H, h->Cs, PH, sd);
  {
    const TransposeJob t{h->Cs, PH, h->CsT, Mt, Mt, H};
    launch_transpose_multi(p, &t, 1, sd);
  }
  {
    // Full slabs of the slab capacity and one remainder (one slab whenever the batch fits), two slab buffer pairs, over the dense rows of
    // the valid target positions.  The host sizes the slabs for all T * Bp rows; every kernel gets the
    // device's count and a slab that lies beyond it costs a few empty launches.  Per slab the main
    // stream takes forward (logits -> e, partials), lse / nll, e -> dz and dz^T, and dH_o = dz W_o (the
    // decoder needs it); the second stream takes dW_o += dz^T H_o and dB_o.
    int nslab;
    const int rows = ce_slab_plan(h, Mt, &nslab);
    std::vector<hipEvent_t> done(nslab, nullptr);
    const float eps = h->ls_eps;
    int sl = 0, n_dbo = 0;
    for (int m0 = 0; m0 < Mt; ++sl) {
      const int Mc = (sl == nslab - 1 || Mt - m0 < rows) ? Mt - m0 : rows;
      const RowLimit lim{h->ce_nvalid, m0};
      char* dz = (sl & 1) ? h->dzs2 : h->dzs;
      char* dzT = (sl & 1) ? h->dzTs2 : h->dzTs;
      // (rows of dz as whole cache lines where the slab's buffer, pitch x vocabulary, holds them: 7170 positions x 50000 ce_scale 634 -> 491 us,
      // dz W_o 1016 -> 848 with those of W_o^T)
      const int line = 128 / (int)esz, whole = round_up(V, line), lddz = (size_t)Mc * whole <= (size_t)h->ce_pitch * V ? whole : V;
      if (sl >= 2 && sd != st) (void)hipStreamWaitEvent(st, done[sl - 2], 0);
      const size_t po = (size_t)sl * np * h->ce_pitch;       // this slab's block of partials
      launch_ce_fwd(p, h->Hoc + (size_t)m0 * PH * esz, PH, h->Pw(h->off_Wo), P + h->off_Bo, h->labels_c + m0, Mc, V, H, dzT,
                    h->ce_pitch, h->pmax + po, h->psum + po, eps > 0.f ? h->psz + po : nullptr, h->zy + m0, st, lim);
      launch_ce_rows(h->pmax + po, h->psum + po, h->psz + po, h->zy + m0, nullptr, Mc, np, h->ce_pitch, eps, V, h->lse + m0,
                     h->nll + m0, st, lim);
      launch_ce_scale(p, dzT, h->ce_pitch, V, Mc, h->pmax + po, h->lse + m0, h->labels_c + m0, h->rowscale + m0, eps, dz, lddz,
                      h->dbo_parts + (size_t)n_dbo * V, st, lim);
      n_dbo += (Mc + 63) / 64;
      stream_after(h, sd, st);
      launch_gemm_nt(p, dz, lddz, h->WoT, h->ldWoT, Mc, H, V, h->dHoCE + (size_t)m0 * H, nullptr, H, nullptr, 0, st, h->gsplit,
                     h->gsplit_floats, lim, 1, 0, 1);                     // dH_o[slab] = dz W_o
      if (m0 + Mc >= Mt) {                                   // the last slab: dB_o and the loss, which nothing of the pass waits for
        launch_sum_parts(h->dbo_parts, n_dbo, (size_t)V, G + h->off_Bo, sd);
        launch_ce_loss(h->nll, Mt, h->loss, h->flags, h->h_loss, sd, RowLimit{h->ce_nvalid, 0});
      }
      // dW_o (+)= dz^T H_o[slab]; the first slab always holds a row, so W_o's gradient is always written
      launch_gemm_nt(p, dzT, h->ce_pitch, h->HocT + (size_t)m0 * esz, Mt, V, H, Mc, G + h->off_Wo, nullptr, H, nullptr, sl > 0,
                     sd, nullptr, 0, lim, 2, sd != st ? h->side_wgs_wo : 0, 1);
      if (sd != st) {
        done[sl] = h->ev[h->ev_next++ % h->ev.size()];
        (void)hipEventRecord(done[sl], sd);
      }
      m0 += Mc;
    }
  }

  phase_mark(h, "decoder backward loop");
  // ---- decoder loop backwards -----------------------------------------------------------------------
  const int kbd = step_kblocks(p, 2 * H, 4 * H, Bp, h->kb_bwd_dec);       // planes written by a decoder layer's backward GEMM
  const size_t pstr = (size_t)Bp * 2 * H;
  const Planes no_planes{nullptr, 0, 0, 0};
  if (loop && (h->bwd_fused & 1) && h->wc_whole_k) {
    sec.open(alone);
    enqueue_dec_loop_bwd(h, S, T);
    enqueue_dec_contexts_bwd(h, T);
    if (split) sec.close();
    h->n_loops++;
    h->ran_loops = LOOP_RAN_FWD | LOOP_RAN_BWD;
  } else if ((h->bwd_fused & 1) && Bp <= 128) {            // (measured at 128 sentences: 8.1 against 8.7 ms for the k-split form)
    // one launch per layer and step (dec_bwd_gemm): no pointwise launches, no planes
    for (int j = T - 1; j >= 0; --j) {
      char* dpre = h->dPre + j * BP * esz;
      const bool last = j == T - 1;
      char* dpreF = h->dPreF ? h->dPreF + j * BH * esz : nullptr;
      if (last)
        launch_tanh_bwd(p, h->dHoCE, h->ce_pos + (size_t)j * Bp, no_planes, h->HoBuf + (j + 1) * BP * esz, PH, dpre, PH, Bp, H,
                        drop_spec(h, DROP_SITE_HO, j), st, dpreF);
      int kbw = step_kblocks(p, 2 * H, H, Bp, h->kb_wc);
      if (proj && (h->att_proj & 1) && h->wc_whole_k) {
        dec_att_bwd_proj(h, j, S, last);
        for (int l = L - 1; l >= 0; --l) {
          const StepBwd gl = dec_bwd_gemm(h, l, j);
          launch_step_bwd_fused(p, gl, Bp, st);
        }
        continue;
      }
      if (h->wc_whole_k) {   // [dC_s ; dH_t] = dpre W_c with the whole (short) k range per workgroup: one plane
        StepBwd g{};
        g.dg = dpre; g.lddg = PH; g.K = H; g.Wt = h->WcT; g.ldw = H;
        g.part[0].kind = BWD_EPI_STORE; g.part[0].ncols = 2 * H; g.part[0].out = h->wcp; g.part[0].ldout = 2 * H;
        g.dg_fm = dpreF; g.Wt_fm = dpreF ? h->WcTF : nullptr; g.wt_tile0 = 0;
        launch_step_bwd_fused(p, g, Bp, st);
        kbw = 1;
      } else {   // the same as k blocks into planes
        StepGemm g{};
        g.a0 = dpre; g.lda0 = PH; g.K0 = H; g.w0_off = 0; g.K1 = 0;
        g.W = h->WcT; g.ldw = H; g.N = 2 * H; g.mode = 1; g.max_kb = h->kb_wc;
        g.out = h->wcp; g.ldout = 2 * H; g.plane_stride = pstr;
        g.W_fm = h->WcTF; g.a0_fm = dpreF;
        launch_step_gemm(p, g, Bp, st);
      }
      // attention backward; the gradient it sends to the top layer's output stays in registers and that
      // layer's cell backward runs in the same launch
      LstmBwdPoint top = dec_cell(h, L - 1, j);
      top.dhrec = Planes{h->dec[L - 1].bwdp, H, last ? 0 : 1, 0};
      launch_att_bwd(p, h->Kmat, H, Hs, ldHs, Planes{h->wcp, 2 * H, kbw, pstr}, h->dCs + j * BH, h->att_a + (size_t)j * Bp * S,
                     h->len_s, S, Bp, H, h->dots, h->att_ds + (size_t)j * Bp * S, h->dHt, st, &top);
      for (int l = L - 1; l >= 0; --l) {
        const StepBwd g = dec_bwd_gemm(h, l, j);
        launch_step_bwd_fused(p, g, Bp, st);
      }
    }
    for (int l = 0; l < L; ++l)
      launch_planes_add(h->dec[l].dh, h->dec[l].dh, Planes{h->dec[l].bwdp, H, 1, 0}, 0, Bp, H, st);
  } else {
  for (int j = T - 1; j >= 0; --j) {
    char* dpre = h->dPre + j * BP * esz;
    const bool last = j == T - 1;
    // dH_o = cross-entropy part + what step j+1's bottom layer sent back through the input feed
    char* dpreF = h->dPreF ? h->dPreF + j * BH * esz : nullptr;
    launch_tanh_bwd(p, h->dHoCE, h->ce_pos + (size_t)j * Bp, Planes{h->dec[0].bwdp, 2 * H, last ? 0 : kbd, pstr}, h->HoBuf + (j + 1) * BP * esz,
                    PH, dpre, PH, Bp, H, drop_spec(h, DROP_SITE_HO, j), st, dpreF);
    const int kbw = step_kblocks(p, 2 * H, H, Bp, h->kb_wc);
    {   // [dC_s ; dH_t] = dpre W_c, as planes
      StepGemm g{};
      g.a0 = dpre; g.lda0 = PH; g.K0 = H; g.w0_off = 0; g.K1 = 0;
      g.W = h->WcT; g.ldw = H; g.N = 2 * H; g.mode = 1; g.max_kb = h->kb_wc;
      g.out = h->wcp; g.ldout = 2 * H; g.plane_stride = pstr;
      g.W_fm = h->WcTF; g.a0_fm = dpreF;
      launch_step_gemm(p, g, Bp, st);
    }
    launch_att_bwd(p, h->Kmat, H, Hs, ldHs, Planes{h->wcp, 2 * H, kbw, pstr}, h->dCs + j * BH, h->att_a + (size_t)j * Bp * S,
                   h->len_s, S, Bp, H, h->dots, h->att_ds + (size_t)j * Bp * S, h->dHt, st);
    for (int l = L - 1; l >= 0; --l) {
      LD& e = h->dec[l];
      LstmBwdPoint q;
      if (l == L - 1) q.dy = Planes{h->dHt, H, 1, 0};
      else { q.dy = Planes{h->dec[l + 1].bwdp, 2 * H, kbd, pstr}; q.drop_dy = drop_spec(h, DROP_SITE_DEC + l, j); }
      q.dy_col = 0;                                                   // dx of the layer above, columns [0, H)
      q.dhrec = Planes{e.bwdp, 2 * H, last ? 0 : kbd, pstr}; q.dhrec_col = H;
      q.dh = e.dh; q.dc = e.dc;
      q.gsave = e.Gs + (size_t)j * Bp * 4 * H;
      q.cprev = e.Cst + j * BH; q.cnext = e.Cst + (j + 1) * BH;
      q.mask = h->mask_t + (size_t)j * Bp;
      q.dg = e.dG + (size_t)j * Bp * e.pg * esz; q.lddg = e.pg;
      if (e.fmb) q.dg_fm = e.dGF + (size_t)j * Bp * 4 * H * esz;
      launch_lstm_bwd_point(p, q, Bp, H, st);
      StepGemm g{};                                  // [dx ; dh_prev] = dgates [W_x ; W_h] (bottom layer: [feed ; h])
      g.a0 = q.dg; g.lda0 = e.pg; g.K0 = 4 * H; g.w0_off = 0; g.K1 = 0;
      g.W = e.Wt + (size_t)(l == 0 ? E : 0) * 4 * H * esz; g.ldw = 4 * H;
      if (e.fmb) { g.W_fm = e.WtF; g.w_tile0 = (l == 0 ? E : 0) / 16; g.a0_fm = q.dg_fm; }
      g.N = 2 * H; g.mode = 1; g.max_kb = h->kb_bwd_dec;
      g.out = e.bwdp; g.ldout = 2 * H; g.plane_stride = pstr;
      launch_step_gemm(p, g, Bp, st);
    }
  }
  // gradient of the decoder's initial state: pass-through part + the last GEMM's recurrent part
  for (int l = 0; l < L; ++l)
    launch_planes_add(h->dec[l].dh, h->dec[l].dh, Planes{h->dec[l].bwdp, 2 * H, kbd, pstr}, H, Bp, H, st);
  }

  phase_mark(h, "deferred attention gradients");
  // ---- second stream: everything that only needed the decoder's dgates and dpre -----------------------
  stream_after(h, sd, st);
  h->dw_tr.push_back({h->dPre, PH, h->dPreT, Mt, Mt, H});
  // encoder layer outputs, transposed: layer 0 -> Y0T (ld Ms); layer l >= 1 -> HstT + Bp (ld (S+1)Bp)
  auto encYT = [&](int l, int* ld) -> const char* {
    if (l == 0) { *ld = Ms; return h->Y0T; }
    if (drop && l + 1 < L) { *ld = Ms; return h->enc[l + 1].YdT; }
    *ld = (S + 1) * Bp; return h->enc[l + 1].HstT + (size_t)Bp * esz;
  };
  // dW_c = dpre^T [C_s ; H_t]
  h->dw_group.push_back(GemmProb{h->dPreT, h->CsT, G + h->off_Wc, Mt, Mt, 2 * H, H, H, Mt, 0});
  h->dw_group.push_back(GemmProb{h->dPreT, h->dec[L - 1].HstT + (size_t)Bp * esz, G + h->off_Wc + H, Mt, (T + 1) * Bp, 2 * H, H, H, Mt, 0});
  for (int l = 0; l < L; ++l) {
    LD& e = h->dec[l];
    if (l == 0)
      weight_grads(h, e, T, {{h->XtT, Mt}, {h->HoBufT, ldHoT}, {e.HstT, (T + 1) * Bp}}, {E, H, H}, sd);
    else
      weight_grads(h, e, T, {drop ? std::pair<const char*, int>{h->dec[l - 1].YdT, Mt}
                                  : std::pair<const char*, int>{h->dec[l - 1].HstT + (size_t)Bp * esz, (T + 1) * Bp},
                             {e.HstT, (T + 1) * Bp}}, {H, H}, sd);
  }
  // W_c and every decoder layer's weight gradient: one launch.  The top encoder layers' recurrences come beside it, one workgroup to
  // a CU; where they take half of the chip at most, the 256 x 256 tiles, which hold a CU for long, are left the rest: 64 sentences, width 1024,
  // first recurrence 267 -> 218 us, the product before it 156 -> 74, this launch 312 -> 506, the step 5.74 -> 5.61 ms.  (128 sentences take
  // every CU: a cap of 128 19.1 -> 19.4; groups of smaller tiles: width 512 2.564 -> 2.574.)  14 steps of widths 512 - 1024, 2 to 4 layers, 16 to
  // 100 sentences of 5 to 110 tokens: 0 - 2.7 % faster with the cap but for one, width 896, 40 sentences, 0.4 % slower.
  const SeqPlan top = seq_bwd_plan(p, 1, Bp, H);
  const int beside = top.groups * top.group;
  flush_dw_group(h, sd, L > 1 && 2 * beside <= h->seq.cus ? h->seq.cus - beside : 0);
  launch_gemm_nt(p, h->dec[0].dG, h->dec[0].pg, h->dec[0].Wt, 4 * H, Mt, E, 4 * H, h->dXt, nullptr, E, nullptr, 0, sd);
  launch_embed_scatter(h->dXt, h->tok_t, Mt, c.tgt_vocab, E, G + h->off_Etgt, sd, false);

  // ---- attention gradients that do not feed the decoder recurrence, batched over all steps ---------
  const char* HtAll = h->dec[L - 1].Hst + BP * esz;      // H_t^{<0..T-1>}
  launch_att_deferred(p, h->att_a, h->att_ds, h->dCs, H, HtAll, PH, S, T, Bp, H, h->dHs, h->dK, st);
  launch_gemm_nt(p, h->dK, H, h->Pw(h->off_Wa), H, Ms, H, H, h->dHs, nullptr, H, nullptr, 1, st);   // dHs += dK W_a^T
  stream_after(h, sd, st);
  h->dw_tr.push_back({h->dK, H, h->dKT, Ms, Ms, H});
  {   // dW_a[r,c] = sum_i H_s[i,r] dK[i,c]
    int ld; const char* HsT = encYT(L - 1, &ld);
    h->dw_group.push_back(GemmProb{HsT, h->dKT, G + h->off_Wa, ld, Ms, H, H, H, Ms, 0});
    flush_dw_group(h, sd);
  }

  phase_mark(h, "encoder upper layers backward");
  // ---- encoder backwards ------------------------------------------------------------------------------
  // Per layer, top first, one launch for the whole recurrence and one GEMM for the gradient it sends to the layer below.
  {   // the exchange slots (the tickets of the forward pass are used up: cleared as well)
    std::vector<FillJob> z;
    for (int l = 0; l <= L; ++l) add_empty(z, h->enc[l].XG, (size_t)Ms * 4 * h->enc[l].Hh, esz);
    add_fill(z, h->tickets, SEQ_TICKETS, 4);
    launch_fill_multi(z.data(), (int)z.size(), st);
  }
  const unsigned long long drop_step = (unsigned long long)h->B * H;
  auto seq_bwd_dir = [&](LD& e, const float* dY) {
    SeqBwdDir d{};
    d.Wt = e.Wt + (size_t)e.Kin * 4 * e.Hh * esz; d.ldw = 4 * e.Hh;
    d.dY = dY; d.lddy = H; d.mask = h->mask_s; d.G = e.Gs; d.C = e.Cst;
    d.X = e.XG; d.dG = e.dG; d.lddg = e.pg; d.ldd0 = H;
    return d;
  };
  SeqBwdArgs sb{};
  sb.again = h->again;
  sec.open(false);
  for (int l = L - 1; l >= 1; --l) {
    LD& e = h->enc[l + 1];
    SeqBwdDir& d = sb.d[0];
    d = seq_bwd_dir(e, l == L - 1 ? h->dHs : h->dYa);
    if (l < L - 1) { d.drop = drop_spec(h, DROP_SITE_ENC + l, 0); d.drop_step = drop_step; }
    d.dh0 = h->dec[l].dh; d.dc0 = h->dec[l].dc;    // gradient of the final state = that of the decoder's initial state
    sb.ticket = h->tickets + 2 * l;
    launch_lstm_seq_bwd(p, sb, 1, S, Bp, H, h->seq, st);
    launch_gemm_nt(p, e.dG, e.pg, e.Wt, 4 * H, Ms, H, 4 * H, h->dYa, nullptr, H, nullptr, 0, st);   // the layer below's dY = dG W_x
  }
  if (L > 1) {
    stream_after(h, sd, st);
    for (int l = L - 1; l >= 1; --l) {
      LD& e = h->enc[l + 1];
      int ld; const char* XT = encYT(l - 1, &ld);
      weight_grads(h, e, S, {{XT, ld}, {e.HstT, (S + 1) * Bp}}, {H, H}, sd);
    }
    flush_dw_group(h, sd);
  }
  phase_mark(h, "encoder bottom layer backward");
  {   // bottom layer: both directions in one launch
    LD& d0 = h->dec[0];
    for (int i = 0; i < 2; ++i) {
      SeqBwdDir& d = sb.d[i];
      d = seq_bwd_dir(i ? eb : ef, L > 1 ? h->dYa : h->dHs);
      d.dy_col = i ? Hd : 0; d.reverse = i;
      if (L > 1) { d.drop = drop_spec(h, DROP_SITE_ENC + 0, 0); d.drop_step = drop_step; }
      d.dh0 = d0.dh + (i ? Hd : 0); d.dc0 = d0.dc + (i ? Hd : 0);
    }
    sb.ticket = h->tickets;
    launch_lstm_seq_bwd(p, sb, 2, S, Bp, Hd, h->seq, st);
    sec.close();
    // What is left after the last recurrent kernel is shared between the two streams: the weight gradients of
    // both directions on the second one, the source-embedding gradient (dX_s, then the scatter) on the caller's.
    stream_after(h, sd, st);
    weight_grads(h, ef, S, {{h->XsT, Ms}, {ef.HstT, (S + 1) * Bp}}, {E, Hd}, sd);
    weight_grads(h, eb, S, {{h->XsT, Ms}, {eb.HstT + (size_t)Bp * esz, (S + 1) * Bp}}, {E, Hd}, sd);
    flush_dw_group(h, sd);
    const GemmProb dx{ef.dG, ef.Wt, h->dXs, ef.pg, 4 * Hd, E, Ms, E, 4 * Hd, 0, nullptr, eb.dG, eb.Wt, eb.pg, 4 * Hd, 4 * Hd};
    launch_gemm_nt_group(p, &dx, 1, st, nullptr, 0);
    if (esrc_cleared) (void)hipStreamWaitEvent(st, esrc_cleared, 0);
    launch_embed_scatter(h->dXs, h->tok_s, Ms, c.src_vocab, E, G + h->off_Esrc, st, false);
  }
  phase_mark(h, "wait for the second stream");
  stream_after(h, st, sd);                         // join: the step is complete on the caller's stream
  phase_mark(h, "end");
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "enqueue");
  h->have_step = true;
  return CMT_OK;
}

}  // namespace

// ================================================================================================
extern "C" {

int cmt_query_sizes(const cmt_config* cfg, size_t* param_bytes, size_t* grad_bytes, size_t* workspace_bytes) {
  if (!config_ok(cfg, nullptr)) return CMT_EINVAL;
  cmt_handle tmp;
  tmp.cfg = *cfg; tmp.prec = cfg->precision; tmp.esz = cfg->precision ? 2 : 4;
  tmp.Bpm = round_up(cfg->max_batch, 16);
  build_table(tmp.cfg, tmp.table, tmp.nparams);
  const size_t ws = layout(&tmp, nullptr);
  if (param_bytes) *param_bytes = tmp.nparams * 4;
  if (grad_bytes) *grad_bytes = tmp.nparams * 4;
  if (workspace_bytes) *workspace_bytes = ws;
  return CMT_OK;
}

int cmt_create(const cmt_config* cfg, void* params_dev, void* grads_dev, void* workspace_dev, void* hip_stream,
               cmt_handle** out) {
  if (!out) return CMT_EINVAL;
  *out = nullptr;
  std::string why;
  if (!config_ok(cfg, &why)) return CMT_EINVAL;
  if (!params_dev || !grads_dev || !workspace_dev) return CMT_EINVAL;
  if (((uintptr_t)params_dev | (uintptr_t)grads_dev | (uintptr_t)workspace_dev) & 255) return CMT_EINVAL;
  cmt_handle* h = new cmt_handle();
  h->cfg = *cfg; h->prec = cfg->precision; h->esz = cfg->precision ? 2 : 4;
  h->st = (hipStream_t)hip_stream;
  h->params = (float*)params_dev; h->grads = (float*)grads_dev; h->ws = (char*)workspace_dev;
  h->Bpm = round_up(cfg->max_batch, 16);
  {
    const char* k1d = getenv("CMT_KB_BWD_DEC"); h->kb_bwd_dec = k1d ? atoi(k1d) : 0;
    const char* k2 = getenv("CMT_KB_WC"); h->kb_wc = k2 ? atoi(k2) : 2;
    const char* ks1 = getenv("CMT_SIDE_WGS"); h->side_wgs = ks1 ? atoi(ks1) : 0;
    const char* ks2 = getenv("CMT_SIDE_WGS_WO"); h->side_wgs_wo = ks2 ? atoi(ks2) : 0;
    const char* kw = getenv("CMT_WC_WHOLE_K"); h->wc_whole_k = kw ? atoi(kw) : 1;
    const char* k3 = getenv("CMT_SIDE_STREAM"); h->use_side = k3 ? atoi(k3) : 1;
    const char* k3p = getenv("CMT_ATT_PROJ"); h->att_proj = k3p ? atoi(k3p) : 1;
    const char* k4 = getenv("CMT_PHASE_TIMING"); h->phase_timing = k4 ? atoi(k4) : 0;
    const char* k5 = getenv("CMT_BWD_FUSED"); h->bwd_fused = k5 ? atoi(k5) : 1;
    const char* k7 = getenv("CMT_DEC_LOOP"); h->loop = k7 ? atoi(k7) : 1;
    const char* k6 = getenv("CMT_RECUR"); h->seq.mode = k6 ? atoi(k6) : SEQ_RUN_TOGETHER;
  }
  build_table(h->cfg, h->table, h->nparams);
  h->ws_bytes = layout(h, h->ws);
  bind_params(h);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&h->seq.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    cmt_destroy(h);
    return CMT_EHIP;
  }
  hipError_t e = hipHostMalloc((void**)&h->h_loss, 256, hipHostMallocDefault);
  if (e != hipSuccess) { cmt_destroy(h); return CMT_EHIP; }
  h->gate = &g_gates[dev % GATES];
  h->section = new Gate::Client();
  h->gate->add(*h->section, h->st);
  for (hipEvent_t* ev : {&h->section->shared, &h->section->alone})
    if (hipEventCreateWithFlags(ev, hipEventDisableTiming) != hipSuccess) { cmt_destroy(h); return CMT_EHIP; }
  // second stream at the default priority, and a pool of events for the hand-offs between the two
  if (hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking) != hipSuccess) { cmt_destroy(h); return CMT_EHIP; }
  h->ev.assign(512, nullptr);
  for (auto& ev : h->ev)
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) { cmt_destroy(h); return CMT_EHIP; }
  h->h_flags = (int*)(h->h_loss + 8);
  h->h_loss[0] = 0.f; h->h_loss[1] = 0.f; *h->h_flags = 0;
  h->again = h->flags + 1;
  launch_fill_f32((float*)h->flags, 2, 0.f, h->st);  // the workspace may hold anything
  *out = h;
  return CMT_OK;
}

void cmt_destroy(cmt_handle* h) {
  if (!h) return;
  if (h->h_loss) (void)hipHostFree(h->h_loss);
  if (h->side) (void)hipStreamSynchronize(h->side);
  if (h->section) {
    h->gate->remove(*h->section);
    for (hipEvent_t ev : {h->section->shared, h->section->alone}) if (ev) (void)hipEventDestroy(ev);
    delete h->section;
  }
  for (auto ev : h->ev) if (ev) (void)hipEventDestroy(ev);
  for (auto ev : h->phase_ev) if (ev) (void)hipEventDestroy(ev);
  if (h->side) (void)hipStreamDestroy(h->side);
  delete h;
}

int cmt_param_count(const cmt_handle* h) { return h ? (int)h->table.size() : CMT_EINVAL; }

int cmt_param_info(const cmt_handle* h, int idx, const char** name, int64_t* rows, int64_t* cols, size_t* offset_elems) {
  if (!h || idx < 0 || idx >= (int)h->table.size()) return CMT_EINVAL;
  const ParamInfo& p = h->table[idx];
  if (name) *name = p.name.c_str();
  if (rows) *rows = p.rows;
  if (cols) *cols = p.cols;
  if (offset_elems) *offset_elems = p.off;
  return CMT_OK;
}

int cmt_init_params(cmt_handle* h, uint64_t seed, float scale) {
  if (!h) return CMT_EINVAL;
  launch_init_uniform(h->params, h->nparams, seed, scale, h->st);
  refresh_params(h);
  hipError_t e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_init_params");
  return CMT_OK;
}

int cmt_set_params(cmt_handle* h, const float* host_src) {
  if (!h || !host_src) return fail(h, CMT_EINVAL, "null pointer");
  hipError_t e = hipMemcpyAsync(h->params, host_src, h->nparams * 4, hipMemcpyHostToDevice, h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_set_params copy");
  refresh_params(h);
  e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_set_params");
  return CMT_OK;
}

int cmt_get_params(cmt_handle* h, float* host_dst) {
  if (!h || !host_dst) return fail(h, CMT_EINVAL, "null pointer");
  hipError_t e = hipMemcpyAsync(host_dst, h->params, h->nparams * 4, hipMemcpyDeviceToHost, h->st);
  if (e == hipSuccess) e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_get_params");
  return CMT_OK;
}

int cmt_get_grads(cmt_handle* h, float* host_dst) {
  if (!h || !host_dst) return fail(h, CMT_EINVAL, "null pointer");
  hipError_t e = hipMemcpyAsync(host_dst, h->grads, h->nparams * 4, hipMemcpyDeviceToHost, h->st);
  if (e == hipSuccess) e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_get_grads");
  return CMT_OK;
}

int cmt_train_step_async(cmt_handle* h, const int32_t* src_ids_dev, const int32_t* src_len_dev,
                         const int32_t* tgt_ids_dev, const int32_t* tgt_len_dev, int32_t B, int32_t S, int32_t T) {
  if (!h) return CMT_EINVAL;
  return enqueue_step(h, src_ids_dev, src_len_dev, tgt_ids_dev, tgt_len_dev, B, S, T, false);
}

int cmt_eval_loss(cmt_handle* h, const int32_t* src_ids_dev, const int32_t* src_len_dev, const int32_t* tgt_ids_dev,
                  const int32_t* tgt_len_dev, int32_t B, int32_t S, int32_t T, float* loss_host, float* n_tok_host) {
  if (!h) return CMT_EINVAL;
  const float keep_p = h->drop_p, keep_eps = h->ls_eps;
  h->drop_p = 0.f; h->ls_eps = 0.f;                 // evaluation: no masks, plain cross-entropy
  int rc = enqueue_step(h, src_ids_dev, src_len_dev, tgt_ids_dev, tgt_len_dev, B, S, T, true);
  h->drop_p = keep_p; h->ls_eps = keep_eps;
  if (rc != CMT_OK) return rc;
  rc = cmt_fetch_loss(h, loss_host);
  if (n_tok_host) *n_tok_host = h->h_loss[1];
  return rc;
}

// ---- evaluation without a caller-provided workspace -------------------------------------------------
// All intermediates of cmt_eval_loss_static live in this array instead of the handle's workspace.  In
// host code the array's name is only a stand-in: the device address comes from hipGetSymbolAddress,
// once per device (every GPU holds its own copy), and only that pointer is handed to kernels.
static __device__ __align__(256) unsigned char scratch[CMT_STATIC_SCRATCH_BYTES];
namespace {
constexpr int STATIC_MAX_DEVICES = 64;
void* g_static_scratch[STATIC_MAX_DEVICES] = {};
// device address of `scratch` on the current device (looked up at the first call on that device)
int static_scratch_ptr(cmt_handle* h, char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(h, e, "hipGetDevice");
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return fail(h, CMT_EINVAL, "device ordinal beyond the static scratch table");
  if (!g_static_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_fail(h, e, "hipGetSymbolAddress(scratch)");
    g_static_scratch[dev] = p;
  }
  *out = (char*)g_static_scratch[dev];
  return CMT_OK;
}
}  // namespace

int cmt_eval_loss_static(cmt_handle* h, const int32_t* src_ids_dev, const int32_t* src_len_dev, const int32_t* tgt_ids_dev,
                         const int32_t* tgt_len_dev, int32_t B, int32_t S, int32_t T, float* loss_host, float* n_tok_host) {
  if (!h) return CMT_EINVAL;
  const cmt_config& c = h->cfg;
  if (B < 1 || B > c.max_batch || S < 1 || S > c.max_src_len || T < 1 || T > c.max_tgt_len)
    return fail(h, CMT_EINVAL, "B, S or T outside [1, configured maximum]");
  // a view of the handle whose workspace is the static array, laid out for exactly this call's shape
  cmt_handle v = *h;
  v.cfg.max_batch = B; v.cfg.max_src_len = S; v.cfg.max_tgt_len = T;
  v.Bpm = round_up(B, 16);
  v.phase_timing = 0; v.phase_ev.clear(); v.phase_name.clear();
  // The kernels of cmt_eval_loss in their order, so that the losses are equal bit by bit.  (The decoder's loop has its slots in
  // buffers that are there already; for one position, or 16 units, one of them is a few KB larger, and a shape that just fits
  // without those gets the launches per position.)
  v.loop_slots = LOOP_SLOTS_EVAL;
  v.pad_lines = false;
  size_t need = layout(&v, nullptr);
  if (need > (size_t)CMT_STATIC_SCRATCH_BYTES) {
    v.loop_slots = LOOP_SLOTS_NONE;
    need = layout(&v, nullptr);
  }
  if (need > (size_t)CMT_STATIC_SCRATCH_BYTES) {
    char msg[160];
    snprintf(msg, sizeof msg, "this shape needs %zu bytes of scratch, the static buffer holds %zu", need,
             (size_t)CMT_STATIC_SCRATCH_BYTES);
    return fail(h, CMT_EINVAL, msg);
  }
  char* base = nullptr;
  int rc = static_scratch_ptr(h, &base);
  if (rc != CMT_OK) return rc;
  v.ws = base;
  v.ws_bytes = layout(&v, base);
  bind_params(&v);
  // the array keeps the last call's contents (perhaps of another shape): start from zeros
  launch_fill_f32((float*)base, (need + 3) / 4, 0.f, v.st);
  refresh_params(&v);                                // working copies of the parameters (casts, transposes) in the array
  v.drop_p = 0.f; v.ls_eps = 0.f;                    // evaluation: no masks, plain cross-entropy
  rc = enqueue_step(&v, src_ids_dev, src_len_dev, tgt_ids_dev, tgt_len_dev, B, S, T, true);
  if (rc == CMT_OK) rc = cmt_fetch_loss(&v, loss_host);
  if (rc != CMT_OK) { h->err = v.err; return rc; }
  if (n_tok_host) *n_tok_host = v.h_loss[1];
  h->ev_next = v.ev_next;
  h->n_loops = v.n_loops;
  return CMT_OK;
}

int cmt_fetch_loss(cmt_handle* h, float* loss_host) {
  if (!h) return CMT_EINVAL;
  if (!h->have_step) return fail(h, CMT_EINVAL, "no step has been run");
  hipError_t e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_fetch_loss");
  if (h->phase_timing && h->phase_n > 1) {          // phases of the last step, as the caller's stream saw them
    float total = 0.f;
    for (size_t i = 0; i + 1 < h->phase_n; ++i) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, h->phase_ev[i], h->phase_ev[i + 1]) != hipSuccess) break;
      fprintf(stderr, "[cytonmt_hip] %-40s %8.3f ms   (enqueued in %6.3f ms)\n", h->phase_name[i], ms,
              h->phase_host[i + 1] - h->phase_host[i]);
      total += ms;
    }
    fprintf(stderr, "[cytonmt_hip] %-40s %8.3f ms\n", "step", total);
  }
  const int flags = *h->h_flags;
  if (loss_host) *loss_host = h->h_loss[0];
  if (flags) {                                       // reported once: clear the device word for the steps to come
    *h->h_flags = 0;
    launch_fill_f32((float*)h->flags, 1, 0.f, h->st);
  }
  if (flags & 3) return fail(h, CMT_ERANGE, (flags & 1) ? "a token id is outside its vocabulary" : "a length is outside [1, padded length]");
  if (flags & 4) return fail(h, CMT_ENONFINITE, "the loss is not finite");
  return CMT_OK;
}

int cmt_wait_counts(cmt_handle* h, int64_t* loops, int64_t* again) {
  if (!h) return CMT_EINVAL;
  int n = 0;
  hipError_t e = hipMemcpyAsync(&n, h->again, sizeof n, hipMemcpyDeviceToHost, h->st);
  if (e == hipSuccess) e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_wait_counts");
  if (loops) *loops = h->n_loops;
  if (again) *again = n;
  return CMT_OK;
}

int cmt_train_step(cmt_handle* h, const int32_t* src_ids_dev, const int32_t* src_len_dev, const int32_t* tgt_ids_dev,
                   const int32_t* tgt_len_dev, int32_t B, int32_t S, int32_t T, float* loss_host) {
  const int rc = cmt_train_step_async(h, src_ids_dev, src_len_dev, tgt_ids_dev, tgt_len_dev, B, S, T);
  if (rc != CMT_OK) return rc;
  return cmt_fetch_loss(h, loss_host);
}

int cmt_greedy_decode(cmt_handle* h, const int32_t* src_ids_dev, const int32_t* src_len_dev, int32_t B, int32_t S,
                      int32_t max_len, int32_t eos_id, int32_t* out_ids_dev, int32_t* out_len_dev) {
  if (!h) return CMT_EINVAL;
  const cmt_config& c = h->cfg;
  if (!src_ids_dev || !src_len_dev || !out_ids_dev || !out_len_dev) return fail(h, CMT_EINVAL, "null pointer");
  if (B < 1 || B > c.max_batch || S < 1 || S > c.max_src_len || max_len < 1 || max_len > c.max_tgt_len)
    return fail(h, CMT_EINVAL, "B, S or max_len outside [1, configured maximum]");
  if (eos_id < 0 || eos_id >= c.tgt_vocab) return fail(h, CMT_EINVAL, "eos_id outside the target vocabulary");
  const int p = h->prec, E = c.emb_dim, H = c.hidden, L = c.layers, V = c.tgt_vocab;
  const int Bp = round_up(B, 16);
  const size_t esz = h->esz;
  hipStream_t st = h->st;
  h->B = B; h->Bp = Bp; h->S = S; h->T = max_len;
  h->have_step = false;                              // the training step's intermediates are overwritten
  h->phase_n = 0;
  const int PH = h->PH;
  const size_t BP = (size_t)Bp * PH, BH = (size_t)Bp * H;
  const float keep_p = h->drop_p;
  h->drop_p = 0.f;                                   // inference: no dropout
  launch_fill_f32((float*)h->flags, 1, 0.f, st);
  const GatherSide side{h->Pw(h->off_Esrc), c.src_vocab, src_ids_dev, src_len_dev, S, 0, 0, h->Xs, h->mask_s, h->tok_s, nullptr, h->len_s};
  launch_gather(p, &side, 1, E, B, Bp, h->flags, st);
  const char* Hs; int ldHs;
  note_capture(h);
  const bool proj = h->att_proj && Bp < 256;
  const LoopFit fit = loop_decode_fits(p, L, Bp, H, S, V, h->seq);
  const bool loop = proj && dec_loop(h, fit), alone = loop && fit.alone;
  const bool split = alone && h->gate->crowded(*h->section);
  Section sec(h);
  sec.open(alone && !split);
  enqueue_encoder(h, S, &Hs, &ldHs, !loop, proj, nullptr);
  if (!loop || split) sec.close();
  launch_dec_init(B, Bp, max_len, c.bos_id, c.pad_id, h->dec_tok, h->dec_done, out_ids_dev, out_len_dev, h->dec_mask, st);
  if (loop) {
    sec.open(alone);
    enqueue_greedy_loop(h, B, S, max_len, eos_id, out_ids_dev, out_len_dev);
    sec.close();
  }
  const bool fm0 = h->xcatF && h->dec[0].fm;                          // bottom layer on fragment-major operands
  if (!loop) {
    launch_fill_T(p, h->xcat, (size_t)Bp * h->ldxcat, st);            // H_o^{<-1>} = 0
    if (fm0) launch_fill_T(p, h->xcatF, (size_t)Bp * (E + H), st);
    // the first step's input embedding; every later one is written by the arg-max kernel of the step before
    launch_dec_embed(p, h->Pw(h->off_Etgt), E, h->dec_tok, B, Bp, h->xcat, h->ldxcat, st, fm0 ? h->xcatF : nullptr, (E + H) >> 5);
  }
  for (int j = loop ? max_len : 0; j < max_len; ++j) {
    for (int l = 0; l < L; ++l) {
      LD& e = h->dec[l];
      LstmFwdDir d;
      if (l == 0) { d.x = h->xcat; d.ldx = h->ldxcat; d.Kx = E + H; d.wx_off = 0; d.wh_off = E + H; d.ldw = E + 2 * H; }
      else { d.x = h->dec[l - 1].Hst + (j + 1) * BP * esz; d.ldx = e.ph; d.Kx = H; d.wx_off = 0; d.wh_off = H; d.ldw = 2 * H; }
      d.gx = nullptr; d.ldgx = 0; d.bias = h->params + e.b_off;
      d.hprev = e.Hst + j * BP * esz; d.ldh = e.ph; d.W = e.W;
      d.cprev = e.Cst + j * BH; d.mask = h->dec_mask;
      d.hnext = e.Hst + (j + 1) * BP * esz; d.ldhn = e.ph; d.cnext = e.Cst + (j + 1) * BH;
      d.gsave = nullptr; d.ycat = nullptr; d.ldy = 0;
      if (e.fm) {
        d.hnext_fm = e.HstF + (j + 1) * BH * esz;
        if (l > 0 && h->dec[l - 1].fm) {
          d.W_fm = e.Wfm; d.x_fm = h->dec[l - 1].HstF + (j + 1) * BH * esz; d.hprev_fm = e.HstF + j * BH * esz;
        } else if (l == 0 && fm0) {
          d.W_fm = h->Wdec0F; d.x_fm = h->xcatF; d.hprev_fm = e.HstF + j * BH * esz;
        }
      }
      launch_lstm_fwd(p, d, Bp, H, st);
    }
    const char* Ht = h->dec[L - 1].Hst + (j + 1) * BP * esz;
    StepGemm g{};                                   // H_o = tanh(W_c [C_s; H_t]) straight into the next step's input
    g.a0 = h->Cs + j * BP * esz; g.lda0 = PH; g.K0 = H; g.w0_off = 0;
    g.a1 = Ht; g.lda1 = PH; g.K1 = H; g.w1_off = H;
    g.W = h->Pw(h->off_Wc); g.ldw = 2 * H; g.N = H; g.mode = 0;
    g.outT = h->xcat + (size_t)E * esz; g.ldo = h->ldxcat;
    g.out = h->wcp; g.ldout = H; g.plane_stride = BH;
    if (h->HoFeedF && h->dec[L - 1].fm) {
      g.W_fm = h->WcF; g.a0_fm = h->CsF + j * BH * esz; g.a1_fm = h->dec[L - 1].HstF + (j + 1) * BH * esz;
      g.outF = h->HoFeedF;                          // H_o of this step, for the logits
      if (fm0) { g.outF2 = h->xcatF; g.outF2_nsteps = (E + H) >> 5; g.outF2_k0 = E; }   // and for the next step's bottom layer
    }
    if (proj) {                                     // on the projected source rows, as in the training step
      AttOut o{};
      o.outT = g.outT; o.ldo = g.ldo; o.outF = g.outF; o.outF2 = g.outF2; o.outF2_nsteps = g.outF2_nsteps; o.outF2_k0 = g.outF2_k0;
      g.mode = 3; g.skip0 = 1; g.a0_fm = g.a1_fm;
      launch_att_fwd_proj(p, h->Kmat, H, h->PmatT, H, Ht, PH, g, o, h->len_s, S, Bp, H, h->dots, h->att_a + (size_t)j * Bp * S, st);
    } else {
      launch_att_fwd(p, h->Kmat, H, Hs, ldHs, Ht, PH, h->len_s, S, Bp, H, h->dots, h->att_a + (size_t)j * Bp * S,
                     h->Cs + j * BP * esz, PH, st, h->CsF ? h->CsF + j * BH * esz : nullptr);
      launch_step_gemm(p, g, Bp, st);
    }
    StepGemm z{};                                   // logits (without the bias) = H_o W_o^T
    z.a0 = h->xcat + (size_t)E * esz; z.lda0 = h->ldxcat; z.K0 = H; z.w0_off = 0; z.K1 = 0;
    // ... of which only the largest per sentence is wanted: every workgroup of the product keeps the best of its 64
    // vocabulary entries (bias included), and the arg-max kernel picks among those
    const int nblk = (V + 63) / 64;
    float* part_v = h->logits; int32_t* part_i = (int32_t*)(h->logits + (size_t)nblk * Bp);
    z.W = h->Pw(h->off_Wo); z.ldw = H; z.N = V; z.mode = 2; z.max_kb = 1;
    if (g.outF && h->WoF) { z.W_fm = h->WoF; z.a0_fm = h->HoFeedF; }
    z.out = part_v; z.best_idx = part_i; z.bias = h->params + h->off_Bo; z.ldout = V; z.plane_stride = (size_t)Bp * V;
    launch_step_gemm(p, z, Bp, st);
    launch_dec_argmax(part_v, Bp, nullptr, nblk, B, j, max_len, eos_id, h->dec_tok, h->dec_done, out_ids_dev,
                      out_len_dev, st, p, h->Pw(h->off_Etgt), E, h->xcat, h->ldxcat, fm0 ? h->xcatF : nullptr, (E + H) >> 5, part_i);
  }
  h->drop_p = keep_p;
  (void)hipMemcpyAsync(h->h_flags, h->flags, sizeof(int), hipMemcpyDeviceToHost, st);
  hipError_t e = hipStreamSynchronize(st);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "cmt_greedy_decode");
  const int flags = *h->h_flags;
  if (flags & 3) return fail(h, CMT_ERANGE, (flags & 1) ? "a token id is outside its vocabulary" : "a length is outside [1, padded length]");
  return CMT_OK;
}

int cmt_beam_decode(cmt_handle* h, const int32_t* src_ids_dev, const int32_t* src_len_dev, int32_t B, int32_t S,
                    int32_t max_len, int32_t beam, float length_penalty, int32_t eos_id, int32_t* out_ids_dev,
                    int32_t* out_len_dev, float* out_score_dev) {
  if (!h) return CMT_EINVAL;
  const cmt_config& c = h->cfg;
  if (!src_ids_dev || !src_len_dev || !out_ids_dev || !out_len_dev || !out_score_dev) return fail(h, CMT_EINVAL, "null pointer");
  if (B < 1 || S < 1 || S > c.max_src_len || max_len < 1 || max_len > c.max_tgt_len)
    return fail(h, CMT_EINVAL, "B, S or max_len outside [1, configured maximum]");
  if (beam < 1 || beam > 16) return fail(h, CMT_EINVAL, "beam must be in [1, 16]");
  if ((long long)B * beam > c.max_batch) return fail(h, CMT_EINVAL, "B * beam exceeds max_batch (one decoder row per hypothesis)");
  if (c.max_tgt_len < 2) return fail(h, CMT_EINVAL, "beam search needs max_tgt_len >= 2 (state double buffer)");
  if (!(length_penalty >= 0.f) || !isfinite(length_penalty)) return fail(h, CMT_EINVAL, "length_penalty must be finite and >= 0");
  if (eos_id < 0 || eos_id >= c.tgt_vocab) return fail(h, CMT_EINVAL, "eos_id outside the target vocabulary");
  const int p = h->prec, E = c.emb_dim, H = c.hidden, L = c.layers, V = c.tgt_vocab, K = beam;
  const int BpE = round_up(B, 16);                   // encoder rows
  const int R = B * K, Rp = round_up(R, 16);         // decoder rows
  const size_t esz = h->esz;
  hipStream_t st = h->st;
  h->B = B; h->Bp = BpE; h->S = S; h->T = max_len;
  h->have_step = false;
  h->phase_n = 0;
  const int PH = h->PH;
  const float keep_p = h->drop_p;
  h->drop_p = 0.f;                                   // inference: no dropout
  launch_fill_f32((float*)h->flags, 1, 0.f, st);
  const GatherSide side{h->Pw(h->off_Esrc), c.src_vocab, src_ids_dev, src_len_dev, S, 0, 0, h->Xs, h->mask_s, h->tok_s, nullptr, h->len_s};
  launch_gather(p, &side, 1, E, B, BpE, h->flags, st);
  const char* Hs; int ldHs;
  note_capture(h);
  Section sec(h);
  sec.open(false);
  enqueue_encoder(h, S, &Hs, &ldHs, false, true, nullptr);                 // also leaves the decoder's initial states in slot 0 (BpE rows)
  sec.close();
  h->drop_p = keep_p;
  // one decoder row per hypothesis: the initial states repeated K times; the attention runs on the projected source rows, as in
  // the training step, and a sentence's hypotheses share them
  BeamState& bs = h->beam;
  bs.hist_ld = Rp;
  launch_beam_init(bs, B, Rp, K, c.bos_id, st);
  const size_t slotT = (size_t)Rp * PH * esz, slotC = (size_t)Rp * H * 4;   // state slots of Rp rows: 1 = read, 2 = written
  const size_t slotF = (size_t)Rp * H * esz;                                // the same slots of the fragment-major copies
  for (int l = 0; l < L; ++l) {
    LD& e = h->dec[l];
    launch_beam_expand((int)esz, e.Hst, e.ph, e.Hst + slotT, e.ph, R, Rp, K, H, st);
    launch_beam_expand(4, e.Cst, H, (char*)e.Cst + slotC, H, R, Rp, K, H, st);
    if (e.fm) launch_fm_pack(e.Hst + slotT, e.ph, Rp, H, e.HstF + slotF, st);   // fragment-major copy of the expanded states
  }
  launch_fill_T(p, h->xcat, (size_t)Rp * h->ldxcat, st);               // H_o^{<-1>} = 0
  const bool fm0 = h->xcatF && h->dec[0].fm;                           // bottom layer on fragment-major operands
  if (fm0) launch_fill_T(p, h->xcatF, (size_t)Rp * (E + H), st);
  BeamReorder ro{};
  for (int l = 0; l < L; ++l) {
    LD& e = h->dec[l];
    ro.h_src[l] = e.Hst + 2 * slotT; ro.h_dst[l] = e.Hst + slotT;
    ro.c_src[l] = (const float*)((char*)e.Cst + 2 * slotC); ro.c_dst[l] = (float*)((char*)e.Cst + slotC);
    if (e.fm && (l == 0 ? fm0 : h->dec[l - 1].fm)) ro.h_dst_fm[l] = e.HstF + slotF;   // (where the step reads it)
  }
  ro.ldh = PH;
  ro.ho_src = h->HoBuf; ro.ldho_src = PH; ro.ho_dst = h->xcat + (size_t)E * esz; ro.ldho_dst = h->ldxcat;
  if (fm0) { ro.ho_dst_fm = h->xcatF; ro.ho_fm_nsteps = (E + H) >> 5; ro.ho_fm_k0 = E; }
  ro.table = h->Pw(h->off_Etgt); ro.E = E; ro.x = h->xcat;
  launch_dec_embed(p, h->Pw(h->off_Etgt), E, bs.tok, R, Rp, h->xcat, h->ldxcat, st, fm0 ? h->xcatF : nullptr, (E + H) >> 5);
  for (int j = 0; j < max_len; ++j) {                  // (the later steps' embeddings come with the reorder)
    for (int l = 0; l < L; ++l) {
      LD& e = h->dec[l];
      LstmFwdDir d;
      if (l == 0) { d.x = h->xcat; d.ldx = h->ldxcat; d.Kx = E + H; d.wx_off = 0; d.wh_off = E + H; d.ldw = E + 2 * H; }
      else { d.x = h->dec[l - 1].Hst + 2 * slotT; d.ldx = PH; d.Kx = H; d.wx_off = 0; d.wh_off = H; d.ldw = 2 * H; }
      d.gx = nullptr; d.ldgx = 0; d.bias = h->params + e.b_off;
      d.hprev = e.Hst + slotT; d.ldh = e.ph; d.W = e.W;
      d.cprev = (const float*)((char*)e.Cst + slotC); d.mask = bs.mask;
      d.hnext = e.Hst + 2 * slotT; d.ldhn = e.ph; d.cnext = (float*)((char*)e.Cst + 2 * slotC);
      d.gsave = nullptr; d.ycat = nullptr; d.ldy = 0;
      if (e.fm) {                                    // as in greedy decoding: the layers above the bottom one
        d.hnext_fm = e.HstF + 2 * slotF;
        if (l > 0 && h->dec[l - 1].fm) { d.W_fm = e.Wfm; d.x_fm = h->dec[l - 1].HstF + 2 * slotF; d.hprev_fm = e.HstF + slotF; }
        else if (l == 0 && fm0) { d.W_fm = h->Wdec0F; d.x_fm = h->xcatF; d.hprev_fm = e.HstF + slotF; }
      }
      launch_lstm_fwd(p, d, Rp, H, st);
    }
    const char* Ht = h->dec[L - 1].Hst + 2 * slotT;
    StepGemm g{};                                    // W_c2 H_t
    g.a0 = g.a1 = Ht; g.lda0 = g.lda1 = PH; g.K0 = g.K1 = H; g.w0_off = 0; g.w1_off = H;
    g.W = h->Pw(h->off_Wc); g.ldw = 2 * H; g.N = H; g.mode = 3; g.skip0 = 1;
    g.out = h->wcp; g.ldout = H;
    if (h->CsF && h->dec[L - 1].fm) { g.W_fm = h->WcF; g.a0_fm = g.a1_fm = h->dec[L - 1].HstF + 2 * slotF; }
    launch_beam_attention(p, h->Kmat, h->PmatT, BpE, Ht, PH, g, h->len_s, S, B, K, H, h->dots, h->HoBuf, PH, st);
    // (the output layer's partials of a training step are of no use here)
    launch_beam_select(p, h->HoBuf, PH, h->Pw(h->off_Wo), h->params + h->off_Bo, Rp, V, H, h->logits, h->pmax, h->psum, bs, B, K, j, max_len,
                       eos_id, length_penalty, st);
    launch_beam_reorder(p, ro, bs, R, H, L, st);
  }
  launch_beam_finish(bs, B, K, max_len, c.pad_id, out_ids_dev, out_len_dev, out_score_dev, st);
  (void)hipMemcpyAsync(h->h_flags, h->flags, sizeof(int), hipMemcpyDeviceToHost, st);
  hipError_t e = hipStreamSynchronize(st);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "cmt_beam_decode");
  const int flags = *h->h_flags;
  if (flags & 3) return fail(h, CMT_ERANGE, (flags & 1) ? "a token id is outside its vocabulary" : "a length is outside [1, padded length]");
  return CMT_OK;
}

int cmt_sgd_update(cmt_handle* h, float lr) {
  if (!h) return CMT_EINVAL;
  if (!isfinite(lr)) return fail(h, CMT_EINVAL, "learning rate is not finite");
  launch_sgd(h->params, h->grads, h->nparams, lr, h->flags, h->prec ? h->Pc : nullptr, h->st);
  refresh_params(h, false);                        // the update wrote the bf16 copy itself: only the transposes are left
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "cmt_sgd_update");
  return CMT_OK;
}

int cmt_set_regularization(cmt_handle* h, float dropout, float label_smoothing, uint64_t dropout_seed) {
  if (!h) return CMT_EINVAL;
  if (!(dropout >= 0.f) || !(dropout < 1.f)) return fail(h, CMT_EINVAL, "dropout must be in [0, 1)");
  if (!(label_smoothing >= 0.f) || !(label_smoothing < 1.f)) return fail(h, CMT_EINVAL, "label_smoothing must be in [0, 1)");
  h->drop_p = dropout;
  h->drop_thresh = (unsigned)floor((double)dropout * 16777216.0);
  h->drop_scale = (float)(1.0 / (1.0 - (double)dropout));
  h->drop_seed = dropout_seed;
  h->ls_eps = label_smoothing;
  return CMT_OK;
}

int cmt_time_kernel(cmt_handle* h, const char* name, int iters, float* us_per_launch, double* algo_work) {
  if (!h || !name || iters < 1 || !us_per_launch || !algo_work) return fail(h, CMT_EINVAL, "bad argument");
  if (!h->have_step) return fail(h, CMT_EINVAL, "no step has been run");
  const cmt_config& c = h->cfg;
  const int p = h->prec, H = c.hidden, L = c.layers, E = c.emb_dim, V = c.tgt_vocab, Bp = h->Bp, T = h->T, S = h->S;
  const int PH = h->PH, Mt = T * Bp;
  const size_t BP = (size_t)Bp * PH, BH = (size_t)Bp * H;
  const double esz = (double)h->esz;
  const size_t es = h->esz;
  hipStream_t st = h->st;
  const std::string s(name);
  const int j = T / 2;                                  // the middle target position
  std::function<void(int)> launch;
  const int* probe_flag = nullptr;                      // set by a probe whose bounded wait may give up
  Section sec(h);                                       // (open until the replays have ended)
  if (s == "dec_loop_fwd" || s == "dec_loop_bwd") {
    // a whole loop as the step enqueues it, with the clears and copies before it and the launch behind it
    const bool bwd = s == "dec_loop_bwd";
    if (!(h->ran_loops & (bwd ? LOOP_RAN_BWD : LOOP_RAN_FWD))) return fail(h, CMT_EINVAL, "the last step took a launch per layer and position");
    const double state = (double)Bp * H, scores = (double)Bp * S;
    *algo_work = (8.0 * L + 1.0) * H * H * esz                         // [input; recurrent] columns of all layers, W_c's H_t half
               + S * state * (esz + (bwd ? 4 : esz))                   // keys and projected rows
               + (bwd ? T * (L * state * (16 + 4 + 4 * esz)            // activations, cell states; gate gradients
                             + state * (4 + 2 * esz) + 8 * scores)     // the output layer's gradient, H_o, dpre; weights, their gradients
                      : T * (state * 16 + L * state * (16 + 4 + esz)   // input part; activations, cell states, states
                             + state * esz + 4 * scores));             // H_o; weights
    sec.open(loop_fits(p, L, Bp, H, S, T, h->seq).alone);
    launch = [=](int) { if (bwd) enqueue_dec_loop_bwd(h, S, T); else enqueue_dec_loop_fwd(h, S, T); };
  } else if (s == "lstm_fwd_dec") {
    // decoder LSTM forward step, cycling over the layers like the real loop (weights not L2-resident)
    const int K = 2 * H;                                // per-step contraction (layer 0: [feed; h], others: [x; h])
    *algo_work = 4.0 * H * K * esz                      // weights, read once
               + (double)Bp * K * esz                   // [x; h_prev]
               + (double)4 * H * 4                      // bias (the layers timed here have no pre-batched input part)
               + (double)Bp * H * 4                     // c_prev
               + (double)Bp * H * (esz + 4)             // h, c out
               + (double)Bp * 4 * H * 4;                // gate activations kept for backward
    launch = [=](int i) { dec_lstm_fwd(h, L > 1 ? 1 + i % (L - 1) : 0, j); };
  } else if (s == "step2d_bwd_dec") {
    // [dx; dh_prev] = dgates [W_x; W_h] of a decoder layer, written as planes
    const int kb = step_kblocks(p, 2 * H, 4 * H, Bp, h->kb_bwd_dec);
    *algo_work = 4.0 * H * 2 * H * esz + (double)Bp * 4 * H * esz + (double)kb * Bp * 2 * H * 4;
    launch = [=](int i) {
      LD& e = h->dec[L > 1 ? 1 + i % (L - 1) : 0];
      StepGemm g{};
      g.a0 = e.dG + (size_t)j * Bp * e.pg * es; g.lda0 = e.pg; g.K0 = 4 * H; g.w0_off = 0; g.K1 = 0;
      g.W = e.Wt + (size_t)(&e == &h->dec[0] ? E : 0) * 4 * H * es; g.ldw = 4 * H;
      g.N = 2 * H; g.mode = 1; g.max_kb = h->kb_bwd_dec;
      g.out = e.bwdp; g.ldout = 2 * H; g.plane_stride = (size_t)Bp * 2 * H;
      if (e.fmb) { g.W_fm = e.WtF; g.w_tile0 = (&e == &h->dec[0] ? E : 0) / 16; g.a0_fm = e.dGF + (size_t)j * Bp * 4 * H * es; }
      launch_step_gemm(p, g, Bp, st);
    };
  } else if (s == "step_bwd_fused_dec") {
    // the same product with the whole contraction inside the workgroup and the cell backward of the layer below
    // in the epilogue (the form the decoder's backward loop runs): weights and dgates read once, dh_prev stored,
    // and the pointwise operands of the fused cell backward (gates, c, dc, dh in and out, dgates out)
    *algo_work = 4.0 * H * 2 * H * esz + (double)Bp * 4 * H * esz + (double)Bp * H * 4
               + (double)Bp * H * (4 * 4 + 2 * 4 + 2 * 4 + 2 * 4 + 4) + (double)Bp * 4 * H * esz;
    launch = [=](int i) {
      const StepBwd g = dec_bwd_gemm(h, L > 1 ? 1 + i % (L - 1) : 0, j);
      launch_step_bwd_fused(p, g, Bp, st);
    };
  } else if (s == "att_fwd") {
    // attention forward of one decoder step as the step launches it.  On the projected rows: scores (with the sums
    // W_c2 H_t in the same launch), softmax, mix and tanh -> H_o: the keys and the projected rows of every sentence
    // once and the H_t half of W_c.  Else scores + softmax + context: the keys and H_s of every sentence once.
    const bool proj = h->att_proj && Bp < 256;
    *algo_work = 2.0 * Bp * S * H * esz + (proj ? (double)H * H * esz : 0.0);
    const char* Hs = L > 1 ? h->enc[L].Hst + BP * es : h->Y0;
    const int ldHs = L > 1 ? PH : H;
    launch = [=](int) {
      if (proj) dec_att_fwd_proj(h, j, S, h->dots);
      else launch_att_fwd(p, h->Kmat, H, Hs, ldHs, h->dec[L - 1].Hst + (j + 1) * BP * es, PH, h->len_s, S, Bp, H, h->dots,
                          h->att_a + (size_t)j * Bp * S, h->Cs + j * BP * es, PH, st);
    };
  } else if (s == "att_bwd") {
    // attention backward of one decoder step as the step launches it (score gradients, the gradient sent to the
    // top layer's output, that layer's cell backward in the same launch).  On the projected rows the launch of
    // dpre W_c is part of it: the fp32 projected rows and the keys of every sentence once, and W_c.  Else H_s and the
    // keys of every sentence once.
    const bool fused = (h->bwd_fused & 1) && Bp <= 128;
    const bool proj = (h->att_proj & 1) && Bp < 256 && fused && h->wc_whole_k;
    *algo_work = proj ? (double)Bp * S * H * (4 + esz) + 2.0 * H * H * esz : 2.0 * Bp * S * H * esz;
    const char* Hs = L > 1 ? h->enc[L].Hst + BP * es : h->Y0;
    const int ldHs = L > 1 ? PH : H;
    // (the planes the step's dpre W_c wrote: one in the fused loop's whole-k form)
    const int kbw = (h->wc_whole_k && fused) ? 1 : step_kblocks(p, 2 * H, H, Bp, h->kb_wc);
    const size_t pstr = (size_t)Bp * 2 * H;
    launch = [=](int) {
      if (proj) { dec_att_bwd_proj(h, j, S, false); return; }
      LstmBwdPoint top = dec_cell(h, L - 1, j);
      top.dhrec = Planes{h->dec[L - 1].bwdp, H, 1, 0};
      launch_att_bwd(p, h->Kmat, H, Hs, ldHs, Planes{h->wcp, 2 * H, kbw, pstr}, h->dCs + j * BH, h->att_a + (size_t)j * Bp * S,
                     h->len_s, S, Bp, H, h->dots, h->att_ds + (size_t)j * Bp * S, h->dHt, st, &top);
    };
  } else if (s == "gemm_gx") {
    // time-batched input-side GEMM of the decoder's bottom layer: [T Bp, E] x [E, 4H]  (flops)
    *algo_work = 2.0 * Mt * 4 * H * E;
    launch = [=](int) {
      LD& d0 = h->dec[0];
      launch_gemm_nt(p, h->Xt, E, d0.W, E + 2 * H, Mt, 4 * H, E, d0.Gx, nullptr, 4 * H, h->params + d0.b_off, 0, st);
    };
  } else if (s == "gemm_dw") {
    // the decoder's weight gradients as the step launches them: W_c (two segments) and every layer's segments,
    // dG^T [4H, T Bp] x X^T [width, T Bp]^T each, one grouped launch  (flops)
    std::vector<GemmProb> probs;
    probs.push_back(GemmProb{h->dPreT, h->CsT, h->grads + h->off_Wc, Mt, Mt, 2 * H, H, H, Mt, 0});
    probs.push_back(GemmProb{h->dPreT, h->dec[L - 1].HstT + (size_t)Bp * es, h->grads + h->off_Wc + H, Mt, (T + 1) * Bp, 2 * H, H, H, Mt, 0});
    for (int l = 0; l < L; ++l) {
      LD& e = h->dec[l];
      float* dW = h->grads + e.w_off;
      if (l == 0) {
        probs.push_back(GemmProb{e.dGT, h->XtT, dW, Mt, Mt, e.Kin + H, 4 * H, E, Mt, 0});
        probs.push_back(GemmProb{e.dGT, h->HoBufT, dW + E, Mt, Mt + Bp, e.Kin + H, 4 * H, H, Mt, 0});
        probs.push_back(GemmProb{e.dGT, e.HstT, dW + E + H, Mt, (T + 1) * Bp, e.Kin + H, 4 * H, H, Mt, 0});
      } else {
        if (h->drop_p > 0.f) probs.push_back(GemmProb{e.dGT, h->dec[l - 1].YdT, dW, Mt, Mt, e.Kin + H, 4 * H, H, Mt, 0});
        else probs.push_back(GemmProb{e.dGT, h->dec[l - 1].HstT + (size_t)Bp * es, dW, Mt, (T + 1) * Bp, e.Kin + H, 4 * H, H, Mt, 0});
        probs.push_back(GemmProb{e.dGT, e.HstT, dW + H, Mt, (T + 1) * Bp, e.Kin + H, 4 * H, H, Mt, 0});
      }
    }
    double fl = 0;
    for (const GemmProb& q : probs) fl += 2.0 * q.M * q.N * q.K;
    *algo_work = fl;
    launch = [=](int) { launch_gemm_nt_group(p, probs.data(), (int)probs.size(), st, h->gsplit2, h->gsplit2_floats); };
  } else if (s == "ce_fwd") {
    // vocabulary projection of one slab of rows with the partial log-sum-exp statistics  (flops)
    int nslab;
    const int rows = ce_slab_plan(h, Mt, &nslab);
    const int Mc = nslab == 1 ? Mt : rows;              // the first slab
    *algo_work = 2.0 * Mc * (double)V * H;
    const char* Ho = (h->drop_p > 0.f ? h->HoDrop : h->HoBuf) + BP * es;
    launch = [=](int) {
      launch_ce_fwd(p, Ho, PH, h->Pw(h->off_Wo), h->params + h->off_Bo, h->labels, Mc, V, H, h->dzTs, h->ce_pitch, h->pmax,
                    h->psum, nullptr, h->zy, st);
    };
  } else if (s == "grid_barrier" || s == "grid_barrier_nofence") {
    // 100 chip-wide barriers between 256 resident workgroups (bounded polling); work = the number of barriers
    const int rounds = 100, fences = s == "grid_barrier" ? 1 : 0;
    unsigned* counter = (unsigned*)h->gsplit;
    int* gave_up = (int*)h->gsplit + 64;
    *algo_work = rounds;
    launch = [=](int) {
      launch_fill_f32(h->gsplit, 128, 0.f, st);
      launch_grid_barrier_probe(counter, gave_up, 256, rounds, fences, 1 << 16, st);
    };
    probe_flag = gave_up;
  } else if (s == "mfma_rate") {
    // matrix cores alone: up to 4096 workgroups x 4 wavefronts x 2048 x 4 bf16 32x32x16 MFMAs on registers  (flops)
    const int it = 2048;
    const int blocks = (int)std::min<size_t>(4096, h->gsplit_floats / 256);   // one float per lane lands in the split-k scratch
    if (blocks < 1) return fail(h, CMT_EINVAL, "workspace too small for the probe");
    *algo_work = (double)blocks * 4 * it * 4.0 * (2.0 * 32 * 32 * 16);
    launch = [=](int) { (void)launch_mfma_rate(h->gsplit, blocks, it, st); };
  } else {
    return fail(h, CMT_EINVAL, "unknown kernel name");
  }
  (void)BH;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return fail(h, CMT_EHIP, "event create");
  for (int i = 0; i < 4; ++i) launch(i);
  (void)hipEventRecord(e0, st);
  for (int i = 0; i < iters; ++i) launch(i);
  (void)hipEventRecord(e1, st);
  hipError_t e = hipEventSynchronize(e1);
  float ms = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_time_kernel");
  *us_per_launch = ms * 1e3f / iters;
  if (probe_flag) {
    int gave = 0;
    e = hipMemcpy(&gave, probe_flag, sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(h, e, "cmt_time_kernel");
    if (gave) return fail(h, CMT_EHIP, "the barrier probe gave up waiting (its workgroups were not all resident)");
  }
  return CMT_OK;
}

int cmt_padded_batch(const cmt_handle* h) { return h ? h->Bp : CMT_EINVAL; }

int cmt_debug_fetch(cmt_handle* h, const char* name, float* host_dst, size_t bytes) {
  if (!h || !name || !host_dst) return fail(h, CMT_EINVAL, "null pointer");
  if (!h->have_step) return fail(h, CMT_EINVAL, "no step has been run");
  const int H = h->cfg.hidden, E = h->cfg.emb_dim, L = h->cfg.layers;
  const size_t Bp = h->Bp, S = h->S, T = h->T, BP = Bp * h->PH;
  // rows x cols elements with a source row pitch (elements); isT: stored in the operand type
  const void* src = nullptr; size_t rows = 0, cols = 0, pitch = 0; bool isT = false;
  const std::string s(name);
  if (s == "x_src") { src = h->Xs; rows = S * Bp; cols = pitch = E; isT = true; }
  else if (s == "x_tgt") { src = h->Xt; rows = T * Bp; cols = pitch = E; isT = true; }
  else if (s == "mask_src") { src = h->mask_s; rows = 1; cols = pitch = S * Bp; }
  else if (s == "mask_tgt") { src = h->mask_t; rows = 1; cols = pitch = T * Bp; }
  else if (s == "h_s") {
    rows = S * Bp; cols = H; isT = true;
    if (L == 1) { src = h->Y0; pitch = H; } else { src = h->enc[L].Hst + BP * h->esz; pitch = h->PH; }
  }
  else if (s == "h_t") { src = h->dec[L - 1].Hst + BP * h->esz; rows = T * Bp; cols = H; pitch = h->PH; isT = true; }
  else if (s == "att_a") { src = h->att_a; rows = 1; cols = pitch = T * Bp * S; }
  else if (s == "att_s") { src = h->att_s; rows = 1; cols = pitch = T * Bp * S; }
  else if ((s.rfind("enc.l", 0) == 0 || s.rfind("dec.l", 0) == 0) && s.size() >= 8) {
    // "<enc|dec>.l<k>[.fwd|.bwd].<h|c|gates>": states after every step and gate activations of one LSTM
    const bool enc = s[0] == 'e';
    size_t pos = 5;
    int l = 0;
    while (pos < s.size() && s[pos] >= '0' && s[pos] <= '9') l = l * 10 + (s[pos++] - '0');
    int dir = -1;
    if (s.compare(pos, 5, ".fwd.") == 0) { dir = 0; pos += 4; }
    else if (s.compare(pos, 5, ".bwd.") == 0) { dir = 1; pos += 4; }
    const std::string what = pos < s.size() ? s.substr(pos + 1) : "";
    if (l >= L || (what != "h" && what != "c" && what != "gates") || (dir >= 0) != (enc && l == 0))
      return fail(h, CMT_EINVAL, "unknown intermediate name");
    const LD& d = enc ? h->enc[l == 0 ? dir : l + 1] : h->dec[l];
    const size_t steps = enc ? S : T;
    // slot 0 of Hst / Cst holds the initial state (the reverse direction: slot S), slot t + 1 (reverse: t)
    // the state after the step at position t
    const size_t first = (enc && l == 0 && dir == 1) ? 0 : 1;
    rows = steps * Bp;
    if (what == "h") { src = d.Hst + first * Bp * d.ph * h->esz; cols = d.Hh; pitch = d.ph; isT = true; }
    else if (what == "c") { src = d.Cst + first * Bp * d.Hh; cols = pitch = d.Hh; }
    else { src = d.Gs; cols = pitch = 4 * (size_t)d.Hh; }
  }
  else if (s == "att_cs") { src = h->Cs; rows = T * Bp; cols = H; pitch = h->PH; isT = true; }
  else if (s == "h_o") { src = h->HoBuf + BP * h->esz; rows = T * Bp; cols = H; pitch = h->PH; isT = true; }
  else if (s == "h_o_drop") {
    src = (h->drop_p > 0.f ? h->HoDrop : h->HoBuf) + BP * h->esz; rows = T * Bp; cols = H; pitch = h->PH; isT = true;
  }
  else if (s == "lse" || s == "nll") {
    // kept per valid target position, densely numbered on the device: spread out to [T, Bp], zero elsewhere
    const size_t n = T * Bp;
    if (bytes != n * 4) return fail(h, CMT_EINVAL, "size mismatch for the requested intermediate");
    hipError_t e = hipStreamSynchronize(h->st);
    std::vector<int32_t> pos(n);
    std::vector<float> dense(n);
    if (e == hipSuccess) e = hipMemcpy(pos.data(), h->ce_pos, n * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(dense.data(), s == "lse" ? h->lse : h->nll, n * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(h, e, "cmt_debug_fetch");
    for (size_t i = 0; i < n; ++i) host_dst[i] = pos[i] >= 0 ? dense[pos[i]] : 0.f;
    return CMT_OK;
  }
  else return fail(h, CMT_EINVAL, "unknown intermediate name");
  const size_t n = rows * cols;
  if (bytes != n * 4) return fail(h, CMT_EINVAL, "size mismatch for the requested intermediate");
  hipError_t e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return hip_fail(h, e, "cmt_debug_fetch");
  if (isT && h->prec) {
    std::vector<uint16_t> tmp(n);
    e = hipMemcpy2D(tmp.data(), cols * 2, src, pitch * 2, cols * 2, rows, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(h, e, "cmt_debug_fetch");
    for (size_t i = 0; i < n; ++i) { uint32_t u = ((uint32_t)tmp[i]) << 16; memcpy(&host_dst[i], &u, 4); }
  } else {
    e = hipMemcpy2D(host_dst, cols * 4, src, pitch * 4, cols * 4, rows, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(h, e, "cmt_debug_fetch");
  }
  return CMT_OK;
}

const char* cmt_last_error(const cmt_handle* h) { return h ? h->err.c_str() : "null handle"; }

}  // extern "C"

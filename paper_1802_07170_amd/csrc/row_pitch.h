// Row pitches of the activations that a position's kernels and the products over all positions read.  No device code, so that the rule
// can be checked with a host compiler.
#pragma once

namespace cmt {

// The step kernels that read row-major operands take 16 sentences x 64 bytes per fragment load; with a power-of-two pitch those 16
// segments fall on the same cache banks (measured: 14.3 -> 11.0 us for the decoder LSTM step with 16 bytes of padding; rows kept 128-byte
// aligned by padding with 64 elements instead: 11.6 us against 9.8 us, 32 / 72 / 136 elements: 10.0 - 10.2 us).
// Where fragment-major copies serve those kernels, what is left to read the rows are the products over all positions, 128 bytes of a row
// at a time: rows of whole lines, or each piece takes two (dX of 3200 positions, 4096 -> 1024: 73 -> 47 us; medium step 5.87 -> 5.78 ms).
constexpr int ACT_PAD = 8, ACT_PAD_LINES = 64;

// Padding in elements: rows of H (states, H_o, contexts, dpre) and of E + H (the bottom decoder layer's input when decoding), the gate
// gradients of any layer, and those of the bottom decoder layer.
struct RowPitch { int states, gates, gates_bottom; };

// The decoders' bottom layer has a copy of its input and states for whole k steps (E a multiple of 32); the gate gradients of the training
// step's have one for whole tiles of columns (E + H a multiple of 16); every other reader's operands have one wherever H is a multiple of
// 32.  Without the copy, us (whole lines | padded by 8): beam search of 16 x 10 rows, embeddings of 1000, two layers of 1024 2373 | 2271;
// training steps, embeddings of 200, 64 sentences, five layers of 1024 | 512 4634 | 4550, 3350 | 3311, six of 256 (32 sentences) 3025 | 2975.
// With it, layers narrower than 256 gain nothing from whole lines, and their chains lose: five layers of 64 | 128 | 192, 64 sentences 2436 | 2395,
// 2595 | 2575, 2713 | 2704.
inline RowPitch row_pitch(int prec, int E, int H, bool lines) {
  const bool whole = lines && prec && H >= 256 && H % 64 == 0;
  RowPitch p;
  p.gates = whole ? ACT_PAD_LINES : ACT_PAD;
  p.gates_bottom = whole && (E + H) % 16 == 0 ? ACT_PAD_LINES : ACT_PAD;
  p.states = whole && E % 32 == 0 ? ACT_PAD_LINES : ACT_PAD;
  return p;
}

}  // namespace cmt

// The memory step of the paper-form memory (SwiGLU per fast-weight head) in one kernel, for bf16
// activations: hidden activations, their gradients, the three weight gradients and the update, for
// one or several consecutive segments.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mone {

// Operands of the step, written by the preprocessing in MFMA fragment order: a fragment is 64
// lanes x 8 values (1 KiB contiguous), so a wave loads one with a single coalesced instruction
// straight into registers.  d_h is padded to 32 * NB channels (zeros), NB = ceil(d_h / 32).
//   token fragments    [B][Tp/32][2 NB][64][8]: lane l of fragment (t, s) holds token
//                      32 t + l % 32, channels 16 s + 8 (l / 32) ..  (contraction over channels)
//   channel fragments  [B][Tp/16][NB][64][8]: lane l of fragment (t, c) holds channel
//                      32 c + l % 32, tokens 16 t + 8 (l / 32) ..    (contraction over tokens)
struct SwStep {
  const uint16_t* kf;  // keys, token fragments
  const uint16_t* kt;  // keys, channel fragments
  const uint16_t* yf;  // dY0 = -v / n, token fragments
  const uint16_t* yt;  // dY0, channel fragments
  long long k_ss, y_ss;       // elements between consecutive segments
  const float* rate;          // [L][Tp] per-token rates of the first segment, or null (lr)
  const float* beta;          // [L] momentum decays (paper's optimiser)
  long long rate_ss, beta_ss;
  float *w_in, *w_gate, *w_out;  // masters [B][d_h][d_h]
  float *m_in, *m_gate, *m_out;  // momenta (paper's optimiser)
  uint16_t* wig;                 // [B][2 d_h][d_hp] interleaved copy of W_in and W_gate (reads)
  const float *n_ig, *n_out;     // initial row norms [B][2 d_h], [B][d_h] (paper's optimiser)
  float* loss_part;              // [B][parts], parts = 4 * row blocks
  int dh, dhp, H, Tp, n, g, B, parts;
  float lr;
};

// g consecutive segments of n tokens each (n <= Tp).
hipError_t launch_sw_step(const SwStep& p, bool paper, hipStream_t s);

}  // namespace mone

// Arguments and constants of the single-launch decode pass (k_decode.hip).
// Part of gvc_kernels.h: include that header, not this one.
#pragma once

namespace gvc {

// ------------------------------------------------------------------ persistent decode pass
// Single-token passes over all layers for one episode (k_decode.hip).
constexpr int kDecodeMaxSeg = 8;       // weight blocks per workgroup per step
constexpr int kDecodeMaxSegs = 5 * kDecodeMaxSeg;   // of a wave in one layer (4 steps) and the LM head
constexpr int kDecodeXccWord = 544;    // barrier words: set when a workgroup is not on XCD blockIdx % 8
constexpr int kDecodePoisonWord = 576; // barrier words: set when a head contribution was not finite
constexpr int kDecodeHeadWord = 1024;  // barrier words: per-head counters, 32 words apart
constexpr int kDecodeMaxHeads = 64;
// Layer steps (passes x layers) of one launch.  Each has a copy of the q, k, v
// exchange of its own, so that no line of it is read twice in a launch; at the
// 7B shape a launch of 8 passes takes 12.6 MB of them, 0.01% of the weights it
// streams.  More passes go to further launches.
constexpr int kDecodeMaxSteps = 256;
constexpr int decode_launch_passes(int L) { return kDecodeMaxSteps / L; }   // L <= 128
constexpr int kDecodeMaxGrid = 1024;   // workgroups of one pass (per-workgroup head records)
// The abort flag is the last barrier word: the others are zeroed before a launch
// sequence, it stays set until the gate that follows has reported it.
constexpr int kDecodeAbortWord = kDecodeHeadWord + 32 * kDecodeMaxHeads;
constexpr int kDecodeBarWords = kDecodeAbortWord + 1;
// grid barriers and per-head barriers of one pass over L layers (one more
// grid barrier when the pass also runs the LM head and the token choice)
constexpr int decode_grid_barriers(int L, bool head) { return 1 + 3 * L + (head ? 1 : 0); }
constexpr int decode_head_barriers(int L) { return L; }

struct DecodeArgs {
  // packed weights of layer 0 (k = q + qkv_stride, v = q + 2 qkv_stride,
  // up = gate + gu_stride); layer l's are l * layer_stride further (bf16x8 units)
  const bf16x8* wq; const bf16x8* wo; const bf16x8* wg; const bf16x8* wd;
  size_t qkv_stride, gu_stride, layer_stride;
  bf16* kc; bf16* vc;          // layer 0 caches (episode 0); layer l at l * kv_layer_elems
  size_t kv_layer_elems;
  const float* gains;          // [L][2][d]: attention norm, FFN norm
  const float2* rope;          // [kv_pad][head_dim/2]
  const bf16* embed;           // [V][d] token embedding table: a pass starts from its token's row
  const int* tok_in;           // token of the first pass; with `forced`, of pass p at tok_in[p]
  int forced;                  // 1: every pass takes its token from tok_in, 0: from the pass before
  int n_pass;                  // passes of this launch, at positions pos, pos + 1, ... (1 without kDecodeHead),
                               // n_pass * L <= kDecodeMaxSteps
  float* x;                    // [d] layer input / output (in place)
  unsigned long long* racc;    // [d] sum of the heads' attention-output contributions, int64 in 2^-32 units
  float* qkv;                  // [n_pass][L][3d] q, k, v before RoPE
  bf16* act;                   // [F] SwiGLU output
  unsigned* bar;               // kDecodeBarWords barrier words
  unsigned bar_base;           // grid barriers completed by earlier launches since the words were zeroed
  unsigned hbar_base;          // per-head barriers completed by earlier launches
  long long timeout_ticks;     // barrier wait limit in wall-clock ticks (100 MHz)
  int L, d, F, H, head_dim, KBd, KBf, kv_pad, pos, act_bytes;
  float eps;
  int flags;                   // kDecodeHead or 0
  // with kDecodeHead: final norm, LM head and the greedy token and margin of
  // this pass (Eq. 1) after the last layer
  const bf16x8* wlm;           // packed LM head, nlm blocks of KBd fragments
  const float* final_gain;     // [d]
  float* logits;               // [V] logits of pass p at logits + p * logits_stride
  size_t logits_stride;
  float* head_part;            // [gridDim <= kDecodeMaxGrid][8] per workgroup: max, sum, v1, i1, v2, i2
  int* tok_out;                // the tokens of the passes (one int each)
  float* margin_out;           // their margins (one float each)
  int nlm, V, bin_lo, full_vocab;
};
constexpr int kDecodeHead = 4;        // the pass ends with the LM head and the token choice

}  // namespace gvc

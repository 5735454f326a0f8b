// The stack of layers as one launch (ad_team.hip): arguments and limits.
#pragma once

#include "ad_internal.h"

namespace ad {

typedef unsigned short bf16_storage;

constexpr int kTeamMembers = 32;                 // workgroups of a team: the compute units of an XCD
constexpr int kTeamD = 512, kTeamF = 2048;       // the model widths the kernel is built for (bf16, head width 64)
constexpr int kTeamMaxRows = 32, kTeamMaxKeys = 128;
constexpr int kTeamXRows = 8 * kTeamMaxRows;     // packed rows of a launch
constexpr int kTeamFormTicks = 30000;            // 0.3 ms: an idle chip has a team together in a few us

// Byte offsets of a layer's entries from its first byte (weight_layout; the launcher's caller checks them).
template <bool DEC>
struct TeamOff {
  static constexpr int kMat = kTeamD * kTeamD * 2, kVec = kTeamD * 4, kAttn = 4 * kMat + 4 * kVec, kFfn = 2 * kTeamD * kTeamF * 2 + kTeamF * 4 + kVec;
  static constexpr int wqkv = 0, wo = 3 * kMat, bqkv = 4 * kMat, bo = bqkv + 3 * kVec;
  static constexpr int ln1g = kAttn, ln1b = ln1g + kVec;
  static constexpr int cwq = ln1b + kVec, cwo = cwq + 3 * kMat, cbq = cwq + 4 * kMat, cbo = cbq + 3 * kVec;   // decoder only
  static constexpr int ln2g = cwq + kAttn, ln2b = ln2g + kVec;                                              // decoder only
  static constexpr int w1 = DEC ? ln2b + kVec : cwq, b1 = w1 + kTeamD * kTeamF * 2, w2 = b1 + kTeamF * 4, b2 = w2 + kTeamD * kTeamF * 2;
  static constexpr int ln_fg = DEC ? ln2g : ln1g, ln_fb = ln_fg + kVec;   // pending ahead of the FFN
  static constexpr int ln_lg = w1 + kFfn, ln_lb = ln_lg + kVec;           // the layer's last
  static constexpr int kLayerBytes = ln_lb + kVec;
};
struct TeamArgs {
  int n_teams, xcd0, layers;          // teams on the XCDs xcd0, xcd0 + 1, ...
  int head_only;                      // in the last layer only segment 0's rows go on after the key / value projection
  int row_lo[2][9];                   // packed rows of team t: segments [row_lo[s][t], row_lo[s][t + 1])
  int prob[9];                        // its attention problems (descriptors)
  int prob2_off;                      // the descriptors of segment 1's problems lie this much further on (0: none)
  unsigned form_ticks;                // how long the first barrier is waited for (10 ns each; 0: not at all)
  float scale;
  const char* w;                      // layer 0 (the others TeamOff::kLayerBytes apart)
  const float* x;                     // the embedded rows, fp32 and bf16
  const bf16_storage* xa;
  float* s;                           // rows passed on inside a layer; in s the last layer's for the LayerNorm that follows
  float *s1, *s2, *xr;                // (kTeamXRows packed rows)
  bf16_storage* att2;
  bf16_storage *q, *att, *f;
  bf16_storage *K, *V;                // keys / values of layer 0
  size_t kv_stride;                   // bytes to the next layer's
  const bf16_storage *Km, *Vm;        // memory keys / values
  size_t m_stride;
  const SeqDesc *self_desc, *cross_desc;
  const int* row_dst;
  unsigned *words, *fail;             // both cleared before the launch
};
// once per device before the first launch: what the kernels need of the runtime; false: they cannot run
bool prepare_team(bool decoder);
// at most kTeamMaxRows rows a team, kTeamMaxKeys keys a problem
void launch_team(const TeamArgs& a, bool decoder, int max_rows, int max_keys, hipStream_t s);

}  // namespace ad

// The stack of layers as one launch (ad_team.hip): arguments and limits.
#pragma once

#include "ad_internal.h"

namespace ad {

typedef unsigned short bf16_storage;

constexpr int kTeamMembers = 32;                 // workgroups of a team: the compute units of an XCD
constexpr int kTeamD = 512, kTeamF = 2048;       // the model widths the kernel is built for (bf16, head width 64)
constexpr int kTeamMaxRows = 32, kTeamMaxKeys = 128;
constexpr int kTeamStations = 2;                 // XCDs that take turns over a team's layers: one requests strips while the other works
constexpr int kTeamXRows = 8 * kTeamMaxRows;     // packed rows of a launch
constexpr int kTeamFormTicks = 30000;            // 0.3 ms: an idle chip has a team together in a few us

// Byte offsets of a layer's entries from its first byte (weight_layout; the launcher's caller checks them).
template <bool DEC, int D = kTeamD, int F = kTeamF, int ESZ = 2>
struct TeamOff {
  static constexpr int kMat = D * D * ESZ, kVec = D * 4, kAttn = 4 * kMat + 4 * kVec, kFfn = 2 * D * F * ESZ + F * 4 + kVec;
  static constexpr int wqkv = 0, wo = 3 * kMat, bqkv = 4 * kMat, bo = bqkv + 3 * kVec;
  static constexpr int ln1g = kAttn, ln1b = ln1g + kVec;
  static constexpr int cwq = ln1b + kVec, cwo = cwq + 3 * kMat, cbq = cwq + 4 * kMat, cbo = cbq + 3 * kVec;   // decoder only
  static constexpr int ln2g = cwq + kAttn, ln2b = ln2g + kVec;                                              // decoder only
  static constexpr int w1 = DEC ? ln2b + kVec : cwq, b1 = w1 + D * F * ESZ, w2 = b1 + F * 4, b2 = w2 + D * F * ESZ;
  static constexpr int ln_fg = DEC ? ln2g : ln1g, ln_fb = ln_fg + kVec;   // pending ahead of the FFN
  static constexpr int ln_lg = w1 + kFfn, ln_lb = ln_lg + kVec;           // the layer's last
  static constexpr int kLayerBytes = ln_lb + kVec;
};
// A team's XCDs (stations) have buffers of their own for the rows on their way inside a layer: bytes from the first of them.
struct TeamSlot {
  static constexpr int kRow16 = kTeamMaxRows * kTeamD * 2, kRow32 = 2 * kRow16;
  static constexpr int q = 0, att = kRow16, att2 = 2 * kRow16, s1 = 3 * kRow16, s2 = s1 + kRow32, s = s2 + kRow32, xr = s + kRow32, f = xr + kRow32;
  static constexpr int kBytes = f + kTeamMaxRows * kTeamF * 2;
};
constexpr int kTeamHopBytes = 8 * kTeamMaxRows * kTeamD * 4;   // a layer's results on their way to the next XCD: [team][row][512] fp32
constexpr int kTeamKvBytes = kTeamXRows * kTeamD * 2;          // a layer's keys (values) where they have no place in a cache: [packed row][512]
struct TeamArgs {
  int n_teams, stations;              // team t's layers l, l + stations, .. run on XCD xcd0 + t + n_teams * (l % stations)
  int xcd0, layers;
  int head_only;                      // in the last layer only segment 0's rows go on after the key / value projection
  int shared;                         // teams read each other's keys and values
  int row_lo[2][8], row_n[2][8];      // packed rows of team t, two segments
  int prob_lo[8], prob_n[8];          // its attention problems (descriptors); the rows of a problem that are another team's are left to that
  int prob2_off;                      // the descriptors of segment 1's problems lie this much further on (0: none)
  unsigned form_ticks;                // how long the first barrier is waited for (10 ns each; 0: not at all)
  float scale;
  const char* w;                      // layer 0 (the others TeamOff::kLayerBytes apart)
  const float* x;                     // the embedded rows, fp32 and bf16
  const bf16_storage* xa;
  float* s;                           // the last layer's rows, for the LayerNorm that follows
  char *slots, *hop;                  // [8] TeamSlot, [layers] kTeamHopBytes
  bf16_storage *K, *V;                // keys / values of layer 0
  size_t kv_stride;                   // bytes to the next layer's
  const bf16_storage *Km, *Vm;        // memory keys / values
  size_t m_stride;
  const SeqDesc *self_desc, *cross_desc;
  const int* row_dst;
  unsigned *words, *fail;             // both cleared before the launch
};
// One team launch: its arguments, the most rows of a team and the most keys of a problem (they select the kernel).
struct TeamRun { TeamArgs a; int max_rows, max_keys; };
// the deal of n problems' rows to teams (ad_api.cpp; max_keys is the caller's)
bool team_deal(const int* rows, const int* rows2, int n, int xcds, int layers, int max_rows, TeamRun* t);

// ---- fp32 (ad_team_f32.hip): widths 128 (FFN 512, heads of 32) and 512 (2048, 64)
constexpr int kTeamF32Rows = 16;                 // rows of a team
template <int D, int F> struct TeamSlotF32 {     // a team's rows in one layer: [16] of these (bytes)
  static constexpr int q = 0, att = D * 4, att2 = 2 * D * 4, s1 = 3 * D * 4, s2 = 4 * D * 4, xr = 5 * D * 4, f = 6 * D * 4, kRow = f + F * 4;
  static constexpr int kBytes = kTeamF32Rows * kRow;
};
inline bool team_f32_widths(int d, int n_heads, int f) { return (d == 128 && n_heads == 4 && f == 512) || (d == 512 && n_heads == 8 && f == 2048); }
inline size_t team_f32_slot_bytes(int d) { return d == 128 ? TeamSlotF32<128, 512>::kBytes : TeamSlotF32<512, 2048>::kBytes; }
// LDS of the row tile: FFN2's operand, or the tile with the attention behind it
__host__ __device__ constexpr size_t team_f32_rows_bytes(int d, int f, int dh) {
  const size_t ffn = 16 * (size_t)(f + 4) * 4, att = (16 * (size_t)(d + 4) + 16 * 132 + 16 + 16 * (dh + 4)) * 4;
  return ffn > att ? ffn : att;
}
bool prepare_team_f32(int d, bool decoder);
void launch_team_f32(const TeamArgs& a, int d, bool decoder, int max_keys, hipStream_t s);

// once per device before the first launch: what the kernels need of the runtime; false: they cannot run
bool prepare_team(bool decoder);
// whether there is a kernel for teams of max_rows rows, problems of max_keys keys and so many XCDs a team: launch_team's condition
bool team_has_kernel(bool decoder, int max_rows, int max_keys, int stations);
// at most kTeamMaxRows rows a team, kTeamMaxKeys keys a problem
void launch_team(const TeamArgs& a, bool decoder, int max_rows, int max_keys, hipStream_t s);

}  // namespace ad

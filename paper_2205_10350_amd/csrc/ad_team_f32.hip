// A whole stack of layers in one launch, fp32: teams as in ad_team.hip, the sums as in ad_gemm_f32.hip and ad_attention_f32.hip.
//
// A forward of a few fp32 rows as a launch per stage is a chain of 17 (two layers of width 128) or 45 launches (six of width 512) of 4.5 to
// 5.5 us, most of it the boundary.  Here up to 16 rows of a sequence are a team of 32 compute units on one XCD, longer blocks are cut into
// pieces that read each other's keys and values, and where XCDs are left over a team has two that take turns over the layers.
// A workgroup's eight waves are two quads; a quad takes strips of 16 columns, its waves the four quarters of K, whose sums meet in LDS as
// (p0 + p1) + (p2 + p3), whatever the launch: a row's bits are those of the other kernels.  Strips are requested ahead
// of the rows they wait for (width 128: all of a layer's; width 512: what the registers hold, the rest a stage ahead).
//
// What bounds it (clock stamps at every workgroup barrier): at width 128 the seven exchanges of a layer, 0.7 to 1.2 us each with what is summed
// in between, 13 us a layer; at width 512 what an XCD takes from the last-level cache, 16.8 MB a layer in 12 us, and the products of
// its 32 units, 7 us for 16 rows, of 25 us a layer.  The decoder at width 512 asks for more registers than there are: 47 spilled (176 bytes of scratch a
// lane) with up to 64 keys, 153 (440) with up to 128, 5 (24) in the encoder with up to 128; at width 128 only the decoder with up to 128 keys, 8 (36).
// Both sides' figures, with the spills in, stand at team_pays in ad_api.cpp.  Not kept: the keys that earlier
// forwards wrote requested ahead (39.0 -> 39.9 us at width 128), FFN1's strips requested in two places, in and beside the attention
// (a branch around loads has them copied, hence waited for, where it ends: 208 -> 310 us at width 512).
//
// Every exchanged row has a place of its own for every layer, all ones until it is written (ad_team_device.h), set back before the team's
// first barrier: at 16 rows of width 512 and six layers 2 MB a team, 0.4 us.  Whoever reads what another XCD writes has seen the arrival of
// all XCDs before: the second XCD of a team, and all where teams share keys, at that barrier, the first XCD after its first layer.
#include <hip/hip_runtime.h>

#include "ad_team_device.h"

namespace ad {

constexpr int kFThreads = 512, kFRows = kTeamF32Rows;

__device__ __forceinline__ f32x4 f32_unit(const float4& a, const float4& b, f32x4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, c, 0, 0, 0);
}
__device__ __forceinline__ float4 as_f4(const uint4& v) { return __builtin_bit_cast(float4, v); }
// units u0 .. u0 + N - 1 (16 k each) of the 16 rows of W [*, K] that are output columns n0 ..; a wave that has no such strip asks for
// nothing (a descriptor of no bytes: zeros without a fetch; a branch around the loads would have them waited for where it ends)
template <int N>
__device__ __forceinline__ void load_units(const float* W, int n0, int K, int u0, int lane, float4 (&w)[N], bool has = true) {
  __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)n0 * K + 16 * u0), 0, has ? 0x7fffffff : 0, 0x00027000);
  const int off = ((lane & 15) * K + 4 * (lane >> 4)) * 4;
#pragma unroll
  for (int u = 0; u < N; ++u) w[u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 64 * u, 0));
}
template <int N>
__device__ __forceinline__ f32x4 dot_units(const float* a_lane, const float4 (&w)[N], f32x4 c) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    c = f32_unit(*(const float4*)(a_lane + 16 * u), w[u], c);
    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (else all operands are read into registers first)
  }
  return c;
}
// N units of which the first R are in w: a unit's registers are refilled as soon as its products are issued
template <int N, int R>
__device__ __forceinline__ f32x4 dot_rolling(const float* a_lane, const float* W, int n0, int K, int u0, int lane, float4 (&w)[R]) {
  f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (N == R) {
    return dot_units<N>(a_lane, w, c);
  } else {
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)n0 * K + 16 * u0), 0, 0x7fffffff, 0x00027000);
    const int off = ((lane & 15) * K + 4 * (lane >> 4)) * 4;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      c = f32_unit(*(const float4*)(a_lane + 16 * u), w[u % R], c);
      if (u + R < N) w[u % R] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 64 * (u + R), 0));
      if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    return c;
  }
}
// a LayerNorm's gains and biases in the layout its rows are held in: 4 lane + 256 j .. (width 512), lane + 64 j (width 128)
template <int D> struct LnRegs { float g[D / 64], b[D / 64]; };
template <int D>
__device__ __forceinline__ void load_ln(const char* g, const char* b, int lane, LnRegs<D>& v) {
  if constexpr (D == 512) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float4 x = gload((const float4*)g + lane + 64 * j), y = gload((const float4*)b + lane + 64 * j);
      v.g[4 * j] = x.x; v.g[4 * j + 1] = x.y; v.g[4 * j + 2] = x.z; v.g[4 * j + 3] = x.w;
      v.b[4 * j] = y.x; v.b[4 * j + 1] = y.y; v.b[4 * j + 2] = y.z; v.b[4 * j + 3] = y.w;
    }
  } else {
    ln_load<2, true>((const float*)g, D, lane, v.g);
    ln_load<2, true>((const float*)b, D, lane, v.b);
  }
}
// rows row0, row0 + 8 (NR of them, clamped to last; pitch in bytes) through LayerNorm into the same rows of At
template <int D, int NR>
__device__ __forceinline__ void stage_ln_rows(TeamWait& tw, const char* src, int pitch, int row0, int last, const LnRegs<D>& v, float* At, int lane) {
  constexpr int LD = D + 4;
  float x[NR][D / 64];
  wait_for(tw, lane, [&]() {
    Seen32 seen;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const unsigned off = (unsigned)min(row0 + 8 * i, last) * pitch;
      if constexpr (D == 512) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint4 u = ld16_l2(src, off + 16 * lane + 1024 * j);
          seen.add(u);
          const float4 f = as_f4(u);
          x[i][4 * j] = f.x; x[i][4 * j + 1] = f.y; x[i][4 * j + 2] = f.z; x[i][4 * j + 3] = f.w;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          x[i][j] = ld4_l2(src, off + 4 * lane + 256 * j);
          seen.m = max(seen.m, __float_as_uint(x[i][j]));
        }
      }
    }
    return seen.all();
  });
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    float mean, rstd;
    if constexpr (D == 512) {
      const float4 xv[2] = {float4{x[i][0], x[i][1], x[i][2], x[i][3]}, float4{x[i][4], x[i][5], x[i][6], x[i][7]}};
      ln_stats4<2>(xv, D, mean, rstd);
    } else {
      ln_stats<2>(x[i], D, lane, mean, rstd);
    }
    float* at = At + (row0 + 8 * i) * LD;
    if constexpr (D == 512) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float4 o;
        o.x = ln_value(x[i][4 * j], mean, rstd, v.g[4 * j], v.b[4 * j]);
        o.y = ln_value(x[i][4 * j + 1], mean, rstd, v.g[4 * j + 1], v.b[4 * j + 1]);
        o.z = ln_value(x[i][4 * j + 2], mean, rstd, v.g[4 * j + 2], v.b[4 * j + 2]);
        o.w = ln_value(x[i][4 * j + 3], mean, rstd, v.g[4 * j + 3], v.b[4 * j + 3]);
        *(float4*)(at + 4 * lane + 256 * j) = o;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) at[lane + 64 * j] = ln_value(x[i][j], mean, rstd, v.g[j], v.b[j]);
    }
  }
}
template <int D>
__device__ __forceinline__ void stage_ln(TeamWait& tw, const char* src, int pitch, int n, const LnRegs<D>& v, float* At, int wave, int lane) {
  if (wave >= n) return;
  if (n > 8) stage_ln_rows<D, 2>(tw, src, pitch, wave, n - 1, v, At, lane);
  else stage_ln_rows<D, 1>(tw, src, pitch, wave, n - 1, v, At, lane);
}
// W floats of rows as they are, into rows of LDW
template <int W, int LDW, int NR>
__device__ __forceinline__ void stage_rows_n(TeamWait& tw, const char* src, int pitch, int row0, int last, float* At, int lane) {
  constexpr int P = (W + 255) / 256;   // 1 KB pieces
  uint4 v[NR][P];
  wait_for(tw, lane, [&]() {
    Seen32 seen;
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int j = 0; j < P; ++j) {
        v[i][j] = ld16_l2(src, (unsigned)min(row0 + 8 * i, last) * pitch + (W < 256 ? min(16 * lane, 4 * W - 16) : 16 * lane + 1024 * j));
        seen.add(v[i][j]);
      }
    return seen.all();
  });
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int j = 0; j < P; ++j)
      if (W >= 256 || 4 * lane < W) *(uint4*)(At + (row0 + 8 * i) * LDW + 4 * lane + 256 * j) = v[i][j];
}
template <int W>
__device__ __forceinline__ void stage_rows(TeamWait& tw, const char* src, int pitch, int n, float* At, int wave, int lane) {
  constexpr int P = W < 1024 ? W : 1024;   // (registers)
  if (wave >= n) return;
#pragma unroll 1
  for (int c = 0; c < W; c += P) {
    if (n > 8) stage_rows_n<P, W + 4, 2>(tw, src + (size_t)wave * pitch + 4 * c, pitch, 0, n - 1 - wave, At + wave * (W + 4) + c, lane);
    else stage_rows_n<P, W + 4, 1>(tw, src + (size_t)wave * pitch + 4 * c, pitch, 0, n - 1 - wave, At + wave * (W + 4) + c, lane);
  }
}

// Attention of a chunk of up to 16 rows, head h, at most 16 NKT keys, by the first four waves; the order of k_attention_f32.
constexpr int kFLds = 132;   // row stride of the scores: four dwords past a multiple of 64 banks
template <int DH, int NKT> struct AttnF { float4 k[NKT / 4][DH / 16]; float v[NKT][4]; };
// (first_new: the first key that this launch writes)
template <int DH, int NKT, bool L2>
__device__ __forceinline__ void attn_request(const float* K, const float* V, int kv0, int nk_all, int D, int h, int wave, int lane, int first_new,
                                             AttnF<DH, NKT>& g, Seen32& seen) {
  const int r = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int t = 0; t < NKT / 4; ++t) {
    const int key = min(16 * (wave + 4 * t) + r, nk_all - 1);
    const unsigned off = ((unsigned)(kv0 + key) * D + h * DH + 4 * kq) * 4;
#pragma unroll
    for (int s = 0; s < DH / 16; ++s) {
      const uint4 u = L2 ? ld16_l2(K, off + 64 * s) : ldg16((const char*)K + off + 64 * s);
      g.k[t][s] = as_f4(u);
      if (L2 && key >= first_new) seen.add(u);
    }
  }
  const int ch = 16 * wave < DH ? 16 * wave : 0;
#pragma unroll
  for (int u = 0; u < NKT; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = min(16 * u + 4 * kq + i, nk_all - 1);
      const unsigned off = ((unsigned)(kv0 + key) * D + h * DH + ch + r) * 4;
      g.v[u][i] = L2 ? ld4_l2(V, off) : gload((const float*)((const char*)V + off));
      if (L2 && key >= first_new) seen.m = max(seen.m, __float_as_uint(g.v[u][i]));
    }
}
// (every wave of the workgroup comes here for the barriers)
template <int DH, int NKT, typename Q>
__device__ __forceinline__ void attn_core(float* S, float* L, const Q& qf, const AttnF<DH, NKT>& g, const float* V, int kv0, int nk_all, int nk_base,
                                          int off, int causal, float scale, int D, char* out, int pitch, int row, int n, int h, int wave, int lane) {
  const int r = lane & 15, kq = lane >> 4, nt = (nk_all + 15) >> 4;
  if (wave < 4) {
#pragma unroll
    for (int t = 0; t < NKT / 4; ++t) {
      const int tile = wave + 4 * t, key = 16 * tile + r;
      if (tile < nt) {
        f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < DH / 16; ++s) s4 = f32_unit(qf[s], g.k[t][s], s4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int nkr = causal ? nk_base + off + 4 * kq + i + 1 : nk_base;
          S[(4 * kq + i) * kFLds + key] = key < nkr ? s4[i] * scale : -INFINITY;
        }
      }
    }
  }
  wg_bar();
  if (wave < 4) {
    float* sr = S + (4 * wave + kq) * kFLds + r;   // row 4 wave + kq, this lane's keys r, r + 16, ..
    float mx = -INFINITY, l = 0.f;
    for (int t = 0; t < nt; ++t) mx = fmaxf(mx, sr[16 * t]);
    mx = row16_max(mx);
    for (int t = 0; t < nt; ++t) {
      const float p = expf(sr[16 * t] - mx);
      l += p;
      sr[16 * t] = p;
    }
    l = row16_sum(l);
    if (r == 0) L[4 * wave + kq] = l;
  }
  wg_bar();
  if (wave < 4 && 16 * wave < DH) {
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NKT; ++u)
      if (u < nt) acc = f32_unit(*(const float4*)(S + r * kFLds + 16 * u + 4 * kq), float4{g.v[u][0], g.v[u][1], g.v[u][2], g.v[u][3]}, acc);
    bool odd = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) odd |= !__builtin_isfinite(acc[i]);
    if (__any(odd)) {   // the product once more, in the same order, with values that are not finite held apart (k_attention_f32)
      const int nk_full = causal ? nk_base + off + 1 : nk_base;
      const unsigned vo = ((unsigned)kv0 * D + h * DH + 16 * wave + r) * 4;
      acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int u = 0; u < nt; ++u) {
        const bool in_part = 16 * (u + 1) > nk_full;
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int key = 16 * u + 4 * kq + i;
          x[i] = ld4_l2(V, vo + (unsigned)min(key, nk_all - 1) * (D * 4));
          if (in_part && (key >= nk_all || !__builtin_isfinite(x[i]))) x[i] = 0.f;
        }
        acc = f32_unit(*(const float4*)(S + r * kFLds + 16 * u + 4 * kq), float4{x[0], x[1], x[2], x[3]}, acc);
        if (!in_part) continue;
#pragma unroll 1
        for (int key = 16 * u; key < min(nk_all, 16 * u + 16); ++key) {
          const float y = ld4_l2(V, vo + (unsigned)key * (D * 4));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int nkr = causal ? nk_base + off + 4 * kq + i + 1 : nk_base;
            if (!__builtin_isfinite(y) && key < nkr) acc[i] += S[(4 * kq + i) * kFLds + key] * y;
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * kq + i < n) put((float*)(out + (size_t)(row + 4 * kq + i) * pitch) + h * DH + 16 * wave + r, acc[i] / L[4 * kq + i]);
  }
}

template <int D, int F, int DH, int NKT, bool DEC>
__global__ __launch_bounds__(kFThreads) void k_team_f32(TeamArgs a) {
  typedef TeamOff<DEC, D, F, 4> O;
  typedef TeamSlotF32<D, F> T;
  constexpr int H = D / DH, LD = D + 4, U = D / 64, UF = F / 64, UR = UF < 16 ? UF : 16;
  constexpr int NS = D / 16, QS = (3 * NS + 63) / 64, FS = (F / 16 + 63) / 64, CS = DH / 32;   // strips: of a width; a quad's of Q, K, V, of FFN1, of a head's queries
  constexpr bool kAll = D == 128;   // all of a layer's strips fit the registers
  constexpr int kAttn = kFRows * LD;   // (floats) behind the row tile: scores, denominators, queries of the cross-attention
  extern __shared__ uint4 team_lds[];
  int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = (int)((xcc_id() - (unsigned)a.xcd0) & 7u);
  if (slot >= a.n_teams * a.stations) return;
  const int team = slot % a.n_teams, station = slot / a.n_teams;
  float* At = (float*)team_lds;
  float* S = At + kAttn;
  float* L = S + 16 * kFLds;
  float* Qt = L + 16;
  f32x4* part = (f32x4*)((char*)team_lds + team_f32_rows_bytes(D, F, DH));   // [quad][strip][quarter][64]
  float* xres = (float*)(part + 2 * 2 * 4 * 64);                   // [16][16]
  TeamChunk* chunks = (TeamChunk*)(xres + 256);
  int* grow = (int*)(chunks + kFRows);
  int* rdst = grow + kFRows;
  int* misc = rdst + kFRows;
  unsigned* gave_up = (unsigned*)(misc + 4);

  unsigned* words = a.words + slot * 64;
  const int n_all = a.row_n[0][team];
  if (threadIdx.x == 256) misc[0] = (int)__hip_atomic_fetch_add(words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x == 64) *gave_up = 0;
  team_lists<kFRows, DEC>(a, team, n_all, 0, chunks, grow, rdst, misc + 1, wave, lane);
  __syncthreads();
  const int idx = __builtin_amdgcn_readfirstlane(misc[0]);
  const int n_chunks = __builtin_amdgcn_readfirstlane(min(misc[1], kFRows));
  if (idx >= kTeamMembers) {   // more workgroups on the XCD than members: not how this grid is dealt out
    if (threadIdx.x == 0) __hip_atomic_store(a.fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  constexpr int CPR = kTeamMembers / H;
  const int c_first = idx / H, h = idx % H, n = n_all;
  const int quad = wave >> 2, quarter = wave & 3, g0 = 2 * idx + quad;   // a quad's strips: g0, g0 + 64, ..
  int r = lane & 15, kq = lane >> 4;
  // what is computed from the lane is computed where it is used, not kept in registers over the whole stack of layers
  auto fresh = [&]() {
    asm volatile("" : "+v"(lane));
    r = lane & 15; kq = lane >> 4;
  };
  TeamWait tw;
  tw.fail = a.fail; tw.gave_up = gave_up; tw.off = false;
  const bool far_hop = a.stations > 1, far_kv = a.shared != 0;
  auto place = [&](int l) { return a.slots + (size_t)(l * 8 + team) * T::kBytes; };
  auto hop = [&](int l) { return a.hop + (size_t)l * kTeamHopBytes + team * (kTeamMaxRows * kTeamD * 4); };
  float* Kc = (float*)a.K;
  float* Vc = (float*)a.V;

  // places to be written, this member's share
#pragma unroll 1
  for (int l = station; l < a.layers; l += a.stations) {
    char* p = place(l);
    for (int i = idx * kFThreads + threadIdx.x; i < n * (T::kRow / 16); i += kTeamMembers * kFThreads) unwrite16(p, 16 * i);
    if (l + 1 < a.layers)
      for (int i = idx * kFThreads + threadIdx.x; i < n * (D / 4); i += kTeamMembers * kFThreads) {
        if (far_hop) unwrite16_far(hop(l), 16 * i);
        else unwrite16(hop(l), 16 * i);
      }
    for (int i = idx * kFThreads + threadIdx.x; i < 2 * n * (D / 4); i += kTeamMembers * kFThreads) {
      const int m = i / (D / 2), c = i % (D / 2);
      char* base = (char*)(c < D / 4 ? Kc : Vc) + (size_t)l * a.kv_stride;
      const unsigned off = (unsigned)rdst[m] * (D * 4) + (c % (D / 4)) * 16;
      if (far_kv) unwrite16_far(base, off);
      else unwrite16(base, off);
    }
  }
  team_put_ready();
  // the embedded rows
  if (station == 0) {
    for (int i = threadIdx.x; i < n * (D / 4); i += kFThreads) {
      const int m = i / (D / 4), c = i % (D / 4);
      *(uint4*)(At + m * LD + 4 * c) = ldg16(a.x + (size_t)grow[m] * D + 4 * c);
    }
    if (idx < NS && threadIdx.x < 16 * n) xres[threadIdx.x] = gload(a.x + (size_t)grow[threadIdx.x >> 4] * D + idx * 16 + (threadIdx.x & 15));
  }
  wg_bar();
  if (wave == 7) {
    team_arrive(a, words, lane);
    team_wait_count(a, words + 32, kTeamMembers, gave_up, lane);
    if (station > 0 || far_kv) team_wait_count(a, a.words + 48, a.n_teams * a.stations, gave_up, lane);
  }
  wg_bar();
  tw.off = __builtin_amdgcn_readfirstlane(__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0;

  auto a_lane = [&]() { return At + r * LD + 4 * kq + 16 * U * quarter; };
  auto mine = [&](int s) { return part + ((quad * 2 + s) * 4) * 64 + lane; };
  auto total = [&](int s) { const f32x4* p = mine(s); return (p[0] + p[64]) + (p[128] + p[192]); };
  // this quad's strip of a product whose strips are the members' (quad 0), and its result: wave 0
  auto one_strip = [&](const float4 (&w)[U]) {
    if (quad == 0 && idx < NS) mine(0)[quarter * 64] = dot_units<U>(a_lane(), w, f32x4{0.f, 0.f, 0.f, 0.f});
    wg_bar();
  };
#pragma unroll 1
  for (int l = station; l < a.layers; l += a.stations) {
    float4 wq[QS][U], wo[U], wc[CS][U], wo2[U], w1[FS][U], w2[UR];
    float bq[QS], b1[FS], bc[CS], b_o, b_o2, b_2;
    const char* wl = a.w + (size_t)l * O::kLayerBytes;
    char* p = place(l);
    const float* Kl = (const float*)((const char*)Kc + (size_t)l * a.kv_stride);
    const float* Vl = (const float*)((const char*)Vc + (size_t)l * a.kv_stride);
    const bool attends = c_first < n_chunks, has_one = quad == 0 && idx < NS;   // a chunk's member; a quad with a strip of a product of width D
    const int col = min(idx, NS - 1);
    auto request_ffn1 = [&]() {
#pragma unroll
      for (int j = 0; j < FS; ++j) {
        const int s = min(g0 + 64 * j, F / 16 - 1);
        b1[j] = gload((const float*)(wl + O::b1) + 16 * s + r);
        load_units((const float*)(wl + O::w1), 16 * s, D, U * quarter, lane, w1[j]);
      }
    };
    auto request_out2 = [&]() {
      b_o2 = gload((const float*)(wl + O::cbo) + 16 * col + r);
      load_units((const float*)(wl + O::cwo), 16 * col, D, U * quarter, lane, wo2, has_one);
    };
    auto request_ffn2 = [&]() {
      b_2 = gload((const float*)(wl + O::b2) + 16 * col + r);
      load_units((const float*)(wl + O::w2), 16 * col, F, UF * quarter, lane, w2, has_one);
    };
    LnRegs<D> ln;
    // ---------------------------------------------------------------- Q, K, V
    fresh();
    if (l > 0) load_ln<D>(wl - O::kLayerBytes + O::ln_lg, wl - O::kLayerBytes + O::ln_lb, lane, ln);
#pragma unroll
    for (int j = 0; j < QS; ++j) {
      const int s = min(g0 + 64 * j, 3 * NS - 1);
      bq[j] = gload((const float*)(wl + O::bqkv) + 16 * s + r);
      load_units((const float*)(wl + O::wqkv), 16 * s, D, U * quarter, lane, wq[j]);
    }
    b_o = gload((const float*)(wl + O::bo) + 16 * col + r);
    load_units((const float*)(wl + O::wo), 16 * col, D, U * quarter, lane, wo, has_one);
    if (DEC) {
#pragma unroll
      for (int j = 0; j < CS; ++j) {
        bc[j] = gload((const float*)(wl + O::cbq) + h * DH + 16 * (quad * CS + j) + r);
        load_units((const float*)(wl + O::cwq), h * DH + 16 * (quad * CS + j), D, U * quarter, lane, wc[j], attends);
      }
    }
    auto request_all = [&]() {
      if (DEC) request_out2();
      request_ffn1(); request_ffn2();
    };
    if (l > 0) stage_ln<D>(tw, hop(l - 1), D * 4, n, ln, At, wave, lane);
    wg_bar();
#pragma unroll
    for (int j = 0; j < QS; ++j) mine(j)[quarter * 64] = dot_units<U>(a_lane(), wq[j], f32x4{0.f, 0.f, 0.f, 0.f});
    wg_bar();
    if (quarter < QS) {
      const int j = quarter, s = g0 + 64 * j;
      if (s < 3 * NS) {
        const f32x4 v = total(j);
        const float bias = j == 0 ? bq[0] : bq[QS - 1];
        const int which = s / NS, col = (s % NS) * 16 + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = 4 * kq + i;
          if (m < n) {
            if (which == 0) {
              put((float*)(p + m * T::kRow + T::q) + col, v[i] + bias);
            } else {
              float* to = (float*)((char*)(which == 1 ? Kc : Vc) + (size_t)l * a.kv_stride) + (size_t)rdst[m] * D + col;
              if (far_kv) put_far(to, v[i] + bias);
              else put(to, v[i] + bias);
            }
          }
        }
      }
    }
    if (l > 0 && idx < NS && threadIdx.x >= 256) xres[threadIdx.x - 256] = At[((threadIdx.x - 256) >> 4) * LD + idx * 16 + (threadIdx.x & 15)];
    wg_bar();
    if (kAll) request_all();   // (the first product's strips ahead of all others; these have the attention's time)
    // ---------------------------------------------------------------- self-attention
    fresh();
#pragma unroll 1
    for (int c = c_first; c < n_chunks; c += CPR) {
      const TeamChunk ch = chunk_at(chunks, c);
      const int nk_all = min(ch.causal ? ch.nk_base + ch.off + ch.n : ch.nk_base, 16 * NKT);
      const int first_new = ch.causal ? ch.nk_base : 0;
      float4 qf[DH / 16];
      AttnF<DH, NKT> g;
      if (wave < 4) {
        wait_for(tw, lane, [&]() {
          Seen32 seen;
          const unsigned off = (unsigned)(ch.row + min(r, ch.n - 1)) * T::kRow + T::q + (h * DH + 4 * kq) * 4;
#pragma unroll
          for (int s = 0; s < DH / 16; ++s) {
            const uint4 u = ld16_l2(p, off + 64 * s);
            seen.add(u);
            qf[s] = as_f4(u);
          }
          attn_request<DH, NKT, true>(Kl, Vl, ch.kv_self, nk_all, D, h, wave, lane, first_new, g, seen);
          return seen.all();
        });
      }
      attn_core<DH, NKT>(S, L, qf, g, Vl, ch.kv_self, nk_all, ch.nk_base, ch.off, ch.causal, a.scale, D, p + T::att, T::kRow, ch.row, ch.n, h, wave, lane);
      wg_bar();
    }
    if (!DEC && !kAll) request_ffn1();
    // ---------------------------------------------------------------- output projection + residual
    fresh();
    if (DEC) load_ln<D>(wl + O::ln1g, wl + O::ln1b, lane, ln);
    else load_ln<D>(wl + O::ln_fg, wl + O::ln_fb, lane, ln);
    stage_rows<D>(tw, p + T::att, T::kRow, n, At, wave, lane);
    wg_bar();
    one_strip(wo);
    if (wave == 0 && idx < NS) {
      const f32x4 v = total(0);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * kq + i < n) put((float*)(p + (4 * kq + i) * T::kRow + T::s1) + idx * 16 + r, v[i] + b_o + xres[(4 * kq + i) * 16 + r]);
    }
    wg_bar();
    if constexpr (DEC) {
      if (!kAll) request_out2();
      const float* Km = (const float*)((const char*)a.Km + (size_t)l * a.m_stride);
      const float* Vm = (const float*)((const char*)a.Vm + (size_t)l * a.m_stride);
      // -------------------------------------------------------------- cross-attention with its query projection
      fresh();
#pragma unroll 1
      for (int c = c_first; c < n_chunks; c += CPR) {
        const TeamChunk ch = chunk_at(chunks, c);
        const int nk_all = min(ch.nk_cross, 16 * NKT);
        AttnF<DH, NKT> g;
        Seen32 none;
        if (wave < 4) attn_request<DH, NKT, false>(Km, Vm, ch.kv_cross, nk_all, D, h, wave, lane, 0, g, none);
        stage_ln<D>(tw, p + T::s1 + ch.row * T::kRow, T::kRow, ch.n, ln, At, wave, lane);
        wg_bar();
#pragma unroll
        for (int j = 0; j < CS; ++j) mine(j)[quarter * 64] = dot_units<U>(a_lane(), wc[j], f32x4{0.f, 0.f, 0.f, 0.f});
        wg_bar();
        if (quarter < CS) {
          const f32x4 v = total(quarter);
          const float bias = quarter == 0 ? bc[0] : bc[CS - 1];
#pragma unroll
          for (int i = 0; i < 4; ++i) Qt[(4 * kq + i) * (DH + 4) + 16 * (quad * CS + quarter) + r] = v[i] + bias;
        } else if (wave == 7) {   // the rows of this head's channels, for the residual of the later projection
#pragma unroll 1
          for (int i = lane; i < ch.n * DH; i += 64)
            put((float*)(p + (ch.row + i / DH) * T::kRow + T::xr) + h * DH + i % DH, At[(i / DH) * LD + h * DH + i % DH]);
        }
        wg_bar();
        float4 qf[DH / 16];
#pragma unroll
        for (int s = 0; s < DH / 16; ++s) qf[s] = *(const float4*)(Qt + min(r, ch.n - 1) * (DH + 4) + 16 * s + 4 * kq);
        attn_core<DH, NKT>(S, L, qf, g, Vm, ch.kv_cross, nk_all, nk_all, 0, 0, a.scale, D, p + T::att2, T::kRow, ch.row, ch.n, h, wave, lane);
        wg_bar();
      }
      // -------------------------------------------------------------- output projection + residual
      fresh();
      if (!kAll) request_ffn1();
      stage_rows<D>(tw, p + T::att2, T::kRow, n, At, wave, lane);
      wg_bar();
      one_strip(wo2);
      if (wave == 0 && idx < NS) {
        float res[4];
        wait_for(tw, lane, [&]() {
          Seen32 seen;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            res[i] = ld4_l2(p, (unsigned)min(4 * kq + i, n - 1) * T::kRow + T::xr + (idx * 16 + r) * 4);
            seen.m = max(seen.m, __float_as_uint(res[i]));
          }
          return seen.all();
        });
        const f32x4 v = total(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * kq + i < n) put((float*)(p + (4 * kq + i) * T::kRow + T::s2) + idx * 16 + r, v[i] + b_o2 + res[i]);
      }
      wg_bar();
      load_ln<D>(wl + O::ln_fg, wl + O::ln_fb, lane, ln);
    }
    if (!kAll) request_ffn2();
    // ---------------------------------------------------------------- FFN1
    fresh();
    stage_ln<D>(tw, p + (DEC ? T::s2 : T::s1), T::kRow, n, ln, At, wave, lane);
    wg_bar();
#pragma unroll
    for (int j = 0; j < FS; ++j) mine(j)[quarter * 64] = dot_units<U>(a_lane(), w1[j], f32x4{0.f, 0.f, 0.f, 0.f});
    wg_bar();
    if (quarter < FS && g0 + 64 * quarter < F / 16) {
      const f32x4 v = total(quarter);
      const float bias = quarter == 0 ? b1[0] : b1[FS - 1];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * kq + i < n) put((float*)(p + (4 * kq + i) * T::kRow + T::f) + 16 * (g0 + 64 * quarter) + r, fmaxf(v[i] + bias, 0.f));
    }
    if (idx < NS && threadIdx.x >= 256) xres[threadIdx.x - 256] = At[((threadIdx.x - 256) >> 4) * LD + idx * 16 + (threadIdx.x & 15)];
    wg_bar();
    // ---------------------------------------------------------------- FFN2 + residual
    fresh();
    stage_rows<F>(tw, p + T::f, T::kRow, n, At, wave, lane);
    wg_bar();
    if (quad == 0 && idx < NS) mine(0)[quarter * 64] = dot_rolling<UF>(At + r * (F + 4) + 4 * kq + 16 * UF * quarter, (const float*)(wl + O::w2), 16 * idx, F, UF * quarter, lane, w2);
    wg_bar();
    if (wave == 0 && idx < NS) {
      const f32x4 v = total(0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = 4 * kq + i;
        if (m < n) {
          const float y = v[i] + b_2 + xres[m * 16 + r];
          if (l + 1 == a.layers) gstore(a.s + (size_t)grow[m] * D + idx * 16 + r, y);
          else if (far_hop) put_far((float*)hop(l) + m * D + idx * 16 + r, y);
          else put((float*)hop(l) + m * D + idx * 16 + r, y);
        }
      }
    }
    // The next rows come from the second XCD: it has set their places back.  (Verify forward of width 512, us, without a wait / here / at the
    // first barrier: 1 row 209.0 / 210.1 / 210.4, 4 sequences of 8 rows 250.0 / 251.7 / 254.2, of 16 rows 288.2 / 290.0 / 290.7.)
    if (wave == 7 && l == 0 && far_hop) team_wait_count(a, a.words + 48, a.n_teams * a.stations, gave_up, lane);
    wg_bar();
  }
}

static size_t team_f32_lds(int D, int F, int DH) {
  const size_t b = team_f32_rows_bytes(D, F, DH) + 2 * 2 * 4 * 64 * 16 + 256 * 4 + kFRows * sizeof(TeamChunk) + 2 * kFRows * 4 + 64;
  return b > 84 * 1024 ? b : 84 * 1024;   // (more than half a CU's: one member per CU)
}
template <typename Fn>
static void each_team_f32(int D, bool dec, const Fn& f) {
  if (D == 128) {
    if (dec) { f(4, &k_team_f32<128, 512, 32, 4, true>); f(8, &k_team_f32<128, 512, 32, 8, true>); }
    else { f(4, &k_team_f32<128, 512, 32, 4, false>); f(8, &k_team_f32<128, 512, 32, 8, false>); }
  } else {
    if (dec) { f(4, &k_team_f32<512, 2048, 64, 4, true>); f(8, &k_team_f32<512, 2048, 64, 8, true>); }
    else { f(4, &k_team_f32<512, 2048, 64, 4, false>); f(8, &k_team_f32<512, 2048, 64, 8, false>); }
  }
}
static size_t lds_of(int D) { return D == 128 ? team_f32_lds(128, 512, 32) : team_f32_lds(512, 2048, 64); }
bool prepare_team_f32(int D, bool dec) {
  bool ok = true;
  each_team_f32(D, dec, [&](int, void (*k)(TeamArgs)) { ok = ok && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of(D)) == hipSuccess; });
  if (!ok) (void)hipGetLastError();
  return ok;
}
void launch_team_f32(const TeamArgs& a, int D, bool dec, int max_keys, hipStream_t s) {
  const int nkt = max_keys <= 64 ? 4 : 8;
  each_team_f32(D, dec, [&](int nk, void (*k)(TeamArgs)) {
    if (nk == nkt) k<<<8 * kTeamMembers, kFThreads, lds_of(D), s>>>(a);
  });
}

}  // namespace ad

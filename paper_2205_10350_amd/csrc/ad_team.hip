// A whole stack of layers in one launch: the rows of a few sequences stay on one XCD.
//
// A forward of a few rows as a launch per stage is a chain of 32-45 launches of 3-8 us whose products take 0.1 us each:
// what they spend is the launch boundary (2.4 us), the trip of the rows from another XCD's writes and the fetch of
// weights that could not be requested earlier.  Here the 32 compute units of an XCD form a team: one workgroup per CU,
// resident for the whole stack, the strips of the next stages requested while the present one's results are on their way.
// Rows pass from stage to stage through the XCD's L2 without a barrier: whoever needs a row reads it until it is there (0.27 us one way
// between two waves of an XCD, 0.45 from a store to the row in the reader's LDS; a barrier over the team with the trip behind it took 1.4).
//
// Sequences of up to 16 rows (a row tile) get a team each; longer ones are cut into pieces of at most 16 rows, a team each, where there are
// XCDs for all: pieces read each other's keys and values (agent-scope stores past the writer's L2, 0.5-0.6 us one way), all else of a row is its own.
// Where XCDs are left over a team has two and they take turns over the layers: one requests a layer's strips (an XCD streams a
// layer's 7.3 MB from the last-level cache in 5.7 us) while the other works on the layer before, and the rows go across as keys do.  (Three or
// more: no faster, 81 us of layers at 1 row with two or three, 83 with six: all members of all XCDs have to be there first.)  Verify forward, us,
// one XCD a team / two, teams of 1, 8, 16 rows: one team 85, 99, 111 / 80, 94, 105; two 86, 99, 112 / 82, 97, 109; three 89, 104, 116 / 83, 98, 109; four
// 97, 110, 121 / 88, 103, 114.
//
// Registers (512 threads, 256 a lane at most): 229 to 256.  Only k_team<1, 8, true, true> (two XCDs, 65 to 128 keys) spills vector registers, 16 of
// them (40 bytes of scratch a lane), once a layer; it has no place for the older keys requested ahead either (kEarly).
//
// What bounds it (clock stamps at every workgroup barrier, base model, a layer of 11.5 / 14 / 16 us at 1 / 8 / 25 rows on two XCDs a team):
// products 2.6 us a layer (FFN2's chain through four slices 0.9, the others 0.25-0.35 each), seven exchanges of 0.4 to 1.2, the two
// attentions 2.2, LayerNorms 0.9; with one XCD a team (32 sequences) strips on their way delay the exchanges by 2 to 3 us a layer.
// Verify forward of the base model, us, with barriers between the stages on one XCD / this way: 1 sequence of 1, 4, 8, 16, 17,
// 25, 32 rows 139, 143, 144, 150, 167, 177, 177 / 80, 89, 94, 105, 106, 110, 109; 8 sequences of 25 rows 207 / 165; 32 sequences of 1, 2, 4, 6, 8 rows
// 164, 166, 176, 196, 206 / 111, 117, 131, 157, 170.  A launch per stage: 159-172, 172, 175, 180, 178, 181, 183; 222; 177, 182, 195, 221, 231
// (the launches replayed as a graph; a call shape's first two appearances go out launch by launch in 223).  33 to 64 rows on one XCD, four row
// tiles, were 240 and more / 184-191 with barriers: hence at most 32 rows a team.
//
// Stages of a layer: QKV | self-attention | output projection | cross-attention with its query projection | output
// projection | FFN1 | FFN2 (the encoder without the middle two).  Members of a team split the columns of a product
// (16-column strips), every member normalises or copies the rows it multiplies into LDS.
//
// Every value is computed as the launch-per-stage kernels compute it (k ascending, 32 at a time, one accumulator; the
// LayerNorm of ad_device.h; attention sums in the same order over keys), so a row's bits do not depend on which path
// serves it.
//
// Exchanged rows are read with loads that miss the vector cache (sc1): a CU's L1 may hold the row of an earlier layer.
// Waiting is bounded everywhere: a team that is not complete within form_ticks, or a row that takes kWaitTicks,
// sets the fail word, the remaining waits return at once, and the caller runs the launches instead.
#include <hip/hip_runtime.h>

#include "ad_team_device.h"

namespace ad {

constexpr int kGW = 4, kTW = 2 * kGW;          // two groups of four waves
constexpr int kTeamThreads = 64 * kTW;
constexpr int kTD = kTeamD, kTF = kTeamF, kTH = kTD / 64;
constexpr int kTLd = kTD + 16;                 // row stride in LDS (elements): 32 bytes past a multiple of 64
constexpr int kSlices = kTF / kTD;             // 512-k slices of FFN2

// barrier over the four waves of a group, through a count in LDS: the other group may be held up by its requests meanwhile
__device__ __forceinline__ void group_wait(unsigned* count, unsigned target) {
  while (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target) {}
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void group_bar(unsigned* count, unsigned& target, int lane) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  target += kGW;
  if (lane == 0) (void)__hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  group_wait(count, target);
}
// a value the compiler cannot see through: what is computed from it is computed where it is used, not kept in registers
// over the whole stack of layers
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ int here_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// the 16 weight fragments (512 k) of the 16-column strip at column n0 of W [*, K], from step u0 (one address register for all of them)
template <int U0 = 0, int U1 = 16>
__device__ __forceinline__ void load_strip(const bf16_t* W, int n0, int K, int u0, int lane, uint4 (&b)[16]) {
  __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)n0 * K + u0 * 512), 0, 16384, 0x00027000);
#pragma unroll
  for (int u = U0; u < U1; ++u) b[u] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, 16 * lane, 1024 * u, 0));
}
// T tiles of 16 x 16 over 512 k, added to acc, a quarter of the operands in registers at a time and the next quarter on its way (where two
// sets of strips fill them)
template <int T>
__device__ __forceinline__ void mm16_lean(const bf16_t* a_lane, const uint4 (&b)[16], f32x4 (&acc)[T]) {
  constexpr int U = 4 / T;
  uint4 af[2][T][U];
  auto read = [&](int u0, uint4 (&f)[T][U]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) f[t][u] = *(const uint4*)(a_lane + t * 16 * kTLd + 32 * (u0 + u));
  };
  read(0, af[0]);
  read(U, af[1]);
#pragma unroll
  for (int g = 0; g < 16 / U; ++g) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[g & 1][t][u]), __builtin_bit_cast(bf16x8, b[g * U + u]), acc[t], 0, 0, 0);
    if (g + 2 < 16 / U) read((g + 2) * U, af[g & 1]);
  }
  __builtin_amdgcn_sched_barrier(0);
}
// The same with the operands of 16 / T steps in registers, read well before the products: left to itself the compiler puts each read next to
// its use and the chain waits for LDS sixteen times (0.7 us instead of 0.3).  ready(): called with the first reads on their way.
template <int T, typename F = NoOp>
__device__ __forceinline__ void mm16(const bf16_t* a_lane, const uint4 (&b)[16], f32x4 (&acc)[T], const F& ready = F{}) {
  constexpr int U = 16 / T;
#pragma unroll
  for (int u0 = 0; u0 < 16; u0 += U) {
    uint4 af[T][U];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) af[t][u] = *(const uint4*)(a_lane + t * 16 * kTLd + 32 * (u0 + u));
    if (u0 == 0) ready();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[t][u]), __builtin_bit_cast(bf16x8, b[u0 + u]), acc[t], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int T>
__device__ __forceinline__ void zero(f32x4 (&acc)[T]) {
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// A LayerNorm's gains and biases go through LDS, [2][512]: a wave of group B brings a quarter (every wave bringing all of them for its
// own rows was a quarter of all a CU requested)
__device__ __forceinline__ uint4 load_ln(const float* g, const float* b, int gw, int lane) {
  return ldg16((gw < 2 ? g : b) + 256 * (gw & 1) + 4 * lane);
}
__device__ __forceinline__ void keep_ln(float* lnv, const uint4& v, int gw, int lane) { *(uint4*)(lnv + 256 * gw + 4 * lane) = v; }
// Rows row0, row0 + step, .. (NR of them; local indices, clamped to `last`) through LayerNorm into the same rows of At;
// xres (nullable): the fp32 values of this member's 16 columns, the residual of its later strip; xr (nullable): those of head h's
// 64 columns, for the others.
template <int NR>
__device__ __forceinline__ void stage_ln_rows(TeamWait& tw, const float* s, int row0, int step, int last, const float* lnv,
                                              bf16_t* At, float* xres, int idx, float* xr, int h, int lane) {
  if (row0 > last) return;
  float4 xv[NR][2], gv[2], bv[2];
  s += (size_t)row0 * kTD;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    gv[j] = *(const float4*)(lnv + 4 * lane + 256 * j);
    bv[j] = *(const float4*)(lnv + kTD + 4 * lane + 256 * j);
  }
  auto load = [&](int i, Seen32& seen) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint4 u = ld16_l2(s, (unsigned)min(step * i, last - row0) * (kTD * 4) + 16 * lane + 1024 * j);
      xv[i][j] = float4{__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w)};
      seen.add(u);
    }
  };
  if (NR > 2) wait_for(tw, lane, [&]() { Seen32 seen; load(NR - 1, seen); return seen.all(); });   // (the others are there about then)
  wait_for(tw, lane, [&]() {
    Seen32 seen;
#pragma unroll
    for (int i = 0; i < NR; ++i) load(i, seen);
    return seen.all();
  });
  float mean[NR], rstd[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) ln_stats4<2>(xv[i], kTD, mean[i], rstd[i]);
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float4& o = xv[i][j];
      o = float4{ln_value(o.x, mean[i], rstd[i], gv[j].x, bv[j].x), ln_value(o.y, mean[i], rstd[i], gv[j].y, bv[j].y),
                 ln_value(o.z, mean[i], rstd[i], gv[j].z, bv[j].z), ln_value(o.w, mean[i], rstd[i], gv[j].w, bv[j].w)};
      *(uint2*)(At + (row0 + step * i) * kTLd + 4 * lane + 256 * j) = uint2{f2bf_pair(o.x, o.y), f2bf_pair(o.z, o.w)};
    }
  if (xres && (lane >> 2) == (idx & 15)) {
    float* xp = xres + row0 * 16 + 4 * (lane & 3);
    if (idx < 16) {
#pragma unroll
      for (int i = 0; i < NR; ++i) *(float4*)(xp + step * i * 16) = xv[i][0];
    } else {
#pragma unroll
      for (int i = 0; i < NR; ++i) *(float4*)(xp + step * i * 16) = xv[i][1];
    }
  }
  if (xr && (lane >> 4) == (h & 3)) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (row0 + step * i <= last) {
        const float4 o = h < 4 ? xv[i][0] : xv[i][1];
        gstore((uint4*)(xr + (size_t)(row0 + step * i) * kTD + (h >> 2) * 256 + 4 * lane), uint4{written(o.x), written(o.y), written(o.z), written(o.w)});
      }
  }
}
// all rows of the team: wave w takes rows w, w + 8, ..; the last round of eight is left out where none of its rows exists
// (a row costs a wave 0.15 us of vector instructions, and every member normalises every row)
template <int NR>
__device__ __forceinline__ void stage_ln(TeamWait& tw, const float* s, int n, const float* lnv,
                                         bf16_t* At, float* xres, int idx, int wave, int lane) {
  if (n > kTW * (NR - 1)) stage_ln_rows<NR>(tw, s, wave, kTW, n - 1, lnv, At, xres, idx, nullptr, 0, lane);
  else stage_ln_rows<NR - 1>(tw, s, wave, kTW, n - 1, lnv, At, xres, idx, nullptr, 0, lane);
}
// the up to 16 rows of a chunk
__device__ __forceinline__ void stage_ln_chunk(TeamWait& tw, const float* s, int n, const float* lnv,
                                               bf16_t* At, float* xr, int h, int wave, int lane) {
  if (n > kTW) stage_ln_rows<2>(tw, s, wave, kTW, n - 1, lnv, At, nullptr, 0, xr, h, lane);
  else stage_ln_rows<1>(tw, s, wave, kTW, n - 1, lnv, At, nullptr, 0, xr, h, lane);
}
// 1 KB pieces of NR bf16 rows, row0, row0 + step, .. of src (piece of row m at m * pitch + off), into rows of 528 at dst
template <int NR>
__device__ __forceinline__ void stage_pieces(TeamWait& tw, const bf16_t* src, unsigned pitch, unsigned off, int row0, int step,
                                             int last, bf16_t* dst, int lane) {
  if (row0 > last) return;
  uint4 v[NR];
  unsigned o[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) o[i] = (unsigned)min(row0 + step * i, last) * pitch + off;
  if (NR > 2) wait_for(tw, lane, [&]() { Seen16 seen; seen.add(v[NR - 1] = ld16_l2(src, o[NR - 1] + 16 * lane)); return seen.all(); });
  wait_for(tw, lane, [&]() {
    Seen16 seen;
#pragma unroll
    for (int i = 0; i < NR; ++i) v[i] = ld16_l2(src, o[i] + 16 * lane);
#pragma unroll
    for (int i = 0; i < NR; ++i) seen.add(v[i]);
    return seen.all();
  });
#pragma unroll
  for (int i = 0; i < NR; ++i) *(uint4*)(dst + (row0 + step * i) * kTLd + 8 * lane) = v[i];
}
// all rows [*, 512] of the team
template <int NR>
__device__ __forceinline__ void stage_rows(TeamWait& tw, const bf16_t* src, int n, bf16_t* At, int wave, int lane) {
  if (n > kTW * (NR - 1)) stage_pieces<NR>(tw, src, kTD * 2, 0, wave, kTW, n - 1, At, lane);
  else stage_pieces<NR - 1>(tw, src, kTD * 2, 0, wave, kTW, n - 1, At, lane);
}

// the embedded rows (written before this launch)
template <int NR>
__device__ __forceinline__ void stage_first(const bf16_t* src, const int* grow, int n, bf16_t* At, int wave, int lane) {
  uint4 v[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) v[i] = ldg16(src + (size_t)__builtin_amdgcn_readfirstlane(grow[min(wave + kTW * i, n - 1)]) * kTD + 8 * lane);
#pragma unroll
  for (int i = 0; i < NR; ++i) *(uint4*)(At + (wave + kTW * i) * kTLd + 8 * lane) = v[i];
}
// the first layer's residual, this member's 16 columns of the embedded rows
template <int ROWS>
__device__ __forceinline__ void stage_first_residual(const float* x, const int* grow, int n, float* xres, int idx, int wave, int lane) {
#pragma unroll
  for (int p = 0; p < (ROWS + 31) / 32; ++p) {
    const int row = 32 * p + wave * 4 + (lane >> 4);
    if (row < n) xres[row * 16 + (lane & 15)] = gload(x + (size_t)grow[row] * kTD + idx * 16 + (lane & 15));
  }
}
// FFN2's operand as [slice][row][528]: a wave takes the rows par, par + 2, .. of slice sl
template <int ROWS>
__device__ __forceinline__ void stage_ffn(TeamWait& tw, const bf16_t* f, int n, bf16_t* At, int sl, int par, int lane) {
  bf16_t* dst = At + sl * ROWS * kTLd;
  if constexpr (ROWS == 16) {
    if (n > 8) stage_pieces<8>(tw, f, kTF * 2, sl * 1024, par, 2, n - 1, dst, lane);
    else if (n > 2) stage_pieces<4>(tw, f, kTF * 2, sl * 1024, par, 2, n - 1, dst, lane);
    else stage_pieces<1>(tw, f, kTF * 2, sl * 1024, par, 2, n - 1, dst, lane);
  } else {
    if (n > 24) stage_pieces<16>(tw, f, kTF * 2, sl * 1024, par, 2, n - 1, dst, lane);
    else stage_pieces<12>(tw, f, kTF * 2, sl * 1024, par, 2, n - 1, dst, lane);
  }
}
// places of this member's next results, set back (a wave; offsets in bytes)
// NP pieces of 16 bytes a row, rows row0, row0 + 1, ..
template <int NP>
__device__ __forceinline__ void unwrite_rows(void* base, unsigned pitch, unsigned off, int row0, int count, int lane) {
#pragma unroll 1
  for (int m = lane / NP; m < count; m += 64 / NP) unwrite16(base, (unsigned)(row0 + m) * pitch + off + (lane % NP) * 16);
}

// One attention problem's chunk of up to 16 rows, head h, at most 16 NKT keys, by the four waves of a group: wave w holds
// the score tiles of keys 16 w .. and 16 (w + 4) .., the waves' maxima and the unrounded exponentials go through LDS,
// every wave sums the denominators in key order and computes 16 output columns.  Same order as attn_tiles_mfma: a score is
// one chain over the head width, a lane's denominator adds its keys in ascending order, the output is one chain over the keys.
struct AttnLds { bf16_t* Vt; bf16_t* Pt; f32x4* Pf; float* xmax; unsigned* count; };
template <int NKT> struct AttnDims { static constexpr int LDV = 16 * NKT + 16, VP = NKT * 16 * 8 / (64 * kGW), KT = NKT / kGW; };
template <int NKT> struct AttnRegs { uint4 kf[AttnDims<NKT>::KT][2], vr[AttnDims<NKT>::VP]; };
// (false: a key or value of the keys first_new.. is not written yet)
// (own keys: lo is first_new where the older ones are there already, else 0)
template <int NKT, bool L2>
__device__ __forceinline__ bool attn_request(const bf16_t* K, const bf16_t* V, int kv0, int nk_all, int h, int wave, int lane, AttnRegs<NKT>& g, int lo = 0, int first_new = 0) {
  const int r = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int t = 0; t < AttnDims<NKT>::KT; ++t) {
    const unsigned off = (unsigned)(kv0 + min(max(16 * (wave + kGW * t) + r, lo), nk_all - 1)) * (kTD * 2) + (h * 64 + kq * 8) * 2;
#pragma unroll
    for (int s = 0; s < 2; ++s) g.kf[t][s] = L2 ? ld16_l2(K, off + 64 * s) : ldg16((const char*)K + off + 64 * s);
  }
#pragma unroll
  for (int it = 0; it < AttnDims<NKT>::VP; ++it) {
    const int i = (wave * 64 + lane) + 64 * kGW * it, t = i % (16 * NKT), c = i / (16 * NKT);   // key t, channels 8 c ..
    const unsigned off = (unsigned)(kv0 + min(max(t, lo), nk_all - 1)) * (kTD * 2) + (h * 64 + c * 8) * 2;
    g.vr[it] = L2 ? ld16_l2(V, off) : ldg16((const char*)V + off);
  }
  if (!L2) return true;
  Seen16 seen;
#pragma unroll
  for (int t = 0; t < AttnDims<NKT>::KT; ++t)
#pragma unroll
    for (int s = 0; s < 2; ++s) seen.add(g.kf[t][s], min(16 * (wave + kGW * t) + r, nk_all - 1) >= first_new);
#pragma unroll
  for (int it = 0; it < AttnDims<NKT>::VP; ++it) seen.add(g.vr[it], min(((wave * 64 + lane) + 64 * kGW * it) % (16 * NKT), nk_all - 1) >= first_new);
  return seen.all();
}
// the keys ahead of first_new from e
template <int NKT>
__device__ __forceinline__ void attn_older(const AttnRegs<NKT>& e, int first_new, int wave, int lane, AttnRegs<NKT>& g) {
  auto pick = [](bool older, const uint4& x, uint4& y) { y = uint4{older ? x.x : y.x, older ? x.y : y.y, older ? x.z : y.z, older ? x.w : y.w}; };
#pragma unroll
  for (int t = 0; t < AttnDims<NKT>::KT; ++t)
#pragma unroll
    for (int s = 0; s < 2; ++s) pick(16 * (wave + kGW * t) + (lane & 15) < first_new, e.kf[t][s], g.kf[t][s]);
#pragma unroll
  for (int it = 0; it < AttnDims<NKT>::VP; ++it) pick(((wave * 64 + lane) + 64 * kGW * it) % (16 * NKT) < first_new, e.vr[it], g.vr[it]);
}
template <int NKT>
__device__ __forceinline__ void attn_values(const AttnLds& L, const AttnRegs<NKT>& g, int nk_all, int wave, int lane) {
  constexpr int LDV = AttnDims<NKT>::LDV;
  const int nkp = (nk_all + 31) & ~31;
#pragma unroll
  for (int it = 0; it < AttnDims<NKT>::VP; ++it) {
    const int i = (wave * 64 + lane) + 64 * kGW * it, t = i % (16 * NKT), c = i / (16 * NKT);
    if (t < nkp) {
      const uint4 v = t < nk_all ? g.vr[it] : uint4{0u, 0u, 0u, 0u};
      bf16_t* dst = L.Vt + (c * 8) * LDV + t;
      dst[0] = (bf16_t)(v.x & 0xffffu); dst[LDV] = (bf16_t)(v.x >> 16);
      dst[2 * LDV] = (bf16_t)(v.y & 0xffffu); dst[3 * LDV] = (bf16_t)(v.y >> 16);
      dst[4 * LDV] = (bf16_t)(v.z & 0xffffu); dst[5 * LDV] = (bf16_t)(v.z >> 16);
      dst[6 * LDV] = (bf16_t)(v.w & 0xffffu); dst[7 * LDV] = (bf16_t)(v.w >> 16);
    }
  }
}
// (two barriers, of the group by its count, of the workgroup without; the values are written ahead of the first)
template <int NKT>
__device__ __forceinline__ void attn_core(const AttnLds& L, unsigned* target, const uint4 (&qf)[2], const AttnRegs<NKT>& g, int nk_all, int nk_base,
                                          int off, int causal, float scale, bf16_t* att, int row, int n_rows,
                                          int h, int wave, int lane) {
  constexpr int LDV = AttnDims<NKT>::LDV, KT = AttnDims<NKT>::KT;
  const int r = lane & 15, kq = lane >> 4;
  const int nb = (nk_all + 31) >> 5, nt2 = 2 * nb;
  f32x4 S[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const int tile = wave + kGW * t;
    S[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s)
      S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qf[s]), __builtin_bit_cast(bf16x8, g.kf[t][s]), S[t], 0, 0, 0);
    const int key = 16 * tile + r;
    float m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int nkr = causal ? nk_base + off + 4 * kq + i + 1 : nk_base;
      S[t][i] = key < nkr ? S[t][i] * scale : -INFINITY;
      m[i] = row16_max(S[t][i]);
    }
    if (r == 0) *(float4*)(L.xmax + tile * 16 + 4 * kq) = float4{m[0], m[1], m[2], m[3]};
  }
  if (target) group_bar(L.count, *target, lane);   // values and maxima
  else wg_bar();
  {
    f32x4 mx = *(const f32x4*)(L.xmax + 4 * kq);
#pragma unroll
    for (int w = 1; w < NKT; ++w) {   // (tiles past the last key: -inf)
      const f32x4 o = *(const f32x4*)(L.xmax + w * 16 + 4 * kq);
#pragma unroll
      for (int i = 0; i < 4; ++i) mx[i] = fmaxf(mx[i], o[i]);
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const int tile = wave + kGW * t;
      if (tile < nt2) {
        f32x4 p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[i] = __builtin_amdgcn_exp2f((S[t][i] - mx[i]) * 1.44269504088896340736f);
          L.Pt[(4 * kq + i) * LDV + r + 16 * tile] = f2bf(p[i]);
        }
        L.Pf[tile * 64 + lane] = p;
      }
    }
  }
  if (target) group_bar(L.count, *target, lane);   // probabilities
  else wg_bar();
  f32x4 O = f32x4{0.f, 0.f, 0.f, 0.f}, ps = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < NKT / 2; ++kb) {
    if (kb < nb) {
      const uint4 pa = *(const uint4*)(L.Pt + r * LDV + 32 * kb + 8 * kq);
      const uint4 vb = *(const uint4*)(L.Vt + (16 * wave + r) * LDV + 32 * kb + 8 * kq);
      const f32x4 p0 = L.Pf[(2 * kb) * 64 + lane], p1 = L.Pf[(2 * kb + 1) * 64 + lane];
      O = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pa), __builtin_bit_cast(bf16x8, vb), O, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) { ps[i] += p0[i]; ps[i] += p1[i]; }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float l = row16_sum(ps[i]);
    if (4 * kq + i < n_rows)
      put(att + (size_t)(row + 4 * kq + i) * kTD + h * 64 + 16 * wave + r, O[i] / l);
  }
}

template <int MT, int NKT, bool DEC, bool AHEAD>
__global__ __launch_bounds__(kTeamThreads) void k_team(TeamArgs a) {
  constexpr int ROWS = 16 * MT, RPW = ROWS / kTW;   // RPW: rows a wave stages
  constexpr int LDV = AttnDims<NKT>::LDV;
  extern __shared__ uint4 team_lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = (int)((xcc_id() - (unsigned)a.xcd0) & 7u), stations = AHEAD ? a.stations : 1;
  if (slot >= a.n_teams * stations) return;
  const int team = AHEAD ? slot % a.n_teams : slot, station = AHEAD ? slot / a.n_teams : 0;
  char* lds = (char*)team_lds;
  bf16_t* At = (bf16_t*)lds;                                     // [ROWS][528], FFN2: [4 slices][ROWS][528]
  float* xres = (float*)(lds + kSlices * ROWS * kTLd * 2);      // [ROWS][16]
  f32x4* accx = (f32x4*)(xres + ROWS * 16);                      // [3 slices][MT][64]
  float* lnv = (float*)(accx + 3 * MT * 64);                     // [2][512]
  TeamChunk* chunks = (TeamChunk*)(lnv + 2 * kTD);               // [ROWS]
  int* grow = (int*)(chunks + ROWS);                             // [ROWS] packed row of the team's row
  int* rdst = grow + ROWS;                                       // [ROWS] its key / value row
  int* misc = rdst + ROWS;                                       // member, chunks, chunks of segment 0
  unsigned* gave_up = (unsigned*)(misc + 4);
  unsigned* met_a = gave_up + 1;                                 // arrivals at group A's barriers
  // attention: the row tile [16][528] and the queries [16][80] of the cross-attention first, then values and probabilities
  bf16_t* Qt = At + 16 * kTLd;
  AttnLds AL;
  AL.Vt = Qt + 16 * kCrossqQld;
  AL.Pt = AL.Vt + 64 * LDV;
  AL.Pf = (f32x4*)(AL.Pt + 16 * LDV);
  AL.xmax = (float*)(AL.Pf + NKT * 64);
  AL.count = met_a;

  unsigned* words = a.words + slot * 64;
  const int n0 = a.row_n[0][team], n1 = a.row_n[1][team];
  // member number, row tables, attention chunks
  if (threadIdx.x == 64 * kGW) misc[0] = (int)__hip_atomic_fetch_add(words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (wave >= kGW) {
#pragma unroll
    for (int i = 0; i < 3 * MT; i += kGW)
      if (i + wave - kGW < 3 * MT) accx[(i + wave - kGW) * 64 + lane] = unwritten4();
  }
  team_lists<ROWS, DEC>(a, team, n0, n1, chunks, grow, rdst, misc + 1, wave, lane);
  if (threadIdx.x == 64) { *gave_up = 0; *met_a = 0; }
  __syncthreads();
  const int idx = __builtin_amdgcn_readfirstlane(misc[0]);
  const int n_chunks_all = __builtin_amdgcn_readfirstlane(min(misc[1], ROWS)), n_chunks0 = __builtin_amdgcn_readfirstlane(min(misc[2], ROWS));
  if (idx >= kTeamMembers) {   // more workgroups on the XCD than members: not how this grid is dealt out
    if (threadIdx.x == 0) __hip_atomic_store(a.fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  constexpr int CPR = kTeamMembers / kTH;   // chunks a team works on at a time
  const int c_first = idx >> 3;
  const TeamChunk ch0 = chunk_at(chunks, min(c_first, ROWS - 1));
  typedef TeamOff<DEC> O;

  TeamWait tw;
  tw.fail = a.fail; tw.gave_up = gave_up; tw.off = false;
  const int gw = wave & (kGW - 1), lane0 = lane, idx0 = idx;

  // this XCD's buffers
  char* sl = a.slots + (size_t)slot * TeamSlot::kBytes;
  bf16_t *xq = (bf16_t*)(sl + TeamSlot::q), *xatt = (bf16_t*)(sl + TeamSlot::att), *xatt2 = (bf16_t*)(sl + TeamSlot::att2), *xf = (bf16_t*)(sl + TeamSlot::f);
  float *xs1 = (float*)(sl + TeamSlot::s1), *xs2 = (float*)(sl + TeamSlot::s2), *xs = (float*)(sl + TeamSlot::s), *xr = (float*)(sl + TeamSlot::xr);
  auto hop = [&](int l) { return (float*)(a.hop + (size_t)l * kTeamHopBytes) + team * (kTeamMaxRows * kTD); };

  // The two groups of waves take turns: one multiplies a stage's rows and stores, then the other requests the next stages' strips
  // into its registers.  A CU takes only so many requests at a time and answers them in order: stores behind 32 to 64 KB of strips
  // (from the last-level cache 64 KB take 0.93 us) left 1.2 us after the product, so the strips go out behind the stores (a barrier
  // says so, which also frees the rows' place in LDS) and return while the results of the others are on their way, or while attention computes.
  // With several XCDs a team (AHEAD) an XCD requests a layer's strips while the others work on the layers before; what the registers
  // do not hold (the second output projection's and FFN2's) follows during the cross-attention.
  // Group A: Q, K, V | self-attention | cross-attention | FFN1.  Group B: output projections | cross queries | FFN2.
  //
  // Exchanges of a layer, who reads them, and when group B sets their places back (the stores are answered for before the member's next
  // data leave; a reader has seen those data whole, or data that took them, before it looks at the place; and whoever read the
  // place's former content has stored data since which the writer has seen):
  //   q, k, v    the members of a problem's chunk                        at FFN2 of the XCD's layer before, or ahead of the first barrier
  //   att        all (those without a chunk have seen FFN2's rows only)  at FFN2 of the XCD's layer before, or ahead of the first barrier
  //   s1         a chunk's members; the encoder: all                     before Q, K, V
  //   att2, xr   all (those without a chunk have seen att)               before Q, K, V
  //   s2         all (seen att2)                                         before Q, K, V
  //   f          all (seen s2; the encoder: s1)                          during self-attention
  //   s          all (seen f)                                            before FFN1 (group A)
  // What other XCDs read (hop; keys and values that teams share) has a place for every layer, set back ahead of the writer's first barrier;
  // its readers have seen the arrival of all XCDs before their first look (wait_all).
  auto unwrite_attn = [&](int n, int idx, int lane) {   // q, att (a wave)
#pragma unroll
    for (int s = 0; s < 3; ++s)
      if (idx * 3 + s < kTD / 16) unwrite_rows<2>(xq, kTD * 2, (idx * 3 + s) * 32, 0, n, lane);
#pragma unroll 1
    for (int c = c_first; c < n_chunks_all; c += CPR) {
      const TeamChunk ch = chunk_at(chunks, c);
      unwrite_rows<8>(xatt, kTD * 2, (idx & (kTH - 1)) * 128, ch.row, ch.n, lane);
    }
  };
  auto unwrite_kv = [&](int l, int n, int idx, int lane) {   // (a wave)
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int strip = idx * 3 + s;
      if (strip >= kTD / 16) {
        char* base = (char*)(strip < 2 * (kTD / 16) ? a.K : a.V) + (size_t)l * a.kv_stride + ((strip * 16) & (kTD - 1)) * 2;
#pragma unroll 1
        for (int m = lane >> 1; m < n; m += 32) {
          const unsigned off = (unsigned)rdst[m] * (kTD * 2) + (lane & 1) * 16;
          if (a.shared) unwrite16_far(base, off);
          else unwrite16(base, off);
        }
      }
    }
  };
  const bool far_kv = a.shared != 0;
  if (wave < kGW) {
    // ------------------------------------------------------------------------------------------ group A
    uint4 b[16], b1[16];                       // strips of Q, K, V | FFN1 (in b too where nothing is requested a layer ahead)
    uint4 (&bw)[16] = *(AHEAD ? &b1 : &b);
    float bias = 0.f, bias1 = 0.f;
    unsigned met = 0;
    auto request_qkv = [&](int l, int idx, int lane) {
      const char* wl = a.w + (size_t)l * O::kLayerBytes;
      if (gw < 3) {
        bias = gload((const float*)(wl + O::bqkv) + (idx * 3 + gw) * 16 + (lane & 15));
        load_strip((const bf16_t*)(wl + O::wqkv), (idx * 3 + gw) * 16, kTD, 0, lane, b);
      }
    };
    auto request_ffn1 = [&](int l, int idx, int lane) {
      const char* wl = a.w + (size_t)l * O::kLayerBytes;
      bias1 = gload((const float*)(wl + O::b1) + (idx * 4 + gw) * 16 + (lane & 15));
      load_strip((const bf16_t*)(wl + O::w1), (idx * 4 + gw) * 16, kTD, 0, lane, bw);
    };
    {
      const int lane = here(lane0), idx = here_s(idx0);
      if (station == 0) {
        stage_first<RPW>(a.xa, grow, n0 + n1, At, wave, lane);
        stage_first_residual<ROWS>(a.x, grow, n0 + n1, xres, idx, wave, lane);
      }
      request_qkv(station, idx, lane);
      wg_bar();   // the team is complete
      tw.off = __builtin_amdgcn_readfirstlane(__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0;
      if (AHEAD && station > 0) request_ffn1(station, idx, lane);
    }
#pragma unroll 1
    for (int l = station; l < a.layers; l += stations) {
      int n = n0 + n1, n_chunks = n_chunks_all;
      const bool in_time = !AHEAD || l == 0;                   // this layer's strips are requested on the way
      const char* wl = a.w + (size_t)l * O::kLayerBytes;       // the layer's matrices and vectors
      AttnRegs<NKT> cg, eg;   // the memory's keys and values; the own ones that earlier forwards wrote (of the first chunk)
      constexpr bool kEarly = AHEAD && DEC && NKT == 4;   // (where the registers hold them beside two sets of strips)
      bool early = false;
      const int h = idx0 & (kTH - 1);
      auto memory_keys = [&](const TeamChunk& ch, int lane) {
        attn_request<NKT, false>((const bf16_t*)((const char*)a.Km + (size_t)l * a.m_stride), (const bf16_t*)((const char*)a.Vm + (size_t)l * a.m_stride),
                                 ch.kv_cross, min(ch.nk_cross, 16 * NKT), h, gw, lane, cg);
      };
      // ---------------------------------------------------------------- Q, K, V
      {
        const int lane = here(lane0), idx = here_s(idx0), r = lane & 15, kq = lane >> 4;
        if (AHEAD && l > 0) {
          // The strips have gone through the L2 and taken the places of the rows to come with them: looked at once they are back
          // (a first look past the L2 takes 0.8 to 1 us, and the row's arrival with it).
          team_put_ready();
          if (gw == kGW - 1) {
            float seen = 0.f;
            if (lane < n) seen = ld4_l2(xatt, lane * (kTD * 2) + (idx & (kTH - 1)) * 128);
            if (c_first < n_chunks) {
              const int first_new = ch0.causal ? ch0.nk_base : 0, nk_all = min(ch0.causal ? ch0.nk_base + ch0.off + ch0.n : ch0.nk_base, 16 * NKT);
              const unsigned at = (idx & (kTH - 1)) * 128;
              if (lane < ch0.n) seen += ld4_l2(xq, (unsigned)(ch0.row + lane) * (kTD * 2) + at);
#pragma unroll
              for (int t = 0; t < NKT / 4; ++t) {
                const int key = first_new + 64 * t + lane;
                const unsigned off = (unsigned)(ch0.kv_self + key) * (kTD * 2) + at;
                if (key < nk_all) {
                  seen += ld4_l2((const char*)a.K + (size_t)l * a.kv_stride, off);
                  seen += ld4_l2((const char*)a.V + (size_t)l * a.kv_stride, off);
                }
              }
            }
            asm volatile("" :: "v"(seen));
          }
        }
        if constexpr (kEarly) {
          if (c_first < n_chunks) {
            const TeamChunk& ch = ch0;
            memory_keys(ch, lane);
            early = ch.causal && ch.nk_base > 0;
            if (early)
              attn_request<NKT, false>((const bf16_t*)((const char*)a.K + (size_t)l * a.kv_stride), (const bf16_t*)((const char*)a.V + (size_t)l * a.kv_stride),
                                       ch.kv_self, min(ch.nk_base, 16 * NKT), idx & (kTH - 1), gw, lane, eg);
          }
        }
        if constexpr (AHEAD) wg_bar();   // the LayerNorm's vectors
        if (l > 0) stage_ln<RPW>(tw, AHEAD ? hop(l - 1) : xs, n, lnv, At, xres, idx, wave, lane);
        wg_bar();
        team_put_ready();
        if (gw < 3) {
          const int strip = idx * 3 + gw, col = (strip * 16 + r) & (kTD - 1), part = strip >> 5;
          bf16_t* out = (part == 0 ? xq : (bf16_t*)((char*)(part == 1 ? a.K : a.V) + (size_t)l * a.kv_stride)) + col;
          int to[MT][4];
#pragma unroll
          for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) to[t][i] = part == 0 ? t * 16 + 4 * kq + i : rdst[t * 16 + 4 * kq + i];
          f32x4 acc[MT];
          zero(acc);
          if constexpr (AHEAD) mm16_lean<MT>(At + r * kTLd + kq * 8, b, acc);
          else mm16<MT>(At + r * kTLd + kq * 8, b, acc);
          if (part > 0 && far_kv) {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if (t * 16 + 4 * kq + i < n) put_far(out + (size_t)to[t][i] * kTD, acc[t][i] + bias);
          } else {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if (t * 16 + 4 * kq + i < n) put(out + (size_t)to[t][i] * kTD, acc[t][i] + bias);
          }
        }
        wg_bar();
      }
      if (a.head_only && l + 1 == a.layers) { n = n0; n_chunks = n_chunks0; }   // only segment 0 goes on
      // ---------------------------------------------------------------- self-attention
      {
        const int lane = here(lane0), r = lane & 15, kq = lane >> 4;
        const bf16_t* Kl = (const bf16_t*)((const char*)a.K + (size_t)l * a.kv_stride);
        const bf16_t* Vl = (const bf16_t*)((const char*)a.V + (size_t)l * a.kv_stride);
#pragma unroll 1
        for (int c = c_first; c < n_chunks; c += CPR) {
          const TeamChunk ch = c == c_first ? ch0 : chunk_at(chunks, c);
          const int nk_all = min(ch.causal ? ch.nk_base + ch.off + ch.n : ch.nk_base, 16 * NKT);
          uint4 qf[2];
          AttnRegs<NKT> g;
          const unsigned qo = (unsigned)(ch.row + min(r, ch.n - 1)) * (kTD * 2) + (h * 64 + kq * 8) * 2;
          wait_for(tw, lane, [&]() {
            Seen16 seen;
#pragma unroll
            for (int s = 0; s < 2; ++s) qf[s] = ld16_l2(xq, qo + 64 * s);
            const int first_new = ch.causal ? ch.nk_base : 0;
            const bool kv = attn_request<NKT, true>(Kl, Vl, ch.kv_self, nk_all, h, gw, lane, g, early && c == c_first ? first_new : 0, first_new);
#pragma unroll
            for (int s = 0; s < 2; ++s) seen.add(qf[s]);
            return kv && seen.all();
          });
          if constexpr (kEarly) {
            if (early && c == c_first) attn_older<NKT>(eg, ch.nk_base, gw, lane, g);
          }
          if constexpr (DEC && !kEarly) {
            if (c == c_first) memory_keys(ch, lane);
          }
          attn_values<NKT>(AL, g, nk_all, gw, lane);
          attn_core<NKT>(AL, in_time ? &met : nullptr, qf, g, nk_all, ch.nk_base, ch.off, ch.causal, a.scale, xatt, ch.row, ch.n, h, gw, lane);
          wg_bar();
        }
      }
      // ---------------------------------------------------------------- output projection (group B multiplies)
      {
        const int lane = here(lane0), idx = here_s(idx0);
        stage_rows<RPW>(tw, xatt, n, At, wave, lane);
        wg_bar();
        wg_bar();
        if (in_time) {
          if constexpr (DEC) {
            bias1 = gload((const float*)(wl + O::b1) + (idx * 4 + gw) * 16 + (lane & 15));
            load_strip<0, 8>((const bf16_t*)(wl + O::w1), (idx * 4 + gw) * 16, kTD, 0, lane, bw);
          } else {
            request_ffn1(l, idx, lane);
          }
        }
      }
      if constexpr (DEC) {
        // -------------------------------------------------------------- cross-attention with its query projection
        {
          const int lane = here(lane0), r = lane & 15, kq = lane >> 4;
#pragma unroll 1
          for (int c = c_first; c < n_chunks; c += CPR) {
            const TeamChunk ch = c == c_first ? ch0 : chunk_at(chunks, c);
            const int nk_all = min(ch.nk_cross, 16 * NKT);
            if (c != c_first) memory_keys(ch, lane);
            stage_ln_chunk(tw, xs1 + ch.row * kTD, ch.n, lnv, At, xr + ch.row * kTD, h, wave ^ kGW, lane);
            attn_values<NKT>(AL, cg, nk_all, gw, lane);
            wg_bar();
            wg_bar();   // group B has left the queries
            uint4 qf[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) qf[s] = *(const uint4*)(Qt + min(r, ch.n - 1) * kCrossqQld + kq * 8 + 32 * s);
            attn_core<NKT>(AL, &met, qf, cg, nk_all, nk_all, 0, 0, a.scale, xatt2, ch.row, ch.n, h, gw, lane);
            wg_bar();
          }
        }
        // -------------------------------------------------------------- output projection (group B multiplies)
        {
          const int lane = here(lane0), idx = here_s(idx0);
          stage_rows<RPW>(tw, xatt2, n, At, wave, lane);
          wg_bar();
          wg_bar();
          if (in_time) load_strip<8, 16>((const bf16_t*)(wl + O::w1), (idx * 4 + gw) * 16, kTD, 0, lane, bw);
        }
      }
      // ---------------------------------------------------------------- FFN1
      {
        const int lane = here(lane0), idx = here_s(idx0), r = lane & 15, kq = lane >> 4;
        if (!AHEAD && gw < MT && l + 1 < a.layers) unwrite_rows<4>(xs, kTD * 4, idx * 64, gw * 16, min(n - gw * 16, 16), lane);
        stage_ln<RPW>(tw, DEC ? xs2 : xs1, n, lnv, At, xres, idx, wave ^ kGW, lane);
        wg_bar();
        team_put_ready();
        bf16_t* out = xf + (idx * 4 + gw) * 16 + r;
        f32x4 acc[MT];
        zero(acc);
        if constexpr (AHEAD) mm16_lean<MT>(At + r * kTLd + kq * 8, bw, acc);
        else mm16<MT>(At + r * kTLd + kq * 8, bw, acc);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          const int m = t * 16 + 4 * kq;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (m + i < n) put(out + (size_t)(m + i) * kTF, fmaxf(acc[t][i] + bias1, 0.f));
        }
        wg_bar();
      }
      // ---------------------------------------------------------------- FFN2 (group B multiplies)
      {
        const int lane = here(lane0), idx = here_s(idx0);
        stage_ffn<ROWS>(tw, xf, n, At, gw, wave >> 2, lane);
        wg_bar();
        if (!AHEAD && l + 1 < a.layers) request_qkv(l + 1, idx, lane);   // (FFN2's chain is long: these are there before it ends)
        wg_bar();
        if (AHEAD && l + stations < a.layers) {
          request_qkv(l + stations, idx, lane);
          request_ffn1(l + stations, idx, lane);
        }
      }
    }
    return;
  }

  // -------------------------------------------------------------------------------------------- group B
  uint4 bo[16], bq[16];   // strips of the output projection, then FFN2 | of the query projection, then the second output projection
  uint4 (&b2)[16] = *(DEC || !AHEAD ? &bo : &bq);
  uint4 ln = {};
  unsigned met = 0;       // group A's barriers so far
  float bias_o = 0.f, bias_q = 0.f, bias_2 = 0.f;
  auto request_out = [&](int l, int idx, int lane) {
    const char* wl = a.w + (size_t)l * O::kLayerBytes;
    if (gw < MT) {
      bias_o = gload((const float*)(wl + O::bo) + idx * 16 + (lane & 15));
      load_strip((const bf16_t*)(wl + O::wo), idx * 16, kTD, 0, lane, bo);
    }
  };
  auto request_queries = [&](int l, int idx, int lane) {
    const char* wl = a.w + (size_t)l * O::kLayerBytes;
    const int col = (idx & (kTH - 1)) * 64 + gw * 16;
    bias_q = gload((const float*)(wl + O::cbq) + col + (lane & 15));
    load_strip((const bf16_t*)(wl + O::cwq), col, kTD, 0, lane, bq);
  };
  auto request_ffn2 = [&](int l, int idx, int lane) {
    const char* wl = a.w + (size_t)l * O::kLayerBytes;
    bias_2 = gload((const float*)(wl + O::b2) + idx * 16 + (lane & 15));
    load_strip((const bf16_t*)(wl + O::w2), idx * 16, kTF, 16 * gw, lane, b2);
  };
  auto request_ahead = [&](int l, int idx, int lane) {
    const char* before = a.w + (size_t)(l - 1) * O::kLayerBytes;
    ln = load_ln((const float*)(before + O::ln_lg), (const float*)(before + O::ln_lb), gw, lane);
    request_out(l, idx, lane);
    if constexpr (DEC) {
      if (c_first < n_chunks_all) request_queries(l, idx, lane);
    } else {
      request_ffn2(l, idx, lane);
    }
  };
  // Before the first look at a place that another XCD writes: all XCDs' members are there, their places set back.  The second XCD of a team
  // looks at the first one's rows at once, the first at the second one's ahead of its second layer (by then the count is complete on an
  // idle chip; without this wait a second XCD that starts late has the rows of an earlier forward taken for its own), all at shared
  // keys and values ahead of the first attention.
  auto wait_all = [&]() { team_wait_count(a, a.words + 48, a.n_teams * stations, gave_up, lane0); };
  {
    const int lane = here(lane0), idx = here_s(idx0);
    if (gw == kGW - 1) {   // this member is here, and its places can be read
      const int n = n0 + n1;
      unwrite_attn(n, idx, lane);
      if (!AHEAD && !far_kv) {
        unwrite_kv(0, n, idx, lane);
      } else {
#pragma unroll 1
        for (int l = station; l < a.layers; l += stations) {
          unwrite_kv(l, n, idx, lane);
          if (AHEAD && l + 1 < a.layers) {
#pragma unroll 1
            for (int m = lane >> 2; m < n; m += 16) unwrite16_far(hop(l), (unsigned)m * (kTD * 4) + idx * 64 + (lane & 3) * 16);
          }
        }
      }
      team_arrive(a, words, lane);
    }
    if (station == 0) {
      stage_first<RPW>(a.xa, grow, n0 + n1, At, wave, lane);
      stage_first_residual<ROWS>(a.x, grow, n0 + n1, xres, idx, wave, lane);
    }
    if (gw == kGW - 1) {
      team_wait_count(a, words + 32, kTeamMembers, gave_up, lane0);
      if (AHEAD && station > 0) wait_all();
    }
    wg_bar();
    tw.off = __builtin_amdgcn_readfirstlane(__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0;
    if (AHEAD && station > 0) request_ahead(station, idx, lane);
  }
#pragma unroll 1
  for (int l = station; l < a.layers; l += stations) {
    int n = n0 + n1, n_chunks = n_chunks_all;
    const bool in_time = !AHEAD || l == 0;
    const char* wl = a.w + (size_t)l * O::kLayerBytes;
    // ------------------------------------------------------------------ Q, K, V
    {
      const int lane = here(lane0), idx = here_s(idx0);
      if (AHEAD && l > 0) team_put_ready();   // (behind the strips: see group A)
      if (gw < MT) {
        unwrite_rows<4>(xs1, kTD * 4, idx * 64, gw * 16, min(n - gw * 16, 16), lane);
        if constexpr (DEC) unwrite_rows<4>(xs2, kTD * 4, idx * 64, gw * 16, min(n - gw * 16, 16), lane);
      } else if (DEC && gw >= kGW - 2) {
#pragma unroll 1
        for (int c = c_first; c < n_chunks; c += CPR) {
          const TeamChunk ch = c == c_first ? ch0 : chunk_at(chunks, c);
          if (gw == kGW - 1) unwrite_rows<8>(xatt2, kTD * 2, (idx & (kTH - 1)) * 128, ch.row, ch.n, lane);
          else unwrite_rows<16>(xr, kTD * 4, (idx & (kTH - 1)) * 256, ch.row, ch.n, lane);
        }
      }
      if constexpr (AHEAD) {
        if (l > 0) keep_ln(lnv, ln, gw, lane);
        if (l == stations && !far_kv && gw == kGW - 1 && !tw.off) wait_all();   // (station 0)
        wg_bar();
      }
      if (l > 0) stage_ln<RPW>(tw, AHEAD ? hop(l - 1) : xs, n, lnv, At, xres, idx, wave, lane);
      team_put_ready();
      wg_bar();
      if (l == 0 && far_kv && gw == kGW - 1) wait_all();
      wg_bar();
      if (in_time) request_out(l, idx, lane);
      ln = load_ln((const float*)(wl + (DEC ? O::ln1g : O::ln_fg)), (const float*)(wl + (DEC ? O::ln1b : O::ln_fb)), gw, lane);
    }
    if (a.head_only && l + 1 == a.layers) { n = n0; n_chunks = n_chunks0; }
    // ------------------------------------------------------------------ self-attention
    {
      const int lane = here(lane0), idx = here_s(idx0);
      if (gw < MT) unwrite_rows<8>(xf, kTF * 2, idx * 128, gw * 16, min(n - gw * 16, 16), lane);
#pragma unroll 1
      for (int c = c_first; c < n_chunks; c += CPR) {
        if constexpr (DEC) {
          if (in_time && c == c_first) {   // (behind the keys and values)
            group_wait(met_a, met + kGW);
            request_queries(l, idx, lane);
          }
        }
        if (in_time) {
          met += 2 * kGW;
        } else {
          wg_bar(); wg_bar();
        }
        wg_bar();
      }
    }
    // ------------------------------------------------------------------ output projection + residual
    {
      const int lane = here(lane0), idx = here_s(idx0), r = lane & 15, kq = lane >> 4;
      stage_rows<RPW>(tw, xatt, n, At, wave, lane);
      keep_ln(lnv, ln, gw, lane);
      wg_bar();
      if (gw < MT && gw * 16 < n) {
        const int m0 = gw * 16 + 4 * kq;
        float res[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) res[i] = xres[(m0 + i) * 16 + r];
        f32x4 acc[1];
        zero(acc);
        team_put_ready();
        mm16<1>(At + (gw * 16 + r) * kTLd + kq * 8, bo, acc);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (m0 + i < n) put(xs1 + (m0 + i) * kTD + idx * 16 + r, acc[0][i] + bias_o + res[i]);
      }
      wg_bar();
    }
    if constexpr (DEC) {
      // ---------------------------------------------------------------- cross-attention: the queries
      {
        const int lane = here(lane0), idx = here_s(idx0), r = lane & 15, kq = lane >> 4, h = idx & (kTH - 1);
        auto next_strips = [&]() {
          if (gw < MT) {
            bias_q = gload((const float*)(wl + O::cbo) + idx * 16 + r);
            load_strip((const bf16_t*)(wl + O::cwo), idx * 16, kTD, 0, lane, bq);
          }
          ln = load_ln((const float*)(wl + O::ln_fg), (const float*)(wl + O::ln_fb), gw, lane);
          if constexpr (AHEAD) {
            request_ffn2(l, idx, lane);
          } else {
            bias_2 = gload((const float*)(wl + O::b2) + idx * 16 + r);
            load_strip<0, 8>((const bf16_t*)(wl + O::w2), idx * 16, kTF, 16 * gw, lane, b2);
          }
        };
        if (c_first >= n_chunks) {
          __builtin_amdgcn_s_sleep(24);   // (0.7 us: the others' rows first, the L2 is this XCD's only one)
          next_strips();
        }
#pragma unroll 1
        for (int c = c_first; c < n_chunks; c += CPR) {
          const TeamChunk ch = c == c_first ? ch0 : chunk_at(chunks, c);
          const int row = ch.row, nr = ch.n;
          stage_ln_chunk(tw, xs1 + row * kTD, nr, lnv, At, xr + row * kTD, h, wave ^ kGW, lane);
          wg_bar();
          {
            f32x4 acc[1];
            zero(acc);
            mm16<1>(At + r * kTLd + kq * 8, bq, acc);
#pragma unroll
            for (int i = 0; i < 4; ++i) Qt[(4 * kq + i) * kCrossqQld + gw * 16 + r] = f2bf(acc[0][i] + bias_q);
          }
          wg_bar();
          if (c + CPR >= n_chunks) next_strips();
          met += 2 * kGW;
          wg_bar();
        }
      }
      // ---------------------------------------------------------------- output projection + residual
      {
        const int lane = here(lane0), idx = here_s(idx0), r = lane & 15, kq = lane >> 4;
        float res[4] = {};
        if (gw < MT && gw * 16 < n) {
          wait_for(tw, lane, [&]() {
            bool there = true;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              res[i] = ld4_l2(xr, (unsigned)min(gw * 16 + 4 * kq + i, n - 1) * (kTD * 4) + (idx * 16 + r) * 4);
              there = there && __float_as_uint(res[i]) != ~0u;
            }
            return __builtin_amdgcn_ballot_w64(!there) == 0;
          });
        }
        stage_rows<RPW>(tw, xatt2, n, At, wave, lane);
        keep_ln(lnv, ln, gw, lane);
        wg_bar();
        if (gw < MT && gw * 16 < n) {
          const int m0 = gw * 16 + 4 * kq;
          f32x4 acc[1];
          zero(acc);
          team_put_ready();
          mm16<1>(At + (gw * 16 + r) * kTLd + kq * 8, bq, acc);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (m0 + i < n) put(xs2 + (m0 + i) * kTD + idx * 16 + r, acc[0][i] + bias_q + res[i]);
        }
        wg_bar();
      }
    }
    // ------------------------------------------------------------------ FFN1
    {
      const int lane = here(lane0), idx = here_s(idx0);
      stage_ln<RPW>(tw, DEC ? xs2 : xs1, n, lnv, At, xres, idx, wave ^ kGW, lane);
      wg_bar();
      wg_bar();
      if constexpr (!DEC) {
        if (in_time) request_ffn2(l, idx, lane);
      } else if constexpr (!AHEAD) {
        load_strip<8, 16>((const bf16_t*)(wl + O::w2), idx * 16, kTF, 16 * gw, lane, b2);
      }
      if constexpr (!AHEAD) ln = load_ln((const float*)(wl + O::ln_lg), (const float*)(wl + O::ln_lb), gw, lane);
    }
    // ------------------------------------------------------------------ FFN2 + residual: a wave per 512-k slice
    {
      const int lane = here(lane0), idx = here_s(idx0), r = lane & 15, kq = lane >> 4;
      if (gw == kGW - 1 && l + stations < a.layers) {
        unwrite_attn(n0 + n1, idx, lane);
        if (!AHEAD && !far_kv) unwrite_kv(l + 1, n0 + n1, idx, lane);
      }
      stage_ffn<ROWS>(tw, xf, n, At, gw, wave >> 2, lane);
      if constexpr (!AHEAD) keep_ln(lnv, ln, gw, lane);
      wg_bar();
      // The sum of an element stays one chain: the accumulators go from wave to wave through LDS, a place that is all ones is not
      // written yet (a wave waits for the one before it only, so the wait ends).
      const bool last = gw + 1 == kSlices;
      float res[MT][4];
      if (last) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) res[t][i] = xres[(t * 16 + 4 * kq + i) * 16 + r];
        team_put_ready();
      }
      f32x4 acc[MT];
      zero(acc);
      mm16<MT>(At + (gw * ROWS + r) * kTLd + kq * 8, b2, acc, [&]() {
        if (gw > 0) {
          f32x4* from = accx + (gw - 1) * MT * 64 + lane;
          bool there;
          do {
            asm volatile("" ::: "memory");
            unsigned m = 0;
#pragma unroll
            for (int t = 0; t < MT; ++t) {
              acc[t] = from[t * 64];
              const uint4 v = __builtin_bit_cast(uint4, acc[t]);
              m = max(max(m, v.x), max(max(v.y, v.z), v.w));
            }
            there = __builtin_amdgcn_ballot_w64(m == ~0u) == 0;
          } while (!there);
        }
      });
      if (!last) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
          accx[(gw * MT + t) * 64 + lane] = f32x4{__uint_as_float(written(acc[t][0])), __uint_as_float(written(acc[t][1])),
                                                  __uint_as_float(written(acc[t][2])), __uint_as_float(written(acc[t][3]))};
      } else if (l + 1 == a.layers) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int m = t * 16 + 4 * kq + i;
            if (m < n) put(a.s + (size_t)grow[m] * kTD + idx * 16 + r, acc[t][i] + bias_2 + res[t][i]);
          }
      } else {
        float* out = (AHEAD ? hop(l) : xs) + idx * 16 + r;
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int m = t * 16 + 4 * kq + i;
            if (m < n) {
              if constexpr (AHEAD) put_far(out + m * kTD, acc[t][i] + bias_2 + res[t][i]);
              else put(out + m * kTD, acc[t][i] + bias_2 + res[t][i]);
            }
          }
      }
      if (gw > 0) {
#pragma unroll
        for (int t = 0; t < MT; ++t) accx[((gw - 1) * MT + t) * 64 + lane] = unwritten4();
      }
      wg_bar();
      if (AHEAD && l + stations < a.layers) request_ahead(l + stations, idx, lane);
    }
  }
}

// (more than half a CU's LDS: one member per CU)
static size_t team_lds_bytes(int mt) {
  const size_t rows = 16 * mt, b = (size_t)kSlices * rows * kTLd * 2 + rows * 16 * 4 + 3 * mt * 64 * 16 + 2 * kTD * 4 + rows * sizeof(TeamChunk) + 2 * rows * 4 + 64;
  return b > 84 * 1024 ? b : 84 * 1024;
}
// MT by the rows of the largest team, NKT by the keys of the longest problem, AHEAD where every team has several XCDs
// (dealt to teams of one row tile only)
template <typename F>
static void each_team_kernel(bool dec, const F& f) {
  if (dec) {
    f(1, 4, false, &k_team<1, 4, true, false>); f(1, 8, false, &k_team<1, 8, true, false>); f(2, 4, false, &k_team<2, 4, true, false>); f(2, 8, false, &k_team<2, 8, true, false>);
    f(1, 4, true, &k_team<1, 4, true, true>); f(1, 8, true, &k_team<1, 8, true, true>);
  } else {
    f(1, 4, false, &k_team<1, 4, false, false>); f(1, 8, false, &k_team<1, 8, false, false>); f(2, 4, false, &k_team<2, 4, false, false>); f(2, 8, false, &k_team<2, 8, false, false>);
    f(1, 4, true, &k_team<1, 4, false, true>); f(1, 8, true, &k_team<1, 8, false, true>);
  }
}
typedef void (*TeamKernel)(TeamArgs);
static TeamKernel team_kernel(bool dec, int max_rows, int max_keys, int stations) {
  TeamKernel found = nullptr;
  if (max_rows < 1 || max_rows > kTeamMaxRows || max_keys < 1 || max_keys > kTeamMaxKeys) return found;
  const int mt = max_rows <= 16 ? 1 : 2, nkt = max_keys <= 64 ? 4 : 8;
  each_team_kernel(dec, [&](int m, int nk, bool ahead, TeamKernel k) {
    if (m == mt && nk == nkt && ahead == (stations > 1)) found = k;
  });
  return found;
}
bool team_has_kernel(bool decoder, int max_rows, int max_keys, int stations) { return team_kernel(decoder, max_rows, max_keys, stations) != nullptr; }
bool prepare_team(bool decoder) {
  bool ok = true;
  each_team_kernel(decoder, [&](int mt, int, bool, TeamKernel k) {
    ok = ok && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)team_lds_bytes(mt)) == hipSuccess;
  });
  if (!ok) (void)hipGetLastError();
  return ok;
}
void launch_team(const TeamArgs& a, bool decoder, int max_rows, int max_keys, hipStream_t s) {
  const TeamKernel k = team_kernel(decoder, max_rows, max_keys, a.stations);
  k<<<8 * kTeamMembers, kTeamThreads, team_lds_bytes(max_rows <= 16 ? 1 : 2), s>>>(a);
}

}  // namespace ad

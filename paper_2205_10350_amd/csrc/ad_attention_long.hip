// Attention beyond 64 keys or 64 rows (bf16, head width 64), keys and values staged once per 128 query rows
// (k_attention_rows), and the cross-attention with its query projection for source capacities of kLongKeys and more.
// A source file, hence a code object, of its own: the attention kernels are larger than the instruction cache, and the
// speed of the short-range ones, which are the batch-1 path, moved with every addition to their code object although
// their own instructions stayed the same (0.5 us per launch at 1152 rows).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ad_device.h"

namespace ad {

// Up to 128 query rows of a (sequence, head), head width 64, at most 544 keys (526 is the most a configuration of that width
// may have): keys and transposed values are staged in LDS once per workgroup of eight waves (read from L2 by every wave, they
// were the bound: 41 us for eight sources of 301..512 tokens), and a wave takes 16 rows from the scores to the output.
//  * The products are taken transposed, S^T = K Q^T and O^T = V^T P^T: a lane then holds one query row (lane % 16) and four
//    consecutive keys of every key tile, so the whole score row stays in registers (NSB super-blocks of 128 keys, 32 registers
//    each; a fifth one ends after 32 keys, as the LDS does), the mask limit is one value per lane, and the probabilities
//    become the right operand of the output product by two lane swaps per 32 keys (permlane32 / permlane16) instead of a
//    trip through LDS.
//  * Same order as attn_tiles_mfma<64, 16, true>: super-block sb adds into accumulator sb % 4, the four are combined as
//    (a0 + a1) + (a2 + a3); a row's denominator adds keys of equal key % 16 in ascending order, then pairs, quads, halves
//    and rows of 16 as row16_sum does (four of the sixteen partial sums sit in each of four lanes).
// Eight sources of 301..512 tokens, 16 heads: 25.7 us (54 us with the four waves of a 64-row chunk splitting the keys).
constexpr int kRowsKeys = 512, kRowsKeysTail = 544;   // most keys without / with the fifth super-block
constexpr int kRowsKld = 64 + 16;                     // row stride of the staged keys (32 bytes past a multiple of 64)
constexpr int rows_key_tiles(int sb) { return sb < 4 ? 8 : 2; }   // 16-key tiles of super-block sb
// (value_block; the up to four blocks past key 512 stay among themselves)
__device__ __forceinline__ int rows_value_block(int b, int c, int r, bool whole) { return whole ? value_block(b, c, r) : b ^ ((2 * c + (r >> 3)) & 3); }
template <int NSB, bool LONGK>
__device__ __forceinline__ void attn_rows_tile(const uint4 (&qf)[2], bf16_t* __restrict__ out, const SeqDesc sd, int row0, int row_end,
                                               int h, int d, float scale, const bf16_t* Ks, const bf16_t* Vt, int ldv) {
  constexpr int DH = 64;
  const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
  const int nkr = sd.causal ? sd.nk_base + row0 + r + 1 : sd.nk_base;   // keys this lane's row sees
  const int nk_full = sd.causal ? sd.nk_base + row0 + 1 : sd.nk_base;   // keys every row of the tile sees
  // the raw products: the scale, 1/8, is a power of two, so scaling them in the subtraction of the maximum rounds as
  // scaling them first does
  f32x4 S[NSB][8];   // (of a fifth super-block: two)
  float m = -INFINITY;
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
#pragma unroll
    for (int j = 0; j < rows_key_tiles(sb); ++j) {
      f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint4 kf = *(const uint4*)(Ks + (128 * sb + 16 * j + r) * kRowsKld + 32 * s + 8 * kq);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf), __builtin_bit_cast(bf16x8, qf[s]), c, 0, 0, 0);
      }
      S[sb][j] = c;
    }
    if (128 * sb + 16 * rows_key_tiles(sb) > nk_full) {   // (the same for the whole wave: super-blocks every row sees whole need no mask)
#pragma unroll
      for (int j = 0; j < rows_key_tiles(sb); ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[sb][j][i] = 128 * sb + 16 * j + 4 * kq + i < nkr ? S[sb][j][i] : -INFINITY;
    }
#pragma unroll
    for (int j = 0; j < rows_key_tiles(sb); ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) m = fmaxf(m, S[sb][j][i]);
  }
  {
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    m = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    m = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1])) * scale;
  }
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 O[LONGK ? 4 : 1][4], psum[LONGK ? 4 : 1];
#pragma unroll
  for (int a = 0; a < (LONGK ? 4 : 1); ++a) {
    psum[a] = zero;
#pragma unroll
    for (int c = 0; c < 4; ++c) O[a][c] = zero;
  }
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
    const int a = LONGK ? sb & 3 : 0;
#pragma unroll
    for (int b = 0; b < rows_key_tiles(sb) / 2; ++b) {
      unsigned x[2][2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[i] = __builtin_amdgcn_exp2f(fmaf(S[sb][2 * b + t][i], scale, -m) * 1.44269504088896340736f);
          psum[a][i] += p[i];
        }
        x[t][0] = f2bf_pair(p[0], p[1]);
        x[t][1] = f2bf_pair(p[2], p[3]);
      }
      uint4 pf;
      {
        auto u = __builtin_amdgcn_permlane32_swap(x[0][0], x[1][0], false, false);
        auto w = __builtin_amdgcn_permlane16_swap(u[0], u[1], false, false);
        pf.x = w[0]; pf.z = w[1];
        u = __builtin_amdgcn_permlane32_swap(x[0][1], x[1][1], false, false);
        w = __builtin_amdgcn_permlane16_swap(u[0], u[1], false, false);
        pf.y = w[0]; pf.w = w[1];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint4 vf = *(const uint4*)(Vt + (16 * c + r) * ldv + 8 * rows_value_block(16 * sb + 4 * b + kq, c, r, sb < 4));
        O[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, pf), O[a][c], 0, 0, 0);
      }
    }
  }
  if constexpr (LONGK) {
    psum[0] = (psum[0] + psum[1]) + (psum[2] + psum[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) O[0][c] = (O[0][c] + O[1][c]) + (O[2][c] + O[3][c]);
  }
  float l = (psum[0][0] + psum[0][1]) + (psum[0][2] + psum[0][3]);
  {
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(l), __float_as_uint(l), false, false);
    l = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
    l = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
  // channels 32 p + 8 kq .. + 7 of the lane's row from the four lanes that hold four of each 16: a store then covers 64
  // consecutive bytes of a row (32 as they are)
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    unsigned x[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f32x4 o = O[0][2 * p + t];
      x[t][0] = f2bf_pair(o[0] / l, o[1] / l);
      x[t][1] = f2bf_pair(o[2] / l, o[3] / l);
    }
    uint4 of;
    auto u = __builtin_amdgcn_permlane32_swap(x[0][0], x[1][0], false, false);
    auto w = __builtin_amdgcn_permlane16_swap(u[0], u[1], false, false);
    of.x = w[0]; of.z = w[1];
    u = __builtin_amdgcn_permlane32_swap(x[0][1], x[1][1], false, false);
    w = __builtin_amdgcn_permlane16_swap(u[0], u[1], false, false);
    of.y = w[0]; of.w = w[1];
    if (row0 + r < row_end) gstore((uint4*)(out + (size_t)(sd.q_row0 + row0 + r) * d + h * DH + 32 * p + 8 * kq), of);
  }
}
__host__ __device__ inline int attn_rows_padded(int nk) { return nk <= kRowsKeys ? (nk + 127) / 128 * 128 : (nk + 31) / 32 * 32; }
__host__ __device__ inline size_t attn_rows_lds_bytes(int nk) {
  const size_t nkp = attn_rows_padded(nk);
  return (nkp * kRowsKld + 64 * (nkp + 16)) * 2;
}
// LONGK: the order of configurations whose key capacity is kLongKeys or more; otherwise one chain for all keys, as in the
// other kernels of such configurations (at most kLongKeys keys then).
// TAIL: key capacities beyond kRowsKeys, whose last keys are a fifth super-block; a kernel of its own, as it takes 236 registers
// and the other 164.  Eight sequences of 40 rows against 512 keys, 16 heads: 9.3 us, 23.3 in the generic attn_block (a wave
// walks all keys of its tile), 12.7 with the four waves of a workgroup splitting the keys; 526 rows against 526 keys 23.6 us,
// 72.7 and 60.4 there.
template <bool LONGK, bool TAIL>
__global__ __launch_bounds__(512) void k_attention_rows(const bf16_t* __restrict__ q, const bf16_t* __restrict__ Kb,
                                                        const bf16_t* __restrict__ Vb, bf16_t* __restrict__ out,
                                                        const SeqDesc* __restrict__ desc, int d, float scale) {
  extern __shared__ uint4 att_rows_lds[];
  const SeqDesc sd = desc[blockIdx.x];
  const int row_begin = blockIdx.z * 128, h = blockIdx.y;
  if (row_begin >= sd.nq) return;
  const int row_end = min(sd.nq, row_begin + 128);
  const int nk_all = min(sd.causal ? sd.nk_base + row_end : sd.nk_base, TAIL ? kRowsKeysTail : LONGK ? kRowsKeys : kLongKeys);   // (the host promises the bound)
  const int n_sb = (nk_all + 127) >> 7, nkp = TAIL ? attn_rows_padded(nk_all) : 128 * n_sb, ldv = nkp + 16;
  bf16_t* Ks = (bf16_t*)att_rows_lds;   // [nkp][kRowsKld]
  bf16_t* Vt = Ks + nkp * kRowsKld;     // [64][ldv]
  const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
  const int row0 = row_begin + 16 * (threadIdx.x >> 6);
  uint4 qf[2], kr[8], vr[8];
  const bf16_t* qp = q + (size_t)(sd.q_row0 + min(row0 + r, row_end - 1)) * d + h * 64 + kq * 8;
#pragma unroll
  for (int s = 0; s < 2; ++s) qf[s] = ldg16(qp + 32 * s);
  // keys: 16-byte pieces, eight per key; values: items of 8 keys x 8 channels, transposed in registers (keys past the last
  // one: the last key again, masked below; values: zeros)
  const int g = threadIdx.x & 7, t0 = (threadIdx.x >> 3) << 3;
  const bf16_t* kg = Kb + (size_t)sd.kv_row0 * d + h * 64 + g * 8;
  const bf16_t* vg = Vb + (size_t)sd.kv_row0 * d + h * 64 + g * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (64 * i < nkp) kr[i] = ldg16(kg + (size_t)min(64 * i + (int)(threadIdx.x >> 3), nk_all - 1) * d);
  if (t0 < nkp) {
#pragma unroll
    for (int i = 0; i < 8; ++i) vr[i] = ldg16(vg + (size_t)min(t0 + i, nk_all - 1) * d);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (64 * i < nkp) *(uint4*)(Ks + (64 * i + (threadIdx.x >> 3)) * kRowsKld + 8 * g) = kr[i];
  auto put_values = [&](int t0) {
    unsigned in[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool there = t0 + i < nk_all;
      in[i][0] = there ? vr[i].x : 0u; in[i][1] = there ? vr[i].y : 0u; in[i][2] = there ? vr[i].z : 0u; in[i][3] = there ? vr[i].w : 0u;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      unsigned o[4];
#pragma unroll
      for (int pr = 0; pr < 4; ++pr) {
        const unsigned lo = in[2 * pr][c >> 1], hi = in[2 * pr + 1][c >> 1];
        o[pr] = (c & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
      }
      *(uint4*)(Vt + (size_t)(g * 8 + c) * ldv + (t0 ^ 8 * (t0 < kRowsKeys ? g : g & 3))) = uint4{o[0], o[1], o[2], o[3]};
    }
  };
  if (t0 < nkp) put_values(t0);
  if constexpr (TAIL) {   // the (at most 32) keys past the first 512: one piece per thread, values by the first four items of keys
    const int key = kRowsKeys + (int)(threadIdx.x >> 3), t1 = kRowsKeys + t0;
    if (key < nkp) *(uint4*)(Ks + key * kRowsKld + 8 * g) = ldg16(kg + (size_t)min(key, nk_all - 1) * d);
    if (t1 < nkp) {
#pragma unroll
      for (int i = 0; i < 8; ++i) vr[i] = ldg16(vg + (size_t)min(t1 + i, nk_all - 1) * d);
      put_values(t1);
    }
  }
  __syncthreads();
  if (row0 >= row_end) return;
  auto tile = [&](auto n_c) { attn_rows_tile<decltype(n_c)::value, LONGK>(qf, out, sd, row0, row_end, h, d, scale, Ks, Vt, ldv); };
  if (n_sb == 1) tile(std::integral_constant<int, 1>{});
  else if (!LONGK || n_sb == 2) tile(std::integral_constant<int, 2>{});
  else if (n_sb == 3) tile(std::integral_constant<int, 3>{});
  else if (!TAIL || n_sb == 4) tile(std::integral_constant<int, 4>{});
  else tile(std::integral_constant<int, 5>{});
}

void launch_attention_long(const void* q, const void* K, const void* V, void* out, const SeqDesc* desc, int n_seq, int max_rows,
                           int H, float scale, int max_keys, hipStream_t s) {
  const size_t lds = attn_rows_lds_bytes(max_keys);   // (at most 155 KB: ad_config_check admits 526 keys)
  const dim3 grid(n_seq, H, (max_rows + 127) / 128);
  auto go = [&](auto long_c, auto tail_c) {
    constexpr bool LONGK = decltype(long_c)::value, TAIL = decltype(tail_c)::value;
    static size_t set_rows = 0;
    if (lds > set_rows) {
      (void)hipFuncSetAttribute((const void*)k_attention_rows<LONGK, TAIL>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      set_rows = lds;
    }
    k_attention_rows<LONGK, TAIL><<<grid, 512, lds, s>>>((const bf16_t*)q, (const bf16_t*)K, (const bf16_t*)V, (bf16_t*)out, desc, H * 64, scale);
  };
  if (max_keys > kRowsKeys) go(std::true_type{}, std::true_type{});
  else if (max_keys >= kLongKeys) go(std::true_type{}, std::false_type{});
  else go(std::false_type{}, std::false_type{});
}

// Cross-attention with its query projection for a source capacity of kLongKeys or more (head width 64, d 512 or 1024,
// bf16: launch_crossq_attention has checked that and chosen the rows per workgroup).  One row tile per workgroup: the
// waves split the keys (k_crossq_attention_split); several: every wave walks all keys with the four accumulators
// (k_crossq_attention<.., LONGK = true>).  false: the tiles do not fit in LDS or two launches are faster, the caller launches
// projection and attention separately.
bool launch_crossq_attention_long(const LnA& ln, const void* A, const void* W, const float* bias, const void* K, const void* V,
                                  void* out, const SeqDesc* desc, int n_seq, int max_rows, int H, int chunk, int max_keys,
                                  hipStream_t s) {
  const int d = H * 64;
  const int mt = (std::min(max_rows, chunk) + 15) / 16;
  const float scale = 1.0f / sqrtf(64.0f);
  if (mt == 1 && 16 * (size_t)(d + 16) * 2 <= 4 * (size_t)kSplitWaveElems * 2) {
    if (n_seq <= 0 || max_rows <= 0) return true;
    const size_t shs = crossq_split_lds_bytes();
    dim3 g(n_seq, H, (max_rows + 15) / 16);
    auto go = [&](auto nv_c) {
      constexpr int NV = decltype(nv_c)::value;
      static bool set = false;
      if (!set) {
        (void)hipFuncSetAttribute((const void*)k_crossq_attention_split<NV>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shs);
        set = true;
      }
      k_crossq_attention_split<NV><<<g, 256, shs, s>>>(desc, scale, (const bf16_t*)W, (const bf16_t*)K, (const bf16_t*)V, ln.x, ln.g,
                                                       ln.b, ln.y, (const bf16_t*)A, bias, (bf16_t*)out);
    };
    if (d == 512) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
    return true;
  }
  // Model width 1024: projection and k_attention_rows as two launches are faster (a workgroup here reads 128 KB of the query
  // matrix and stages one head's values for 32 or 64 rows, k_attention_rows for 128 with twice the waves).  Verify forward, one
  // launch / two, us: 8 x 40 rows 555 / 498, 16 x 25 rows 588 / 525, 4 x 72 rows 539 / 488 (512 source tokens), 479 / 469 for
  // 16 x 25 rows of 100; drafter forward, 8 sources of 512, 502 / 451.  Width 512 goes on with one: half the matrix, and 16 x 40 rows
  // take 409 / 368 with 512 source tokens but 324 / 334 with 100.
  if (d == 1024) return false;
  const size_t sh = crossq_lds_bytes(max_keys, mt, d);
  if (sh > 160 * 1024) return false;
  if (n_seq <= 0 || max_rows <= 0) return true;
  dim3 g(n_seq, H, (max_rows + chunk - 1) / chunk);
  static size_t set_for = 0;
  if (sh > set_for) {
    (void)hipFuncSetAttribute((const void*)k_crossq_attention<2, 0, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    set_for = sh;
  }
  k_crossq_attention<2, 0, true><<<g, 256, sh, s>>>(desc, chunk, scale, (const bf16_t*)W, (const bf16_t*)K, (const bf16_t*)V, ln.x, ln.g,
                                                    ln.b, ln.y, (const bf16_t*)A, bias, (bf16_t*)out);
  return true;
}

}  // namespace ad

// Attention of the fp32 mode on the matrix cores (v_mfma_f32_16x16x4_f32).  A code object of its own, as the fp32 GEMMs.
#include <hip/hip_runtime.h>

#include "ad_device.h"

namespace ad {

// One workgroup per (sequence, head, 16 query rows); bound by the latency of a short chain of loads and products, so its
// four waves share each step: the score tiles (16 keys each, wave w: tiles w, w + 4, ..) go to LDS scaled and masked; the
// softmax, four rows per wave, takes the exact row maximum, p = exp(s - max), and a denominator whose 16 lanes each add
// their keys (key % 16 = lane) in ascending order; the output product walks all keys in ascending order, wave w for
// channels 16 w .. + 15 (and 64 further on), its first values requested at the kernel's start.
// A fragment is one 16-byte load (4 consecutive channels or probabilities) or four 4-byte loads (values) per lane, and
// MFMA i multiplies element i of both, as in the fp32 GEMM.  Keys a row does not see have probability 0; should a result not be
// finite, the product is taken once more with the values that are not finite held out of the units that rows see in part (0 x Inf
// is NaN) and added for the rows that see them only: a row's result depends on the keys it sees alone, not on the block it
// is verified in.
// (base model, 4 sequences of 10..60 keys, kernel trace average: 4.4 us; one wave per query row on the vector units with
// keys and values staged in LDS, which this replaces: 14.5 us)
template <int DH>
__global__ __launch_bounds__(256) void k_attention_f32(const float* __restrict__ q, const float* __restrict__ Kb,
                                                       const float* __restrict__ Vb, float* __restrict__ out,
                                                       const SeqDesc* __restrict__ desc, int d, float scale, int ld) {
  constexpr int KS = DH / 16, CW = (DH + 63) / 64, PRE = 4;   // 16-channel units, channel tiles per wave, key units requested ahead
  extern __shared__ float4 f32_scores[];
  float* S = (float*)f32_scores;   // [16][ld]
  float* L = S + 16 * ld;          // [16] denominators
  const SeqDesc sd = desc[blockIdx.x];
  const int row_begin = blockIdx.z * 16, h = blockIdx.y;
  if (row_begin >= sd.nq) return;
  const int row_end = min(sd.nq, row_begin + 16);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, kq = lane >> 4;
  const int nk_all = sd.causal ? sd.nk_base + row_end : sd.nk_base, nt = (nk_all + 15) >> 4;
  const int nk_full = sd.causal ? sd.nk_base + row_begin + 1 : sd.nk_base;   // keys every row of the tile sees
  auto f4 = [](const float* p) { return __builtin_bit_cast(float4, ldg16(p)); };
  float4 qf[KS], kf[KS];
  const float* qp = q + (size_t)(sd.q_row0 + min(row_begin + r, row_end - 1)) * d + h * DH + 4 * kq;
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = f4(qp + 16 * s);
  auto request_keys = [&](int t) {   // (indices clamped to the last key: what lies past it is masked)
    const float* kp = Kb + (size_t)(sd.kv_row0 + min(16 * t + r, nk_all - 1)) * d + h * DH + 4 * kq;
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = f4(kp + 16 * s);
  };
  request_keys(wave);
  const bool has_ch = 16 * wave < DH;
  const float* vp = Vb + (size_t)sd.kv_row0 * d + h * DH + 16 * (has_ch ? wave : 0) + r;
  float v[PRE][CW][4];
  auto request_values = [&](int p, int u) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < CW; ++c) v[p][c][i] = gload(vp + (size_t)min(16 * u + 4 * kq + i, nk_all - 1) * d + 64 * c);
  };
#pragma unroll
  for (int p = 0; p < PRE; ++p) request_values(p, p);
  auto unit = [](const float4& a, const float4& b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, c, 0, 0, 0);
  };
  for (int t = wave; t < nt; t += 4) {
    f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) s4 = unit(qf[s], kf[s], s4);
    if (t + 4 < nt) request_keys(t + 4);
    const int key = 16 * t + r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int nkr = sd.causal ? sd.nk_base + row_begin + 4 * kq + i + 1 : sd.nk_base;
      S[(4 * kq + i) * ld + key] = key < nkr ? s4[i] * scale : -INFINITY;
    }
  }
  __syncthreads();
  {
    float* sr = S + (4 * wave + kq) * ld + r;   // row 4 wave + kq, this lane's keys r, r + 16, ..
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
  __syncthreads();
  if (!has_ch) return;
  f32x4 acc[CW];
#pragma unroll
  for (int c = 0; c < CW; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int u0 = 0; u0 < nt; u0 += PRE) {
#pragma unroll
    for (int p = 0; p < PRE; ++p) {
      if (u0 + p < nt) {
        const float4 pf = *(const float4*)(S + r * ld + 16 * (u0 + p) + 4 * kq);
#pragma unroll
        for (int c = 0; c < CW; ++c) acc[c] = unit(pf, float4{v[p][c][0], v[p][c][1], v[p][c][2], v[p][c][3]}, acc[c]);
      }
    }
    if (u0 + PRE < nt) {
#pragma unroll
      for (int p = 0; p < PRE; ++p) request_values(p, u0 + PRE + p);
    }
  }
  bool odd = false;
#pragma unroll
  for (int c = 0; c < CW; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) odd |= !__builtin_isfinite(acc[c][i]);
  if (__any(odd)) {   // the product once more, in the same order, with those values held apart
#pragma unroll
    for (int c = 0; c < CW; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int u = 0; u < nt; ++u) {
      const bool in_part = 16 * (u + 1) > nk_full;   // (the same for the whole workgroup)
      float x[CW][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = 16 * u + 4 * kq + i;
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          x[c][i] = gload(vp + (size_t)min(key, nk_all - 1) * d + 64 * c);
          if (in_part && (key >= nk_all || !__builtin_isfinite(x[c][i]))) x[c][i] = 0.f;
        }
      }
      const float4 pf = *(const float4*)(S + r * ld + 16 * u + 4 * kq);
#pragma unroll
      for (int c = 0; c < CW; ++c) acc[c] = unit(pf, float4{x[c][0], x[c][1], x[c][2], x[c][3]}, acc[c]);
      if (!in_part) continue;
#pragma unroll 1
      for (int key = 16 * u; key < min(nk_all, 16 * u + 16); ++key) {
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const float y = gload(vp + (size_t)key * d + 64 * c);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int nkr = sd.causal ? sd.nk_base + row_begin + 4 * kq + i + 1 : sd.nk_base;
            if (!__builtin_isfinite(y) && key < nkr) acc[c][i] += S[(4 * kq + i) * ld + key] * y;
          }
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = row_begin + 4 * kq + i;
    if (row < row_end) {
#pragma unroll
      for (int c = 0; c < CW; ++c) gstore(out + (size_t)(sd.q_row0 + row) * d + h * DH + 16 * wave + 64 * c + r, acc[c][i] / L[4 * kq + i]);
    }
  }
}

void launch_attention_f32(const float* q, const float* K, const float* V, float* out, const SeqDesc* desc, int n_seq,
                          int max_rows, int H, int dh, int max_keys, hipStream_t s) {
  const int ld = (max_keys + 63) / 64 * 64 + 4;   // four dwords past a multiple of 64 banks
  const size_t lds = (16 * (size_t)ld + 16) * 4;
  const dim3 g(n_seq, H, (max_rows + 15) / 16);
  const float scale = 1.0f / sqrtf((float)dh);
#define AD_ATT(DH)                                                                                                        \
  do {                                                                                                                    \
    static size_t set_for = 0;                                                                                            \
    if (lds > set_for) {                                                                                                  \
      (void)hipFuncSetAttribute((const void*)k_attention_f32<DH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);  \
      set_for = lds;                                                                                                      \
    }                                                                                                                     \
    k_attention_f32<DH><<<g, 256, lds, s>>>(q, K, V, out, desc, H * dh, scale, ld);                                       \
  } while (0)
  switch (dh) {
    case 16: AD_ATT(16); break;
    case 32: AD_ATT(32); break;
    case 64: AD_ATT(64); break;
    default: AD_ATT(128); break;
  }
#undef AD_ATT
}

}  // namespace ad

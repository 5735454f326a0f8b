// fp32 GEMMs on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation).
// A source file, hence a code object, of its own: the bf16 kernels' speed follows the size of theirs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ad_device.h"

namespace ad {

// C[M,N] = A[M,K] . W[N,K]^T, both row-major.  A workgroup of four waves owns MT*16 rows x SP*16 columns and its waves
// split K: wave w takes the w-th quarter of the 16-wide k units (f32_quarter), so that a 16 x 16 tile of K = 512 is four
// chains of 32 MFMAs (0.4 us) instead of one of 128, and the four partial sums are combined through LDS as
// (p0 + p1) + (p2 + p3).  Within a unit an operand fragment is one 16-byte load per lane (lane = row or column l%16,
// k = 4 (l/16) .. + 3) and MFMA i of the unit multiplies element i of both fragments, i.e. the k values i, 4 + i, 8 + i, 12 + i:
// no lane exchange and no trip through LDS lies between memory and the matrix cores.  The order of an element's sum
// depends on K alone: every launch shape (and f32_dot_tile) gives the same bits.
// D units are in flight per wave; a unit's registers are refilled as soon as its MFMAs are issued.
// LNV >= 0: A is LayerNorm(ln.x), the LayerNorm kernel's statistics and values: the waves normalise the workgroup's rows
// into LDS (behind the request of the first weights) and the fragments come from there; the workgroups of group 0 also
// keep the fp32 rows.  LNV: ln_vector_width(K), 0 also standing for K <= 128.
struct F32Quarter { int begin, end; };
__device__ __forceinline__ F32Quarter f32_quarter(int K, int w) {
  const int units = K >> 4, per = (units + 3) >> 2;
  return F32Quarter{min(units, w * per), min(units, (w + 1) * per)};
}
__device__ __forceinline__ f32x4 f32_mfma_unit(const float4& a, const float4& b, f32x4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, c, 0, 0, 0);
}
__device__ __forceinline__ float4 ldg_f4(const float* p) { return __builtin_bit_cast(float4, ldg16(p)); }

// Rows row0 .. row0 + NR - 1 of the workgroup's tile into LDS through LayerNorm, by one wave.
template <int LNV, int NR, typename F>
__device__ __forceinline__ void f32_stage_ln(const LnA& ln, float* At, int ld, int row0, int m0, int M, int K, int lane,
                                             bool keep_y, const F& after_loads) {
  constexpr int NV = LNV > 0 ? LNV : 1;
  float4 x4[NR][NV];
  float x2[NR][2];
  float mean[NR], rstd[NR];
  float4 g4[NV], b4[NV];
  float g2[2], b2[2];
  if constexpr (LNV > 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) { g4[j] = ldg_f4(ln.g + 4 * lane + 256 * j); b4[j] = ldg_f4(ln.b + 4 * lane + 256 * j); }
  } else {
    ln_load<2>(ln.g, K, lane, g2);
    ln_load<2>(ln.b, K, lane, b2);
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const float* xr = ln.x + (size_t)min(m0 + row0 + i, M - 1) * K;
    if constexpr (LNV > 0) ln_load4<NV>(xr, lane, x4[i]);
    else ln_load<2>(xr, K, lane, x2[i]);
  }
  after_loads();
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    if constexpr (LNV > 0) ln_stats4<NV>(x4[i], K, mean[i], rstd[i]);
    else ln_stats<2>(x2[i], K, lane, mean[i], rstd[i]);
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int m = m0 + row0 + i;
    const bool keep = keep_y && m < M;
    if constexpr (LNV > 0) {
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int c = 4 * lane + 256 * j;
        const float4 o = float4{ln_value(x4[i][j].x, mean[i], rstd[i], g4[j].x, b4[j].x), ln_value(x4[i][j].y, mean[i], rstd[i], g4[j].y, b4[j].y),
                                ln_value(x4[i][j].z, mean[i], rstd[i], g4[j].z, b4[j].z), ln_value(x4[i][j].w, mean[i], rstd[i], g4[j].w, b4[j].w)};
        *(float4*)(At + (row0 + i) * ld + c) = o;
        if (keep) *(float4*)(ln.y + (size_t)m * K + c) = o;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = lane + 64 * j;
        if (c < K) {
          const float o = ln_value(x2[i][j], mean[i], rstd[i], g2[j], b2[j]);
          At[(row0 + i) * ld + c] = o;
          if (keep) gstore(ln.y + (size_t)m * K + c, o);
        }
      }
    }
  }
}

// KIND 0: layer epilogues, 1: arg max (and logits, where asked for), 2: EPI_COUNT
template <int MT, int SP, int D, int KIND, int LNV>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ A, const float* __restrict__ W, int M, int N,
                                                  int K, int groups, int chunks, const float* __restrict__ ln_x,
                                                  const float* __restrict__ ln_g, const float* __restrict__ ln_b,
                                                  float* __restrict__ ln_y, Epi e) {
  __shared__ f32x4 part[4][MT * SP][64];
  extern __shared__ float4 f32_rows[];   // LNV >= 0: [MT * 16][K + 4]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  // workgroup -> (strip group, row chunk): a group's row chunks back to back on one XCD, whose L2 then holds its weights
  int group, chunk;
  if (groups >= 8) {
    const int t = blockIdx.x >> 3;
    chunk = t % chunks;
    group = (t / chunks) * 8 + (blockIdx.x & 7);
    if (group >= groups) return;
  } else {
    group = blockIdx.x % groups;
    chunk = blockIdx.x / groups;
  }
  const int m0 = chunk * MT * 16, n_strips = N >> 4, s0 = group * SP;
  const F32Quarter qu = f32_quarter(K, wave);
  const int n = qu.end - qu.begin;
  const float *ap[MT], *wp[SP];
#pragma unroll
  for (int t = 0; t < MT; ++t) ap[t] = A + (size_t)min(m0 + 16 * t + r, M - 1) * K + 4 * kq;   // (rows past M: computed, never stored)
#pragma unroll
  for (int j = 0; j < SP; ++j) wp[j] = W + (size_t)(16 * min(s0 + j, n_strips - 1) + r) * K + 4 * kq;
  float4 a[D][MT], b[D][SP];
  float* At = (float*)f32_rows;
  const int ld = K + 4;   // (four dwords past a multiple of 64 banks: a fragment read meets no bank twice)
  // unit u (clamped: a unit past the end is requested again and not used)
  auto request_a = [&](int i, int u) {
    const int k0 = 16 * max(0, min(u, qu.end - 1));
#pragma unroll
    for (int t = 0; t < MT; ++t) a[i][t] = LNV >= 0 ? *(const float4*)(At + (16 * t + r) * ld + 4 * kq + k0) : ldg_f4(ap[t] + k0);
  };
  auto request_b = [&](int i, int u) {
    const int k0 = 16 * max(0, min(u, qu.end - 1));
#pragma unroll
    for (int j = 0; j < SP; ++j) b[i][j] = ldg_f4(wp[j] + k0);
  };
  if constexpr (LNV >= 0) {
    LnA ln;
    ln.x = ln_x; ln.g = ln_g; ln.b = ln_b; ln.y = ln_y;
    f32_stage_ln<LNV, MT * 4>(ln, At, ld, wave * MT * 4, m0, M, K, lane, KIND == 0 && group == 0, [&]() {
#pragma unroll
      for (int i = 0; i < D; ++i) request_b(i, qu.begin + i);
    });
    __syncthreads();
#pragma unroll
    for (int i = 0; i < D; ++i) request_a(i, qu.begin + i);
  } else {
#pragma unroll
    for (int i = 0; i < D; ++i) { request_a(i, qu.begin + i); request_b(i, qu.begin + i); }
  }
  // tile x = j * MT + t is finished by wave x % 4 (KIND 0) or wave t % 4 (a row's columns meet in one wave)
  constexpr int NT = (MT * SP + 3) / 4;
  EpiRegs<1> g[NT];
  if constexpr (KIND == 0) {
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const int x = wave + 4 * q, t = x % MT, j = x / MT;
      if (x < MT * SP && s0 + j < n_strips) epi_preload<1>(e, 1, m0 + 16 * t, (s0 + j) << 4, M, N, lane, g[q]);
    }
  }
  f32x4 acc[SP][MT];
#pragma unroll
  for (int j = 0; j < SP; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int rounds = (n + D - 1) / D;
  for (int rd = 0; rd + 1 < rounds; ++rd) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int j = 0; j < SP; ++j)
            acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32((&a[i][t].x)[c], (&b[i][j].x)[c], acc[j][t], 0, 0, 0);
      request_a(i, qu.begin + (rd + 1) * D + i);
      request_b(i, qu.begin + (rd + 1) * D + i);
    }
  }
  const int rem = n - (rounds - 1) * D;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    if (i < rem && n > 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int j = 0; j < SP; ++j)
            acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32((&a[i][t].x)[c], (&b[i][j].x)[c], acc[j][t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < SP; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t) part[wave][j * MT + t][lane] = acc[j][t];
  __syncthreads();
  auto total = [&](int x) { return (part[0][x][lane] + part[1][x][lane]) + (part[2][x][lane] + part[3][x][lane]); };
  if constexpr (KIND == 0) {
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const int x = wave + 4 * q, t = x % MT, j = x / MT;
      if (x < MT * SP && s0 + j < n_strips) {
        const f32x4 c[1] = {total(x)};
        epi_apply<float, 1>(e, c, g[q], 1, m0 + 16 * t, (s0 + j) << 4, M, N, lane);
      }
    }
  } else {
    for (int t = wave; t < MT; t += 4) {
      float bv[4];
      int bi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + 16 * t + 4 * kq + i;
        bv[i] = KIND == 2 ? e.thr[min(m, M - 1)] : -INFINITY;
        bi[i] = KIND == 2 ? 0 : (s0 << 4) + r;
      }
#pragma unroll
      for (int j = 0; j < SP; ++j) {
        if (s0 + j >= n_strips) break;
        const f32x4 v = total(j * MT + t);
        const int col = ((s0 + j) << 4) + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = m0 + 16 * t + 4 * kq + i;
          const bool better = v[i] > bv[i];   // (columns ascend: the lowest of equal ones stays)
          if constexpr (KIND == 2) {
            bi[i] += better ? 1 : 0;
          } else {
            bv[i] = better ? v[i] : bv[i];
            bi[i] = better ? col : bi[i];
            if (e.logits && m < M) gstore(e.logits + (size_t)m * N + col, v[i]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (KIND == 2) bi[i] = row16_sum_i(bi[i]);
        else argmax_row16(bv[i], bi[i]);
      }
      if (r == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = m0 + 16 * t + 4 * kq + i;
          if (m < M) {
            if constexpr (KIND == 1) gstore(e.part_val + (size_t)m * e.n_strips + group, bv[i]);
            gstore(e.part_idx + (size_t)m * e.n_strips + group, bi[i]);
          }
        }
      }
    }
  }
}

template <int MT, int SP, int D, int KIND, int LNV = -1>
static int launch_f32(const float* A, const float* W, int M, int N, int K, const Epi& e, hipStream_t s, const LnA& ln = LnA{}) {
  const int groups = (N / 16 + SP - 1) / SP, chunks = (M + 16 * MT - 1) / (16 * MT);
  const int grid = (groups >= 8 ? (groups + 7) / 8 * 8 : groups) * chunks;
  const size_t lds = LNV >= 0 ? (size_t)MT * 16 * (K + 4) * 4 : 0;
  if constexpr (LNV >= 0) {
    static size_t set_for = 0;
    if (lds > set_for) {
      (void)hipFuncSetAttribute((const void*)k_gemm_f32<MT, SP, D, KIND, LNV>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      set_for = lds;
    }
  }
  k_gemm_f32<MT, SP, D, KIND, LNV><<<grid, 256, lds, s>>>(A, W, M, N, K, groups, chunks, ln.x, ln.g, ln.b, ln.y, e);
  return groups;
}
static bool f32_fuses_ln(int K, int MT) { return (K <= 128 || K == 256 || K == 512 || K == 1024) && MT * 16 * (K + 4) * 4 <= 130 * 1024; }
// Rows x columns of a workgroup by the number of 16 x 16 tiles of the product: while those are fewer than the CUs' waves
// the smallest workgroup wins (latency: a tile's chain), with more of them operand traffic does and a fragment has to feed
// more MFMAs.  Measured at K = 512, us for <1,1> / <2,1> / <2,2> / <4,4>: N 512 x 240 rows 5.8 / 6.8 / 7.5 / 15.0, N 2048 x 60
// rows 5.8 / 5.4 / 6.2 / 15.1, x 120 rows 9.4 / 8.1 / 6.5 / 15.2, x 480 rows 29 / 24 / 18 / 16; vocabulary of 32000, <1,2> / <2,2> /
// <4,4>: 16 rows 14.5 / 16.6 / 28, 32 rows 25 / 19 / 27, 120 rows 87 / 60 / 51.
// (One thread per output element behind LDS tiles, which this replaces, took 18-29 us per launch at 1..60 rows of the base model.)
int launch_gemm_f32(const float* A, const float* W, int M, int N, int K, const Epi& e, hipStream_t s, const LnA& ln) {
  const int tiles = N / 16 * ((M + 15) / 16);
  auto with_ln = [&](auto mt_c, auto sp_c, auto kind_c) {
    constexpr int MT = decltype(mt_c)::value, SP = decltype(sp_c)::value, KIND = decltype(kind_c)::value;
    if (!ln.x) return launch_f32<MT, SP, 8, KIND>(A, W, M, N, K, e, s);
    if (K <= 128) return launch_f32<MT, SP, 8, KIND, 0>(A, W, M, N, K, e, s, ln);
    if (K == 256) return launch_f32<MT, SP, 8, KIND, 1>(A, W, M, N, K, e, s, ln);
    if (K == 512) return launch_f32<MT, SP, 8, KIND, 2>(A, W, M, N, K, e, s, ln);
    return launch_f32<MT, SP, 8, KIND, 4>(A, W, M, N, K, e, s, ln);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  if (e.mode == EPI_ARGMAX || e.mode == EPI_COUNT) {
    auto go = [&](auto kind_c) {
      constexpr int KIND = decltype(kind_c)::value;
      if (tiles <= 256) return with_ln(I1{}, I1{}, kind_c);
      if (M <= 16) return with_ln(I1{}, I2{}, kind_c);
      if (M <= 32 || tiles <= 1536) return launch_f32<2, 2, 4, KIND>(A, W, M, N, K, e, s);
      return launch_f32<4, 4, 2, KIND>(A, W, M, N, K, e, s);
    };
    return e.mode == EPI_ARGMAX ? go(I1{}) : go(I2{});
  }
  if (tiles <= 320) return with_ln(I1{}, I1{}, I0{});
  if (tiles <= 640) return with_ln(I2{}, I1{}, I0{});
  return launch_f32<2, 2, 4, 0>(A, W, M, N, K, e, s);
}
// Whether that launch normalises the rows itself: the few-row shapes do (a launch less); with more rows than that
// every strip group would normalise them again, and a LayerNorm launch ahead is the shorter way.
bool gemm_f32_takes_ln(int M, int N, int K, const Epi& e) {
  const int tiles = N / 16 * ((M + 15) / 16);
  if (e.mode == EPI_ARGMAX || e.mode == EPI_COUNT) return (tiles <= 256 || M <= 16) && f32_fuses_ln(K, 1);
  return tiles <= 640 && f32_fuses_ln(K, tiles <= 320 ? 1 : 2);
}

// Score of each row's drafted token (GAD++).  One workgroup per 16 rows: the tile whose column j holds the weight row of
// row j's drafted token, its diagonal is what is asked for.  Fragments, quarters and combination are the kernel's above,
// and an MFMA output element is a dot product of its own, so lp[m] is the score that kernel computes for (m, token), bit for bit.
__global__ __launch_bounds__(256) void k_draft_logit_f32(const float* __restrict__ A, const float* __restrict__ W, int M,
                                                         int N, int K, const int* __restrict__ row_seq,
                                                         const int* __restrict__ row_start, const int* __restrict__ draft,
                                                         int k_max, float* __restrict__ lp, int* __restrict__ col) {
  __shared__ f32x4 part[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int m = min((int)blockIdx.x * 16 + r, M - 1), b = row_seq[m];
  const int tok = draft[b * k_max + (m - row_start[b])];
  const float* ap = A + (size_t)m * K + 4 * kq;
  const float* wp = W + (size_t)min(max(tok, 0), N - 1) * K + 4 * kq;
  const F32Quarter qu = f32_quarter(K, wave);
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int u = qu.begin; u < qu.end; ++u) acc = f32_mfma_unit(ldg_f4(ap + 16 * u), ldg_f4(wp + 16 * u), acc);
  part[wave][lane] = acc;
  __syncthreads();
  // lane (r, kq) holds rows 4 kq .. 4 kq + 3 of column r: row r's diagonal element sits in the lane with kq = r / 4
  if (wave == 0 && kq == (r >> 2) && (int)blockIdx.x * 16 + r < M) {
    const f32x4 c = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    const int i = r & 3;
    lp[m] = i == 0 ? c[0] : i == 1 ? c[1] : i == 2 ? c[2] : c[3];
    col[m] = tok;
  }
}
void launch_draft_logit_f32(const float* A, const float* W, int M, int N, int K, const int* row_seq, const int* row_start,
                            const int* draft, int k_max, float* lp, int* col, hipStream_t s) {
  k_draft_logit_f32<<<(M + 15) / 16, 256, 0, s>>>(A, W, M, N, K, row_seq, row_start, draft, k_max, lp, col);
}

}  // namespace ad

// bf16 GEMM for many rows (v_mfma_f32_16x16x32_bf16), a code object of its own.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ad_device.h"

namespace ad {

// C[M,N] = A[M,K] . W[N,K]^T, A row-major, W in operand tiles.  A workgroup of NW waves owns BM = 16*MT rows x BN = 16*SP*NW
// columns: every wave all the rows, SP of the 16-column strips.  K is walked 64 U at a time; a stage's rows go through registers
// into LDS (two buffers), its weights straight into operand registers, D stages requested ahead.
// The products are taken with the weights as the left operand, so that a lane holds four consecutive columns of one row:
// acc[t][i] = row m0 + 16 t + lane % 16, column n0 + 4 (lane / 16) + i.  Same value per element as strip_epilogue.
// tile_request: what the epilogue reads and the product does not decide (bias, residual values, destination rows).
template <int MT> struct TileRegs {
  f32x4 bias;
  uint4 res[MT];   // RESID: the residual values' bits; QKV / KV: .x = the destination row
};
template <int MT, int EM>
__device__ __forceinline__ void tile_request(const Epi& e, int m0, int n0, int M, int N, int lane, TileRegs<MT>& g) {
  const int r = lane & 15, c0 = 4 * (lane >> 4);
  g.bias = f32x4{0.f, 0.f, 0.f, 0.f};
  if (e.bias) g.bias = __builtin_bit_cast(f32x4, ldg16(e.bias + n0 + c0));
  const bool by_dst = EM == EPI_KV || (EM == EPI_QKV && n0 >= e.d);
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int m = min(m0 + 16 * t + r, M - 1);
    if constexpr (EM == EPI_RESID) g.res[t] = ldg16(e.resid + (size_t)m * N + n0 + c0);
    else g.res[t].x = by_dst ? (unsigned)gload(e.row_dst + m) : (unsigned)m;
  }
}
template <int MT, int EM>
__device__ __forceinline__ void tile_apply(const Epi& e, const f32x4 (&acc)[MT], const TileRegs<MT>& g, int m0, int n0, int M, int N,
                                           int lane) {
  const int r = lane & 15, c0 = 4 * (lane >> 4), d = e.d;
  bf16_t* base = (bf16_t*)e.out0;
  int ld = N, col = n0;
  if constexpr (EM == EPI_QKV) {
    const int part = n0 / d;   // (a strip lies inside one of the q / k / v ranges)
    ld = d; col = n0 - part * d;
    base = (bf16_t*)(part == 0 ? e.out0 : part == 1 ? e.out1 : e.out2);
  } else if constexpr (EM == EPI_KV) {
    const int layer = n0 / (2 * d), c = n0 - layer * 2 * d;
    ld = d; col = c < d ? c : c - d;
    base = (bf16_t*)((char*)(c < d ? e.out1 : e.out2) + layer * e.layer_stride);
  }
  base += col + c0;
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int m = m0 + 16 * t + r;
    if (m >= M) continue;
    f32x4 v = acc[t];
    if (e.bias) v += g.bias;
    if constexpr (EM == EPI_RESID) {
      v += __builtin_bit_cast(f32x4, g.res[t]);
      gstore((uint4*)((float*)e.out0 + (size_t)m * N + n0 + c0), __builtin_bit_cast(uint4, v));
    } else {
      if constexpr (EM == EPI_RELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
      }
      gstore((uint2*)(base + (size_t)g.res[t].x * ld), uint2{f2bf_pair(v[0], v[1]), f2bf_pair(v[2], v[3])});
    }
  }
}
// The same for a wave's SP strips together, by way of its own part of the LDS that held the rows: there a lane has 16 bytes of
// one row, and a store covers 64 (bf16, SP = 2) to 256 (fp32, SP = 4) consecutive bytes of a row where tile_apply's covers 32 or
// 64.  A tile's results leave all at once when its products are done, so these bytes are not hidden behind anything: of the
// 36.8 us of 3249 rows x N 4096 x K 1024 (27 MB of results) 12 were theirs.  tile_apply / this, us: that product 36.5 / 31.5,
// N 3072 32.6 / 28.9, N 12288 91.0 / 77.8, N 1024 with fp32 residuals 16.7 / 15.2 and K 4096 43.3 / 41.4; K = 512, 1120 rows, N
// 1536 / 2048 / 6144 6.1 / 8.4 / 17.3 and 5.3 / 7.1 / 13.9, N 512 with residuals 4.3 and 4.4.  (Whole rows of the workgroup's
// tile, 256 to 1024 bytes a row behind two barriers, measured the same as a wave's own part.)  The kernels of one strip a
// wave, whose operands are requested before the products, stay with tile_apply: their results are few.
// Everything a lane reads (bias, residual values, destination rows) is requested before the first result is put down.
// (The SP strips lie inside one of the q / k / v ranges, or one layer's key or value range: those are multiples of 512 columns,
// the width K, wide.)
template <int MT, int SP, int EM, int BYTES>
__device__ __forceinline__ void tile_finish(const Epi& e, const f32x4 (&acc)[SP][MT], char* tmp, int m0, int s0, int n_strips, int M,
                                            int N, int lane) {
  constexpr int EB = EM == EPI_RESID ? 4 : 2, LDB = SP * 16 * EB + 16;   // bytes of an element and of a row (16 apart: banks)
  constexpr int PL = SP * EB, RW = 64 / PL;                              // 16-byte pieces of a row, rows a store covers
  constexpr int CT = BYTES >= MT * 16 * LDB ? MT : BYTES >= MT * 8 * LDB ? MT / 2 : MT / 4;   // row tiles put down at once
  static_assert(CT >= 1 && CT * 16 * LDB <= BYTES, "a chunk fits the wave's part");
  constexpr int NI = CT * 16 / RW;
  if (s0 >= n_strips) return;
  const int r = lane & 15, c0 = 4 * (lane >> 4), d = e.d, n0 = s0 << 4;
  const int row = lane / PL, piece = lane % PL, col = piece * (16 / EB);
  const bool in_n = s0 + piece / EB < n_strips;
  f32x4 bias[SP];
#pragma unroll
  for (int j = 0; j < SP; ++j) {
    bias[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (e.bias) bias[j] = __builtin_bit_cast(f32x4, ldg16(e.bias + (min(s0 + j, n_strips - 1) << 4) + c0));
  }
  char* base = (char*)e.out0;
  size_t ld = (size_t)N * EB;
  bool by_dst = false;
  if constexpr (EM == EPI_QKV) {
    const int part = n0 / d;
    ld = (size_t)d * 2; by_dst = part > 0;
    base = (char*)(part == 0 ? e.out0 : part == 1 ? e.out1 : e.out2) + (n0 - part * d) * 2;
  } else if constexpr (EM == EPI_KV) {
    const int layer = n0 / (2 * d), c = n0 - layer * 2 * d;
    ld = (size_t)d * 2; by_dst = true;
    base = (char*)(c < d ? e.out1 : e.out2) + layer * e.layer_stride + (c < d ? c : c - d) * 2;
  } else {
    base += (size_t)n0 * EB;
  }
  base += piece * 16;
#pragma unroll
  for (int k0 = 0; k0 < MT; k0 += CT) {
    const int mr = m0 + 16 * k0 + row;
    uint4 res[NI];   // the residual values, or .x = the destination row
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int m = min(mr + i * RW, M - 1);
      if constexpr (EM == EPI_RESID) res[i] = ldg16(e.resid + (size_t)m * N + min(n0 + col, N - 4));
      else res[i].x = by_dst ? (unsigned)gload(e.row_dst + m) : (unsigned)m;
    }
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int j = 0; j < SP; ++j) {
        f32x4 v = acc[j][k0 + t];
        if (e.bias) v += bias[j];
        if constexpr (EM == EPI_RELU) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
        }
        char* at = tmp + (16 * t + r) * LDB + (16 * j + c0) * EB;
        if constexpr (EM == EPI_RESID) *(uint4*)at = __builtin_bit_cast(uint4, v);
        else *(uint2*)at = uint2{f2bf_pair(v[0], v[1]), f2bf_pair(v[2], v[3])};
      }
    // (a wave's LDS accesses take effect in order: only the compiler has to keep them so)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      uint4 v = *(const uint4*)(tmp + (i * RW + row) * LDB + piece * 16);
      if constexpr (EM == EPI_RESID) v = __builtin_bit_cast(uint4, __builtin_bit_cast(f32x4, v) + __builtin_bit_cast(f32x4, res[i]));
      const int m = mr + i * RW;
      if (in_n && m < M) gstore((uint4*)(base + (EM == EPI_RESID ? (size_t)m : (size_t)res[i].x) * ld), v);
    }
    asm volatile("" ::: "memory");
  }
}
template <int MT, int SP, int D, int U, int NW, int EM>
__global__ __launch_bounds__(64 * NW) void k_gemm_bf16_tile(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M,
                                                        int N, int K, int m_tiles, int n_tiles, Epi e) {
  constexpr int BM = 16 * MT, BK = 64 * U, NA = BM * U / (8 * NW), LD = BK + 16;   // NA 16-byte pieces of a stage's rows per thread
  static_assert(8 / U % D == 0, "D divides the stages of every K that is a multiple of 512");
  __shared__ __align__(16) bf16_t At[2][BM * LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  // consecutive workgroups go to consecutive XCDs: XCD x works through the x-th eighth of the tiles, column tile by column
  // tile, so that a column tile's weights stay in its L2 while the row tiles pass
  const int per = (m_tiles * n_tiles + 7) >> 3, lin = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || lin >= m_tiles * n_tiles) return;
  const int tn = lin / m_tiles, tm = lin - tn * m_tiles;
  const int m0 = tm * BM, n_strips = N >> 4, s0 = tn * NW * SP + wave * SP;
  const bf16_t* ap[NA];
  int a_lds[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int row = threadIdx.x / (8 * U) + 8 * NW / U * i, c = threadIdx.x % (8 * U);
    ap[i] = A + (size_t)min(m0 + row, M - 1) * K + 8 * c;
    a_lds[i] = row * LD + 8 * c;
  }
  const bf16_t* wp[SP];
#pragma unroll
  for (int j = 0; j < SP; ++j) wp[j] = W + (size_t)min(s0 + j, n_strips - 1) * 16 * K + lane * 8;
  const int n_st = K / BK, rounds = n_st / D;
  uint4 ra[D][NA], rb[D][SP][2 * U], af[2][2 * U][MT];
  auto req_a = [&](int q, int st) {
#pragma unroll
    for (int i = 0; i < NA; ++i) ra[q][i] = ldg16(ap[i] + BK * st);
  };
  auto req_b = [&](int q, int st) {
#pragma unroll
    for (int u = 0; u < 2 * U; ++u)
#pragma unroll
      for (int j = 0; j < SP; ++j) rb[q][j][u] = ldg16(wp[j] + (size_t)st * 1024 * U + u * 512);
  };
  auto put_a = [&](int q, int buf) {
#pragma unroll
    for (int i = 0; i < NA; ++i) *(uint4*)(At[buf] + a_lds[i]) = ra[q][i];
  };
  auto get_a = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 2 * U; ++u)
#pragma unroll
      for (int t = 0; t < MT; ++t) af[buf][u][t] = *(const uint4*)(At[buf] + (16 * t + r) * LD + 32 * u + 8 * kq);
  };
  // in the order of the loop's requests, so that its waits are exact from the first round on: rows of stages 0 and 1, then for
  // every stage q its weights and the rows of stage q + 2
  uint4 rp[2][NA];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int i = 0; i < NA; ++i) rp[q][i] = ldg16(ap[i] + BK * q);
#pragma unroll
  for (int q = 0; q < D; ++q) {
    req_a((q + 2) % D, min(q + 2, n_st - 1));
    req_b(q, q);
    __builtin_amdgcn_sched_barrier(0);
  }
  // (the small tiles have the registers to request the epilogue's operands here)
  constexpr bool PRE = MT * SP <= 4;
  TileRegs<MT> g[SP];
  if constexpr (PRE) {
#pragma unroll
    for (int j = 0; j < SP; ++j) tile_request<MT, EM>(e, m0, min(s0 + j, n_strips - 1) << 4, M, N, lane, g[j]);
    __builtin_amdgcn_sched_barrier(0);
  }
  f32x4 acc[SP][MT];
#pragma unroll
  for (int j = 0; j < SP; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int i = 0; i < NA; ++i) *(uint4*)(At[q] + a_lds[i]) = rp[q][i];
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  get_a(0);
  __syncthreads();
  // stage st: its row fragments are in registers; the next stage's are read, the one after that is written into the
  // buffer the present one came from, and the registers are refilled D stages ahead
  auto round = [&](auto more_c, int st0) {
    constexpr bool MORE = decltype(more_c)::value;
#pragma unroll
    for (int q = 0; q < D; ++q) {
      const int st = st0 + q;
      __builtin_amdgcn_sched_barrier(0);
      if (MORE || q + 2 < D) put_a((q + 2) % D, q & 1);
      if (MORE || q + 1 < D) get_a((q + 1) & 1);
      if (MORE) req_a((q + 2) % D, q + 2 < D ? st + 2 + D : min(st + 2 + D, n_st - 1));
#pragma unroll
      for (int u = 0; u < 2 * U; ++u)
#pragma unroll
        for (int j = 0; j < SP; ++j) {
#pragma unroll
          for (int t = 0; t < MT; ++t)
            acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, rb[q][j][u]), __builtin_bit_cast(bf16x8, af[q & 1][u][t]), acc[j][t], 0, 0, 0);
          if (MORE) rb[q][j][u] = ldg16(wp[j] + (size_t)(st + D) * 1024 * U + u * 512);
        }
      if (MORE || q + 2 < D) __builtin_amdgcn_sched_group_barrier(0x200, NA, 0);
#pragma unroll
      for (int g = 0; g < 2 * U * SP; ++g) {
#pragma unroll
        for (int i = 0; i < MT / 2; ++i) {
          const int at = g * (MT / 2) + i;   // of U * SP * MT steps
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          if ((MORE || q + 1 < D) && at < U * MT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          if (MORE && at < NA) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        if (MORE) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (MORE || q + 1 < D) __syncthreads();
    }
  };
  for (int rd = 0; rd + 1 < rounds; ++rd) round(std::true_type{}, rd * D);
  round(std::false_type{}, (rounds - 1) * D);
  if constexpr (PRE) {
#pragma unroll
    for (int j = 0; j < SP; ++j)
      if (s0 + j < n_strips) tile_apply<MT, EM>(e, acc[j], g[j], m0, (s0 + j) << 4, M, N, lane);
  } else {   // (the last stage's fragments were read before its barrier: the rows' LDS is free)
    constexpr int BYTES = 2 * BM * LD * 2 / NW;
    tile_finish<MT, SP, EM, BYTES>(e, acc, (char*)At + wave * BYTES, m0, s0, n_strips, M, N, lane);
  }
}

// The same product for many rows, where the matrix cores and not latencies are the bound: one register set per operand,
// refilled as soon as its last MFMA is issued (a row fragment from LDS for the next 32 k, the weights and the rows' pieces for the
// next stage), so that a 128 x 256 tile fits 256 registers and two workgroups a CU, which cover each other's waits.
// Three LDS buffers: one being read, the next one ready, one being written.
template <int MT, int SP, int EM>
__global__ __launch_bounds__(256, 2) void k_gemm_bf16_roll(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M,
                                                           int N, int K, int m_tiles, int n_tiles, Epi e) {
  constexpr int BM = 16 * MT, NA = BM / 32, LD = 64 + 16, BUF = BM * LD;
  __shared__ __align__(16) bf16_t At[3 * BUF];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int per = (m_tiles * n_tiles + 7) >> 3, lin = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || lin >= m_tiles * n_tiles) return;
  const int tn = lin / m_tiles, tm = lin - tn * m_tiles;
  const int m0 = tm * BM, n_strips = N >> 4, s0 = tn * 4 * SP + wave * SP;
  const bf16_t* ap[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) ap[i] = A + (size_t)min(m0 + (int)(threadIdx.x >> 3) + 32 * i, M - 1) * K + 8 * (threadIdx.x & 7);
  bf16_t* a_put = At + (threadIdx.x >> 3) * LD + 8 * (threadIdx.x & 7);
  const bf16_t* a_get = At + r * LD + 8 * kq;
  const bf16_t* wp[SP];
#pragma unroll
  for (int j = 0; j < SP; ++j) wp[j] = W + (size_t)min(s0 + j, n_strips - 1) * 16 * K + lane * 8;
  const int n_st = K >> 6;
  uint4 ra[NA], rb[2][SP], af[MT];
  {
    uint4 r1[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) ra[i] = ldg16(ap[i]);
#pragma unroll
    for (int i = 0; i < NA; ++i) r1[i] = ldg16(ap[i] + 64);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < SP; ++j) rb[u][j] = ldg16(wp[j] + u * 512);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NA; ++i) *(uint4*)(a_put + 32 * i * LD) = ra[i];
#pragma unroll
    for (int i = 0; i < NA; ++i) *(uint4*)(a_put + BUF + 32 * i * LD) = r1[i];
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) ra[i] = ldg16(ap[i] + 64 * min(2, n_st - 1));
  f32x4 acc[SP][MT];
#pragma unroll
  for (int j = 0; j < SP; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
#pragma unroll
  for (int t = 0; t < MT; ++t) af[t] = *(const uint4*)(a_get + 16 * t * LD);
  int cur = 0, nxt = BUF, wrt = 2 * BUF;
  for (int st = 0; st < n_st; ++st) {
    const int st1 = min(st + 1, n_st - 1), st3 = min(st + 3, n_st - 1);   // (past the end: requested again, not used)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NA; ++i) *(uint4*)(a_put + wrt + 32 * i * LD) = ra[i];
#pragma unroll
    for (int i = 0; i < NA; ++i) ra[i] = ldg16(ap[i] + 64 * st3);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bf16_t* an = u == 0 ? a_get + cur + 32 : a_get + nxt;
#pragma unroll
      for (int t = 0; t < MT; ++t) {
#pragma unroll
        for (int j = 0; j < SP; ++j)
          acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, rb[u][j]), __builtin_bit_cast(bf16x8, af[t]), acc[j][t], 0, 0, 0);
        af[t] = *(const uint4*)(an + 16 * t * LD);
      }
#pragma unroll
      for (int j = 0; j < SP; ++j) rb[u][j] = ldg16(wp[j] + (size_t)st1 * 1024 + u * 512);
    }
    __builtin_amdgcn_sched_group_barrier(0x200, NA, 0);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x008, SP, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (u == 0 && t < NA) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x020, SP, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    const int x = cur;
    cur = nxt; nxt = wrt; wrt = x;
  }
  constexpr int BYTES = 3 * BUF * 2 / 4;
  tile_finish<MT, SP, EM, BYTES>(e, acc, (char*)At + wave * BYTES, m0, s0, n_strips, M, N, lane);
}

template <int MT, int SP, int NW = 4, typename Go>
static void with_tile_shape(int M, int N, const Epi& e, const Go& go) {
  const int m_tiles = (M + 16 * MT - 1) / (16 * MT), n_tiles = (N / 16 + NW * SP - 1) / (NW * SP);
  const int grid = (m_tiles * n_tiles + 7) / 8 * 8;
  switch (e.mode) {
    case EPI_QKV: go(std::integral_constant<int, EPI_QKV>{}, grid, m_tiles, n_tiles); break;
    case EPI_KV: go(std::integral_constant<int, EPI_KV>{}, grid, m_tiles, n_tiles); break;
    case EPI_STORE: go(std::integral_constant<int, EPI_STORE>{}, grid, m_tiles, n_tiles); break;
    case EPI_RELU: go(std::integral_constant<int, EPI_RELU>{}, grid, m_tiles, n_tiles); break;
    default: go(std::integral_constant<int, EPI_RESID>{}, grid, m_tiles, n_tiles); break;
  }
}
template <int MT, int SP, int D, int U = 1, int NW = 4>
static void launch_tile(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epi& e, hipStream_t s) {
  with_tile_shape<MT, SP, NW>(M, N, e, [&](auto em_c, int grid, int m_tiles, int n_tiles) {
    k_gemm_bf16_tile<MT, SP, D, U, NW, decltype(em_c)::value><<<grid, 64 * NW, 0, s>>>(A, W, M, N, K, m_tiles, n_tiles, e);
  });
}
template <int MT, int SP>
static void launch_roll(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epi& e, hipStream_t s) {
  with_tile_shape<MT, SP>(M, N, e, [&](auto em_c, int grid, int m_tiles, int n_tiles) {
    k_gemm_bf16_roll<MT, SP, decltype(em_c)::value><<<grid, 256, 0, s>>>(A, W, M, N, K, m_tiles, n_tiles, e);
  });
}

// Which layer GEMMs come here rather than to the kernels that keep all of K of their rows in LDS.  Measured, us there / here, launches back
// to back with their operands in the last-level cache; a pending LayerNorm, 2.5-3 us as a launch of its own, is inside both figures:
//  K = 1024, LayerNorm pending: 64 / 80 / 96 / 97 / 130 / 250 / 626 rows x N 3072 4.9 / 5.1 / 6.9 / 6.8 / 7.1 / 9.7 / 21.2 there, 6.2 / 6.5 / 6.5 /
//    6.6 / 6.7 / 8.3 / 10.5 here; 64 / 65 / 130 / 250 / 626 rows x N 4096 4.7 / 6.3 / 8.3 / 12.2 / 26.2 there, 5.7 / 6.1 / 7.5 / 7.8 / 13.3
//    here; N 12288 (memory keys and values) 16 / 17 / 25 / 626 / 3249 rows 5.4 / 7.2 / 7.6 / 77 / 366 there, 6.0 / 6.0 / 6.1 / 23 / 84 here
//  K = 1024, none: N 1024 80 / 128 / 129 / 626 / 3249 rows 3.0 / 3.1 / 4.2 / 7.6 / 25.9 there, 3.4 / 3.3 / 3.3 / 5.3 / 14.7 here; N 512 and 768
//    128 / 160 / 161 rows 2.6 / 2.9 / 4.0 and 3.0 / 3.1 / 5.4 there, 3.3 / 3.3 / 3.3 and 3.4 / 3.4 / 3.4 here
//  K = 4096: beyond the two rounds of one workgroup per CU that k_gemm_bf16_kchain makes (its comment); N 1024 64 / 65 / 80 / 128 / 129 / 626 /
//    3249 rows 5.5 / 7.1 / 7.8 / 8.0 / 11.9 / 21.1 / 73.8 there, 7.1 / 7.2 / 7.2 / 7.1 / 7.2 / 13.4 / 39.9 here.  (So the second round no longer
//    pays with the matrix in the last-level cache: 8-11 % from 80 to 128 rows; the line stands as measured in a forward, where the matrix
//    comes from memory: 160 rows 15.3 / 13.6)
//  K = 512, LayerNorm pending: below 1408 columns never (N 512 520 / 2048 / 4000 rows 5.2 / 8.1 / 10.3 there, 5.6 / 9.3 / 12.5 here, N 1024 520 /
//    1345 / 2048 / 4000 rows 7.0 / 8.0 / 8.9 / 15.0 there, 6.4 / 8.8 / 10.5 / 16.1 here, N 1280 520 / 2048 / 3000 / 4000 rows 6.7 / 10.8 / 16.1 /
//    17.9 there, 6.5 / 11.6 / 14.5 / 19.0 here); below 2048 from 1400 rows (N 1408 1120 / 1345 / 1400 rows 8.8 / 9.1 / 11.9 there, 8.4 /
//    9.0 / 9.1 here, N 1536 1280 / 1345 / 1400 / 2048 rows 7.6 / 10.3 / 13.0 / 14.3 there, 8.9 / 9.9 / 10.1 / 11.8 here); below 3072 from 600
//    rows where the 16-wave workgroups need a second round (N 2048 512 / 600 / 800 / 1024 / 1025 / 1120 rows 6.7 / 7.7 / 8.0 / 8.8 / 10.8 / 10.9
//    there, 6.7 / 7.4 / 7.8 / 8.4 / 9.4 / 9.7 here, N 2080 567 / 599 / 620 / 900 rows 6.5 / 8.7 / 8.8 / 9.3 there, 7.4 / 7.5 / 7.5 / 8.1 here, N 2560
//    400 / 600 / 800 / 801 rows 6.8 / 12.6 / 13.2 / 10.6 there, 7.1 / 7.7 / 9.1 / 9.0 here); below 4096 from 513 rows (N 3072 256 / 400 / 512 / 513 /
//    1024 rows 5.8 / 7.4 / 7.8 / 10.1 / 12.4 there, 6.4 / 7.2 / 7.4 / 7.4 / 9.8 here); N 4096 160 / 256 / 257 / 300 rows 5.7 / 6.2 / 8.0 / 8.3 there
//    with the ReLU, whose epilogue is a constant there, 6.2 / 6.4 / 7.1 / 7.2 here, 130 / 161 / 211 rows of keys and values 6.7 / 6.9 / 7.1 there,
//    6.3 / 6.4 / 6.5 here; N 6144 96 / 128 / 160 / 161 / 1120 rows 6.7 / 6.9 / 7.0 / 9.6 / 28.0 there, 6.3 / 6.4 / 6.9 / 6.9 / 16.7 here
//  K = 512, none: N 512 400 / 519 / 576 / 1120 rows 2.6 / 3.2 / 3.2 / 5.1 there, 2.8 / 2.9 / 2.9 / 4.0 here, N 1536 256 / 400 / 520 / 1120 rows 3.4 /
//    4.7 / 6.1 / 8.3 there, 3.3 / 4.3 / 4.4 / 5.1 here
//  K = 2048: N 512 192 / 400 / 519 / 576 / 1024 rows 5.2 / 5.3 / 6.9 / 7.8 / 8.0 there, 4.6 / 4.7 / 4.9 / 4.9 / 7.2 here, 1025 / 1365 / 2048 / 2049
//    rows 8.0 / 8.7 / 11.4 / 17.2 there, 8.5 / 9.8 / 12.5 / 11.8 here: beyond 1024 rows the eight-wave workgroups while they make one round;
//    past it N 1024 1025 / 2048 rows 19.4 / 19.4 there, 11.8 / 14.6 here, N 2048 1365 rows 28.3 / 19.7.  (Below 520 rows the line was drawn
//    before the 32 x 32 tiles: N 1024 192 / 400 rows 5.3 / 7.1 there, 4.6 / 5.0 here, N 2048 192 / 400 rows 7.1 / 11.4 and 4.9 / 7.8)
//  K = 1536: the same from 1600 rows, N 512 1300 / 1600 / 1800 / 2048 / 2049 rows 8.5 / 8.6 / 8.9 / 9.4 / 12.7 there, 7.4 / 9.2 / 9.8 / 10.7 / 9.6 here;
//    N 512 / 1024 / 1536 128 rows 4.6 / 4.7 / 4.8 there, 3.9 / 4.0 / 4.1 here
// Where "here" is ahead on the near side of a line, the line is as it was drawn with tile_apply's stores.
bool gemm_tile_takes(int M, int N, int K, bool has_ln, int mode) {
  if (K % 512 || K < 512 || mode == EPI_ARGMAX || mode == EPI_COUNT) return false;
  if (K == 512 && has_ln) {
    if (N < 2048) return N >= 1408 && M >= 1400;
    if (N < 3072) return M >= 600 && !gemm_one_round(M, N, 16);
    return M > (N < 4096 ? 512 : N < 6144 && mode == EPI_RELU ? 256 : 160);
  }
  if (K == 512) return M >= 520;
  if (K == 2048) return M >= 520 && !(M > 1024 && gemm_one_round(M, N, 8));
  if (K == 4096) return M > 160 || (N / 16) * ((M + 15) / 16) > 512;
  if (K == 1536 && M > 1600 && gemm_one_round(M, N, 8)) return false;
  return has_ln ? M > (N > 4096 ? 16 : N == 4096 ? 64 : 96) : M > (K == 1024 && N < 1024 ? 160 : 128);
}
// Tile by the number of workgroups w(rows x columns of a tile): the smallest while they fit the CUs at once (a stage's latency is
// the bound), larger ones as soon as there are enough of them (operand traffic from L2 and then the matrix cores are).
// 32 x 32 (two waves) while those fit: the small tiles are bound by what a CU takes from L2 (32 x 64: 12 KB per 64 k in 82 ns, 95 % of
// 64 bytes a clock), and 32 x 32 takes 8 KB on twice the CUs.  Both walk 128 k a stage, half the barriers.  32 x 64 with 64 k a
// stage / with 128 / 32 x 32, us: N 1024 x 200 rows, K 1024 3.65 / 3.57 / 3.45, K 4096 8.04 / 7.63 / 7.23, K 1536 4.42 / 4.26 / 4.08; N 512 x
// 400 rows, K 2048 5.14 / 4.94 / 4.69; past the line N 1024 x 400 rows, K 1024 3.84 / 3.76 / 4.45, K 4096 9.76 / 9.72 / 11.2.  Eight stages of
// 64 k ahead 3.89 and 8.13 at 200 rows; the 64-row tiles gained nothing from longer stages.
// 64 x 128: four stages ahead while there is one workgroup per CU, two (and two workgroups per CU) beyond: K = 1536, N 1536 x 700 /
// 1024 / 1600 rows (w 132 / 192 / 300) 10.5 / 11.8 / 19.5 us with four, 12.6 / 13.8 / 18.0 with two; K = 512, N 3072 x 519 rows (216)
// 8.9 / 9.4; K = 2048, N 1024 x 2049 rows (264) 21.9 / 19.3.
// 128 x 128 rolling: two workgroups per CU; up to 640 of them a second round is nearly empty and the 64 x 128 rolling shape
// wins: K = 512, N 3072 x 3000 rows (w(128, 128) 576) 28.5 / 26.2 us, K = 1536, N 6144 x 1300 (528) 54.0 / 44.0; but K = 2048,
// N 2048 x 4096 (512) 45.1 / 49.7, K = 1024, N 3072 x 3531 (672) 40.8 / 43.1.
// (These figures are of all kernels with tile_apply's stores.)  With tile_finish at K = 1024 (64 x 128
// two stages ahead / 64 x 128 rolling / 128 x 128 / 128 x 256): N 3072 x 626 rows (w 240) 7.3 / 8.4 / 10.9 / 15.9 us (four stages
// 7.1), x 2000 (768) 18.6 / 19.0 / 19.7 / 21.0, x 3249 (1224) 29.1 / 29.4 / 30.4 / 29.6; N 4096 x 2000 (1024) 24.2 / 24.0 / 21.6 /
// 23.2, x 3249 (1632) 39.1 / 39.3 / 38.1 / 32.1 (850 TFLOP/s); N 12288 x 3249 107 / 109 / 100 / 81 (1010 TFLOP/s).
void launch_gemm_tile(const void* A_, const void* W_, int M, int N, int K, const Epi& e, hipStream_t s) {
  const bf16_t *A = (const bf16_t*)A_, *W = (const bf16_t*)W_;
  auto w = [&](int rows, int cols) { return ((M + rows - 1) / rows) * ((N + cols - 1) / cols); };
  if (w(32, 32) <= 256) launch_tile<2, 1, 2, 2, 2>(A, W, M, N, K, e, s);
  else if (w(32, 64) <= 256) launch_tile<2, 1, 2, 2>(A, W, M, N, K, e, s);
  else if (w(64, 64) <= 256) launch_tile<4, 1, 4>(A, W, M, N, K, e, s);
  else if (w(64, 128) <= 256) launch_tile<4, 2, 4>(A, W, M, N, K, e, s);
  else if (w(64, 128) <= 450) launch_tile<4, 2, 2>(A, W, M, N, K, e, s);
  else if (w(64, 128) > 900 && w(128, 256) >= 350) launch_roll<8, 4>(A, W, M, N, K, e, s);
  else if (w(64, 128) > 900 && (w(128, 128) <= 512 || w(128, 128) > 640)) launch_roll<8, 2>(A, W, M, N, K, e, s);
  else launch_roll<4, 2>(A, W, M, N, K, e, s);
}

}  // namespace ad

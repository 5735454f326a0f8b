// bf16 GEMMs of few rows whose K is several 512-slices: a workgroup's waves share K.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ad_device.h"

namespace ad {

// ---------------------------------------------------------------- rows as they are: K = 1024, 2048, 4096, up to 160 rows
// C = A . W^T for FFN2 and the attention output projections of the wide model.  The A-in-LDS kernel (k_gemm_bf16_astat) walks a strip's
// 512-slices one after the other in one wave, a round trip to memory per slice.  Here a workgroup
// owns one 16-column strip of one 16-row chunk and every wave one slice: every
// wave requests its slice of the rows (into an LDS tile of its own: no barrier before the first
// MFMA; fragments requested straight from the row-major rows, 16 rows x 64 bytes per wave
// instruction, measured 1 us slower per launch) and of the weights at once, so the workgroup waits
// for memory once.  The sum itself stays one chain: the accumulators go from
// wave to wave through LDS in slice order (k ascending, 32 at a time, one accumulator per element:
// the same bits as every other GEMM kernel here), and the wave of the last slice runs the epilogue.
// Rows past M are not requested, four at a time (what the tile holds in their place reaches no row that is stored): with one
// row a workgroup takes in a fifth of the bytes, 4.26 -> 3.54 us at K = 2048.
// K = 4096: eight waves, a wave per slice, while that is at most one workgroup per CU (136 KB of LDS each); four waves of two
// slices, the second requested once the first is multiplied, two workgroups per CU, up to twice as many.  Wide model, N 1024,
// matrix from memory / from the last-level cache, eight waves / four, us: 64 rows 6.8 / 6.4 and 9.1 / 8.0, 80 rows 10.9 / 10.6
// and 9.9 / 8.7, 100 rows 11.1 / 10.8 and 10.1 / 8.9, 128 rows 11.5 / 11.1 and 10.5 / 9.3; in a verify forward of 4 x 25 rows (kernel
// trace) 12.2 and 10.4.  The tiled kernel's few workgroups wait for memory stage after stage: 11.8 / 8.9 at 100 rows, 12.7 in the
// forward, but with more workgroups than that it wins (N 2048, 96 rows 14.0 / 9.2 against 17.2 / 15.8).
constexpr int kChainLd = 512 + 16;   // row stride of a wave's tile (elements): 32 bytes past a multiple of 64
static size_t kchain_lds_bytes(int nw) { return (size_t)nw * 16 * kChainLd * 2 + 64 * 16; }
template <int NS, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_gemm_bf16_kchain(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                              int M, int N, int K, int n_strips, Epi e) {
  extern __shared__ uint4 kchain_lds[];   // [wave][16 rows][LD], the accumulators handed on
  f32x4* hand = (f32x4*)((bf16_t*)kchain_lds + NW * 16 * kChainLd);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int strip = blockIdx.x % n_strips, m0 = (blockIdx.x / n_strips) * 16, n0 = strip << 4;
  bf16_t* At = (bf16_t*)kchain_lds + wave * 16 * kChainLd;
  const bf16_t* a_lane = At + r * kChainLd + kq * 8;
  uint4 b[16];
  auto request = [&](int slice) {
    uint4 av[16];
    const bf16_t* ap = A + slice * 512 + lane * 8;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q == 0 || m0 + 4 * q < M) {
#pragma unroll
        for (int i = 4 * q; i < 4 * q + 4; ++i) av[i] = ldg16(ap + (size_t)min(m0 + i, M - 1) * K);
      } else {
#pragma unroll
        for (int i = 4 * q; i < 4 * q + 4; ++i) av[i] = uint4{0u, 0u, 0u, 0u};
      }
    }
    const bf16_t* wp = W + (size_t)n0 * K + (size_t)slice * 8192 + lane * 8;
#pragma unroll
    for (int u = 0; u < 16; ++u) b[u] = ldg16(wp + u * 512);
#pragma unroll
    for (int i = 0; i < 16; ++i) *(uint4*)(At + i * kChainLd + lane * 8) = av[i];
  };
  if (NS >= NW || wave < NS) request(wave);
  constexpr int LAST = (NS - 1) % NW;
  EpiRegs<1> g;
  if (wave == LAST) epi_preload<1>(e, 1, m0, n0, M, N, lane, g);
  f32x4 acc[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int p = 0; p < NS; ++p) {
    if (wave == p % NW) {
      if (p > 0) acc[0] = hand[lane];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, *(const uint4*)(a_lane + 32 * u)), __builtin_bit_cast(bf16x8, b[u]), acc[0], 0, 0, 0);
      if (p + 1 < NS) hand[lane] = acc[0];
      if (p + NW < NS) request(p + NW);   // (the wave's own tile and registers: no barrier)
    }
    if (p + 1 < NS) __syncthreads();
  }
  if (wave == LAST) epi_apply<bf16_t, 1>(e, acc, g, 1, m0, n0, M, N, lane);
}
void launch_kchain(const void* A, const void* W, int M, int N, int K, const Epi& e, hipStream_t s) {
  const int n_strips = N / 16, grid = n_strips * ((M + 15) / 16);
  auto go = [&](auto ns_c, auto nw_c) {
    constexpr int NS = decltype(ns_c)::value, NW = decltype(nw_c)::value;
    const size_t lds = kchain_lds_bytes(NW);
    (void)hipFuncSetAttribute((const void*)k_gemm_bf16_kchain<NS, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k_gemm_bf16_kchain<NS, NW><<<grid, 64 * NW, lds, s>>>((const bf16_t*)A, (const bf16_t*)W, M, N, K, n_strips, e);
  };
  using I2 = std::integral_constant<int, 2>;
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  if (K == 1024) go(I2{}, I4{});
  else if (K == 2048) go(I4{}, I4{});
  else if (grid <= 256) go(I8{}, I8{});
  else go(I8{}, I4{});
}

// ---------------------------------------------------------------- rows through the pending LayerNorm: K = 1024
// Workgroup = (16 rows, SW strips of 16 columns): eight waves normalise two rows each, then KH = 8 / SW waves share a strip's
// K, the accumulator passing from one to the next through LDS (the same chain as above).  Every weight is requested at the
// start, behind the rows; the A-in-LDS kernel (four waves of four rows and one strip, the second 512 of K requested while the
// first is multiplied) took 8.4 us for N = 4096 and 8.2 for N = 3072 at 25 rows, this one 5.9 and 6.0: 8 and 6 MB of weights.
// Two strips per workgroup while that makes at most one workgroup per CU, four beyond (wide model, 8 / 17 / 64 rows: within
// 1 % of each other).
template <int SW, int EM>
__global__ __launch_bounds__(512, 2) void k_gemm_bf16_lnchain(const float* __restrict__ ln_x, const float* __restrict__ ln_g,
                                                           const float* __restrict__ ln_b, const bf16_t* __restrict__ W, int M, int N,
                                                           int groups, float* __restrict__ ln_y, Epi e) {
  constexpr int K = 1024, KH = 8 / SW, FR = K / 32 / KH, LD = K + 16;
  __shared__ uint4 tile[16 * LD / 8];
  __shared__ f32x4 hand[SW * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int group = blockIdx.x % groups, m0 = (blockIdx.x / groups) * 16;
  const int sl = wave % SW, part = wave / SW, n0 = (group * SW + sl) << 4;
  bf16_t* At = (bf16_t*)tile;
  LnA ln;
  ln.x = ln_x; ln.g = ln_g; ln.b = ln_b; ln.y = ln_y;
  uint4 b[FR];
  EpiRegs<1> g;
  auto behind_rows = [&]() {
    const bf16_t* wp = W + (size_t)n0 * K + (size_t)part * FR * 512 + lane * 8;
#pragma unroll
    for (int u = 0; u < FR; ++u) b[u] = ldg16(wp + u * 512);
  };
  astat_stage_ln<4, 2, 2>(ln, At, LD, wave * 2, m0, M, lane, group == 0, behind_rows);
  if (part == KH - 1) epi_preload<1, EM>(e, 1, m0, n0, M, N, lane, g);
  __syncthreads();
  const bf16_t* a_lane = At + r * LD + kq * 8 + part * FR * 32;
  f32x4 acc[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int p = 0; p < KH; ++p) {
    if (part == p) {
      if (p > 0) acc[0] = hand[sl * 64 + lane];
#pragma unroll
      for (int u = 0; u < FR; ++u)
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, *(const uint4*)(a_lane + 32 * u)), __builtin_bit_cast(bf16x8, b[u]), acc[0], 0, 0, 0);
      if (p + 1 < KH) hand[sl * 64 + lane] = acc[0];
    }
    if (p + 1 < KH) __syncthreads();
  }
  if (part == KH - 1) epi_apply<bf16_t, 1, EM>(e, acc, g, 1, m0, n0, M, N, lane);
}
bool launch_lnchain(const void* W, int M, int N, int K, const Epi& e, hipStream_t s, const LnA& ln) {
  const int n_strips = N / 16, chunks = (M + 15) / 16;
  if (K != 1024 || !ln.x || N % 64 || e.mode == EPI_ARGMAX || e.mode == EPI_COUNT) return false;
  auto go = [&](auto sw_c, auto em_c) {
    constexpr int SW = decltype(sw_c)::value, EM = decltype(em_c)::value;
    const int groups = n_strips / SW;
    k_gemm_bf16_lnchain<SW, EM><<<groups * chunks, 512, 0, s>>>(ln.x, ln.g, ln.b, (const bf16_t*)W, M, N, groups, ln.y, e);
  };
  auto by_mode = [&](auto sw_c) {
    if (e.mode == EPI_QKV) go(sw_c, std::integral_constant<int, EPI_QKV>{});
    else if (e.mode == EPI_RELU) go(sw_c, std::integral_constant<int, EPI_RELU>{});
    else go(sw_c, std::integral_constant<int, -1>{});
  };
  if (n_strips / 2 * chunks <= 256) by_mode(std::integral_constant<int, 2>{});
  else by_mode(std::integral_constant<int, 4>{});
  return true;
}

}  // namespace ad

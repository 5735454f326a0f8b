// Device code shared by the kernels that run a stack of layers in one launch (ad_team.hip, ad_team_f32.hip): exchanges between the
// members of a team, and the lists a member needs.
#pragma once

#include "ad_device.h"
#include "ad_team.h"

namespace ad {

constexpr unsigned long long kWaitTicks = 200000;   // 100 MHz ticks: 2 ms

struct TeamChunk { int row, n, off, causal, nk_base, kv_self, kv_cross, nk_cross; };   // up to 16 query rows of one attention problem

__device__ __forceinline__ unsigned xcc_id() {
  unsigned v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & 15;
}
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// loads of rows another CU of the XCD wrote during this launch: past the vector cache, from the L2
__device__ __forceinline__ uint4 ld16_l2(const void* base, unsigned off) {
  __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00027000);
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 16));
}
__device__ __forceinline__ float ld4_l2(const void* base, unsigned off) {
  __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00027000);
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 16));
}
// workgroup barrier that leaves memory requests in flight
__device__ __forceinline__ void wg_bar() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// A row goes from the CU that computes it to those that multiply it without a barrier: its place is set to all ones ahead of time,
// nothing computed is stored as that, and whoever needs the row reads it until no piece of it is all ones.  (All ones is one of
// the NaNs; a NaN with these bits is stored as its neighbour.)  Who sets a place back, and when: its writer, no later than the
// store of an earlier exchange that every reader of the place has seen whole, and after an exchange that every reader of its former
// content had to pass; the stores are answered for before the writer's next data leave (team_put_ready).
__device__ __forceinline__ void unwrite16(void* base, unsigned off) { gstore((uint4*)((char*)base + off), uint4{~0u, ~0u, ~0u, ~0u}); }
__device__ __forceinline__ f32x4 unwritten4() { return __builtin_bit_cast(f32x4, uint4{~0u, ~0u, ~0u, ~0u}); }
__device__ __forceinline__ unsigned written(float v) { return min(__float_as_uint(v), 0xfffffffeu); }
__device__ __forceinline__ void put(float* p, float v) { gstore((unsigned*)p, written(v)); }
// for readers on other XCDs: past this one's L2
__device__ __forceinline__ void put_far(float* p, float v) { __hip_atomic_store((unsigned*)p, written(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put_far(bf16_t* p, float v) { __hip_atomic_store(p, (bf16_t)min((unsigned)f2bf(v), 0xfffeu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void unwrite16_far(void* base, unsigned off) {
  __hip_atomic_store((unsigned long long*)((char*)base + off), ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store((unsigned long long*)((char*)base + off + 8), ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put(bf16_t* p, float v) { gstore(p, (bf16_t)min((unsigned)f2bf(v), 0xfffeu)); }
__device__ __forceinline__ void team_put_ready() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// has this wave seen a piece that is not written yet?  (fp32 words / bf16 halves)
struct Seen32 {
  unsigned m = 0;
  __device__ __forceinline__ void add(const uint4& v) { m = max(max(m, v.x), max(max(v.y, v.z), v.w)); }
  __device__ __forceinline__ bool all() const { return __builtin_amdgcn_ballot_w64(m == ~0u) == 0; }
};
struct Seen16 {
  typedef unsigned short half2 __attribute__((ext_vector_type(2)));
  half2 m = {0, 0};
  __device__ __forceinline__ void add(const uint4& v, bool counts = true) {
    half2 x = __builtin_elementwise_max(__builtin_elementwise_max(__builtin_bit_cast(half2, v.x), __builtin_bit_cast(half2, v.y)),
                                        __builtin_elementwise_max(__builtin_bit_cast(half2, v.z), __builtin_bit_cast(half2, v.w)));
    m = __builtin_elementwise_max(m, counts ? x : half2{0, 0});
  }
  __device__ __forceinline__ bool all() const { return __builtin_amdgcn_ballot_w64(m.x == 0xffff || m.y == 0xffff) == 0; }
};
struct TeamWait {
  unsigned *fail, *gave_up;   // the launch's fail word; this workgroup's (LDS)
  bool off;                   // wait no more
};
// attempt(): loads, and whether everything was there
template <typename F>
__device__ __forceinline__ void wait_for(TeamWait& tw, int lane, const F& attempt) {
  unsigned long long t0 = 0;
#pragma unroll 1
  for (unsigned spin = 0;; ++spin) {
    asm volatile("" ::: "memory");
    if (attempt() || tw.off) return;
    if ((spin & 15) == 0) {
      const unsigned long long now = __builtin_amdgcn_s_memrealtime();
      if (spin == 0) t0 = now;
      else if (now - t0 >= kWaitTicks || __builtin_amdgcn_readfirstlane(__hip_atomic_load(tw.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))) {
        tw.off = true;
        if (lane == 0) {
          __hip_atomic_store(tw.gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_store(tw.fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
      }
    }
  }
}
__device__ __forceinline__ TeamChunk chunk_at(const TeamChunk* chunks, int c) {
  TeamChunk t = chunks[c];
  t.row = __builtin_amdgcn_readfirstlane(t.row); t.n = __builtin_amdgcn_readfirstlane(t.n);
  t.off = __builtin_amdgcn_readfirstlane(t.off); t.causal = __builtin_amdgcn_readfirstlane(t.causal);
  t.nk_base = __builtin_amdgcn_readfirstlane(t.nk_base); t.kv_self = __builtin_amdgcn_readfirstlane(t.kv_self);
  t.kv_cross = __builtin_amdgcn_readfirstlane(t.kv_cross); t.nk_cross = __builtin_amdgcn_readfirstlane(t.nk_cross);
  return t;
}
// The lists of a team's rows (n0 of segment 0, then n1 of segment 1) and of its attention problems' chunks, by the first two waves:
// grow, rdst: packed row and key / value row; counts[0], [1]: chunks, chunks of segment 0.  (Its reader's barrier follows.)
template <int ROWS, bool DEC>
__device__ __forceinline__ void team_lists(const TeamArgs& a, int team, int n0, int n1, TeamChunk* chunks, int* grow, int* rdst, int* counts,
                                           int wave, int lane) {
  if (wave == 0) {
    const int p0 = a.prob_lo[team], np = a.prob_n[team], np2 = a.prob2_off ? np : 0;
    SeqDesc sd = {}, cd = {};
    if (lane < np + np2) {
      const int p = lane < np ? p0 + lane : a.prob2_off + p0 + lane - np;
      sd = gload(a.self_desc + p);
      if (DEC) cd = gload(a.cross_desc + p);
    }
    // the problem's rows that are this team's
    const int lo = a.row_lo[lane < np ? 0 : 1][team], first = max(sd.q_row0, lo);
    const int off = first - sd.q_row0, nq = max(0, min(sd.q_row0 + sd.nq, lo + (lane < np ? n0 : n1)) - first);
    const int nc = (nq + 15) >> 4;
    int before = nc;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(before, o);
      if (lane >= o) before += up;
    }
    if (lane == 63) counts[0] = before;
    if (lane == np - 1) counts[1] = before;
    before -= nc;
    const int row = (lane < np ? 0 : n0) + first - lo;
    for (int c = 0; c < nc; ++c)
      if (before + c < ROWS) {
        TeamChunk t;
        t.row = row + 16 * c; t.n = min(16, nq - 16 * c); t.off = off + 16 * c; t.causal = sd.causal; t.nk_base = sd.nk_base;
        t.kv_self = sd.kv_row0; t.kv_cross = cd.kv_row0; t.nk_cross = cd.nk_base;
        chunks[before + c] = t;
      }
  } else if (wave == 1 && lane < ROWS) {
    const int row = min(lane, n0 + n1 - 1), g = row < n0 ? a.row_lo[0][team] + row : a.row_lo[1][team] + row - n0;
    grow[lane] = g;
    rdst[lane] = gload(a.row_dst + g);
  }
}
// A member (one wave of it) says it is here and its places can be read; the last of an XCD says so for the XCD.
__device__ __forceinline__ void team_arrive(const TeamArgs& a, unsigned* words, int lane) {
  team_put_ready();
  if (lane == 0 && __hip_atomic_fetch_add(words + 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kTeamMembers - 1)
    (void)__hip_atomic_fetch_add(a.words + 48, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void team_wait_count(const TeamArgs& a, unsigned* count, unsigned target, unsigned* gave_up, int lane) {
  if (lane == 0) {
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    bool late = a.form_ticks == 0;
    for (unsigned spin = 0; !late && __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target; ++spin)
      late = (spin & 15) == 15 && __builtin_amdgcn_s_memrealtime() - t0 >= a.form_ticks;
    if (late) {
      __hip_atomic_store(a.fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
}

}  // namespace ad

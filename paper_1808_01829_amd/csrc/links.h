// Loads of 3 x 3 links from a caller's gauge field U[mu][idx][3][3], one link per lane.
//
// A lane's own link is 144 contiguous bytes, so nine loads at a stride of 144 bytes
// touch 64 cache lines each, and such kernels were bound by the L1's line rate. Here the
// wave's 64 links are read as 576 consecutive entries instead: lane l takes entry
// (64 k + l) % 9 of link (64 k + l) / 9 in load k, so runs of neighbouring links (the
// usual case: an x-row, shifted or not) are whole lines, and the entries reach their lanes
// through LDS. The reads back are at a pitch of 144 bytes, an odd multiple of 16: no bank
// conflicts.
#pragma once

#include "common.h"

constexpr int WL_ENTRIES = 64 * 9;  // LDS of one wave, complex

struct M3 {
  double2 e[9];
};

// LDS and global accesses by a vector type: copies of double2, a struct, through LDS left
// whole matrices in scratch memory
typedef double wl2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void wl_st(double2* p, double2 v) { *(wl2*)p = wl2{v.x, v.y}; }
__device__ __forceinline__ double2 wl_ld(const double2* p) {
  const wl2 v = *(const wl2*)p;
  return make_double2(v.x, v.y);
}

// Entries of the wave's 64 links (lane j's is number `link` = mu * vol + idx); every lane of
// the wave takes part, with a valid link.
__device__ __forceinline__ void wl_fetch(const double2* __restrict__ U, int link, M3& r) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int i = 64 * k + lane, j = (i * 7282) >> 16;  // i / 9 for i < 576
    r.e[k] = wl_ld(U + (size_t)__shfl(link, j) * 9 + (i - 9 * j));
  }
  // one set of entries in flight: hoisted further, they would take 36 registers each
  __builtin_amdgcn_sched_barrier(0);
}
// what wl_fetch brought, as this lane's own link
__device__ __forceinline__ M3 wl_own(const M3& r, double2* lds) {
  const int lane = threadIdx.x & 63;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 9; ++k) wl_st(lds + 64 * k + lane, r.e[k]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  M3 m;
#pragma unroll
  for (int k = 0; k < 9; ++k) m.e[k] = wl_ld(lds + 9 * lane + k);
  __builtin_amdgcn_wave_barrier();
  return m;
}
// the reverse: this lane's link as the entries it stores
__device__ __forceinline__ M3 wl_spread(const M3& m, double2* lds) {
  const int lane = threadIdx.x & 63;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 9; ++k) wl_st(lds + 9 * lane + k, m.e[k]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  M3 r;
#pragma unroll
  for (int k = 0; k < 9; ++k) r.e[k] = wl_ld(lds + 64 * k + lane);
  __builtin_amdgcn_wave_barrier();
  return r;
}

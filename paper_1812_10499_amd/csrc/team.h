// Teams of workgroups that share one XCD's L2: stores, words and waits between
// them.  What a team shares goes through agent-scope relaxed loads and atomics
// (they pass over the L1) and the stores below, so nothing needs a cache
// write-back or invalidation.
#pragma once

#include "sssp_dev.h"

namespace sssp {

// A wait ends after this many reads (some seconds; a round takes
// microseconds) and the solve with an internal error.
constexpr int kSpinLimit = 1 << 24;

// A store the team's other waves are to read: within one XCD it only has to
// reach the shared L2 (about 440 cycles until done, against 830 for an
// agent-scope store; with the latter a 1024 x 1024 grid takes 45 ms in a team
// of 64 waves, 22.4 without).
// same_l2 is narrower than the sharing: HIP promises a workgroup-scope store to
// the workgroup alone.  Relied on is its form on gfx950, a store with sc0 and
// not sc1 (a CPU test reads it from the compiler's output): the L1 writes every
// store through, so that once vmcnt has counted it (stores_done) it lies in the
// L2 of the XCD, where the agent-scope loads of that XCD's other workgroups look.
// That they are on that XCD is established by xcd_id() when a team starts.
// Read-modify-writes need nothing of the kind: they are at agent scope, where
// the instruction is the same.
__device__ __forceinline__ void put(int32_t *p, int32_t v, bool same_l2) {
  if (same_l2) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put64(unsigned long long *p, unsigned long long v, bool same_l2) {
  if (same_l2) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// every store of this wave has reached the point the other waves read
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ unsigned long long tagged(unsigned tag, int32_t v) {
  return ((unsigned long long)tag << 32) | (uint32_t)v;
}

// A published word: the round's low two bits (no member is more than one round
// ahead of another), minD's key and thr's (non-negative).
__device__ __forceinline__ unsigned long long offers(unsigned ep, int32_t md, int32_t th) {
  return ((unsigned long long)(ep & 3u) << 62) | ((unsigned long long)(uint32_t)md << 31) |
         (unsigned long long)(uint32_t)th;
}
__device__ __forceinline__ int32_t offers_md(unsigned long long x) {
  return (int32_t)((x >> 31) & 0x7fffffffu);
}
__device__ __forceinline__ int32_t offers_th(unsigned long long x) {
  return (int32_t)(x & 0x7fffffffu);
}

// Lane l's word of `words` once every lane's carries round ep (whole wave).
// *lost: the limit was reached first.
__device__ __forceinline__ unsigned long long await_offers(const unsigned long long *words, int l,
                                                           unsigned ep, bool *lost) {
  unsigned long long x = 0;
  int spins = 0;
  do {
    x = ld_relaxed64(&words[l]);
    *lost = ++spins > kSpinLimit;
  } while (!*lost && __ballot((unsigned)(x >> 62) != (ep & 3u)));
  asm volatile("" ::: "memory");  // nothing below is read before the words
  return x;
}

// the XCD this wave runs on
__device__ __forceinline__ int32_t xcd_id() {
  return (int32_t)(__builtin_amdgcn_s_getreg((31 << 11) | 20) & 0xffu);
}

}  // namespace sssp

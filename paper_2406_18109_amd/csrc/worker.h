// Persistent workers over independent streams of work pinned to XCDs: what
// the batched executor (batch.hip) and the solve server's rounds (serve.hip)
// share on the device.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "claim.h"
#include "vm.h"

namespace dfx {

// Synchronisation.  Streams are pinned to XCDs, so every wave that reads a
// stream's data runs on the XCD whose L2 holds it.  A run's stores are
// released by waiting for their completion (s_waitcnt: they have reached
// the L2), without writing the L2 back to memory as an agent-scope release
// would; a claim or a completed count is followed by the agent-scope
// acquire (it invalidates the CU's caches above the L2).  Control words are
// agent-scope atomics.  A message-passing test between waves of one XCD on
// MI355X (writer: plain stores, wait, flag; reader: flag, acquire, loads)
// saw no stale value over 8 x 10^5 messages with this pair, and stale values
// with an L1-only invalidate (buffer_inv sc0) as the acquire.
__device__ __forceinline__ void xcd_release() {
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
}
// By one wave, before a block barrier: for every wave of the block.
__device__ __forceinline__ void block_acquire() {
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
}
template <typename U> __device__ __forceinline__ U xload(U* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U> __device__ __forceinline__ void xstore(U* p, U v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U> __device__ __forceinline__ U xadd(U* p, U v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long bcast64(unsigned long long v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

// Stall detector: a wave that finds nothing to claim while no pass of its
// XCD's streams has completed for this many ticks of the 100 MHz constant
// clock (2 s) ends the launch with an error.
#ifndef DFX_BATCH_STALL_TICKS
#define DFX_BATCH_STALL_TICKS 200000000ull
#endif

// Looks for a stream of this XCD with a run left, 64 at a time (lane l at
// stream s + l of ns, so the stream served last comes first): claim_of(q) is
// stream q's claim word.  Lane 0 claims from the candidates in lane order.
// Called by one wave; returns the stream's index and its word at the claim,
// or -1.
template <class F>
__device__ __forceinline__ int find_run(const uint32_t s, const uint32_t ns, F claim_of, unsigned long long& word) {
  const int lane = threadIdx.x & (WAVE - 1);
  for (uint32_t base = 0; base < ns; base += WAVE) {
    const uint32_t j = base + lane;
    uint32_t q = s + j;
    q = q < ns ? q : q - ns;   // s < ns and j < ns below, so one wrap suffices
    bool can = false;
    if (j < ns) can = claimable(xload(claim_of(q)));
    unsigned long long m = __ballot(can);
    while (m != 0ull) {
      const int L = (int)__builtin_ctzll(m);
      m &= m - 1ull;
      const uint32_t qL = __builtin_amdgcn_readfirstlane(__shfl(q, L, WAVE));
      unsigned long long w = 0;
      if (lane == 0) w = xadd(claim_of(qL), 1ull);
      w = bcast64(w);
      if (claimable(w)) {
        word = w;
        return (int)qL;
      }
    }
  }
  return -1;
}

// Nothing to claim: whether the block should leave (every stream has
// settled, or an error), else the stall detector and a short sleep.
__device__ __forceinline__ bool idle(XcdCtl& X, uint32_t& seen_progress, unsigned long long& since) {
  const int lane = threadIdx.x & (WAVE - 1);
  uint32_t settled = 0, prog = 0;
  int err = 0;
  if (lane == 0) {
    settled = xload(&X.n_settled);
    prog = xload(&X.progress);
    err = xload(&X.error);
  }
  settled = __builtin_amdgcn_readfirstlane(settled);
  prog = __builtin_amdgcn_readfirstlane(prog);
  err = __builtin_amdgcn_readfirstlane(err);
  if (settled >= X.n_streams || err) return true;
  const unsigned long long now = __builtin_amdgcn_s_memrealtime();
  if (prog != seen_progress) {
    seen_progress = prog;
    since = now;
  } else if (now - since > DFX_BATCH_STALL_TICKS) {
    if (lane == 0) xstore(&X.error, 1);
    return true;
  }
  __builtin_amdgcn_s_sleep(1);
  return false;
}

}  // namespace dfx

// Control words of the persistent workers (worker.h), shared with the host.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dfx {

// A stream's claim word: passes completed << 32 | runs of the current pass
// << 16 | next run to claim, so that one load tells whether a run is left.
// A settled (done or paused) stream has no runs.  Claimers add one after
// seeing a run left, so the next-run field passes the runs by at most one
// per block of the launch and never reaches the runs field.  While a block
// keeps a stream to itself (passes of one run) the word stays that of the
// last published pass, all of whose runs are taken.
__host__ __device__ inline unsigned long long claim_word(uint32_t gen, uint32_t runs, uint32_t next) {
  return (unsigned long long)gen << 32 | (unsigned long long)runs << 16 | next;
}
__host__ __device__ inline bool claimable(unsigned long long w) {
  return ((uint32_t)w & 0xffffu) < ((uint32_t)w >> 16);
}

// Streams of work are pinned to XCDs: the L2 of its XCD is the coherence
// point of everything a stream's waves exchange inside a launch.  Each XCD's
// counters sit in their own 256-byte line.
constexpr int MAX_XCD = 8;
struct XcdCtl {
  uint32_t n_streams;            // streams of this XCD
  uint32_t n_settled;            // of them, settled in this launch
  uint32_t progress;             // passes completed: the stall detector's clock
  int32_t error;                 // 1: the stall detector fired (idle blocks left early)
  uint32_t first;                // (solve server) its first entry of the round's list
  uint32_t pad[59];
};

// Whether a launch settled every stream: after it, the one thing that says so.
// An XCD that got no block sets no error, and the stall detector's error loses
// nothing by itself: a block leaves on it only with nothing taken and nothing
// to claim, and what is published later is carried on by the block that
// publishes it.  (The detector's clock runs on while a shared GPU has another
// process's work in the queue's place.)
inline bool all_settled(const XcdCtl* x, uint32_t n_xcd) {
  for (uint32_t k = 0; k < n_xcd; ++k)
    if (x[k].n_settled != x[k].n_streams) return false;
  return true;
}

}  // namespace dfx

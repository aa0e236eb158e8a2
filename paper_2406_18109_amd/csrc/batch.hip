// The persistent batched executor (see batch.h): one launch runs many
// independent task streams of fused passes.  Each block of 16 waves is an
// independent worker.  It claims a work item (stream, current pass, run of
// tiles) with an atomic on the stream's claim word, executes the run tile by
// tile with all its waves (coop_tile), writes one sum per tile and
// reduction, and counts the run done.  The block that finishes a pass's last
// run reduces the tile sums with the canonical pairwise tree (the same tree
// the two-launch path evaluates, so every result is bit-identical to a solo
// run), writes the 0-d results, advances the stream to its next pass and
// takes that pass's first run itself.  A stream runs on one XCD; its passes
// are ordered by agent-scope release/acquire (xcd_release, block_acquire);
// values written inside the launch (0-d results, tile sums) are read with
// vector or atomic loads, never through the scalar cache.
//
// What bounds it is the latency of a pass: claim, acquire, the pass's
// dependent loads, release, count, publish.  Three things decide it, measured
// over 32 CG solves of sides 32 to 256 to 1e-8.  With single waves as workers
// a tile was one wave's 32 rows in sequence and every idle wave of the chip
// polled the claim words: about 97 us per pass of 16 tiles, 403 ms in all;
// with blocks 84 ms.  One wave's acquire for its block instead of sixteen:
// 34 ms.  Passes of one run are kept by the block that completed the pass
// before: no claim, and no wait for stores, between them (a one-tile CG
// iteration of five passes takes 18 us at 256 unknowns, 27 us at 4096).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "batch.h"
#include "dev_common.h"
#include "coop_exec.h"
#include "worker.h"
#include "vm_exec.h"

namespace dfx {

namespace {

// One instantiation serves every pass of a batch: FP64, 8 registers, up to
// 6 input streams, the SpMV prologue taken when the pass has one; with the
// transcendental op set (HV 1) when any pass needs it, else the arithmetic
// one (HV 0, two rows per step).
typedef double BT;

// Pass index (into the batch's pass table) of the g-th pass a stream runs;
// -1 past the end of a stream without a repeated body.
__device__ __forceinline__ int pass_of(const BatchStream& st, uint32_t g) {
  if ((int64_t)g < st.n_pre) return st.pass0 + (int)g;
  if (st.n_body == 0) return -1;
  return st.pass0 + st.n_pre + (int)((g - (uint32_t)st.n_pre) % (uint32_t)st.n_body);
}

// The canonical tree over a[0..n) (any n >= 1) evaluated by one wave:
// aligned chunks of 256 are complete subtrees (block_tree), their sums are
// written to `scratch` and reduced the same way until one chunk remains.
// `a` and `scratch` are global; the result is valid in every lane.
__device__ double wave_tree(const double* a, int64_t n, double* scratch, int lane) {
  const double* src = a;
  double* dst = scratch;
  while (n > 4 * WAVE) {
    const int64_t m = (n + 4 * WAVE - 1) / (4 * WAVE);
    for (int64_t c = 0; c < m; ++c) {
      const int cnt = (int)min((int64_t)4 * WAVE, n - c * 4 * WAVE);
      const double v = block_tree(src + c * 4 * WAVE, cnt, lane);
      if (lane == 0) dst[c] = v;
    }
    __threadfence_block();
    src = dst;
    dst = (dst == scratch) ? scratch + ((m + 255) & ~(int64_t)255) : scratch;
    n = m;
  }
  const double v = block_tree(src, (int)n, lane);
  return __shfl(v, 0, WAVE);
}

// What wave 0 found, or decided, for its block.
struct BatchItem {
  int32_t sid, pidx;   // sid < 0: leave; pidx < 0: nothing taken, search
  uint32_t run, gen;
  int32_t status;      // the stream's after a completed pass
  int32_t publish;     // ... whose next pass other blocks may claim (or that has settled)
};

template <int BHV>
__global__ __launch_bounds__(COOP_BLOCK) void batch_kernel(const BatchPass* __restrict__ passes,
                                                           BatchStream* __restrict__ streams,
                                                           BatchCtl* __restrict__ ctl) {
  extern __shared__ __attribute__((aligned(16))) char coop_dyn_lds[];
  __shared__ BatchItem item;
  __shared__ double tot[VM_MAXRED];
  __shared__ uint32_t last_run;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  // this block's XCD (hardware register XCC_ID)
  const uint32_t xcc = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_s_getreg((20) | (0 << 6) | (3 << 11)));
  const uint32_t nxcd = ctl->n_xcd;
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_or(&ctl->xcc_seen, 1u << (xcc & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&ctl->waves[xcc & 15], (uint32_t)COOP_WAVES, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (xcc >= nxcd) return;
  XcdCtl& X = ctl->x[xcc];
  const uint32_t ns = X.n_streams;   // streams xcc, xcc + nxcd, ...
  if (ns == 0) return;
  // (wave 0 alone searches and decides; these are its own)
  uint32_t s = (blockIdx.x / nxcd) % ns;   // index among this XCD's streams
  uint32_t seen_progress = 0;
  unsigned long long since = __builtin_amdgcn_s_memrealtime();
  int32_t own_it = -1, own_rit = 0;   // the stream's repetition counts while this block keeps it (-1: not known)
  bool have = false;                  // item holds a run this block took when it completed a pass
  // stream and pass up to which this block's last acquire made every earlier
  // pass visible (passes before acq_gen of stream acq_sid)
  int acq_sid = -1;
  uint32_t acq_gen = 0;
  for (;;) {
    if (wib == 0 && !have) {
      BatchItem it = {-1, -1, 0u, 0u, BS_RUNNING, 0};
      own_it = -1;
      for (;;) {
        unsigned long long w = 0;
        const int q = find_run(s, ns, [&](uint32_t k) { return &streams[(size_t)k * nxcd + xcc].claim; }, w);
        if (q >= 0) {
          s = (uint32_t)q;
          it.sid = (int)((size_t)q * nxcd + xcc);
          it.gen = (uint32_t)(w >> 32);
          it.run = (uint32_t)w & 0xffffu;
          it.pidx = pass_of(const_table(streams[it.sid]), it.gen);
          // acquire for the block: the stream's earlier passes are visible.
          // A block whose last acquire already followed the completion of
          // every pass before this one (another run of the same pass) skips
          // it.  One wave is enough, and all that is affordable: the waves
          // of a compute unit share the caches above the L2 and their
          // accesses pass them in order, and with every wave of 16 blocks
          // invalidating, the first load of a pass took 9 us.
          if (it.sid != acq_sid || it.gen > acq_gen) {
            block_acquire();
            acq_sid = it.sid;
            acq_gen = it.gen;
          }
          break;
        }
        if (idle(X, seen_progress, since)) break;
      }
      if (lane == 0) item = it;
    }
    __syncthreads();
    const int sid = __builtin_amdgcn_readfirstlane(item.sid);
    if (sid < 0) return;
    const int pidx = __builtin_amdgcn_readfirstlane(item.pidx);
    const uint32_t run = __builtin_amdgcn_readfirstlane(item.run), gen = __builtin_amdgcn_readfirstlane(item.gen);
    BatchStream& st = streams[sid];
    const BatchStream& sc = const_table(st);   // for the fields no launch writes
    const BatchPass& B = const_table(passes[pidx]);
    const VmParams& P = B.P;
    const uint32_t n_runs = (uint32_t)B.n_runs;
    const int64_t t_begin = (int64_t)run * P.tiles_per_wave;
    const int64_t t_end = min(t_begin + P.tiles_per_wave, P.n_tiles);
    for (int64_t t = t_begin; t < t_end; ++t) {
      coop_tile<BT, BHV>(P, t, coop_dyn_lds, tot);
      if (P.n_red > 0) {
        // (lane 0 of wave k holds sum k; a one-tile pass keeps it in LDS)
        if (P.n_tiles > 1 && wib < P.n_red && lane == 0) global_ptr<double>(sc.tsum)[wib * sc.tsum_stride + t] = tot[wib];
        if (t + 1 < t_end) __syncthreads();   // the summands' LDS is written again
      }
    }
    since = __builtin_amdgcn_s_memrealtime();
    if (n_runs > 1) {
      // release every wave's stores of this run, then count it
      xcd_release();
      __syncthreads();
      if (wib == 0) {
        uint32_t d = 0;
        if (lane == 0) d = xadd(&st.done, 1u);
        const bool last = __builtin_amdgcn_readfirstlane(d) + 1 == n_runs;
        if (last) block_acquire();   // the other runs' tile sums and outputs
        if (lane == 0) last_run = last ? 1u : 0u;
      }
      __syncthreads();
      have = false;
      if (!__builtin_amdgcn_readfirstlane(last_run)) continue;
    }
    acq_sid = sid;
    acq_gen = gen + 1;
    // ---- the pass is complete: reductions, then advance the stream ------------
    if (P.n_red > 0) {
      if (P.n_tiles <= 4 * WAVE) {
        if (wib < P.n_red) {
          const double v = P.n_tiles == 1 ? tot[wib] : block_tree(global_ptr<double>(sc.tsum) + wib * sc.tsum_stride, (int)P.n_tiles, lane);
          if (lane == 0) {
            double* res = global_ptr<double>(B.result[wib]);
            *res = B.init[wib] ? v : load_0d<double>(res) + v;
          }
        }
      } else if (wib == 0) {
        // (the chunk sums' scratch is one per stream)
        double* tsum = global_ptr<double>(sc.tsum);
        double* chunk = tsum + (int64_t)VM_MAXRED * sc.tsum_stride;
        for (int k = 0; k < P.n_red; ++k) {
          const double v = wave_tree(tsum + k * sc.tsum_stride, P.n_tiles, chunk, lane);
          if (lane == 0) {
            double* res = global_ptr<double>(B.result[k]);
            *res = B.init[k] ? v : load_0d<double>(res) + v;
          }
        }
      }
    }
    __syncthreads();
    if (wib == 0) {
      int32_t status = BS_RUNNING;
      const int body0 = sc.pass0 + sc.n_pre, end = body0 + sc.n_body;
      int np = pidx + 1;
      if (np == end && sc.n_body > 0) {
        np = body0;
        // a repetition of the body is complete (only this block touches the
        // counters now: the stream's next pass is not yet published)
        if (own_it < 0) {
          own_it = __builtin_amdgcn_readfirstlane(xload(&st.iters));
          own_rit = __builtin_amdgcn_readfirstlane(xload(&st.round_iters));
        }
        own_it += 1;
        own_rit += 1;
        if (lane == 0) {
          xstore(&st.iters, own_it);
          xstore(&st.round_iters, own_rit);
        }
        bool stop = own_it >= sc.max_iter;
        if (!stop && sc.conv_a) {
          const double a = load_0d<double>(sc.conv_a), b = load_0d<double>(sc.conv_b);
          stop = a <= sc.tol * b;
        }
        if (stop) status = BS_DONE;
        else if (ctl->round_limit > 0 && own_rit >= ctl->round_limit) status = BS_PAUSED;
      } else if (np == body0 && (sc.n_body == 0 || sc.max_iter <= 0)) {
        status = BS_DONE;
      }
      if (status != BS_RUNNING) np = -1;
      if (lane == 0) {
        item.pidx = np;
        item.run = 0u;
        item.gen = gen + 1;
        item.status = status;
        // a next pass of one run is this block's alone: nothing to tell
        // anyone, and no store has to be waited for
        item.publish = np < 0 || const_table(passes[np]).n_runs > 1;
        xadd(&X.progress, 1u);
      }
    }
    __syncthreads();
    have = __builtin_amdgcn_readfirstlane(item.pidx) >= 0;
    if (__builtin_amdgcn_readfirstlane(item.publish)) {
      xcd_release();   // every wave's stores since the stream was last published
      __syncthreads();
      if (threadIdx.x == 0) {
        const int32_t status = item.status, np = item.pidx;
        xstore(&st.done, 0u);
        if (status != BS_RUNNING) xstore(&st.status, status);
        xcd_release();
        // the next pass opens with its first run taken by this block
        xstore(&st.claim, claim_word(item.gen, np < 0 ? 0u : (uint32_t)const_table(passes[np]).n_runs, 1u));
        if (status != BS_RUNNING) xadd(&X.n_settled, 1u);
      }
    }
  }
}

}  // namespace

// Allows the batch kernels the dynamic LDS that any pass may need and returns
// how many of their blocks a compute unit holds with `lds` bytes (heavy: the
// transcendental variant), 0 on failure.  (The allowance belongs to the
// kernel, not to the launch: one that followed each batch's need could be
// lowered by another thread's batch between this one's setting and launch.)
int batch_blocks_per_cu(int heavy, uint32_t lds) {
  int blocks = 0;
  const void* f = heavy ? (const void*)&batch_kernel<1> : (const void*)&batch_kernel<0>;
  if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)coop_lds(VM_MAXRED, true)) != hipSuccess)
    return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, COOP_BLOCK, lds) != hipSuccess) return 0;
  return blocks;
}

int launch_batch(const BatchPass* passes, BatchStream* streams, BatchCtl* ctl, int grid, int heavy, uint32_t lds,
                 hipStream_t stream) {
  if (heavy) hipLaunchKernelGGL(batch_kernel<1>, dim3(grid), dim3(COOP_BLOCK), lds, stream, passes, streams, ctl);
  else hipLaunchKernelGGL(batch_kernel<0>, dim3(grid), dim3(COOP_BLOCK), lds, stream, passes, streams, ctl);
  return (int)hipGetLastError();
}

}  // namespace dfx

// Batched CG for the continuous-batching server: a round of iterations is one
// persistent launch (serve_round_kernel, below), or with many tiles one
// launch per CG phase that covers the tiles of every resident solve (solves
// of different sizes share a launch).  In a phase launch each (solve, tile)
// work item is processed by one wave in the
// canonical order of the op-list kernel (lane l owns columns 2l, 2l+1 of each
// 128-element row; 32 rows per tile), so the tile sums -- and, through the
// same pairwise tree, every dot product -- are identical whatever else is in
// the batch.  A second launch, one block per solve of the phase, reduces the
// solve's tile sums and forms its scalars: rho and ||b|| (init),
// alpha = rho/(p.q), or beta = rho'/rho and the convergence test.
#include <hip/hip_runtime.h>
#include <math.h>

#include "coop_exec.h"
#include "dev_common.h"
#include "serve.h"
#include "worker.h"

namespace dfx {

constexpr int S_TW = 128;   // FP64 row width of the canonical tiling
constexpr int S_TH = RED_TH;
// tile rows whose SpMV groups one csr_rows call walks together
#ifndef DFX_SERVE_SPMV_ROWS
#define DFX_SERVE_SPMV_ROWS 2
#endif
constexpr int SR = DFX_SERVE_SPMV_ROWS;
// 1: the SpMV phase stages each 64-row group's CSR range in LDS (csr_group)
#ifndef DFX_SERVE_SPMV_STAGE
#define DFX_SERVE_SPMV_STAGE 0
#endif

// One instantiation per phase, so the elementwise phases do not carry the
// SpMV phase's registers (and keep more waves per SIMD).
template <int PHASE>
__global__ __launch_bounds__(BLOCK) void serve_phase_kernel(const ServeLaunch L) {
  const int lane = threadIdx.x & (WAVE - 1);
  int lb = blockIdx.x;
  if ((L.grid & 7) == 0) lb = (blockIdx.x & 7) * (L.grid >> 3) + (blockIdx.x >> 3);
  const int64_t gw = (int64_t)lb * (BLOCK / WAVE) + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int64_t i0 = gw * L.items_per_wave;
  const int64_t i1 = min(i0 + L.items_per_wave, L.n_items);
  constexpr int phase = PHASE;

  for (int64_t it = i0; it < i1; ++it) {
    const int slot = L.item_slot[it];
    const int tile = L.item_tile[it];
    SolveDev* S = L.solves + slot;
    const int status = __builtin_nontemporal_load(&S->status);
    if (phase == PH_INIT ? status != SOLVE_INIT : status != SOLVE_RUN) continue;
    const int64_t n = S->n;
    const double* __restrict__ b = S->b;
    double* __restrict__ x = S->x;
    double* __restrict__ r = S->r;
    double* __restrict__ p = S->p;
    double* __restrict__ q = S->q;
    const double alpha = S->alpha, beta = S->beta;
    const int64_t t0 = (int64_t)tile * S_TH * S_TW;
    const int nrows = (int)min((int64_t)S_TH, (n - t0 + S_TW - 1) / S_TW);  // rows of the tile inside n
    double acc = 0.0;
    if constexpr (phase == PH_SPMV_DOT && DFX_SERVE_SPMV_STAGE) {
      // q = A p, one 64-row group at a time with its CSR range staged in
      // LDS, then p.q in the canonical order (lane l owns elements 2l, 2l+1
      // of each row)
      __shared__ int32_t sp_col[BLOCK / WAVE][SP_CAP];
      __shared__ double sp_val[BLOCK / WAVE][SP_CAP];
      const int wib = threadIdx.x / WAVE;
      const int32_t nnz = S->rowptr[n];
      for (int rr = 0; rr < nrows; ++rr) {
        const int64_t rb = t0 + (int64_t)rr * S_TW;
        double y[2], pv[2], qo[4];
#pragma unroll
        for (int v = 0; v < 2; ++v) pv[v] = rb + 2 * lane + v < n ? p[rb + 2 * lane + v] : 0.0;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int64_t g0 = rb + m * WAVE;
          y[m] = g0 < n ? csr_group<double>(S->rowptr, S->col, S->val, p, g0, n, nnz, (uint32_t)n, sp_col[wib],
                                            sp_val[wib])
                        : 0.0;
          if (g0 + lane < n) q[g0 + lane] = y[m];
        }
        rows_to_owners<double, 2>(y, qo);
#pragma unroll
        for (int v = 0; v < 2; ++v)
          if (rb + 2 * lane + v < n) {
            const double t = pv[v] * qo[v];
            acc = acc + t;
          }
      }
    } else if constexpr (phase == PH_SPMV_DOT) {
      // q = A p with consecutive rows on consecutive lanes (two tile rows,
      // four 64-row groups, per call), then p.q in the canonical order (lane
      // l owns elements 2l, 2l+1 of each row)
      const int32_t nnz = S->rowptr[n];
      for (int r0 = 0; r0 < nrows; r0 += SR) {
        int64_t gi[2 * SR];
        bool gok[2 * SR];
        double y[2 * SR], pv[SR][2];
#pragma unroll
        for (int m = 0; m < 2 * SR; ++m) {
          gi[m] = t0 + (int64_t)(r0 + m / 2) * S_TW + (m % 2) * WAVE + lane;
          gok[m] = r0 + m / 2 < nrows && gi[m] < n;
        }
#pragma unroll
        for (int h = 0; h < SR; ++h)
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const int64_t i = t0 + (int64_t)(r0 + h) * S_TW + 2 * lane + v;
            pv[h][v] = r0 + h < nrows && i < n ? p[i] : 0.0;
          }
        csr_rows<double, 2 * SR>(S->rowptr, S->col, S->val, p, gi, gok, nnz, (uint32_t)n, y);
#pragma unroll
        for (int m = 0; m < 2 * SR; ++m)
          if (gok[m]) q[gi[m]] = y[m];
#pragma unroll
        for (int h = 0; h < SR; ++h) {
          if (r0 + h >= nrows) break;
          const double yy[2] = {y[2 * h], y[2 * h + 1]};
          double qo[4];
          rows_to_owners<double, 2>(yy, qo);
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const int64_t i = t0 + (int64_t)(r0 + h) * S_TW + 2 * lane + v;
            if (i < n) {
              const double t = pv[h][v] * qo[v];
              acc = acc + t;
            }
          }
        }
      }
    } else {
      // RU rows' loads in flight together, then the rows in order
      constexpr int RU = 4;
      for (int r0 = 0; r0 < nrows; r0 += RU) {
        double va[RU][2], vb[RU][2], vc[RU][2], vd[RU][2];
        bool ok[RU][2];
        int64_t ix[RU][2];
#pragma unroll
        for (int u = 0; u < RU; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const int64_t i = t0 + (int64_t)(r0 + u) * S_TW + 2 * lane + v;
            ix[u][v] = i;
            ok[u][v] = r0 + u < nrows && i < n;
            va[u][v] = vb[u][v] = vc[u][v] = vd[u][v] = 0.0;
            if (!ok[u][v]) continue;
            if (phase == PH_INIT) {
              va[u][v] = b[i];
            } else if (phase == PH_AXPY_DOT) {
              va[u][v] = p[i];
              vb[u][v] = x[i];
              vc[u][v] = q[i];
              vd[u][v] = r[i];
            } else {
              va[u][v] = p[i];
              vb[u][v] = r[i];
            }
          }
#pragma unroll
        for (int u = 0; u < RU; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            if (!ok[u][v]) continue;
            const int64_t i = ix[u][v];
            if (phase == PH_INIT) {
              const double bi = va[u][v];
              r[i] = bi;
              p[i] = bi;
              x[i] = 0.0;
              const double t = bi * bi;
              acc = acc + t;
            } else if (phase == PH_AXPY_DOT) {
              const double t1 = alpha * va[u][v];
              x[i] = vb[u][v] + t1;
              const double t2 = alpha * vc[u][v];
              const double ri = vd[u][v] - t2;
              r[i] = ri;
              const double t = ri * ri;
              acc = acc + t;
            } else {
              const double t = beta * va[u][v];
              p[i] = t + vb[u][v];
            }
          }
      }
    }
    if (phase == PH_UPDATE_P) continue;
    const double ts = wave_sum(acc);
    if (lane == 0) S->partials[tile] = ts;
  }
}

// One block per listed solve: the pairwise tree over its tile sums (as the
// op-list executor's tile tree), then the phase's scalar update.
__global__ __launch_bounds__(BLOCK) void serve_final_kernel(SolveDev* solves, const int32_t* slots, int phase) {
  __shared__ double sh[S_MAXTILES];
  SolveDev* S = solves + slots[blockIdx.x];
  const int status = S->status;
  if (phase == PH_INIT ? status != SOLVE_INIT : status != SOLVE_RUN) return;
  const int L = S->n_tiles;
  for (int i = threadIdx.x; i < L; i += BLOCK) sh[i] = __builtin_nontemporal_load(S->partials + i);
  __syncthreads();
  lds_tree(sh, L);
  if (threadIdx.x != 0) return;
  const double total = L > 0 ? sh[0] : 0.0;
  if (phase == PH_INIT) {
    S->rho = total;
    S->bnorm = sqrt(total);
    S->status = !isfinite(total) ? SOLVE_BREAKDOWN : (total == 0.0 ? SOLVE_CONVERGED : SOLVE_RUN);
  } else if (phase == PH_SPMV_DOT) {
    S->pq = total;
    if (!(total > 0.0) || !isfinite(total)) S->status = SOLVE_BREAKDOWN;
    else S->alpha = S->rho / total;
  } else {
    const double rho_new = total;
    S->beta = rho_new / S->rho;
    S->rho = rho_new;
    S->iters = S->iters + 1;
    if (!isfinite(rho_new)) S->status = SOLVE_BREAKDOWN;
    else if (sqrt(rho_new) <= S->tol * S->bnorm) S->status = SOLVE_CONVERGED;
    else if (S->iters >= S->max_iter) S->status = SOLVE_MAXITER;
  }
}

// ---- a round as one persistent launch ---------------------------------------
// The matrix of a solve as coop_spmv reads it.
struct ServeMat {
  const int32_t* rowptr;
  const int32_t* colidx;
  const double* val;
  const double* x;
  int32_t nnz;
  int64_t nx, n1d;
};

// One tile of a phase by the 16 waves of a block, two canonical rows each
// (coop_tile's shape, the phase's arithmetic written out).  The summands of
// the phase's dot product go to dsum in their places; the caller adds them.
template <int PHASE>
__device__ __forceinline__ void serve_tile(const SolveDev& S, const int64_t n, const int tile, double* dsum) {
  constexpr int U = COOP_RPW, W = U * S_TW;   // elements of one wave
  typedef double v2 __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & (WAVE - 1);
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int64_t i0 = (int64_t)tile * S_TH * S_TW + wib * W;
  if (i0 >= n) return;
  const int left = (int)min(n - i0, (int64_t)W);
  const bool full = left == W;
  double* ds = dsum + wib * W;
  auto get = [&](const double* base, double (&o)[U][2]) {
    const double* b = global_ptr<const double>(base) + i0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = u * S_TW + 2 * lane;
      if (full) {
        const v2 w = *(const v2*)(b + e);
        o[u][0] = w[0];
        o[u][1] = w[1];
      } else {
        o[u][0] = b[min(e, left - 1)];
        o[u][1] = b[min(e + 1, left - 1)];
      }
    }
  };
  auto put = [&](double* base, const double (&o)[U][2]) {
    double* b = global_ptr<double>(base) + i0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = u * S_TW + 2 * lane;
      if (full) {
        *(v2*)(b + e) = v2{o[u][0], o[u][1]};
      } else {
        if (e < left) b[e] = o[u][0];
        if (e + 1 < left) b[e + 1] = o[u][1];
      }
    }
  };
  auto stage = [&](const double (&a)[U][2], const double (&b)[U][2]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double t0 = a[u][0] * b[u][0], t1 = a[u][1] * b[u][1];
      *(v2*)(ds + u * S_TW + 2 * lane) = v2{t0, t1};
    }
  };
  if constexpr (PHASE == PH_INIT) {
    double b[U][2], z[U][2] = {};
    get(S.b, b);
    put(S.r, b);
    put(S.p, b);
    put(S.x, z);
    stage(b, b);
  } else if constexpr (PHASE == PH_SPMV_DOT) {
    double p[U][2], q[U][2];
    get(S.p, p);
    const ServeMat M{S.rowptr, S.col, S.val, S.p, S.nnz, n, n};
    coop_spmv<double, W / WAVE>(M, i0, ds);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) q[u][v] = ds[u * S_TW + 2 * lane + v];
    put(S.q, q);
    stage(p, q);
  } else if constexpr (PHASE == PH_AXPY_DOT) {
    const double alpha = load_0d<double>(&S.alpha);
    double p[U][2], x[U][2], q[U][2], r[U][2];
    get(S.p, p);
    get(S.x, x);
    get(S.q, q);
    get(S.r, r);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const double t1 = alpha * p[u][v];
        x[u][v] = x[u][v] + t1;
        const double t2 = alpha * q[u][v];
        r[u][v] = r[u][v] - t2;
      }
    put(S.x, x);
    put(S.r, r);
    stage(r, r);
  } else {
    const double beta = load_0d<double>(&S.beta);
    double p[U][2], r[U][2];
    get(S.p, p);
    get(S.r, r);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const double t = beta * p[u][v];
        p[u][v] = t + r[u][v];
      }
    put(S.p, p);
  }
}

// What wave 0 found, or decided, for its block.
struct ServeItem {
  int32_t slot;        // < 0: leave
  uint32_t gen, tile;
  int32_t have;        // the block goes on with the solve's next phase
  int32_t publish;     // ... which other blocks may claim tiles of (or the solve has settled)
};

// The solves' rounds: blocks as workers, as in the batched executor
// (batch.hip), with the three CG phases compiled in and the scalar updates
// (alpha; beta, rho, the tests) made by the block that completes a phase, so
// an iteration is three passes with no launch between them.  Solves of one
// tile stay with their block for the whole round.  The phase launches this
// replaces there (seven an iteration, one wave per tile) left most of the chip
// idle: 48 solves of sides 32 to 256 to 1e-8 took 111 ms, against 48 ms.
// (Five waves per SIMD: a block's four leave room for another stream's; 96
// registers instead of 116, and no slower.)
__global__ __launch_bounds__(COOP_BLOCK) __attribute__((amdgpu_waves_per_eu(5))) void serve_round_kernel(SolveDev* __restrict__ solves,
                                                                 ServeClaim* __restrict__ claims,
                                                                 const int32_t* __restrict__ list,
                                                                 ServeRound* __restrict__ ctl) {
  __shared__ __attribute__((aligned(16))) double dsum[S_TH * S_TW];
  __shared__ ServeItem item;
  __shared__ double tot, csum[COOP_WAVES];
  __shared__ uint32_t last_tile;
  static_assert(S_MAXTILES <= COOP_WAVES * 4 * WAVE, "a wave for each chunk of tile sums");
  const int lane = threadIdx.x & (WAVE - 1);
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const uint32_t xcc = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_s_getreg((20) | (0 << 6) | (3 << 11)));
  if (xcc >= ctl->n_xcd) return;
  XcdCtl& X = ctl->x[xcc];
  const uint32_t ns = X.n_streams;
  if (ns == 0) return;
  const int32_t* mine = list + X.first;
  uint32_t s = (blockIdx.x / ctl->n_xcd) % ns, seen_progress = 0;
  unsigned long long since = __builtin_amdgcn_s_memrealtime();
  bool have = false;
  int acq_slot = -1;   // as acq_sid, acq_gen of the batched executor
  uint32_t acq_gen = 0;
  for (;;) {
    if (wib == 0 && !have) {
      ServeItem it = {-1, 0u, 0u, 0, 0};
      for (;;) {
        unsigned long long w = 0;
        const int q = find_run(s, ns, [&](uint32_t k) { return &claims[mine[k]].claim; }, w);
        if (q >= 0) {
          s = (uint32_t)q;
          it.slot = mine[q];
          it.gen = (uint32_t)(w >> 32);
          it.tile = (uint32_t)w & 0xffffu;
          if (it.slot != acq_slot || it.gen > acq_gen) {
            block_acquire();
            acq_slot = it.slot;
            acq_gen = it.gen;
          }
          break;
        }
        if (idle(X, seen_progress, since)) break;
      }
      if (lane == 0) item = it;
    }
    __syncthreads();
    const int slot = __builtin_amdgcn_readfirstlane(item.slot);
    if (slot < 0) return;
    const uint32_t gen = __builtin_amdgcn_readfirstlane(item.gen), tile = __builtin_amdgcn_readfirstlane(item.tile);
    const int phase = (int)(gen & 3u);
    SolveDev& D = solves[slot];
    const SolveDev& S = const_table(D);   // for the fields no round writes
    ServeClaim& C = claims[slot];
    const int64_t n = S.n;
    const int n_tiles = S.n_tiles;
    switch (phase) {
      case PH_INIT: serve_tile<PH_INIT>(S, n, (int)tile, dsum); break;
      case PH_SPMV_DOT: serve_tile<PH_SPMV_DOT>(S, n, (int)tile, dsum); break;
      case PH_AXPY_DOT: serve_tile<PH_AXPY_DOT>(S, n, (int)tile, dsum); break;
      default: serve_tile<PH_UPDATE_P>(S, n, (int)tile, dsum); break;
    }
    if (phase != PH_UPDATE_P) {
      __syncthreads();
      if (wib == 0) {
        const double v = wave_sum(tile_lane_sum<double, 8>(dsum, lane, 1, (int64_t)tile * S_TH, n, 0, 0, 0));
        if (lane == 0) {
          tot = v;
          if (n_tiles > 1) global_ptr<double>(S.partials)[tile] = v;
        }
      }
    }
    since = __builtin_amdgcn_s_memrealtime();
    if (n_tiles > 1) {
      xcd_release();
      __syncthreads();
      if (wib == 0) {
        uint32_t d = 0;
        if (lane == 0) d = xadd(&C.done, 1u);
        const bool last = __builtin_amdgcn_readfirstlane(d) + 1 == (uint32_t)n_tiles;
        if (last) block_acquire();
        if (lane == 0) last_tile = last ? 1u : 0u;
      }
      __syncthreads();
      have = false;
      if (!__builtin_amdgcn_readfirstlane(last_tile)) continue;
      if (phase != PH_UPDATE_P && n_tiles > 4 * WAVE) {
        // chunks of 256 tile sums are complete subtrees of the tile tree
        const int c0 = wib * 4 * WAVE;
        if (c0 < n_tiles) {
          const double v = block_tree(global_ptr<const double>(S.partials) + c0, min(4 * WAVE, n_tiles - c0), lane);
          if (lane == 0) csum[wib] = v;
        }
        __syncthreads();
      }
    } else {
      __syncthreads();
    }
    acq_slot = slot;
    acq_gen = gen + 1;
    // ---- the phase is complete: the solve's scalars, then its next phase ----
    if (wib == 0) {
      double total = 0.0;
      if (phase != PH_UPDATE_P)
        total = n_tiles == 1 ? tot
              : n_tiles > 4 * WAVE ? block_tree(csum, (n_tiles + 4 * WAVE - 1) / (4 * WAVE), lane)
                                   : block_tree(global_ptr<const double>(S.partials), n_tiles, lane);
      if (lane == 0) {
        int32_t status = SOLVE_RUN;
        bool pause = false;
        uint32_t next = gen + 1;
        if (phase == PH_INIT) {
          D.rho = total;
          D.bnorm = sqrt(total);
          status = !isfinite(total) ? SOLVE_BREAKDOWN : (total == 0.0 ? SOLVE_CONVERGED : SOLVE_RUN);
        } else if (phase == PH_SPMV_DOT) {
          D.pq = total;
          if (!(total > 0.0) || !isfinite(total)) status = SOLVE_BREAKDOWN;
          else D.alpha = load_0d<double>(&D.rho) / total;
        } else if (phase == PH_AXPY_DOT) {
          const double rho_new = total;
          D.beta = rho_new / load_0d<double>(&D.rho);
          D.rho = rho_new;
          const int32_t iters = xload(&D.iters) + 1;
          D.iters = iters;
          if (!isfinite(rho_new)) status = SOLVE_BREAKDOWN;
          else if (sqrt(rho_new) <= S.tol * load_0d<double>(&D.bnorm)) status = SOLVE_CONVERGED;
          else if (iters >= S.max_iter) status = SOLVE_MAXITER;
        } else {
          next = gen + 2;   // (phase 0 of a generation is the set-up, run once)
          const int32_t it = xload(&C.round_iters) + 1;
          xstore(&C.round_iters, it);
          pause = it >= ctl->iters;
        }
        if (status != SOLVE_RUN || phase == PH_INIT) xstore(&D.status, status);
        const bool settled = status != SOLVE_RUN || pause;
        item.gen = next;
        item.tile = 0u;
        item.have = settled ? 0 : 1;
        item.publish = settled || n_tiles > 1;
        xadd(&X.progress, 1u);
      }
    }
    __syncthreads();
    have = __builtin_amdgcn_readfirstlane(item.have) != 0;
    if (__builtin_amdgcn_readfirstlane(item.publish)) {
      xcd_release();   // every wave's stores since the solve was last published
      __syncthreads();
      if (threadIdx.x == 0) {
        xstore(&C.done, 0u);
        xcd_release();
        // the next phase opens with its first tile taken by this block
        xstore(&C.claim, claim_word(item.gen, item.have ? (uint32_t)n_tiles : 0u, 1u));
        if (!item.have) xadd(&X.n_settled, 1u);
      }
    }
  }
}

int launch_serve_round(SolveDev* solves, ServeClaim* claims, const int32_t* list, ServeRound* ctl, int grid,
                       hipStream_t stream) {
  hipLaunchKernelGGL(serve_round_kernel, dim3(grid), dim3(COOP_BLOCK), 0, stream, solves, claims, list, ctl);
  return (int)hipGetLastError();
}

int launch_serve_phase(const ServeLaunch& L, hipStream_t stream) {
  switch (L.phase) {
    case PH_INIT: hipLaunchKernelGGL(serve_phase_kernel<PH_INIT>, dim3(L.grid), dim3(BLOCK), 0, stream, L); break;
    case PH_SPMV_DOT: hipLaunchKernelGGL(serve_phase_kernel<PH_SPMV_DOT>, dim3(L.grid), dim3(BLOCK), 0, stream, L); break;
    case PH_AXPY_DOT: hipLaunchKernelGGL(serve_phase_kernel<PH_AXPY_DOT>, dim3(L.grid), dim3(BLOCK), 0, stream, L); break;
    default: hipLaunchKernelGGL(serve_phase_kernel<PH_UPDATE_P>, dim3(L.grid), dim3(BLOCK), 0, stream, L); break;
  }
  if (L.phase != PH_UPDATE_P && L.n_fin > 0)
    hipLaunchKernelGGL(serve_final_kernel, dim3(L.n_fin), dim3(BLOCK), 0, stream, L.solves, L.fin_slots, L.phase);
  return (int)hipGetLastError();
}

}  // namespace dfx

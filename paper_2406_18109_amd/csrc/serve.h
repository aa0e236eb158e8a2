// Device-side state of the batched CG executor (continuous-batching server).
#pragma once
#include <stdint.h>

#include "claim.h"

namespace dfx {

// One resident solve.  Vectors follow the canonical 1-D tiling of the
// op-list kernel (rows of 128 FP64 elements, tiles of 32 rows), so every
// reduction is the same tree the unbatched path computes.
struct SolveDev {
  const int32_t* rowptr;
  const int32_t* col;
  const double* val;
  const double* b;
  double* x;
  double* r;
  double* p;
  double* q;
  double* partials;     // n_tiles tile sums
  int64_t n;
  int32_t nnz;
  int32_t n_tiles;
  int32_t max_iter;
  double tol;
  double rho, pq, alpha, beta, bnorm;
  int32_t iters;
  int32_t status;       // SOLVE_* below
};

constexpr int S_MAXTILES = 64 * 64;  // tiles per solve (the tile tree fits one block's LDS)

enum SolveStatus {
  SOLVE_INIT = 0,       // admitted, r = b and rho not yet formed
  SOLVE_RUN = 1,
  SOLVE_CONVERGED = 2,
  SOLVE_MAXITER = 3,
  SOLVE_BREAKDOWN = 4
};

enum ServePhase { PH_INIT = 0, PH_SPMV_DOT = 1, PH_AXPY_DOT = 2, PH_UPDATE_P = 3 };

// Work list of one phase: item i is tile item_tile[i] of solve item_slot[i].
struct ServeLaunch {
  SolveDev* solves;
  const int32_t* item_slot;
  const int32_t* item_tile;
  int64_t n_items;
  int64_t items_per_wave;
  int32_t phase;
  int32_t grid;
  const int32_t* fin_slots;  // the solves of this phase, one block each in the scalar update
  int32_t n_fin;
};

// A round as one persistent launch (serve_round_kernel): every listed solve
// runs up to `iters` iterations, its phases claimed tile by tile by the
// blocks of the XCD it is pinned to for the round.
struct ServeClaim {
  unsigned long long claim;  // claim_word; the generation counts the solve's phases: 4 * iteration + phase
  uint32_t done;             // tiles finished of the current phase
  int32_t round_iters;       // iterations completed in this launch
};
struct ServeRound {
  XcdCtl x[MAX_XCD];         // n_streams listed solves from `first` on
  uint32_t n_xcd;
  int32_t iters;
};

// How a round ended: every solve run; or some XCD got no block and its solves
// are as they were (an XCD of the list may have no block where the hardware's
// ids are not 0 to n_xcd - 1); or some solve was begun and not settled.
// given: the claims that the round started with, now: those it left.
enum RoundEnd { ROUND_WHOLE, ROUND_UNSERVED, ROUND_BROKEN };
inline RoundEnd round_end(const ServeRound& R, const int32_t* list, const ServeClaim* given, const ServeClaim* now) {
  if (all_settled(R.x, R.n_xcd)) return ROUND_WHOLE;
  for (uint32_t k = 0; k < R.n_xcd; ++k) {
    if (R.x[k].n_settled == R.x[k].n_streams) continue;
    for (uint32_t j = 0; j < R.x[k].n_streams; ++j) {
      const int32_t i = list[R.x[k].first + j];
      if (now[i].claim != given[i].claim || now[i].done != 0) return ROUND_BROKEN;
    }
  }
  return ROUND_UNSERVED;
}

// Blocks of a round on each XCD: as many as the fullest one has tiles, and at
// most seven eighths of its compute units, unless a solve alone on its XCD
// then takes its tiles in one pass more (solves that share one fill in for
// each other).  A block holds its compute unit for the whole round; with one
// on every unit, the device's other streams waited for rounds to end.  Beside
// sixteen solves of 16 tiles, with phase launches, with blocks of 116
// registers on every unit, and as here with 96 registers: ten CG iterations
// over 300^2 0.88, 6.2 and 0.62 ms, four Jacobi sweeps of 4096^2 0.73, 4.3 and
// 1.45, eight scaled copies of 2^24 doubles 0.65, 3.8 and 1.6; beside one such
// solve the CG 0.66, 3.7 and 0.44.  The fewer registers alone: 5.0, 1.43 and
// 2.2 ms beside the sixteen.  48 requests take 47.6 ms with every unit, 47.6
// with seven eighths, 48.3 with three quarters and 54.5 with half; one solve
// of 32 tiles 36.5 us an iteration with 32 blocks, 51.6 with 28.
struct XcdLoad { int64_t tiles; int32_t solves; };
inline int blocks_per_xcd(const XcdLoad* load, int n_xcd, int units) {
  const int64_t few = units - units / 8;
  int64_t fullest = 1;
  bool all = false;
  for (int x = 0; x < n_xcd; ++x) {
    const int64_t t = load[x].tiles;
    if (t > fullest) fullest = t;
    if (load[x].solves == 1 && (t + few - 1) / few > (t + units - 1) / units) all = true;
  }
  const int64_t most = all ? units : few;
  return (int)(fullest < most ? fullest : most);
}

}  // namespace dfx

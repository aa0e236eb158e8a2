// A tile run by a whole block: the device side of the batched executor
// (batch.hip) and of chained small passes (chain.hip).
//
// Where few tiles are in flight, one wave walking a tile's 32 rows is bound
// by the latency of each row (an SpMV row alone is three dependent loads).
// Here the 16 waves of a block take two rows each, loaded together.  The
// canonical lane sums follow the tile's rows in order, so reductions write
// their summands to LDS at their places in the tile and one wave per
// reduction adds them in that order (tile_lane_sum): the tile sum has the
// bits of the wave that would have owned the tile.
#pragma once
#include "vm_exec.h"

namespace dfx {

// A 0-d value that this launch may have written: never the scalar cache.
template <typename T> __device__ __forceinline__ T load_0d(const void* p);
template <> __device__ __forceinline__ double load_0d<double>(const void* p) {
  return __builtin_bit_cast(double, __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT));
}
template <> __device__ __forceinline__ float load_0d<float>(const void* p) {
  return __builtin_bit_cast(float, __hip_atomic_load((const unsigned int*)p, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT));
}

// Entries of a row summed per round of x loads: a five-point row in one
// (with more the batch kernel's 128 registers spill).
constexpr int COOP_NZ = 5;

// One 64-row group's CSR range on its way to LDS: entries [a0, a0 + cnt) as
// 16-byte vectors in registers.
template <typename T> struct CoopStage {
  static constexpr int VE = 16 / (int)sizeof(T);
  static constexpr int CC = (COOP_CAP + 4 * WAVE - 1) / (4 * WAVE), VC = (COOP_CAP + VE * WAVE - 1) / (VE * WAVE);
  typedef int32_t i4 __attribute__((ext_vector_type(4)));
  typedef T vv __attribute__((ext_vector_type(VE)));
  i4 cb[CC];
  vv vb[VC];
};

// Rows [base, base + 64 * NG64) of y = A x, NG64 64-row groups by one wave,
// row base + 64 m + l by lane l, left at yt[64 m + l].  Each group's CSR
// range goes through this wave's LDS slice (coalesced 16-byte loads, the
// next group's in flight while this one is summed); a longer range, or no
// slice (scol null), is read directly.  A row is summed in CSR order either
// way.  Row pointers and columns are clamped as in csr_row.
template <typename T, int NG64, class PT>
__device__ __forceinline__ void coop_spmv(const PT& P, const int64_t base, T* yt, int32_t* scol, T* sval) {
  typedef CoopStage<T> CS;
  const int lane = threadIdx.x & (WAVE - 1);
  const int32_t* __restrict__ rowptr = P.rowptr;
  const int32_t* __restrict__ colidx = P.colidx;
  const T* __restrict__ val = (const T*)P.val;
  const T* x = (const T*)P.x;
  const int32_t nnz = P.nnz;
  const uint32_t nx = (uint32_t)P.nx;
  const int64_t n = P.n1d;
  // row pointers of the group in hand and of the next one
  auto pointers = [&](const int m, int32_t& rb, int32_t& re) {
    const int64_t i = base + m * WAVE + lane;
    const bool ok = m < NG64 && i < n;
    rb = ok ? rowptr[i] : 0;
    re = ok ? rowptr[i + 1] : 0;
  };
  // the group's range of entries
  auto bounds = [&](const int m, const int32_t rb, const int32_t re, int32_t& nb, int32_t& ne) {
    const int last = (int)(min(base + (m + 1) * WAVE, n) - (base + m * WAVE)) - 1;
    nb = min(max(__builtin_amdgcn_readfirstlane(rb), 0), nnz);
    ne = min(max(__builtin_amdgcn_readlane(re, last), nb), nnz);
  };
  CS st;
  // its loads into st (none when it is too long)
  auto fetch = [&](const int m, const int32_t rb, const int32_t re) {
    if (!scol || m >= NG64 || base + m * WAVE >= n) return;
    int32_t nb, ne;
    bounds(m, rb, re, nb, ne);
    const int32_t a0 = nb & ~3, cnt = ne - a0;
    if (cnt > COOP_CAP) return;
#pragma unroll
    for (int u = 0; u < CS::CC; ++u) {
      const int j = (u * WAVE + lane) * 4;
      if (j < cnt) {
        if (a0 + j + 3 < nnz) st.cb[u] = *(const typename CS::i4*)(colidx + a0 + j);
        else
          for (int t = 0; t < 4; ++t) st.cb[u][t] = a0 + j + t < nnz ? colidx[a0 + j + t] : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < CS::VC; ++u) {
      const int j = (u * WAVE + lane) * CS::VE;
      if (j < cnt) {
        if (a0 + j + CS::VE - 1 < nnz) st.vb[u] = *(const typename CS::vv*)(val + a0 + j);
        else
          for (int t = 0; t < CS::VE; ++t) st.vb[u][t] = a0 + j + t < nnz ? val[a0 + j + t] : (T)0;
      }
    }
  };
  int32_t rbr, rer, rbn, ren;
  pointers(0, rbr, rer);
  pointers(1, rbn, ren);
  fetch(0, rbr, rer);
#pragma unroll 1
  for (int m = 0; m < NG64; ++m) {
    const int64_t g0 = base + m * WAVE, i = g0 + lane;
    if (g0 >= n) break;
    int32_t nb, ne;
    bounds(m, rbr, rer, nb, ne);
    const int32_t a0 = nb & ~3, cnt = ne - a0;
    const bool slice = scol && cnt <= COOP_CAP;
    if (slice) {
#pragma unroll
      for (int u = 0; u < CS::CC; ++u) {
        const int j = (u * WAVE + lane) * 4;
        if (j < cnt && j < COOP_CAP) *(typename CS::i4*)(scol + j) = st.cb[u];
      }
#pragma unroll
      for (int u = 0; u < CS::VC; ++u) {
        const int j = (u * WAVE + lane) * CS::VE;
        if (j < cnt && j < COOP_CAP) *(typename CS::vv*)(sval + j) = st.vb[u];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    fetch(m + 1, rbn, ren);
    int32_t rb2, re2;
    pointers(m + 2, rb2, re2);
    T s = (T)0;
    if (!slice) {
      if (i < n) s = csr_row<T, 4>(rowptr, colidx, val, x, i, nnz, nx);
    } else {
      if (i < n) {
        // clamped into the staged window: a malformed rowptr reads wrong
        // values, never outside it
        const int32_t rb = min(max(rbr, nb), ne);
        const int32_t re = min(max(rer, rb), ne);
        const int32_t b = rb - a0, e = re - a0;
        for (int32_t k = b; k < e; k += COOP_NZ) {
          int32_t c[COOP_NZ];
          T av[COOP_NZ], xv[COOP_NZ];
#pragma unroll
          for (int t = 0; t < COOP_NZ; ++t) {
            const int32_t kk = k + t < e ? k + t : b;
            c[t] = scol[kk];
            av[t] = sval[kk];
          }
#pragma unroll
          for (int t = 0; t < COOP_NZ; ++t) xv[t] = x[(uint32_t)c[t] < nx ? c[t] : 0];
#pragma unroll
          for (int t = 0; t < COOP_NZ; ++t)
            if (k + t < e) {
              const T tv = av[t] * xv[t];
              s = (k + t == b) ? tv : s + tv;
            }
        }
      }
      // every lane's reads are done before the slice is written again
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    yt[m * WAVE + lane] = s;
    rbr = rbn;
    rer = ren;
    rbn = rb2;
    ren = re2;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Tile t of pass P (a VmParams, or any type with its fields) by every wave
// of the block; lds: laid out as coop_lds says, tot: VM_MAXRED values in LDS that
// receive the tile's sums (from lane 0 of wave k; the caller's next barrier
// publishes them).  The pass's global stores are issued, not waited for.
template <typename T, int HV, class PT>
__device__ __forceinline__ void coop_tile(const PT& P, const int64_t t, char* lds, const int slots, const int staged,
                                          T* tot) {
  // rows per step: both of the wave's in arithmetic kernels; one in the
  // transcendental ones (their handlers need the registers: 1024 threads
  // leave 128 per lane)
  typedef Shape<T, HV, false, VM_NREG_LIGHT, (HV > 0 ? 1 : COOP_RPW)> S;
  constexpr bool HEAVY = S::HEAVY;
  constexpr int V = S::V, U = S::U, TW = S::TW, E = S::E, GS = S::GS, NG = S::NG, NR = VM_NREG_LIGHT, NINB = 6;
  typedef typename GVec<T, GS>::type gvec;
  typedef T vecA __attribute__((ext_vector_type(V), aligned(sizeof(T))));
  const int lane = threadIdx.x & (WAVE - 1);
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  T* dsum = (T*)lds;
  const int64_t tr = t / P.strips;
  const int64_t ts = t - tr * P.strips;
  const int64_t cbase = ts * TW;
  const int64_t c0 = cbase + (int64_t)lane * V;
  const int64_t row_w = tr * RED_TH + wib * COOP_RPW;
  const bool is1d = P.is1d != 0;
  const int64_t rows = P.rows, cols = P.cols, n1d = P.n1d;
  if (row_w < rows) {
    gvec R0[NR], R1[NR], R2[NR], R3[NR];
    VmState<T, NG, GS> G;
    T* yt = dsum + wib * COOP_RPW * TW;   // this wave's rows of slot 0
    if (P.spmv) {
      char* sl = lds + COOP_TILE_BYTES * (size_t)slots;
      coop_spmv<T, COOP_RPW * TW / WAVE>(P, row_w * TW, yt, staged ? (int32_t*)sl + wib * COOP_CAP : nullptr,
                                         (T*)(sl + (size_t)COOP_WAVES * COOP_CAP * 4) + wib * COOP_CAP);
    }
    for (int k = 0; k < P.n_bc; ++k) {
      const gvec v = (gvec)load_0d<T>(P.bc[k]);
      const int r = P.bc_reg[k];
      FOR_G(Rg[r] = v;)
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) G.z[g] = (gvec)(T)0;
    G.dsum = dsum;
    for (int u0 = 0; u0 < COOP_RPW; u0 += U) {
      const int64_t row0 = row_w + u0;
      if (row0 >= rows) break;
      const bool fast = P.unit_cols && (is1d ? ((row0 + U) * TW <= n1d) : (row0 + U <= rows && cbase + TW <= cols));
      unsigned vmask = (1u << E) - 1;
      if (!fast) {
        vmask = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int64_t row = row0 + e / V, col = c0 + e % V;
          const bool ok = is1d ? (row * TW + col < n1d) : (row < rows && col < cols);
          vmask |= (ok ? 1u : 0u) << e;
        }
      }
      // every stream's loads issued together, straight into the register
      // file (elements outside the space load the stream's first element:
      // they are never stored nor added); the scheduling barriers keep one
      // stream's addresses live at a time
#define COOP_RSET(a, e, x) { const int g_ = (e) / GS; \
    if (g_ == 0) gset<T, GS>(R0[a], (e) % GS, x); else if (g_ == 1) gset<T, GS>(R1[a], (e) % GS, x); \
    else if (g_ == 2) gset<T, GS>(R2[a], (e) % GS, x); else gset<T, GS>(R3[a], (e) % GS, x); }
#pragma unroll
      for (int a = 0; a < NINB; ++a) {
        if (a >= P.n_in) break;
        const T* b = (const T*)P.in[a].base;
        const int64_t sr = P.in[a].s_row, sc = P.in[a].s_col;
        if (fast) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const vecA w = *(const vecA*)(b + (row0 + u) * sr + c0);
#pragma unroll
            for (int v = 0; v < V; ++v) COOP_RSET(a, u * V + v, w[v]);
          }
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const T q = b[((vmask >> e) & 1) ? (row0 + e / V) * sr + (c0 + e % V) * sc : 0];
            COOP_RSET(a, e, q);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (P.spmv) {
#pragma unroll
        for (int e = 0; e < E; ++e) COOP_RSET(NR - 1, e, yt[(u0 + e / V) * TW + lane * V + e % V]);
      }
#undef COOP_RSET
      G.drow = wib * COOP_RPW + u0;
      {
        constexpr bool DEFER_OK = true;
        VmInstr nx = P.code[0];
        for (int pc = 0; pc < P.n_code; ++pc) {
          const unsigned w0 = __builtin_amdgcn_readfirstlane(nx.w0), w1 = __builtin_amdgcn_readfirstlane(nx.w1);
          const unsigned w2 = __builtin_amdgcn_readfirstlane(nx.w2), w3 = __builtin_amdgcn_readfirstlane(nx.w3);
          nx = P.code[pc + 1];
          const unsigned flags = (w0 >> 8) & 0xff, slot = (w0 >> 16) & 0xff, post = w0 >> 24;
          const unsigned d = w1 & 0xff, ia = (w1 >> 8) & 0xff, ib = (w1 >> 16) & 0xff, ic = w1 >> 24;
          const unsigned op = w0 & 0xff;
          T k;
          if constexpr (sizeof(T) == 8) k = __builtin_bit_cast(double, ((uint64_t)w3 << 32) | w2);
          else k = __builtin_bit_cast(float, w2);
#include "vm_instr.inc"
        }
      }
      for (int s = 0; s < P.n_out; ++s) {
        const int o = P.out_reg[s];
        gvec ev[NG];
        FOR_G(ev[g] = Rg[o];)
        T* b = (T*)P.out[s].base;
        const int64_t sr = P.out[s].s_row, sc = P.out[s].s_col;
        if (fast) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            vecA w;
#pragma unroll
            for (int v = 0; v < V; ++v) w[v] = gget<T, GS>(ev[(u * V + v) / GS], (u * V + v) % GS);
            *(vecA*)(b + (row0 + u) * sr + c0) = w;
          }
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e)
            if ((vmask >> e) & 1) b[(row0 + e / V) * sr + (c0 + e % V) * sc] = gget<T, GS>(ev[e / GS], e % GS);
        }
      }
    }
  }
  if (P.n_red == 0) return;
  __syncthreads();
  if (wib < P.n_red) {
    const T acc = tile_lane_sum<T, 8>(dsum + (size_t)wib * RED_TH * TW, lane, P.is1d, tr * RED_TH, n1d, rows, cols, cbase);
    const T v = wave_sum(acc);
    if (lane == 0) tot[wib] = v;
  }
}

}  // namespace dfx

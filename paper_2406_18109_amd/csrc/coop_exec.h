// A tile run by a whole block: the device side of the batched executor
// (batch.hip) and of single passes of few tiles (coop_kernel).
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

// A pass's parameters live in a table that a launch only reads, and name
// global memory.  Saying so matters: around fences and atomics the compiler
// reads such a table with vector loads (a memory latency for every field and
// every instruction of the op list, about 3 us a pass) and data behind a
// pointer loaded from it with flat accesses.
// (Both pointers are wave-uniform; the empty asm keeps the casts from being
// folded away.)
template <typename U> __device__ __forceinline__ const U& const_table(const U& p) {
  const __attribute__((address_space(4))) U* q = (const __attribute__((address_space(4))) U*)&p;
  asm("" : "+s"(q));
  return *(const U*)q;
}
template <typename U> __device__ __forceinline__ U* global_ptr(const void* p) {
  __attribute__((address_space(1))) U* q = (__attribute__((address_space(1))) U*)p;
  asm("" : "+s"(q));
  return (U*)q;
}

// A 0-d value that this launch may have written: never the scalar cache.
template <typename T> __device__ __forceinline__ T load_0d(const void* p);
template <> __device__ __forceinline__ double load_0d<double>(const void* p) {
  return __builtin_bit_cast(double, __hip_atomic_load(global_ptr<const unsigned long long>(p),
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
template <> __device__ __forceinline__ float load_0d<float>(const void* p) {
  return __builtin_bit_cast(float, __hip_atomic_load(global_ptr<const unsigned int>(p), __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT));
}

// Entries [f, f + COOP_NZ) of a CSR row, read as 16-byte vectors.
constexpr int COOP_NZ = 8;   // (a seven-point row in one round)
template <typename T> struct CoopEntries {
  int32_t c[COOP_NZ];
  T a[COOP_NZ];
  __device__ __forceinline__ void load(const int32_t* __restrict__ colidx, const T* __restrict__ val, const int32_t f) {
    constexpr int VE = 16 / (int)sizeof(T);
    typedef int32_t i4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef T vv __attribute__((ext_vector_type(VE), aligned(sizeof(T))));
#pragma unroll
    for (int j = 0; j < COOP_NZ; j += 4) {
      const i4 w = *(const i4*)(colidx + f + j);
#pragma unroll
      for (int t = 0; t < 4; ++t) c[j + t] = w[t];
    }
#pragma unroll
    for (int j = 0; j < COOP_NZ; j += VE) {
      const vv w = *(const vv*)(val + f + j);
#pragma unroll
      for (int t = 0; t < VE; ++t) a[j + t] = w[t];
    }
  }
  // s + a0 x0 + a1 x1 ..., the first n entries in order.  Columns are
  // clamped to [0, nx); the x of entries past n is read and not added.
  __device__ __forceinline__ T add(T s, const T* x, const uint32_t nx, const int32_t n) const {
    T xv[COOP_NZ];
#pragma unroll
    for (int j = 0; j < COOP_NZ; ++j) {
      if (__ballot(j < n) == 0ull) break;
      xv[j] = x[min((uint32_t)c[j], nx - 1u)];
    }
#pragma unroll
    for (int j = 0; j < COOP_NZ; ++j) {
      if (__ballot(j < n) == 0ull) break;
      const T t = a[j] * xv[j];
      if (j < n) s = s + t;
    }
    return s;
  }
};

// Rows [base, base + 64 * NG64) of y = A x by one wave, row base + 64 m + l
// by lane l, left at yt[64 m + l], each summed in CSR order as csr_row sums
// it.  Every lane reads its row as 16-byte vectors, eight entries a round,
// all rows' pointers at once and the next row's entries while this one's x
// is gathered, so few memory latencies follow one another.  -0.0 is the
// neutral start of the sequential sum: the first product is the row's first
// partial sum, sign of zero included.  Row pointers are clamped to [0, nnz];
// the matrix's last rows, whose rounds of COOP_NZ entries would read past
// the arrays, are read by csr_row.
template <typename T, int NG64, class PT>
__device__ __forceinline__ void coop_spmv(const PT& P, const int64_t base, T* yt) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int32_t* __restrict__ rowptr = global_ptr<const int32_t>(P.rowptr);
  const int32_t* __restrict__ colidx = global_ptr<const int32_t>(P.colidx);
  const T* __restrict__ val = global_ptr<const T>(P.val);
  const T* x = global_ptr<const T>(P.x);
  const uint32_t nx = (uint32_t)P.nx;
  const int32_t nnz = nx ? P.nnz : 0;
  const int left = (int)min(P.n1d - base, (int64_t)NG64 * WAVE);   // rows of this wave
  const int32_t* rp = rowptr + base;
  int32_t rb[NG64], len[NG64];
  bool tail = false;
#pragma unroll
  for (int m = 0; m < NG64; ++m) {
    const int i = m * WAVE + lane;
    const int32_t b0 = i < left ? rp[i] : 0, e0 = i < left ? rp[i + 1] : 0;
    rb[m] = min(max(b0, 0), nnz);
    len[m] = min(max(e0, rb[m]), nnz) - rb[m];
    const bool past = (uint32_t)rb[m] + (((uint32_t)len[m] + COOP_NZ - 1) & ~(uint32_t)(COOP_NZ - 1)) > (uint32_t)nnz;
    len[m] = past ? -1 : len[m];
    rb[m] = len[m] > 0 ? rb[m] : 0;   // (loaded all the same; nnz >= COOP_NZ below)
    tail = tail || past;
  }
  const bool any = nnz >= COOP_NZ;   // else every row is read by csr_row
  CoopEntries<T> e[2];
  if (any) e[0].load(colidx, val, rb[0]);
#pragma unroll
  for (int m = 0; m < NG64; ++m) {
    if (!any || m * WAVE >= left) break;
    if (m + 1 < NG64) e[(m + 1) & 1].load(colidx, val, rb[m + 1]);
    T s = e[m & 1].add(-(T)0, x, nx, len[m]);
    for (int32_t k = COOP_NZ; __ballot(k < len[m]) != 0ull; k += COOP_NZ) {
      CoopEntries<T> q;
      q.load(colidx, val, k < len[m] ? rb[m] + k : 0);
      s = q.add(s, x, nx, len[m] - k);
    }
    yt[m * WAVE + lane] = len[m] > 0 ? s : (T)0;
  }
  if (!any || __ballot(tail) != 0ull) {
#pragma unroll 1
    for (int m = 0; m < NG64; ++m) {
      const int i = m * WAVE + lane;
      bool past = false;
#pragma unroll
      for (int q = 0; q < NG64; ++q) past = q == m ? len[q] < 0 : past;
      if (past) yt[i] = csr_row<T>(rowptr, colidx, val, x, base + i, nnz, nx);
      else if (!any) yt[i] = (T)0;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Tile t of pass P (a VmParams, or any type with its fields) by every wave
// of the block; lds: coop_lds bytes, tot: VM_MAXRED values in LDS that
// receive the tile's sums (from lane 0 of wave k; the caller's next barrier
// publishes them).  The pass's global stores are issued, not waited for.
template <typename T, int HV, class PG = VmInterp, class PT>
__device__ __forceinline__ void coop_tile(const PT& P, const int64_t t, char* lds, T* tot) {
  constexpr int RPW = COOP_RPW;
  // rows per step: two in arithmetic kernels; one in the transcendental ones
  // (their handlers need the registers: 1024 threads leave 128 per lane)
  typedef Shape<T, HV, false, VM_NREG_LIGHT, (HV > 0 ? 1 : 2)> S;
  constexpr bool HEAVY = S::HEAVY;
  constexpr int V = S::V, U = S::U, TW = S::TW, E = S::E, GS = S::GS, NG = S::NG, NR = VM_NREG_LIGHT, NINB = 6;
  typedef typename GVec<T, GS>::type gvec;
  typedef T vecA __attribute__((ext_vector_type(V), aligned(sizeof(T))));
  const int lane = threadIdx.x & (WAVE - 1);
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  T* dsum = (T*)lds;
  // (a space has at most 2^20 tiles)
  const int64_t tr = P.strips == 1 ? t : (int64_t)((uint32_t)t / (uint32_t)P.strips);
  const int64_t cbase = (t - tr * P.strips) * TW;
  const int64_t row_w = tr * RED_TH + wib * RPW;   // this wave's first row
  const bool is1d = P.is1d != 0;
  if (row_w < P.rows) {
    gvec R0[NR], R1[NR], R2[NR], R3[NR];
    VmState<T, NG, GS> G;
    T* yt = dsum + wib * RPW * TW;   // this wave's rows of slot 0
    if (P.spmv) coop_spmv<T, RPW * TW / WAVE>(P, row_w * TW, yt);
    if constexpr (PG::COMPILED) {
#pragma unroll
      for (int k = 0; k < VM_MAXBC; ++k) {
        if (k >= P.n_bc) break;
        const gvec v = (gvec)load_0d<T>(P.bc[k]);
        FOR_G(Rg[PG::bc_reg[k]] = v;)
      }
    } else {
      for (int k = 0; k < P.n_bc; ++k) {
        const gvec v = (gvec)load_0d<T>(P.bc[k]);
        const int r = P.bc_reg[k];
        FOR_G(Rg[r] = v;)
      }
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) G.z[g] = (gvec)(T)0;
    G.dsum = dsum;
    // 1-D passes of unit stride: every stream at one 32-bit offset from its
    // scalar base (the wave's first element)
    const bool line = is1d && P.unit_cols;
    const int left = is1d ? (int)min(P.n1d - row_w * TW, (int64_t)RPW * TW) : 0;
    for (int u0 = 0; u0 < RPW; u0 += U) {
      const int64_t row0 = row_w + u0;
      if (row0 >= P.rows) break;
      const int i0 = u0 * TW + lane * V;   // the lane's first element from the wave's
      bool fast;
      unsigned vmask = (1u << E) - 1;
      if (is1d) {
        fast = P.unit_cols && left >= (u0 + U) * TW;
        if (!fast) {
          vmask = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) vmask |= (i0 + (e / V) * TW + e % V < left ? 1u : 0u) << e;
        }
      } else {
        const int64_t c0 = cbase + (int64_t)lane * V;
        fast = P.unit_cols && row0 + U <= P.rows && cbase + TW <= P.cols;
        if (!fast) {
          vmask = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) vmask |= (row0 + e / V < P.rows && c0 + e % V < P.cols ? 1u : 0u) << e;
        }
      }
      // every stream's loads issued together, straight into the register
      // file (elements outside the space load some element inside it: they
      // are never stored nor added); the scheduling barriers keep one
      // stream's addresses live at a time
#define COOP_RSET(a, e, x) { const int g_ = (e) / GS; \
    if (g_ == 0) gset<T, GS>(R0[a], (e) % GS, x); else if (g_ == 1) gset<T, GS>(R1[a], (e) % GS, x); \
    else if (g_ == 2) gset<T, GS>(R2[a], (e) % GS, x); else gset<T, GS>(R3[a], (e) % GS, x); }
#pragma unroll
      for (int a = 0; a < NINB; ++a) {
        if (a >= (PG::COMPILED ? PG::N_IN : P.n_in)) break;
        const int64_t sr = P.in[a].s_row, sc = P.in[a].s_col;
        const T* b = global_ptr<const T>(P.in[a].base) + row0 * sr;
        if (fast) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const vecA w = *(const vecA*)(b + u * sr + cbase + lane * V);
#pragma unroll
            for (int v = 0; v < V; ++v) COOP_RSET(a, u * V + v, w[v]);
          }
        } else if (line) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const T q = b[(uint32_t)(min(i0 + (e / V) * TW + e % V, left - 1) - u0 * TW)];
            COOP_RSET(a, e, q);
          }
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const T q = b[((vmask >> e) & 1) ? (e / V) * sr + (cbase + lane * V + e % V) * sc : cbase * sc];
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
      G.drow = wib * RPW + u0;
      if constexpr (PG::COMPILED) {
        PG::template run<T, HV, NR, NG, GS, E>(R0, R1, R2, R3, G, vmask);
      } else {
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
      // (one loop for both: a shared lambda spilled the batched executor's
      // registers, 34 -> 40 ms for 32 solves)
#pragma unroll(PG::COMPILED ? VM_MAXOUT : 1)
      for (int s = 0; s < (PG::COMPILED ? PG::N_OUT : P.n_out); ++s) {
        const int o = PG::COMPILED ? PG::out_reg[s] : P.out_reg[s];
        gvec ev[NG];
        FOR_G(ev[g] = Rg[o];)
        const int64_t sr = P.out[s].s_row, sc = P.out[s].s_col;
        T* b = global_ptr<T>(P.out[s].base) + row0 * sr;
        if (fast) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            vecA w;
#pragma unroll
            for (int v = 0; v < V; ++v) w[v] = gget<T, GS>(ev[(u * V + v) / GS], (u * V + v) % GS);
            *(vecA*)(b + u * sr + cbase + lane * V) = w;
          }
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e)
            if ((vmask >> e) & 1) {
              if (line) b[(uint32_t)((e / V) * TW + lane * V + e % V)] = gget<T, GS>(ev[e / GS], e % GS);
              else b[(e / V) * sr + (cbase + lane * V + e % V) * sc] = gget<T, GS>(ev[e / GS], e % GS);
            }
        }
      }
    }
  }
  if (P.n_red == 0) return;
  __syncthreads();
  if (wib < P.n_red) {
    const T acc = tile_lane_sum<T, 8>(dsum + (size_t)wib * RED_TH * TW, lane, P.is1d, tr * RED_TH, P.n1d, P.rows,
                                      P.cols, cbase);
    const T v = wave_sum(acc);
    if (lane == 0) tot[wib] = v;
  }
}

// One ordinary pass with a block of 16 waves for every tile (the rule and its
// measurements: coop_pass in core.cpp), interpreted or compiled.  Bound: with
// a wave per tile the chain of 32 rows' loads (and, in SpMV, the row walks)
// of one wave; here a wave has two rows, the lane sums run in their order
// from LDS, and 16 waves per tile keep the gathers of x in flight (BiCGSTAB
// over 150 cubed, 8 iterations: 4039 -> 2370 us).  The tile's sum has the
// ordinary pass's bits; a lone block finishes its results itself
// (red_direct), otherwise the block-sum reduction gets one sum per tile.
template <typename T, class PG = VmInterp>
__global__ __launch_bounds__(COOP_BLOCK) void coop_kernel(const VmParams P) {
  extern __shared__ __attribute__((aligned(16))) char coop_dyn_lds[];
  __shared__ T tot[VM_MAXRED];
  coop_tile<T, 0, PG>(P, (int64_t)blockIdx.x, coop_dyn_lds, tot);
  // (wave k holds reduction k's tile sum)
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  if (wib < P.n_red && (threadIdx.x & (WAVE - 1)) == 0) {
    const T v = tot[wib];
    if (P.red_direct) {
      T* res = (T*)P.red_result[wib];
      *res = P.red_init[wib] ? v : *res + v;
    } else {
      ((T*)P.red_partials[wib])[blockIdx.x] = v;
    }
  }
}

}  // namespace dfx

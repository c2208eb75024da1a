// Device helpers shared by the HIP kernels: stored-type loads of X, fixed-tree
// reductions, affine-map scans (the linear recurrences of the tridiagonal
// LDL^T sweeps) and Moebius-map scans (its pivots).
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "flr_internal.h"

namespace flr {

// ---------------------------------------------------------------------------
// stored-type loads: 16 bytes per lane, widened to double
// ---------------------------------------------------------------------------
template <typename XT> struct XV;
template <> struct XV<double> {
  static constexpr int V = 2;
  using raw = double2;
  __device__ static inline void cvt(const raw& v, double* o) { o[0] = v.x; o[1] = v.y; }
  __device__ static inline void cvt(const raw& v, float* o) { o[0] = (float)v.x; o[1] = (float)v.y; }
};
template <> struct XV<float> {
  static constexpr int V = 4;
  using raw = float4;
  __device__ static inline void cvt(const raw& v, double* o) {
    o[0] = (double)v.x; o[1] = (double)v.y; o[2] = (double)v.z; o[3] = (double)v.w;
  }
  __device__ static inline void cvt(const raw& v, float* o) { o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
};
template <> struct XV<uint16_t> {  // bfloat16 bit patterns
  static constexpr int V = 8;
  using raw = uint4;
  __device__ static inline double lo(uint32_t w) { return (double)__uint_as_float(w << 16); }
  __device__ static inline double hi(uint32_t w) { return (double)__uint_as_float(w & 0xffff0000u); }
  __device__ static inline void cvt(const raw& v, double* o) {
    o[0] = lo(v.x); o[1] = hi(v.x); o[2] = lo(v.y); o[3] = hi(v.y);
    o[4] = lo(v.z); o[5] = hi(v.z); o[6] = lo(v.w); o[7] = hi(v.w);
  }
  __device__ static inline float lof(uint32_t w) { return __uint_as_float(w << 16); }
  __device__ static inline float hif(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
  __device__ static inline void cvt(const raw& v, float* o) {
    o[0] = lof(v.x); o[1] = hif(v.x); o[2] = lof(v.y); o[3] = hif(v.y);
    o[4] = lof(v.z); o[5] = hif(v.z); o[6] = lof(v.w); o[7] = hif(v.w);
  }
};

template <typename XT>
__device__ inline typename XV<XT>::raw load16(const XT* p) {
  return *reinterpret_cast<const typename XV<XT>::raw*>(p);
}

// ---------------------------------------------------------------------------
// reductions and scans over one 256-thread workgroup (fixed trees)
// ---------------------------------------------------------------------------
// Butterfly sum over the wave, distances 32, 16, 8, 4, 2, 1, in the vector
// registers: lane halves and rows by permlane swaps (both results hold one
// operand each, so their sum is the pair's), the rest by DPP moves (after the
// distance 8 every row repeats with period 8, so a rotation by 4 pairs the
// right values).  The same additions as with __shfl_xor, whose LDS round trips
// take about five times as long.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double wave_sum(double v) {
  {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  }
  {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  }
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x4e>(v);   // quad_perm [2,3,0,1]
  v += dpp_f64<0xb1>(v);   // quad_perm [1,0,3,2]
  return v;
}

// Values that workgroups of one launch pass to the last one to arrive.  They
// are written and read at the device's coherence point (agent-scope atomics
// bypass the XCDs' own L2), so the publisher only waits for those stores: a
// release fence writes the whole dirty L2 back instead.  With the sums above the
// block kernel went from 10.2 to 9.1 us at 40 blocks and 17.3 to 13.4 at 391.
__device__ inline void put_shared(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double get_shared(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The wave's own stores have completed.  A barrier does not wait for another
// wave's, so where several waves publish each calls this before the barrier that
// precedes arrive().
__device__ inline void published() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_s_waitcnt(0x0f70);  // gfx9 encoding: vmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}
// Called by one thread after everything its workgroup published has completed (its
// own wave's stores are waited for here); true for the last of `count` arrivals,
// which may then read every publisher's values.
__device__ inline bool arrive(unsigned* counter, int count) {
  published();
  const unsigned prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return prev == (unsigned)(count - 1);
}

// The sums and scans below run over groups of 256 threads: the workgroup, or each
// half of one of 512 (with LDS of its own; the barriers are the workgroup's).

// Sum over the group; every thread receives the result.  lds: 4 doubles.
__device__ inline double wg_sum(double v, double* lds) {
  v = wave_sum(v);
  const int w = (threadIdx.x >> 6) & 3, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) lds[w] = v;
  __syncthreads();
  return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// Four sums over the group at once (one pair of barriers).  lds: 16 doubles.
__device__ inline void wg_sum4(double* v, double* lds) {
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = wave_sum(v[k]);
  const int w = (threadIdx.x >> 6) & 3, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) lds[4 * w + k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = (lds[k] + lds[4 + k]) + (lds[8 + k] + lds[12 + k]);
}

// Workgroup barrier that orders LDS only: each wave waits for its own LDS
// operations (lgkmcnt 0) but not for its outstanding global loads, which may
// stay in flight across the barrier (a plain __syncthreads waits for them,
// which defeats loads issued ahead).  The wavefront-scope fences generate no
// code; they keep the compiler from moving memory operations across.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // gfx9 encoding: lgkmcnt(0), vmcnt and expcnt left at their maximum
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (B v)_j for the weighted Laplacian of E, row j of its CSR: the first four
// entries are requested at once and ahead of the values of v (a loop over the row
// waits for its index and then for its value, entry by entry).  In steps, so that
// a caller can put other work between the loads: rows(), entries(), then lap().
struct EdgeRow {
  int q0, q1;
  int col[4];
  double w[4];
  __device__ inline void rows(const int32_t* __restrict__ rowptr, int64_t j) {
    q0 = rowptr[j];
    q1 = rowptr[j + 1];
  }
  // indices past the row stay inside the arrays (nnz >= 1 entries are allocated)
  __device__ inline void entries(const int32_t* __restrict__ c, const double* __restrict__ ws, int64_t nnz) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = min(q0 + e, (int)nnz - 1);
      col[e] = c[q];
      w[e] = ws[q];
    }
  }
  // sum over the row of w (v_j - v_k), in the row's order
  __device__ inline double lap(const int32_t* __restrict__ c, const double* __restrict__ ws, const double* v,
                               double vj) const {
    double vk[4], s = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) vk[e] = v[col[e]];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (q0 + e < q1) s = fma(w[e], vj - vk[e], s);
    for (int q = q0 + 4; q < q1; ++q) s = fma(ws[q], vj - v[c[q]], s);
    return s;
  }
};

// Affine map t -> a t + b.  compose(E, L) applies E first, then L.
struct Aff {
  double a, b;
};
__device__ inline Aff compose(Aff E, Aff Lm) { return {Lm.a * E.a, Lm.a * E.b + Lm.b}; }

// Inclusive scan in thread order 0..255 (recurrence t_j = a_j t_{j-1} + b_j).
// lds: 8 doubles.
__device__ inline Aff wg_scan_fwd(Aff m, double* lds) {
  const int l = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    double pa = __shfl_up(m.a, d, 64), pb = __shfl_up(m.b, d, 64);
    if (l >= d) m = compose({pa, pb}, m);
  }
  __syncthreads();
  if (l == 63) { lds[2 * w] = m.a; lds[2 * w + 1] = m.b; }
  __syncthreads();
  Aff pre = {1.0, 0.0};
  for (int v = 0; v < w; ++v) pre = compose(pre, {lds[2 * v], lds[2 * v + 1]});
  return compose(pre, m);
}

// Inclusive scan in thread order 255..0 (recurrence t_j = a_j t_{j+1} + b_j).
__device__ inline Aff wg_scan_rev(Aff m, double* lds) {
  const int l = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    double pa = __shfl_down(m.a, d, 64), pb = __shfl_down(m.b, d, 64);
    if (l + d < 64) m = compose({pa, pb}, m);
  }
  __syncthreads();
  if (l == 0) { lds[2 * w] = m.a; lds[2 * w + 1] = m.b; }
  __syncthreads();
  Aff pre = {1.0, 0.0};
  for (int v = 3; v > w; --v) pre = compose(pre, {lds[2 * v], lds[2 * v + 1]});
  return compose(pre, m);
}

// Inclusive scans over the 64 lanes of one wave (no barriers).
__device__ inline Aff wave_scan_fwd(Aff m) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    double pa = __shfl_up(m.a, d, 64), pb = __shfl_up(m.b, d, 64);
    if (l >= d) m = compose({pa, pb}, m);
  }
  return m;
}
__device__ inline Aff wave_scan_rev(Aff m) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    double pa = __shfl_down(m.a, d, 64), pb = __shfl_down(m.b, d, 64);
    if (l + d < 64) m = compose({pa, pb}, m);
  }
  return m;
}

// LDL^T of the tridiagonal part of M as a scan.  With e_j >= 0 the coupling of
// (j-1, j) (M_{j,j-1} = -e_j) and alpha_j >= 0 the rest of the diagonal
// (M_jj = alpha_j + e_j + e_{j+1}), the pivots are D_j = t_j + e_{j+1} where
//   t_j = alpha_j + e_j t_{j-1} / (t_{j-1} + e_j),   L_j = -e_j / (t_{j-1} + e_j):
// t_{j-1} -> t_j is a Moebius map with a nonnegative 2 x 2 matrix.  Products of
// such matrices add nonnegative terms only, so nothing cancels and every
// prefix has full relative accuracy in any association, over weights of any
// spread (the textbook form D_j = M_jj - e_j^2 / D_{j-1} cancels where e_j is
// near 1/eps, and a scan of its products loses every digit).  The serial chain
// this replaces took 41 ns per element.
struct Mob {
  double a, b, c, d;  // t -> (a t + b) / (c t + d), all >= 0
};
// Exactness has an end: with lambda1 below 1e-16 lambda2 the exact M is singular to
// working precision, M^-1 as large as 1 / lambda1 and PCG with it breaks down, while
// the textbook form's own rounding kept the pivots near half an ulp of the couplings.
// alpha gets that as its least value (lambda1 = 1e-30, p = 1500, X = I: 6000 steps to
// the cap and a wrong iterate without, 3500 with it, 3780 with the textbook form);
// where lambda1 / |b| is above 1e-16 lambda2 / eps no value changes.
__device__ inline Mob mob_leaf(double alpha, double e) {
  if (!(e > 0.0)) return {0.0, alpha, 0.0, 1.0};  // no coupling: the map is constant
  if (alpha < 0x1p-53 * e) alpha = 0x1p-53 * e;  // not fmax, which would drop a NaN
  if (e >= 1.0) return {alpha / e + 1.0, alpha, 1.0 / e, 1.0};
  return {alpha + e, alpha * e, 1.0, e};
}
// E first, then L; scaled by a power of two (exact) so that long products stay in range.
__device__ inline Mob mob_compose(const Mob& E, const Mob& L) {
  Mob r = {fma(L.a, E.a, L.b * E.c), fma(L.a, E.b, L.b * E.d), fma(L.c, E.a, L.d * E.c), fma(L.c, E.b, L.d * E.d)};
  const int k = -__builtin_amdgcn_frexp_exp(fmax(fmax(r.a, r.b), fmax(r.c, r.d)));
  r.a = __builtin_amdgcn_ldexp(r.a, k);
  r.b = __builtin_amdgcn_ldexp(r.b, k);
  r.c = __builtin_amdgcn_ldexp(r.c, k);
  r.d = __builtin_amdgcn_ldexp(r.d, k);
  return r;
}
__device__ inline double mob_apply(const Mob& m, double t) { return fma(m.a, t, m.b) / fma(m.c, t, m.d); }

// Inclusive scan of the workgroup's maps in thread order 0..255.  lds: 16 doubles.
__device__ inline Mob wg_scan_mob(Mob m, double* lds) {
  const int l = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const Mob pm = {__shfl_up(m.a, d, 64), __shfl_up(m.b, d, 64), __shfl_up(m.c, d, 64), __shfl_up(m.d, d, 64)};
    if (l >= d) m = mob_compose(pm, m);
  }
  __syncthreads();
  if (l == 63) {
    lds[4 * w] = m.a;
    lds[4 * w + 1] = m.b;
    lds[4 * w + 2] = m.c;
    lds[4 * w + 3] = m.d;
  }
  __syncthreads();
  if (w > 0) {
    Mob pre = {lds[0], lds[1], lds[2], lds[3]};
    for (int v = 1; v < w; ++v) pre = mob_compose(pre, {lds[4 * v], lds[4 * v + 1], lds[4 * v + 2], lds[4 * v + 3]});
    m = mob_compose(pre, m);
  }
  return m;
}

// LDL^T of a symmetric tridiagonal matrix (diagonal d, sub-diagonal
// e_j = M_{j,j-1}, e_0 = 0): L_j = e_j / D_{j-1}, D_j = d_j - e_j L_j.  The
// pivots form one dependent chain, so a single wave runs it: the lanes stage
// 64 (d, e) pairs at a time through this wave's LDS and prefetch the next 64
// from memory while the chain runs on broadcast reads; lane t keeps element t
// of the chunk for one coalesced store.  1/D_j is the hardware reciprocal
// refined by two Newton steps (within an ulp or two of the quotient), so the
// chain carries one multiply, one fma, the reciprocal and four fmas per
// element.  Called by all 64 lanes of one wave; stage: 128 doubles of LDS
// that no other wave touches meanwhile.
__device__ inline void tri_factor_wave(const double* d, const double* e, double* L, double* invD, int64_t p,
                                       double* stage) {
  const int lane = threadIdx.x & 63;
  double rprev = 0.0;  // 1/D_{-1}: e_0 = 0 makes L_0 = 0, D_0 = d_0
  double dn = lane < p ? d[lane] : 1.0;
  double en = lane < p ? e[lane] : 0.0;
  for (int64_t c0 = 0; c0 < p; c0 += 64) {
    stage[2 * lane] = dn;
    stage[2 * lane + 1] = en;
    const int64_t jn = c0 + 64 + lane;
    dn = jn < p ? d[jn] : 1.0;
    en = jn < p ? e[jn] : 0.0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double Lout = 0.0, Iout = 0.0;
#pragma unroll 16
    for (int t = 0; t < 64; ++t) {
      const double dt = stage[2 * t], et = stage[2 * t + 1];
      const double Lt = et * rprev;
      const double Dt = fma(-et, Lt, dt);
      double r = __builtin_amdgcn_rcp(Dt);
      r = fma(r, fma(-Dt, r, 1.0), r);
      r = fma(r, fma(-Dt, r, 1.0), r);
      rprev = r;
      Lout = lane == t ? Lt : Lout;
      Iout = lane == t ? r : Iout;
    }
    const int64_t j = c0 + lane;
    if (j < p) {
      L[j] = Lout;
      invD[j] = Iout;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

__device__ inline void copy_state(const State* sin, State* sout, const State& s) {
  (void)sin;
  if (blockIdx.x == 0 && threadIdx.x == 0) *sout = s;
}

}  // namespace flr

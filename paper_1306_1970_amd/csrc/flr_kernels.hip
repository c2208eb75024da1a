// HIP kernels (gfx950) of the device-resident MM / PCG loop for fused lasso
// regression.  Method: section 3.1 (perturbed objective, majorizer, linear
// system with A and B), Algorithm 2 (MM with PCG, preconditioner
// M = lambda1 A + lambda2 B).  See flr_internal.h for the launch rotation.
//
// Numerics: all p-scale arithmetic, dot products, the objective and every
// stopping test are FP64.  X is read in its stored type (f64 / f32 / bf16)
// and widened exactly; products accumulate in FP64.  Every reduction has a
// fixed tree, so a solve is bitwise repeatable and does not depend on what
// else runs on the device.
#include <hip/hip_runtime.h>

#include <cmath>

#include "flr_device.h"
#include "flr_band.h"
#include "flr_internal.h"
#include "flr_nest.h"

namespace flr {

// v[first * stride] + ... + v[(count - 1) * stride] in that order, eight loads
// in flight at a time (one load per add leaves each waiting for the last:
// the block kernel's launch 35 us with 128 partials, 9.3 us with 31 in such batches).
__device__ inline double sum_parts(const double* __restrict__ v, int64_t stride, int first, int count) {
  double sum = 0.0;
  for (int q = first; q < count; q += 8) {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = q + u < count ? v[(int64_t)(q + u) * stride] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += t[u];
  }
  return sum;
}

// ---------------------------------------------------------------------------
// Setup: partial column sums of X_ij y_i and X_ij^2 over row panels
// ---------------------------------------------------------------------------
template <typename XT>
__global__ __launch_bounds__(kWG) void k_setup_partial(Dims D, const XT* __restrict__ X, const double* __restrict__ y,
                                                        double* __restrict__ cpart, double* __restrict__ spart) {
  constexpr int V = XV<XT>::V;
  const int wg = blockIdx.x, cb = wg % D.cb2, rb = wg / D.cb2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)rb * D.r2, r1 = min<int64_t>(D.n, r0 + D.r2);
  const int64_t c0 = (int64_t)cb * D.c2 + lane * V;
  double ac[V], as[V];
#pragma unroll
  for (int v = 0; v < V; ++v) { ac[v] = 0.0; as[v] = 0.0; }
  for (int64_t i = r0 + wave; i < r1; i += 4) {
    double xv[V];
    XV<XT>::cvt(load16(X + i * D.ldx + c0), xv);
    const double yi = y[i];
#pragma unroll
    for (int v = 0; v < V; ++v) { ac[v] = fma(xv[v], yi, ac[v]); as[v] = fma(xv[v], xv[v], as[v]); }
  }
  __shared__ double red[2][4][64 * 8];
#pragma unroll
  for (int v = 0; v < V; ++v) { red[0][wave][lane * V + v] = ac[v]; red[1][wave][lane * V + v] = as[v]; }
  __syncthreads();
  for (int t = threadIdx.x; t < 64 * V; t += kWG) {
    const int64_t j = (int64_t)cb * D.c2 + t;
    cpart[(int64_t)rb * D.p_pad + j] = (red[0][0][t] + red[0][1][t]) + (red[0][2][t] + red[0][3][t]);
    spart[(int64_t)rb * D.p_pad + j] = (red[1][0][t] + red[1][1][t]) + (red[1][2][t] + red[1][3][t]);
  }
}

__global__ __launch_bounds__(kWG) void k_setup_final(Dims D, const double* __restrict__ cpart,
                                                      const double* __restrict__ spart, double* __restrict__ c,
                                                      double* __restrict__ s) {
  const int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (j >= D.p_pad) return;
  const double sc = sum_parts(cpart + j, D.p_pad, 0, D.rb2), ss = sum_parts(spart + j, D.p_pad, 0, D.rb2);
  c[j] = j < D.p ? sc : 0.0;
  s[j] = j < D.p ? ss : 0.0;
}

// Initial iterate (initialization of Algorithms 1 and 2: b_j = X_j^T y / X_j^T X_j,
// 0 for a zero column) or a warm start; both state buffers start at the MM
// boundary so the first rotation evaluates f(b0) and sets up the first PCG.
__global__ __launch_bounds__(kWG) void k_init(Dims D, Bufs B, const double* __restrict__ warm, int use_warm) {
  const int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (j < D.p_pad) {
    double v = 0.0;
    if (j < D.p) v = use_warm ? warm[j] : (B.s[j] > 0.0 ? B.c[j] / B.s[j] : 0.0);
    B.x[j] = v;
    B.r[j] = 0.0;
    B.yv[j] = 0.0;
    B.pbuf[j] = 0.0;
    B.pbuf[D.p_pad + j] = 0.0;
    // the banded mode rebuilds z from yv alone (gains and carries stay zero)
    B.sig[j] = 0.0;
    B.psi[j] = 0.0;
  }
  if (j < 2 * (D.p_pad / kBlk)) B.carry[j] = 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    State s;
    s.phase = PH_END;
    s.status = ST_OK;
    s.first = 1;
    s.first_cg = 1;
    s.mm_iter = 0;
    s.cg_iter = 0;
    s.cg_total = 0;
    s.rz = 0.0;
    s.f_old = 0.0;
    s.f_new = 0.0;
    s.rel_change = 0.0;
    s.rel_res = 0.0;
    s.nu = 0.0;
    s.gamma = 0.0;
    s.rres = 0.0;
    s.fstage = 0;
    s.fin = 0;
    B.st[0] = s;
    B.st[1] = s;
  }
}

// Rows r0..r1 of one column panel: u_part[cb][i] = sum_j X_ij v_j, with the
// first pair of rows already in registers and the next pair always in flight.
// ACC = double (FP64 path) or float (the inner PCG products of the mixed path).
template <typename XT, typename ACC>
__device__ inline void rows_a(const Dims& D, const Bufs& B, const XT* Xb, int cb, int64_t r0, int64_t r1, int64_t c0,
                              int lane, int wave, const double* sh_v, typename XV<XT>::raw (&cur0)[4],
                              typename XV<XT>::raw (&cur1)[4]) {
  constexpr int V = XV<XT>::V;
  constexpr int NV = 4;
  using RAW = typename XV<XT>::raw;
  ACC pl[NV][V];
#pragma unroll
  for (int t = 0; t < NV; ++t)
#pragma unroll
    for (int v = 0; v < V; ++v) pl[t][v] = (ACC)sh_v[(t * 64 + lane) * V + v];
  for (int64_t i = r0 + wave; i < r1; i += 8) {
    const int64_t i1 = i + 4, in0 = i + 8, in1 = i + 12;
    const bool has1 = i1 < r1;
    RAW nx0[NV], nx1[NV];
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      const int64_t col = c0 + (int64_t)(t * 64 + lane) * V;
      if (in0 < r1) nx0[t] = load16(Xb + in0 * D.ldx + col);
      if (in1 < r1) nx1[t] = load16(Xb + in1 * D.ldx + col);
    }
    ACC acc0 = 0, acc1 = 0;
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      ACC xv[V];
      XV<XT>::cvt(cur0[t], xv);
#pragma unroll
      for (int v = 0; v < V; ++v) acc0 = fma(xv[v], pl[t][v], acc0);
      if (has1) {
        ACC xw[V];
        XV<XT>::cvt(cur1[t], xw);
#pragma unroll
        for (int v = 0; v < V; ++v) acc1 = fma(xw[v], pl[t][v], acc1);
      }
    }
    const double s0 = wave_sum((double)acc0);
    const double s1 = wave_sum((double)acc1);
    if (lane == 0) {
      B.upart[(int64_t)cb * D.n + i] = s0;
      if (has1) B.upart[(int64_t)cb * D.n + i1] = s1;
    }
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      cur0[t] = nx0[t];
      cur1[t] = nx1[t];
    }
  }
}

// Nothing to do for A, B and C: done, or M is being factored by later launches.
__device__ inline bool idle(const State& s) { return s.phase == PH_DONE || s.phase == PH_BANDMM; }

// Reduction of the true residual that one refinement round asks of the
// FP32-product PCG (its products carry errors near 1e-7 relative, so it
// cannot be trusted much further in one round).
constexpr double kRoundReduction = 1e-4;

// Phase after a new residual (its squared norm rr, relative norm rn); also
// records the FP64 residual of a boundary or refresh in o.rres.
// Algorithm 2's inner loop is repeat-until: after the first residual of an
// MM step at least one PCG step runs unless that residual is exactly zero (nu
// would be 0/0).  After a PCG step the inner test decides.  With FP32
// products (mixed precision) a round of PCG stops once its recursive residual
// is kRoundReduction below the round's FP64 starting residual (or meets the
// inner tolerance); then the true residual c - Q x is recomputed in FP64 and
// the MM step ends only if that passes the inner test - else PCG restarts
// from it (iterative refinement).  Refinement also ends when a refresh has
// cut the true residual by less than 10 % (FP32 products can resolve no more
// on this system) or at the PCG step cap.
__device__ __forceinline__ int32_t next_phase(const Params& prm, State& o, int mode, double rr, double rn) {
  const bool capped = o.cg_iter >= prm.max_cg;
  if (mode == CM_FIRST) {
    o.rres = rn;
    return rr > 0.0 ? PH_CG : PH_END;
  }
  // A refinement round that starts within 25 % of the tolerance aims at half of
  // it: aiming at the tolerance itself, the FP32 products' error can leave the
  // true residual just above, and the small cut would pass for a stall.
  const bool close = prm.mixed && mode == CM_STEP && o.rres < 1.25 * prm.inner_tol;
  const bool met = !(rn > (close ? 0.5 : 1.0) * prm.inner_tol);
  if (mode == CM_REFRESH) {
    const bool stalled = !(rn < 0.9 * o.rres);
    o.rres = rn;
    return (met || capped || stalled) ? PH_END : PH_CG;
  }
  if (capped) return PH_END;
  if (!prm.mixed) return met ? PH_END : PH_CG;
  return (met || !(rn > kRoundReduction * o.rres)) ? PH_RES : PH_CG;
}

// The end of a step whose M^-1 r came from K1..K3 (flr_nest.h): every workgroup of
// the next A sums the shares of r^T z and r^T r in the same order and takes the
// inner stopping test and gamma for itself.  The loads are issued with the state's
// and before any of X; as a launch of one workgroup of its own this took 4.2 us, here
// 1.1 (a PCG step of the 32 x 32 lattice 28.3 -> 25.2 us, of the 100 x 100 one 96 -> 93).
__device__ __forceinline__ void nest_finish(const Bufs& B, State& s) {
  __shared__ double red[16];
  double sums[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int q = threadIdx.x; q < B.nest.nparts; q += kWG) {
    sums[0] += B.nest.part[2 * q];
    sums[1] += B.nest.part[2 * q + 1];
  }
  if (!__builtin_amdgcn_readfirstlane(s.fin)) return;
  wg_sum4(sums, red);
  const Params prm = *B.prm;
  const double rz_prev = s.rz, rn = sqrt(sums[1]) / prm.cnorm;
  const int mode = s.phase == PH_BANDSOLVE ? CM_FIRST : s.phase == PH_BANDRES ? CM_REFRESH : CM_STEP;
  s.phase = __builtin_amdgcn_readfirstlane(next_phase(prm, s, mode, sums[1], rn));
  s.rel_res = rn;
  s.gamma = mode != CM_STEP ? 0.0 : sums[0] / rz_prev;
  s.rz = sums[0];
  s.fin = 0;
}

// ---------------------------------------------------------------------------
// A: row-panel GEMV u_part[cb] = X[rb, cb] v[cb].  In a PCG step v is the new
// direction p = z + gamma p_old, where z = M^-1 r is rebuilt from the local
// block solutions and the carries that the last C workgroup combined
// (z_j = y_j + sigma_j G_k + psi_j Z_k).  Once PCG has converged, or at the
// MM boundary, v is the iterate x.  The state is read through a restrict
// pointer (scalar loads), so it does not wait behind the X loads.  NEST: M^-1 may
// come from nested inverses (B.nest.S > 0), whose step this launch ends.
// ---------------------------------------------------------------------------
template <typename XT, bool MX, bool NEST>
__device__ __forceinline__ void gemv_a_body(const Dims& D, const Bufs& B, const State* __restrict__ sin,
                                            State* __restrict__ sout, const int wg) {
  constexpr int V = XV<XT>::V;
  constexpr int NV = 4;  // 16-byte loads per lane per row (the panel is 256 V columns)
  using RAW = typename XV<XT>::raw;
  State s = *sin;
  if (NEST && B.nest.S) nest_finish(B, s);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cb = wg % D.cb1, rb = wg / D.cb1;
  if (wg == 0 && tid == 0) {
    State o = *sin;  // read again, so that s stays in registers
    if (NEST) {
      o.phase = s.phase;
      o.fin = s.fin;
      o.rz = s.rz;
      o.gamma = s.gamma;
      o.rel_res = s.rel_res;
      o.rres = s.rres;
    }
    *sout = o;
  }
  if (idle(s)) return;
  const int64_t c0 = (int64_t)cb * D.c1;
  const int64_t r0 = (int64_t)rb * D.r1, r1 = min<int64_t>(D.n, r0 + D.r1);
  const XT* Xb = reinterpret_cast<const XT*>(B.X);

  // operand-slice inputs first (small, needed first), then the wave's first
  // two X rows, so that waiting for the former does not wait for the latter
  __shared__ double sh_v[kMaxC1];
  const bool cg = s.phase == PH_CG;
  const double* pold = B.pbuf + (int64_t)(s.cg_iter & 1) * D.p_pad;
  double* pnew = B.pbuf + (int64_t)((s.cg_iter + 1) & 1) * D.p_pad;
  const int K = D.nblk;
  double fy[V], fs[V], fp[V], fo[V], fg[V], fz[V];
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int64_t j = c0 + tid + u * kWG;
    const int k = (int)(j / kBlk);
    if (cg) {
      fy[u] = B.yv[j];
      fs[u] = B.sig[j];
      fp[u] = B.psi[j];
      fo[u] = pold[j];
      fg[u] = B.carry[k];
      fz[u] = B.carry[K + k];
    } else {
      fy[u] = B.x[j];
    }
  }
  RAW cur0[NV], cur1[NV];
  if (!D.flsa) {
    const int64_t i0 = r0 + wave, i1 = i0 + 4;
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      const int64_t col = c0 + (int64_t)(t * 64 + lane) * V;
      if (i0 < r1) cur0[t] = load16(Xb + i0 * D.ldx + col);
      if (i1 < r1) cur1[t] = load16(Xb + i1 * D.ldx + col);
    }
  }
  if (cg) {
    const double gamma = s.gamma;
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t j = c0 + tid + u * kWG;
      const double z = fma(fs[u], fg[u], fma(fp[u], fz[u], fy[u]));
      const double v = fma(gamma, fo[u], z);
      if (rb == 0) pnew[j] = v;
      sh_v[tid + u * kWG] = v;
    }
  } else {
#pragma unroll
    for (int u = 0; u < V; ++u) sh_v[tid + u * kWG] = fy[u];
  }
  __syncthreads();
  if (D.flsa) return;  // X = I: the column-panel kernel uses the operand itself

  if (MX && s.phase == PH_CG)
    rows_a<XT, float>(D, B, Xb, cb, r0, r1, c0, lane, wave, sh_v, cur0, cur1);
  else
    rows_a<XT, double>(D, B, Xb, cb, r0, r1, c0, lane, wave, sh_v, cur0, cur1);
}

template <typename XT, bool MX, bool NEST>
__global__ __launch_bounds__(kWG) void k_gemv_a(Dims D, Bufs B, const State* __restrict__ sin,
                                                State* __restrict__ sout) {
  gemv_a_body<XT, MX, NEST>(D, B, sin, sout, blockIdx.x);
}

// (M v)_j = lambda1 a_j v_j + lambda2 sum_k w_jk (v_j - v_k)  (A and B of the linear system)
__device__ inline double apply_m(const Bufs& B, const Params& prm, int64_t j, const double* v) {
  const double vj = v[j];
  double lap = 0.0;
  for (int q = B.rowptr[j]; q < B.rowptr[j + 1]; ++q) lap = fma(B.w[q], vj - v[B.col[q]], lap);
  return prm.lam1 * B.a[j] * vj + prm.lam2 * lap;
}

// Rows r0..r1 of one column panel for this lane's V columns:
// out[v] = sum_i X_{i, c0+v} u_i (rows of this wave, RU rows in flight).
template <typename XT, typename ACC, int RU>
__device__ inline void cols_b(const Dims& D, const XT* Xb, int64_t r0, int64_t r1, int64_t c0, int wave,
                              const double* sh_u, typename XV<XT>::raw (&cur)[RU], double* out) {
  constexpr int V = XV<XT>::V;
  using RAW = typename XV<XT>::raw;
  ACC acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0;
  for (int64_t i = r0 + wave; i < r1; i += 4 * RU) {
    RAW nxt[RU];
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int64_t ii = i + 4 * RU + 4 * u;
      if (ii < r1) nxt[u] = load16(Xb + ii * D.ldx + c0);
    }
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int64_t ii = i + 4 * u;
      if (ii < r1) {
        ACC xv[V];
        XV<XT>::cvt(cur[u], xv);
        const ACC uu = (ACC)sh_u[ii - r0];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = fma(xv[v], uu, acc[v]);
      }
    }
#pragma unroll
    for (int u = 0; u < RU; ++u) cur[u] = nxt[u];
  }
#pragma unroll
  for (int v = 0; v < V; ++v) out[v] = (double)acc[v];
}

// ---------------------------------------------------------------------------
// B: column-panel GEMV q_part[rb] = X[rb, :]^T u[rb] (u summed from the A
// partials).  PCG step: panel row 0 adds M p and each workgroup emits its
// share of p^T Q p.  MM boundary: the same product for the new residual, the
// loss partials 1/2 ||y - X b||^2, and (first nblk workgroups) reweighting
// a_j = 1/(|b_j|+eps), w_jk = 1/(|b_j - b_k|+eps), the tridiagonal part of M,
// the penalty sums of f, and each block's product of the tridiagonal
// factorization (the last block to arrive combines them).
// ---------------------------------------------------------------------------
template <typename XT, bool MX>
__device__ __forceinline__ void gemv_b_body(const Dims& D, const Bufs& B, const State* __restrict__ sin,
                                            State* __restrict__ sout, const Params* __restrict__ prmp,
                                            const int wg) {
  constexpr int V = XV<XT>::V;
  constexpr int RU = 8;  // rows per wave in flight
  using RAW = typename XV<XT>::raw;
  const State s = *sin;
  const int tid = threadIdx.x;
  if (wg == 0 && tid == 0) *sout = s;
  if (idle(s)) return;
  const int lane = tid & 63, wave = tid >> 6;
  const int ngemm = D.cb2 * D.rb2;
  const int cb = wg % D.cb2, rb = wg / D.cb2;
  const int64_t r0 = (int64_t)rb * D.r2, r1 = wg < ngemm ? min<int64_t>(D.n, r0 + D.r2) : r0;
  const int64_t c0 = (int64_t)cb * D.c2 + lane * V;
  const XT* Xb = reinterpret_cast<const XT*>(B.X);
  const Params prm = *prmp;
  const bool cg = s.phase == PH_CG;
  const double* pv = cg ? (B.pbuf + (int64_t)((s.cg_iter + 1) & 1) * D.p_pad) : B.x;

  __shared__ double sh_u[kMaxR2];
  __shared__ double sh_red[4][64 * 8];
  __shared__ double sh_s[16];

  // u for the first 256 panel rows (sum of the A partials), issued before
  // the X rows so that waiting for it does not wait for them
  constexpr int CBMAX = 12;
  const int nr = (int)(r1 - r0);
  double upre[CBMAX];
  RAW cur[RU];
  if (!D.flsa) {
#pragma unroll
    for (int q = 0; q < CBMAX; ++q) upre[q] = (tid < nr && q < D.cb1) ? B.upart[(int64_t)q * D.n + r0 + tid] : 0.0;
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int64_t i = r0 + wave + 4 * u;
      if (i < r1) cur[u] = load16(Xb + i * D.ldx + c0);
    }
  }

  if (D.flsa && wg < ngemm) {
    // X = I (one row panel): X^T X v = v; at an MM boundary the loss partial
    // 1/2 ||y - x||^2 runs over this panel's coordinates
    double dotp = 0.0, loss = 0.0;
    for (int t = tid; t < 64 * V; t += kWG) {
      const int64_t j = (int64_t)cb * D.c2 + t;
      double q = 0.0;
      if (j < D.p) {
        q = pv[j];
        if (cg) q += apply_m(B, prm, j, pv);
        if (!cg) {
          const double dlt = B.y[j] - pv[j];
          loss = fma(dlt, dlt, loss);
        }
      }
      B.qpart[j] = q;
      if (cg) dotp = fma(pv[j], q, dotp);
    }
    if (cg) {
      const double tot = wg_sum(dotp, sh_s);
      if (tid == 0) B.pqpart[wg] = tot;
    } else {
      const double tot = wg_sum(loss, sh_s);
      if (tid == 0) B.losspart[cb] = tot;
    }
  } else if (wg < ngemm) {
    double loss = 0.0;
    for (int t = tid; t < nr; t += kWG) {
      double u = 0.0;
      if (t == tid) {
#pragma unroll
        for (int q = 0; q < CBMAX; ++q) u += upre[q];
        for (int q = CBMAX; q < D.cb1; ++q) u += B.upart[(int64_t)q * D.n + r0 + t];
      } else {
        for (int q = 0; q < D.cb1; ++q) u += B.upart[(int64_t)q * D.n + r0 + t];
      }
      sh_u[t] = u;
      if (!cg && cb == 0) {  // loss partials (used at an MM boundary)
        const double dlt = B.y[r0 + t] - u;
        loss = fma(dlt, dlt, loss);
      }
    }
    __syncthreads();
    if (MX && cg)
      cols_b<XT, float, RU>(D, Xb, r0, r1, c0, wave, sh_u, cur, &sh_red[wave][lane * V]);
    else
      cols_b<XT, double, RU>(D, Xb, r0, r1, c0, wave, sh_u, cur, &sh_red[wave][lane * V]);
    __syncthreads();
    double dotp = 0.0;
    for (int t = tid; t < 64 * V; t += kWG) {
      const int64_t j = (int64_t)cb * D.c2 + t;
      double q = (sh_red[0][t] + sh_red[1][t]) + (sh_red[2][t] + sh_red[3][t]);
      if (cg && rb == 0 && j < D.p) q += apply_m(B, prm, j, pv);
      B.qpart[(int64_t)rb * D.p_pad + j] = q;
      if (cg) dotp = fma(pv[j], q, dotp);
    }
    if (cg) {
      const double tot = wg_sum(dotp, sh_s);
      if (tid == 0) B.pqpart[wg] = tot;
    } else if (cb == 0) {
      const double tot = wg_sum(loss, sh_s);
      if (tid == 0) B.losspart[rb] = tot;
    }
  } else if (cg) {
    if (tid == 0) B.pqpart[wg] = 0.0;
  }

  const bool mmb = s.phase == PH_END;  // an MM boundary (not a refinement's residual refresh)
  if (mmb && wg < D.nblk) {
    // reweighting and the tridiagonal part of M, penalties.  d: the diagonal of
    // M (banded mode), or its part beside the couplings e_j of (j-1, j)
    const int64_t j = (int64_t)wg * kBlk + tid;
    double pen = 0.0, dj = 1.0, ej = 0.0;
    if (j < D.p) {
      const double xj = B.x[j];
      const double aj = 1.0 / (fabs(xj) + prm.eps);
      B.a[j] = aj;
      double wsum = 0.0;
      double pen2 = 0.0;
      for (int q = B.rowptr[j]; q < B.rowptr[j + 1]; ++q) {
        const int k = B.col[q];
        const double dlt = fabs(xj - B.x[k]);
        const double wq = 1.0 / (dlt + prm.eps);
        B.w[q] = wq;
        const bool coupled = !prm.band && !prm.jacobi && (k == j - 1 || k == j + 1);
        if (!coupled) wsum += wq;
        if (coupled && k == j - 1) ej = prm.lam2 * wq;
        if (k > j) pen2 += dlt;
      }
      pen = prm.lam1 * fabs(xj) + prm.lam2 * pen2;
      dj = prm.lam1 * aj + prm.lam2 * wsum;
      if (prm.jacobi) dj += B.s[j];
    }
    if (j < D.p_pad) {
      B.d[j] = dj;
      B.e[j] = ej;
    }
    const double tot = wg_sum(pen, sh_s);
    if (tid == 0) B.penpart[wg] = tot;
    if (!prm.band) {
      // Tridiagonal factor: each block's Moebius product; the last of the
      // nblk workgroups to arrive scans them to the value before each block,
      // and the C launch scans inside the blocks.  One wave walking the p
      // pivots here took 41 ns each: this launch was 408 us at an MM boundary
      // with p = 10^4 and 3.9 ms with p = 10^5, now 15 and 38.
      const int K = D.nblk;
      const Mob mb = wg_scan_mob(mob_leaf(dj, ej), sh_s);
      if (tid == kWG - 1) {
        double* o = B.mob + 4 * (int64_t)wg;
        put_shared(o, mb.a);
        put_shared(o + 1, mb.b);
        put_shared(o + 2, mb.c);
        put_shared(o + 3, mb.d);
      }
      __shared__ int sh_flag;
      __syncthreads();
      if (tid == kWG - 1) sh_flag = arrive(B.counter + 16, K);
      __syncthreads();
      if (sh_flag) {
        // thread t: blocks t e4 .. t e4 + e4 - 1
        constexpr int EMAX = kMaxBlocks / kWG;
        const int e4 = (K + kWG - 1) / kWG;
        Mob bm[EMAX], pr = {1.0, 0.0, 0.0, 1.0};
#pragma unroll
        for (int i = 0; i < EMAX; ++i) {
          const int k = tid * e4 + i;
          const bool in = i < e4 && k < K;
          const double* o = B.mob + 4 * (int64_t)(in ? k : 0);
          bm[i] = {get_shared(o), get_shared(o + 1), get_shared(o + 2), get_shared(o + 3)};
          if (in) pr = i == 0 ? bm[0] : mob_compose(pr, bm[i]);
        }
        const Mob inc = wg_scan_mob(pr, sh_s);
        // t after this thread's last block (the first element's map is constant, so any inflow gives it)
        sh_red[0][tid] = inc.b / inc.d;
        __syncthreads();
        double t = tid == 0 ? 0.0 : sh_red[0][tid - 1];
#pragma unroll
        for (int i = 0; i < EMAX; ++i) {
          const int k = tid * e4 + i;
          if (i < e4 && k < K) {
            B.mob[4 * (int64_t)K + k] = t;
            t = mob_apply(bm[i], t);
          }
        }
        if (tid == 0) B.counter[16] = 0u;
      }
    }
  }
}

template <typename XT, bool MX>
__global__ __launch_bounds__(kWG) void k_gemv_b(Dims D, Bufs B, const State* __restrict__ sin,
                                                State* __restrict__ sout, const Params* __restrict__ prmp) {
  gemv_b_body<XT, MX>(D, B, sin, sout, prmp, blockIdx.x);
}

// Solver blocks that one workgroup of the block kernel can take (groups of 256
// threads).
constexpr int kMaxGroup = 2;

// Zero-inflow local solve of the block for the current residual r_j and the
// block scalars that the next A launch combines into the global solution:
//   forward  g_j = r_j - L_j g_{j-1}           (L D L^T, forward sweep)
//   backward y_j = g_j / D_j - L_{j+1} y_{j+1}   (backward sweep)
// loc (not null): the scalars stay in this workgroup's LDS (it holds every block).
__device__ inline void block_local_solve(const Dims& D, const Bufs& B, int b, int64_t j, double rj, double Lj,
                                         double Lnext, double invDj, double sigj, double psij, double* lds,
                                         double* lds2, double* loc) {
  const int tid = threadIdx.x & (kBlk - 1);
  const Aff gf = wg_scan_fwd({-Lj, rj}, lds);
  const double g = gf.b;
  const Aff yb = wg_scan_rev({-Lnext, g * invDj}, lds);
  const double yj = yb.b;
  if (j < D.p_pad) B.yv[j] = yj;
  const int K = D.nblk;
  __syncthreads();
  if (tid == kBlk - 1) lds2[0] = g;
  if (tid == 0) lds2[1] = yj;
  double sums[4] = {rj * yj, rj * sigj, rj * psij, rj * rj};
  wg_sum4(sums, lds);
  if (tid == 0 && b < K) {
    auto put = [&](int field, double v) {
      if (loc)
        loc[field * kMaxGroup + b] = v;
      else
        put_shared(B.blk + field * K + b, v);
    };
    put(BK_B, lds2[0]);
    put(BK_YS, lds2[1]);
    put(BK_RY, sums[0]);
    put(BK_RS, sums[1]);
    put(BK_RP, sums[2]);
    put(BK_RR, sums[3]);
  }
}

// Wave-level variant of combine_blocks for K <= 64 E (E blocks per lane), run by
// wave 0 alone: shuffles only, no barriers.  get(field, k): block scalars.
template <int E, typename Get>
__device__ void combine_blocks_wave(const Dims& D, const Bufs& B, const Params& prm, State o, double rz_prev,
                                    int mode, State* __restrict__ sout, Get get) {
  const int l = threadIdx.x & 63;
  const int K = D.nblk;
  const int e = (K + 63) / 64;
  const int k0 = l * e;
  double fA[E], fB[E], fRY[E], fRS[E], fRP[E], fRR[E], nPS[E], nYS[E], nSS[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int k = k0 + i;
    const bool ok = i < e && k < K;
    const bool okn = i < e && k + 1 < K;
    fA[i] = ok ? get(BK_A, k) : 1.0;
    fB[i] = ok ? get(BK_B, k) : 0.0;
    fRY[i] = ok ? get(BK_RY, k) : 0.0;
    fRS[i] = ok ? get(BK_RS, k) : 0.0;
    fRP[i] = ok ? get(BK_RP, k) : 0.0;
    fRR[i] = ok ? get(BK_RR, k) : 0.0;
    nPS[i] = okn ? get(BK_PSIS, k + 1) : 0.0;
    nYS[i] = okn ? get(BK_YS, k + 1) : 0.0;
    nSS[i] = okn ? get(BK_SIGS, k + 1) : 0.0;
  }
  Aff m = {1.0, 0.0};
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (i < e && k0 + i < K) m = compose(m, {fA[i], fB[i]});
  const Aff fin = wave_scan_fwd(m);
  double G = __shfl_up(fin.b, 1, 64);
  if (l == 0) G = 0.0;
  double Gk[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    Gk[i] = G;
    if (i < e && k0 + i < K) G = fma(fA[i], G, fB[i]);
  }
  Aff mb = {1.0, 0.0};
#pragma unroll
  for (int i = E - 1; i >= 0; --i) {
    const int k = k0 + i;
    const double Gn = (i + 1 < e) ? Gk[(i + 1) < E ? i + 1 : 0] : G;
    if (i < e && k < K - 1) {
      mb = compose(mb, {nPS[i], fma(nSS[i], Gn, nYS[i])});
    } else if (i < e && k == K - 1) {
      mb = compose(mb, {0.0, 0.0});
    }
  }
  const Aff finb = wave_scan_rev(mb);
  double Z = __shfl_down(finb.b, 1, 64);
  if (l == 63) Z = 0.0;
  double rzp = 0.0, rrp = 0.0;
#pragma unroll
  for (int i = E - 1; i >= 0; --i) {
    const int k = k0 + i;
    if (i < e && k < K) {
      const double Gn = (i + 1 < e) ? Gk[(i + 1) < E ? i + 1 : 0] : G;
      Z = (k < K - 1) ? fma(nPS[i], Z, fma(nSS[i], Gn, nYS[i])) : 0.0;
      B.carry[k] = Gk[i];
      B.carry[K + k] = Z;
      rzp += fRY[i] + Gk[i] * fRS[i] + Z * fRP[i];
      rrp += fRR[i];
    }
  }
  const double rz = wave_sum(rzp);
  const double rr = wave_sum(rrp);
  if (l == 0) {
    const double rn = sqrt(rr) / prm.cnorm;
    o.phase = next_phase(prm, o, mode, rr, rn);
    o.rel_res = rn;
    o.rz = rz;
    o.gamma = mode != CM_STEP ? 0.0 : rz / rz_prev;
    *sout = o;
    *B.counter = 0u;
  }
}

// Called by every thread of the last C workgroup to finish, once the block
// scalars of all blocks are visible: carries of the partitioned tridiagonal
// solve over the blocks (forward G_k = forward-sweep value entering block k,
// backward Z_k = solution value entering block k from the right), r^T z,
// ||r||, the inner stopping test of Algorithm 2 and gamma = r^T z / r_old^T z_old.
__device__ void combine_blocks(const Dims& D, const Bufs& B, const Params& prm, State o, double rz_prev,
                               int mode, State* __restrict__ sout, double* sh_m, double* sh_G, double* sh_Z) {
  constexpr int EMAX = kMaxBlocks / kWG;
  const int tid = threadIdx.x & (kWG - 1);  // a larger workgroup's groups do the same
  const int K = D.nblk;
  const int e4 = (K + kWG - 1) / kWG;
  const double* bk = B.blk;
  const int k0 = tid * e4;
  double fA[EMAX], fB[EMAX], fRY[EMAX], fRS[EMAX], fRP[EMAX], fRR[EMAX], nPS[EMAX], nYS[EMAX], nSS[EMAX];
#pragma unroll
  for (int i = 0; i < EMAX; ++i) {
    const int k = k0 + i;
    const bool ok = i < e4 && k < K;
    const bool okn = i < e4 && k + 1 < K;
    fA[i] = ok ? get_shared(bk + BK_A * K + k) : 1.0;
    fB[i] = ok ? get_shared(bk + BK_B * K + k) : 0.0;
    fRY[i] = ok ? get_shared(bk + BK_RY * K + k) : 0.0;
    fRS[i] = ok ? get_shared(bk + BK_RS * K + k) : 0.0;
    fRP[i] = ok ? get_shared(bk + BK_RP * K + k) : 0.0;
    fRR[i] = ok ? get_shared(bk + BK_RR * K + k) : 0.0;
    nPS[i] = okn ? get_shared(bk + BK_PSIS * K + k + 1) : 0.0;
    nYS[i] = okn ? get_shared(bk + BK_YS * K + k + 1) : 0.0;
    nSS[i] = okn ? get_shared(bk + BK_SIGS * K + k + 1) : 0.0;
  }
  Aff m = {1.0, 0.0};
#pragma unroll
  for (int i = 0; i < EMAX; ++i)
    if (i < e4 && k0 + i < K) m = compose(m, {fA[i], fB[i]});
  const Aff fin = wg_scan_fwd(m, sh_m + 8);
  __syncthreads();
  sh_G[kMaxBlocks - 1 - tid] = fin.b;  // scratch: inclusive result per thread
  __syncthreads();
  double G = tid == 0 ? 0.0 : sh_G[kMaxBlocks - tid];
  __syncthreads();
  double Gk[EMAX];
#pragma unroll
  for (int i = 0; i < EMAX; ++i) {
    Gk[i] = G;
    if (i < e4 && k0 + i < K) G = fma(fA[i], G, fB[i]);
  }
  // Z_k = psis_{k+1} Z_{k+1} + ys_{k+1} + sigs_{k+1} G_{k+1},  Z_{K-1} = 0
  Aff mb = {1.0, 0.0};
#pragma unroll
  for (int i = EMAX - 1; i >= 0; --i) {
    const int k = k0 + i;
    const double Gn = (i + 1 < e4) ? Gk[(i + 1) < EMAX ? i + 1 : 0] : G;
    if (i < e4 && k < K - 1) {
      mb = compose(mb, {nPS[i], fma(nSS[i], Gn, nYS[i])});
    } else if (i < e4 && k == K - 1) {
      mb = compose(mb, {0.0, 0.0});
    }
  }
  const Aff finb = wg_scan_rev(mb, sh_m + 8);
  __syncthreads();
  sh_Z[kMaxBlocks - 1 - tid] = finb.b;
  __syncthreads();
  double Z = tid == kWG - 1 ? 0.0 : sh_Z[kMaxBlocks - 2 - tid];
  double rzp = 0.0, rrp = 0.0;
#pragma unroll
  for (int i = EMAX - 1; i >= 0; --i) {
    const int k = k0 + i;
    if (i < e4 && k < K) {
      const double Gn = (i + 1 < e4) ? Gk[(i + 1) < EMAX ? i + 1 : 0] : G;
      Z = (k < K - 1) ? fma(nPS[i], Z, fma(nSS[i], Gn, nYS[i])) : 0.0;
      B.carry[k] = Gk[i];
      B.carry[K + k] = Z;
      rzp += fRY[i] + Gk[i] * fRS[i] + Z * fRP[i];
      rrp += fRR[i];
    }
  }
  const double rz = wg_sum(rzp, sh_m + 8);
  const double rr = wg_sum(rrp, sh_m + 8);
  if (tid == 0) {
    const double rn = sqrt(rr) / prm.cnorm;
    o.phase = next_phase(prm, o, mode, rr, rn);
    o.rel_res = rn;
    o.rz = rz;
    o.gamma = mode != CM_STEP ? 0.0 : rz / rz_prev;
    *sout = o;
    *B.counter = 0u;
  }
}

// True in the one workgroup that finishes last, which may then read every
// block's scalars.  The first thread of each group of 256 wrote its block's; thread
// 0 arrives for all VB of them.  No workgroup waits for another.
template <int VB>
__device__ inline bool arrive_last(const Bufs& B, int nblocks, int* flag) {
  if (VB > 1) published();  // thread 256 publishes from another wave than the one that arrives
  __syncthreads();
  if (threadIdx.x == 0) *flag = arrive(B.counter, nblocks);
  __syncthreads();
  return *flag != 0;
}

// ---------------------------------------------------------------------------
// C: per solver block (256 elements).  PCG step: nu = r^T z / p^T Q p,
// x += nu p, r -= nu Q p (the residual update with the minus sign), then the
// local solve of the new residual.  MM boundary: f of the iterate, the
// relative-change test of Algorithm 2, and - if continuing - the block's part
// of the LDL^T factorization of the tridiagonal M (a scan from the value that
// the B launch left for it), the gain vectors, r0 = c - Q x0 and its
// local solve.  The last workgroup to finish combines the blocks.
// ---------------------------------------------------------------------------
//
// VB blocks per workgroup, one per group of 256 threads, each with the arithmetic
// of a workgroup of its own.  SOLO: one workgroup holds every block; their scalars
// stay in LDS and it combines them itself, without the round trips of publishing
// and arriving.
template <int VB, bool SOLO>
__device__ __forceinline__ void block_body(const Dims& D, const Bufs& B, const State* __restrict__ sin,
                                           State* __restrict__ sout, const Params* __restrict__ prmp,
                                           const int wg) {
  constexpr int QMAX = 16;  // row panels whose partial products are prefetched
  const int tid = threadIdx.x & (kBlk - 1);
  const int vb = VB == 1 ? 0 : threadIdx.x >> 8;
  const int b = wg * VB + vb;
  const int64_t j = (int64_t)b * kBlk + tid;
  const bool real = j < D.p;
  __shared__ double lds_g[VB][24];
  __shared__ double lds2_g[VB][4];
  __shared__ double sh_L_g[VB][kBlk + 1];
  __shared__ double sh_G[SOLO ? 1 : kMaxBlocks], sh_Z[SOLO ? 1 : kMaxBlocks];
  __shared__ double sh_blk[SOLO ? BK_N * kMaxGroup : 1];
  __shared__ int sh_flag;
  double* lds = lds_g[vb];
  double* lds2 = lds2_g[vb];
  double* sh_L = sh_L_g[vb];
  double* loc = SOLO ? sh_blk : nullptr;

  // every input of a PCG step in one round of loads, requested before the state
  // that says whether this is one arrives (both parities of p)
  // (indices clamped into range and the surplus dropped afterwards: a load under a
  // condition is a branch around it)
  const int64_t jc = min(j, D.p - 1);
  double pq0 = B.pqpart[min(tid, D.gridB - 1)], pq1 = B.pqpart[min(tid + kWG, D.gridB - 1)];
  double qp[QMAX];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) qp[rb] = B.qpart[(int64_t)min(rb, D.rb2 - 1) * D.p_pad + jc];
  if (D.rb2 > 4) {
#pragma unroll
    for (int rb = 4; rb < QMAX; ++rb) qp[rb] = B.qpart[(int64_t)min(rb, D.rb2 - 1) * D.p_pad + jc];
  } else {
#pragma unroll
    for (int rb = 4; rb < QMAX; ++rb) qp[rb] = 0.0;
  }
  const double pj0 = B.pbuf[jc], pj1 = B.pbuf[D.p_pad + jc], xj = B.x[jc], rj0 = B.r[jc];
  double Lj = B.L[jc], invDj = B.invD[jc], sigj = B.sig[jc], psij = B.psi[jc];
  const double Lnb = j + kBlk < D.p ? B.L[j + kBlk] : 0.0;  // thread 0: L of the next block's first element
  // SOLO: the scalars that stay for the whole MM step, for lane k of the combining wave
  double kA = 0.0, kSS = 0.0, kPS = 0.0;
  if (SOLO) {
    const int k = min((int)(threadIdx.x & 63), D.nblk - 1), kn = min(k + 1, D.nblk - 1);
    kA = B.blk[BK_A * D.nblk + k];
    kSS = B.blk[BK_SIGS * D.nblk + kn];
    kPS = B.blk[BK_PSIS * D.nblk + kn];
  }
  // the last workgroup to finish combines the blocks (SOLO: the only one)
  auto combine = [&](State o, double rz_prev, int mode) {
    if constexpr (SOLO) {
      __syncthreads();
      if (threadIdx.x < 64)
        combine_blocks_wave<1>(D, B, *prmp, o, rz_prev, mode, sout, [&](int field, int k) {
          const bool kept = field == BK_A || field == BK_SIGS || field == BK_PSIS;
          if (kept && mode != CM_FIRST) return field == BK_A ? kA : field == BK_SIGS ? kSS : kPS;
          return sh_blk[field * kMaxGroup + k];
        });
    } else if (arrive_last<VB>(B, (D.nblk + VB - 1) / VB, &sh_flag)) {
      const double* bk = B.blk;
      const int K = D.nblk;
      if (K > 4 * 64)
        combine_blocks(D, B, *prmp, o, rz_prev, mode, sout, lds, sh_G, sh_Z);
      else if (threadIdx.x < 64)
        combine_blocks_wave<4>(D, B, *prmp, o, rz_prev, mode, sout,
                            [&](int field, int k) { return get_shared(bk + field * K + k); });
    }
  };
  const State s = *sin;
  if (idle(s)) {
    if (b == 0 && tid == 0) *sout = s;
    return;
  }
  const Params prm = *prmp;
  if (tid >= D.gridB) pq0 = 0.0;
  if (tid + kWG >= D.gridB) pq1 = 0.0;
  if (!real) Lj = invDj = sigj = psij = 0.0;

  if (s.phase == PH_CG) {
    const double pj = s.cg_iter & 1 ? pj0 : pj1;  // p of this step: parity (cg_iter + 1) & 1
    double part = pq0 + pq1;
    for (int q = tid + 2 * kWG; q < D.gridB; q += kWG) part += B.pqpart[q];
    const double qrest = real ? sum_parts(B.qpart + j, D.p_pad, QMAX, D.rb2) : 0.0;
    const double pq = wg_sum(part, lds);
    const double nu = s.rz / pq;
    if (!(pq > 0.0) || !isfinite(nu)) {
      if (b == 0 && tid == 0) {
        State o = s;
        o.phase = PH_DONE;
        o.status = ST_NUMERICAL;
        *sout = o;
      }
      return;
    }
    double rj = 0.0;
    if (real) {
      double q = 0.0;
#pragma unroll
      for (int rb = 0; rb < QMAX; ++rb) q += rb < D.rb2 ? qp[rb] : 0.0;
      q += qrest;
      B.x[j] = fma(nu, pj, xj);
      rj = fma(-nu, q, rj0);
      B.r[j] = rj;
    }
    if (prm.band) {  // the K launches solve with the new residual
      if (b == 0 && tid == 0) {
        State o = s;
        o.cg_iter = s.cg_iter + 1;
        o.cg_total = s.cg_total + 1;
        o.nu = nu;
        *sout = o;
      }
      return;
    }
    sh_L[tid] = Lj;
    if (tid == 0) sh_L[kBlk] = Lnb;
    __syncthreads();
    block_local_solve(D, B, b, j, rj, Lj, sh_L[tid + 1], invDj, sigj, psij, lds, lds2, loc);
    State o = s;
    o.cg_iter = s.cg_iter + 1;
    o.cg_total = s.cg_total + 1;
    o.nu = nu;
    combine(o, s.rz, CM_STEP);
    return;
  }

  // ---- MM boundary, or an FP64 residual refresh (refinement) ----
  // inputs that do not depend on the decision, loaded up front
  double cj = 0.0, qsum = 0.0;
  if (real) {
    cj = B.c[j];
    qsum = sum_parts(B.qpart + j, D.p_pad, 0, D.rb2);
  }
  if (s.phase == PH_RES) {
    // true residual c - (X^T X + M) x of this MM step's system, in FP64 (the
    // weights and the factorization of M are the ones the PCG used)
    double rj = 0.0;
    if (real) {
      rj = cj - (qsum + apply_m(B, prm, j, B.x));
      B.r[j] = rj;
    }
    if (prm.band) {  // the K launches solve with the existing factor
      if (b == 0 && tid == 0) {
        State o = s;
        o.phase = PH_BANDRES;
        *sout = o;
      }
      return;
    }
    sh_L[tid] = Lj;
    if (tid == 0) sh_L[kBlk] = Lnb;
    __syncthreads();
    block_local_solve(D, B, b, j, rj, Lj, sh_L[tid + 1], invDj, sigj, psij, lds, lds2, loc);
    combine(s, 0.0, CM_REFRESH);
    return;
  }
  // f(b) = loss + penalties (identical arithmetic in every workgroup)
  double fpart = 0.0;
  for (int q = tid; q < D.nloss; q += kWG) fpart += B.losspart[q];
  const double loss = wg_sum(fpart, lds);
  double ppart = 0.0;
  for (int q = tid; q < D.nblk; q += kWG) ppart += B.penpart[q];
  const double pen = wg_sum(ppart, lds);
  const double f_new = 0.5 * loss + pen;
  State o = s;
  o.f_new = f_new;
  bool finish = false;
  if (!isfinite(f_new)) {
    o.status = ST_NUMERICAL;
    finish = true;
  } else if (s.first) {
    o.first = 0;
  } else {
    o.mm_iter = s.mm_iter + 1;
    const double re = s.f_old != 0.0 ? fabs(f_new - s.f_old) / fabs(s.f_old) : fabs(f_new - s.f_old);
    o.rel_change = re;
    if (re <= prm.tol) {
      o.status = ST_OK;
      finish = true;
    } else if (o.mm_iter >= prm.max_iter) {
      o.status = ST_MAX_ITER;
      finish = true;
    }
  }
  if (finish) {
    o.phase = PH_DONE;
    if (b == 0 && tid == 0) *sout = o;
    return;
  }
  o.f_old = f_new;
  o.first_cg = 1;
  o.cg_iter = 0;
  if (prm.band) {  // r0 = c - (X^T X + M) x0; the K launches factor M and solve
    if (real) B.r[j] = cj - (qsum + apply_m(B, prm, j, B.x));
    if (b == 0 && tid == 0) {
      B.counter[32] = 0u;  // failed pivot
      o.phase = PH_BANDMM;
      o.fstage = 0;
      *sout = o;
    }
    return;
  }
  // L and 1/D of this block: scan of its Moebius maps from t before the block
  // (past p: d = 1, e = 0)
  const bool inpad = j < D.p_pad;
  const double alj = inpad ? B.d[j] : 1.0, ej = inpad ? B.e[j] : 0.0;
  const double en = j + 1 < D.p ? B.e[j + 1] : 0.0;
  const double tin = B.mob[4 * (int64_t)D.nblk + min(b, D.nblk - 1)];
  const double tj = mob_apply(wg_scan_mob(mob_leaf(alj, ej), lds), tin);
  invDj = real ? 1.0 / (tj + en) : 0.0;
  const double Lnext = real ? -en * invDj : 0.0;
  sh_L[tid + 1] = Lnext;
  if (tid == 0) sh_L[0] = ej > 0.0 ? -ej / (tin + ej) : 0.0;
  __syncthreads();
  Lj = real ? sh_L[tid] : 0.0;
  // phi_j = prod_{i=start..j} (-L_i); psi_j = prod_{i=j+1..end+1} (-L_i);
  // sigma = zero-inflow backward sweep of phi / D
  const double phi = wg_scan_fwd({-Lj, 0.0}, lds).a;
  const double psi = wg_scan_rev({-Lnext, 0.0}, lds).a;
  const double sig = wg_scan_rev({-Lnext, phi * invDj}, lds).b;
  psij = real ? psi : 0.0;
  sigj = real ? sig : 0.0;
  if (j < D.p_pad) {
    B.L[j] = Lj;
    B.invD[j] = invDj;
    B.sig[j] = sigj;
    B.psi[j] = psij;
  }
  __syncthreads();
  if (tid == kBlk - 1) lds2[0] = phi;
  if (tid == 0) { lds2[1] = sigj; lds2[3] = psij; }
  __syncthreads();
  if (tid == 0 && b < D.nblk) {
    const int K = D.nblk;
    put_shared(B.blk + BK_A * K + b, lds2[0]);
    put_shared(B.blk + BK_SIGS * K + b, lds2[1]);
    put_shared(B.blk + BK_PSIS * K + b, lds2[3]);
    if (loc) {
      loc[BK_A * kMaxGroup + b] = lds2[0];
      loc[BK_SIGS * kMaxGroup + b] = lds2[1];
      loc[BK_PSIS * kMaxGroup + b] = lds2[3];
    }
  }
  // r0 = c - (X^T X + M) x0 with x0 the MM iterate (Algorithm 2)
  double rj = 0.0;
  if (real) {
    rj = cj - (qsum + apply_m(B, prm, j, B.x));
    B.r[j] = rj;
  }
  block_local_solve(D, B, b, j, rj, Lj, Lnext, invDj, sigj, psij, lds, lds2, loc);
  combine(o, 0.0, CM_FIRST);
}

template <int VB, bool SOLO>
__global__ __launch_bounds__(kBlk * VB) void k_block(Dims D, Bufs B, const State* __restrict__ sin,
                                                     State* __restrict__ sout, const Params* __restrict__ prmp) {
  block_body<VB, SOLO>(D, B, sin, sout, prmp, blockIdx.x);
}

// ---------------------------------------------------------------------------
// K (banded M, one workgroup): z = M^-1 r through the banded Cholesky factor,
// r^T z, ||r||, the inner stopping test of Algorithm 2 and gamma.  After an
// MM boundary (PH_BANDMM) it first assembles M from the new weights and
// factors it.  A then rebuilds p from z = yv (gains and carries are zero).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void band_body(const Dims& D, const Bufs& B, const State* __restrict__ sin,
                                          State* __restrict__ sout, const Params* __restrict__ prmp) {
  __shared__ double lds[kBandLds];
  __shared__ double red[24];
  const State s = *sin;
  const int tid = threadIdx.x;
  if (s.phase != PH_CG && s.phase != PH_BANDMM && s.phase != PH_BANDRES) {  // nothing to solve
    if (tid == 0) *sout = s;
    return;
  }
  const Params prm = *prmp;
  const int W = prm.band;
  const bool mm = s.phase == PH_BANDMM;
  State o = s;
  if (mm) {
    band_assemble(B.d, B.rowptr, B.col, B.w, prm.lam2, D.p, W, B.Lb);
    if (!band_factor(B.Lb, B.LbT, B.invdb, D.p, W, lds)) {
      if (tid == 0) {
        o.phase = PH_DONE;
        o.status = ST_NUMERICAL;
        *sout = o;
      }
      return;
    }
    __syncthreads();
  }
  band_solve(B.r, B.btmp, B.yv, B.Lb, B.LbT, B.invdb, D.p, W, lds);
  double rzp = 0.0, rrp = 0.0;
  for (int64_t j = tid; j < D.p; j += kWG) {
    const double rj = B.r[j];
    rzp = fma(rj, B.yv[j], rzp);
    rrp = fma(rj, rj, rrp);
  }
  double sums[4] = {rzp, rrp, 0.0, 0.0};
  wg_sum4(sums, red);
  if (tid == 0) {
    const double rz = sums[0], rn = sqrt(sums[1]) / prm.cnorm;
    const int mode = mm ? CM_FIRST : s.phase == PH_BANDRES ? CM_REFRESH : CM_STEP;
    o.phase = next_phase(prm, o, mode, sums[1], rn);
    o.rel_res = rn;
    o.gamma = mode != CM_STEP ? 0.0 : rz / s.rz;
    o.rz = rz;
    *sout = o;
  }
}

__global__ __launch_bounds__(kWG) void k_band(Dims D, Bufs B, const State* __restrict__ sin,
                                              State* __restrict__ sout, const Params* __restrict__ prmp) {
  band_body(D, B, sin, sout, prmp);
}

// ---------------------------------------------------------------------------
// K1..K3 (banded M through nested inverses, flr_nest.h).  In the factorization
// phase each does the next stage; with all stages done K1 starts the solve for
// the new residual.  They leave shares of r^T z and r^T r, which the next A sums
// (nest_finish).  Summed by their last workgroup to arrive instead, a step of the
// 32 x 32 lattice took 32 us against 26: hundreds of arrivals at one counter.
// ---------------------------------------------------------------------------
template <int WHICH>
__device__ __forceinline__ void nest_body(const NestView& B, const State* __restrict__ sin, State* __restrict__ sout,
                                          const Params* __restrict__ prmp, const int wg) {
  __shared__ __align__(32) double lds[kNestLds];
  State s = *sin;
  // the same in every lane, and said so: the tile loop's control flow and
  // addresses depend on it (as vector values they spill 140 registers)
  s.phase = __builtin_amdgcn_readfirstlane(s.phase);
  s.fstage = __builtin_amdgcn_readfirstlane(s.fstage);
  const bool lead = wg == 0 && threadIdx.x == 0;
  if (s.phase == PH_BANDMM) {
    if (s.fstage < B.nest.stages) {
      if (lead) {
        State o = s;
        o.fstage = s.fstage + 1;
        *sout = o;
      }
      nest_stage(B, prmp->lam2, s.fstage, wg, lds);
      return;
    }
    if (WHICH != LN_NEST1 || B.counter[32]) {  // the solve starts at K1; a failed pivot ends it all
      if (lead) {
        State o = s;
        if (WHICH == LN_NEST1) {
          o.phase = PH_DONE;
          o.status = ST_NUMERICAL;
        }
        *sout = o;
      }
      return;
    }
  }
  const bool solve = s.phase != PH_DONE && s.phase != PH_END && s.phase != PH_RES;
  if (lead) {
    State o = s;
    if (s.phase == PH_BANDMM) o.phase = PH_BANDSOLVE;
    // K1 without separators or K3 ends the step
    if (solve && WHICH == (B.nest.S == 1 ? LN_NEST1 : LN_NEST3)) o.fin = 1;
    *sout = o;
  }
  if (!solve) return;
  if (WHICH == LN_NEST1) {
    if (B.nest.cols == 16)
      nest_apply_segments<16>(B, wg, lds);
    else
      nest_apply_segments<32>(B, wg, lds);
  } else if (WHICH == LN_NEST2) {
    if (B.nest.S > 1) nest_apply_top(B, wg, lds);
  } else if (B.nest.S > 1) {
    if (B.nest.cols == 16)
      nest_apply_back<16>(B, wg, lds);
    else
      nest_apply_back<32>(B, wg, lds);
  }
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// Grouped launches of the ragged batch: one launch of each rotation kernel
// covers every problem of the batch that stores X in the same type; a
// workgroup finds its problem from the offsets of the problems' shares and
// runs that problem's kernel body on its own operands, so each problem's
// arithmetic is that of its solo launch.
// ---------------------------------------------------------------------------
__device__ inline int group_of(const GroupEntry* __restrict__ e, int count, int wg, int which) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int start = which == LN_A   ? e[mid].wg_a
                      : which == LN_B ? e[mid].wg_b
                      : which == LN_C ? e[mid].wg_c
                                      : e[mid].wg_k;
    if (start <= wg) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <typename XT, bool MX>
__global__ __launch_bounds__(kWG) void k_gemv_a_grp(const GroupEntry* __restrict__ e, int count, int par) {
  const GroupEntry& g = e[group_of(e, count, (int)blockIdx.x, LN_A)];
  gemv_a_body<XT, MX, true>(g.D, g.B, g.B.st + par, g.B.st + (par ^ 1), (int)blockIdx.x - g.wg_a);
}

template <typename XT, bool MX>
__global__ __launch_bounds__(kWG) void k_gemv_b_grp(const GroupEntry* __restrict__ e, int count, int par) {
  const GroupEntry& g = e[group_of(e, count, (int)blockIdx.x, LN_B)];
  gemv_b_body<XT, MX>(g.D, g.B, g.B.st + par, g.B.st + (par ^ 1), g.B.prm, (int)blockIdx.x - g.wg_b);
}

__global__ __launch_bounds__(kWG) void k_block_grp(const GroupEntry* __restrict__ e, int count, int par) {
  const GroupEntry& g = e[group_of(e, count, (int)blockIdx.x, LN_C)];
  block_body<1, false>(g.D, g.B, g.B.st + par, g.B.st + (par ^ 1), g.B.prm, (int)blockIdx.x - g.wg_c);
}

__global__ __launch_bounds__(kWG) void k_band_grp(const GroupEntry* __restrict__ e, int par) {
  const GroupEntry& g = e[blockIdx.x];
  if (g.band != BAND_FACTOR) {
    if (threadIdx.x == 0) g.B.st[par ^ 1] = g.B.st[par];
    return;
  }
  band_body(g.D, g.B, g.B.st + par, g.B.st + (par ^ 1), g.B.prm);
}

template <int WHICH>
__global__ __launch_bounds__(kNT, 2) void k_nest(NestView v, const State* __restrict__ sin, State* __restrict__ sout,
                                                 const Params* __restrict__ prmp) {
  nest_body<WHICH>(v, sin, sout, prmp, (int)blockIdx.x);
}

template <int WHICH>
__global__ __launch_bounds__(kNT, 2) void k_nest_grp(const GroupEntry* __restrict__ e, int count, int par) {
  const GroupEntry& g = e[group_of(e, count, (int)blockIdx.x, WHICH)];
  if (g.band != BAND_NEST) {
    if (threadIdx.x == 0) g.B.st[par ^ 1] = g.B.st[par];
    return;
  }
  const NestView v = nest_view(g.D, g.B);
  nest_body<WHICH>(v, g.B.st + par, g.B.st + (par ^ 1), g.B.prm, (int)blockIdx.x - g.wg_k);
}

// State of every problem of a batch after a graph launch (slot 0 of each).
__global__ __launch_bounds__(kWG) void k_gather_states(const GroupEntry* __restrict__ e, int count,
                                                       State* __restrict__ out) {
  const int i = (int)blockIdx.x * kWG + threadIdx.x;
  if (i < count) out[i] = e[i].B.st[0];
}

template <typename XT, bool MX>
static hipError_t launch_grouped_t(const GroupEntry* e, int count, int wgs, int par, int which, hipStream_t st) {
  const dim3 g(wgs);
  switch (which) {
    case LN_A: hipLaunchKernelGGL((k_gemv_a_grp<XT, MX>), g, dim3(kWG), 0, st, e, count, par); break;
    case LN_B: hipLaunchKernelGGL((k_gemv_b_grp<XT, MX>), g, dim3(kWG), 0, st, e, count, par); break;
    case LN_C: hipLaunchKernelGGL(k_block_grp, g, dim3(kWG), 0, st, e, count, par); break;
    case LN_BAND: hipLaunchKernelGGL(k_band_grp, dim3(count), dim3(kWG), 0, st, e, par); break;
    case LN_NEST1: hipLaunchKernelGGL(k_nest_grp<LN_NEST1>, g, dim3(kNT), 0, st, e, count, par); break;
    case LN_NEST2: hipLaunchKernelGGL(k_nest_grp<LN_NEST2>, g, dim3(kNT), 0, st, e, count, par); break;
    default: hipLaunchKernelGGL(k_nest_grp<LN_NEST3>, g, dim3(kNT), 0, st, e, count, par); break;
  }
  return hipGetLastError();
}

hipError_t launch_grouped(int dtype, bool mixed, const GroupEntry* e, int count, int wgs, int par, int which,
                          hipStream_t st) {
  switch (dtype) {
    case 0: return mixed ? launch_grouped_t<double, true>(e, count, wgs, par, which, st)
                         : launch_grouped_t<double, false>(e, count, wgs, par, which, st);
    case 1: return mixed ? launch_grouped_t<float, true>(e, count, wgs, par, which, st)
                         : launch_grouped_t<float, false>(e, count, wgs, par, which, st);
    default: return mixed ? launch_grouped_t<uint16_t, true>(e, count, wgs, par, which, st)
                          : launch_grouped_t<uint16_t, false>(e, count, wgs, par, which, st);
  }
}

hipError_t launch_gather_states(const GroupEntry* e, int count, State* out, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_states, dim3((unsigned)((count + kWG - 1) / kWG)), dim3(kWG), 0, st, e, count, out);
  return hipGetLastError();
}

template <typename XT, bool MX>
static hipError_t launch_rotation_t(const Dims& D, const Bufs& B, int par, int which, hipStream_t st) {
  const State* sin = B.st + par;
  State* sout = B.st + (par ^ 1);
  switch (which) {
    case LN_A:
      if (B.nest.S)
        hipLaunchKernelGGL((k_gemv_a<XT, MX, true>), dim3(D.cb1 * D.rb1), dim3(kWG), 0, st, D, B, sin, sout);
      else
        hipLaunchKernelGGL((k_gemv_a<XT, MX, false>), dim3(D.cb1 * D.rb1), dim3(kWG), 0, st, D, B, sin, sout);
      break;
    case LN_B:
      hipLaunchKernelGGL((k_gemv_b<XT, MX>), dim3(D.gridB), dim3(kWG), 0, st, D, B, sin, sout, B.prm);
      break;
    case LN_C:
      // one or two blocks (p <= 512) in one workgroup, which combines them without the
      // device round trips (8.5 -> 7.0 us at p = 200; four in one of 1024 threads
      // were slower, its scans share one CU's LDS); two per workgroup where the
      // arrivals of as many workgroups as blocks bound the launch (one and two per
      // workgroup: 8.4 and 8.9 us at 64 blocks, 9.1 and 9.1 at 96, 9.5 and 9.3 at 128,
      // 12.0 and 10.8 at 256, 13.8 and 13.4 at 391, 15.3 and 14.2 at 512)
      if (D.nblk == 1)
        hipLaunchKernelGGL((k_block<1, true>), dim3(1), dim3(kBlk), 0, st, D, B, sin, sout, B.prm);
      else if (D.nblk == 2)
        hipLaunchKernelGGL((k_block<2, true>), dim3(1), dim3(2 * kBlk), 0, st, D, B, sin, sout, B.prm);
      else if (D.nblk >= 128)
        hipLaunchKernelGGL((k_block<2, false>), dim3((D.nblk + 1) / 2), dim3(2 * kBlk), 0, st, D, B, sin, sout, B.prm);
      else
        hipLaunchKernelGGL((k_block<1, false>), dim3(D.nblk), dim3(kBlk), 0, st, D, B, sin, sout, B.prm);
      break;
    case LN_BAND:
      hipLaunchKernelGGL(k_band, dim3(1), dim3(kWG), 0, st, D, B, sin, sout, B.prm);
      break;
    case LN_NEST1:
      hipLaunchKernelGGL(k_nest<LN_NEST1>, dim3(B.nest.wgs), dim3(kNT), 0, st, nest_view(D, B), sin, sout, B.prm);
      break;
    case LN_NEST2:
      hipLaunchKernelGGL(k_nest<LN_NEST2>, dim3(B.nest.wgs), dim3(kNT), 0, st, nest_view(D, B), sin, sout, B.prm);
      break;
    default:
      hipLaunchKernelGGL(k_nest<LN_NEST3>, dim3(B.nest.wgs), dim3(kNT), 0, st, nest_view(D, B), sin, sout, B.prm);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_rotation(const Dims& D, const Bufs& B, int par, int which, hipStream_t st, bool mixed) {
  switch (D.dtype) {
    case 0: return mixed ? launch_rotation_t<double, true>(D, B, par, which, st)
                         : launch_rotation_t<double, false>(D, B, par, which, st);
    case 1: return mixed ? launch_rotation_t<float, true>(D, B, par, which, st)
                         : launch_rotation_t<float, false>(D, B, par, which, st);
    default: return mixed ? launch_rotation_t<uint16_t, true>(D, B, par, which, st)
                          : launch_rotation_t<uint16_t, false>(D, B, par, which, st);
  }
}

template <typename XT>
static hipError_t launch_setup_t(const Dims& D, const void* X, const double* y, double* cpart, double* spart,
                                 double* c, double* s, hipStream_t st) {
  hipLaunchKernelGGL(k_setup_partial<XT>, dim3(D.cb2 * D.rb2), dim3(kWG), 0, st, D, reinterpret_cast<const XT*>(X),
                     y, cpart, spart);
  hipLaunchKernelGGL(k_setup_final, dim3((unsigned)((D.p_pad + kWG - 1) / kWG)), dim3(kWG), 0, st, D, cpart, spart,
                     c, s);
  return hipGetLastError();
}

hipError_t launch_setup(const Dims& D, const void* X, const double* y, double* cpart, double* spart, double* c,
                        double* s, hipStream_t st) {
  switch (D.dtype) {
    case 0: return launch_setup_t<double>(D, X, y, cpart, spart, c, s, st);
    case 1: return launch_setup_t<float>(D, X, y, cpart, spart, c, s, st);
    default: return launch_setup_t<uint16_t>(D, X, y, cpart, spart, c, s, st);
  }
}

hipError_t launch_init(const Dims& D, const Bufs& B, const double* warm, int use_warm, hipStream_t st) {
  hipLaunchKernelGGL(k_init, dim3((unsigned)((D.p_pad + kWG - 1) / kWG)), dim3(kWG), 0, st, D, B, warm, use_warm);
  return hipGetLastError();
}

// Non-finite scan of the stored X (validation at creation).
template <typename XT>
__global__ __launch_bounds__(kWG) void k_check_finite(const XT* __restrict__ X, int64_t count, int* flag) {
  const int64_t stride = (int64_t)gridDim.x * kWG;
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < count; i += stride) {
    if constexpr (sizeof(XT) == 2) {
      bad |= (X[i] & 0x7f80u) == 0x7f80u;
    } else {
      bad |= !isfinite((double)X[i]);
    }
  }
  if (bad) *flag = 1;
}

hipError_t launch_check_finite(const void* X, int dtype, int64_t count, int* flag, hipStream_t st) {
  const dim3 g(1024), b(kWG);
  switch (dtype) {
    case 0: hipLaunchKernelGGL(k_check_finite<double>, g, b, 0, st, reinterpret_cast<const double*>(X), count, flag); break;
    case 1: hipLaunchKernelGGL(k_check_finite<float>, g, b, 0, st, reinterpret_cast<const float*>(X), count, flag); break;
    default: hipLaunchKernelGGL(k_check_finite<uint16_t>, g, b, 0, st, reinterpret_cast<const uint16_t*>(X), count, flag); break;
  }
  return hipGetLastError();
}

}  // namespace flr

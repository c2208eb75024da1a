// Exact preconditioner solve for graphs whose index bandwidth bw = max |j - k|
// over E is at least 2 (the 2-D lattice, all-pairs fusion): M = lambda1 A +
// lambda2 B is banded with bandwidth bw, and Algorithm 2 applies M^-1 through
// its banded Cholesky factor M = L L^T (section 3.1, where the PCG
// preconditioner is solved with a banded Cholesky factorization; the lattice
// of the paper's 2-D experiments has bw = q).  M changes once per MM iteration, so
// the factor is computed once per MM iteration and every PCG step applies it
// with two triangular sweeps.
//
// Two forms, by W = bw + 1 (band_blocks): blocks of NB rows whose diagonal
// blocks of L are inverted (16 <= W <= 107, below), and for the other widths a
// chain of single rows.  Layouts of the latter (W entries per row / column),
// stored as the sweeps use them, i.e. divided by the diagonal of the step that
// applies them:
//   Lb  column-major band, Lb[j*W + k]  = L_{j+k, j} / L_jj  (column j; k >= 1)
//   LbT row-major band,    LbT[i*W + k] = L_{i, i-k} / L_ii  (row i; k >= 1)
//   Lb[j*W] = LbT[j*W] = L_jj, invd[j] = 1 / L_jj
// Both sweeps walk one dependent chain of length p, so one wave runs each:
// the not-yet-final right-hand sides of the next bw elements sit in a ring of
// 64*NR registers across the wave's lanes (element t in slot t mod 64*NR),
// each step reads the current element's right-hand side b_j from its lane and
// subtracts b_j times (multiplier / L_jj) from the ring with one fma per
// register; the solution b_j / L_jj of a chunk of 64 elements is formed once
// the chunk is done.  The other three waves of the workgroup stage the
// coming steps' multipliers into LDS in the ring's slot order, straight from
// Lb / LbT: each staging thread owns fixed ring distances k and walks the
// steps of a sub-chunk (one row of W multipliers per step, read coalesced
// across threads), with its loads issued a sub-chunk ahead.
#pragma once
#include <type_traits>

#include "flr_device.h"

namespace flr {

constexpr int kBandLds = 13312;   // doubles of LDS the band routines use (104 KiB)
constexpr int kBandMaxW = 1025;   // widest band the sweeps handle (NR = 17 ring registers)
constexpr int kPanelMaxW = 107;   // widest band the register-panel factorization takes (its LDS window)

// Rows per block of the blocked sweeps, 0 for the row-by-row ones.  NB <= W, so
// that a block's inverse fits into the unused corner of its band.  Narrower
// bands have too little work per block for its two barriers (at NB = 8 no better
// than the 50 ns per row of the chain); wider ones are factored in place
// in global memory (band_factor_blocked), which needs the plain layout.
__host__ __device__ inline int band_blocks(int W) {
  return W > kPanelMaxW || W < 16 ? 0 : W < 32 ? 16 : W < 64 ? 32 : 64;
}

// Ring registers per lane: 64*NR slots must hold the bw elements ahead of the
// current one plus the 64 of the chunk being consumed.
__host__ __device__ inline int band_nr(int W) {
  const int need = (W + 63 + 63) / 64;
  const int opts[] = {2, 3, 5, 8, 17};  // a few ring sizes keep the code (and compile time) small
  for (int o : opts)
    if (o >= need) return o;
  return 0;
}

// Band of M below the diagonal, column-major: Lb[k*W] = d_k (the diagonal
// lambda1 a_k + lambda2 sum_q w_q), Lb[k*W + (c - k)] = -lambda2 w_q for every
// edge (k, c) with k < c, zero elsewhere.  Whole workgroup; ends with a barrier.
__device__ inline void band_assemble(const double* __restrict__ d, const int32_t* __restrict__ rowptr,
                                     const int32_t* __restrict__ col, const double* __restrict__ w, double lam2,
                                     int64_t p, int W, double* __restrict__ Lb) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t tot = p * (int64_t)W;
  for (int64_t i = tid; i < tot; i += nt) Lb[i] = 0.0;
  __syncthreads();
  for (int64_t k = tid; k < p; k += nt) {
    Lb[k * W] = d[k];
    for (int q = rowptr[k]; q < rowptr[k + 1]; ++q) {
      const int64_t c = col[q];
      if (c > k && c - k < W) Lb[k * W + (c - k)] = -lam2 * w[q];
    }
  }
  __syncthreads();
}

__device__ inline double readlane_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// Blocked right-looking Cholesky of the assembled band for bands too wide for
// the register-panel factorization's LDS window (below).  Panels of nb columns (nb = 16, fewer for very wide
// bands so that a panel fits the band LDS) are loaded into LDS and factored
// there, one pivot per step; the panel's columns of L are written out (Lb
// scaled by 1/L_jj, LbT unscaled, rescaled by the caller), and the triangle
// of the band that the panel reaches - columns j0 + nb .. j0 + nb + W - 2 -
// is updated with one rank-nb pass in global memory (wave w takes every
// fourth column, lanes its rows, coalesced), instead of one pass per pivot.
// 256 threads; returns false in every thread on a pivot that is not
// positive and finite.
__device__ inline bool band_factor_blocked(double* __restrict__ Lb, double* __restrict__ LbT,
                                           double* __restrict__ invd, int64_t p, int W, double* __restrict__ P) {
  __shared__ double sh_inv[16];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
  const int nb = kBandLds / W < 16 ? kBandLds / W : 16;
  for (int64_t j0 = 0; j0 < p; j0 += nb) {
    const int w = (int)((p - j0) < (int64_t)nb ? (p - j0) : (int64_t)nb);
    const double* src = Lb + j0 * W;  // the panel's columns are contiguous
    for (int e = tid; e < w * W; e += nt) P[e] = src[e];
    __syncthreads();
    for (int jj = 0; jj < w; ++jj) {
      const double piv = P[jj * W];
      if (!(piv > 0.0) || !isfinite(piv)) return false;  // the same value in every thread
      const double ljj = sqrt(piv), inv = 1.0 / ljj;
      __syncthreads();  // every thread has the pivot before it is overwritten
      for (int k = tid; k < W; k += nt) P[jj * W + k] = k ? P[jj * W + k] * inv : ljj;
      if (tid == 0) sh_inv[jj] = inv;
      __syncthreads();
      // later panel columns: M(j' + k, j') -= L(j' + k, j) L(j', j), j' = j + d
      const int rem = w - 1 - jj;
      for (int e = tid; e < rem * W; e += nt) {
        const int d = 1 + e / W, k = e - (d - 1) * W;
        if (k < W - d) P[(jj + d) * W + k] = fma(-P[jj * W + k + d], P[jj * W + d], P[(jj + d) * W + k]);
      }
      __syncthreads();
    }
    for (int e = tid; e < w * W; e += nt) {
      const int jj = e / W, k = e - jj * W;
      const int64_t j = j0 + jj;
      const double v = P[e];
      if (k == 0) {
        Lb[j * W] = v;
        LbT[j * W] = v;
        invd[j] = sh_inv[jj];
      } else if (j + k < p) {
        Lb[j * W + k] = v * sh_inv[jj];
        LbT[(j + k) * W + k] = v;
      }
    }
    // trailing triangle: column c = j0 + dcol, row c + di gets the sum over
    // the panel columns whose band reaches both c and c + di
    const int64_t cend = (j0 + w + W - 2) < p - 1 ? (j0 + w + W - 2) : p - 1;
    for (int64_t c = j0 + w + wave; c <= cend; c += 4) {
      const int dcol = (int)(c - j0);
      int dimax = W - 1 < w + W - 2 - dcol ? W - 1 : w + W - 2 - dcol;
      if ((int64_t)dimax > p - 1 - c) dimax = (int)(p - 1 - c);
      for (int di = lane; di <= dimax; di += 64) {
        const int jlo = dcol + di - (W - 1) > 0 ? dcol + di - (W - 1) : 0;
        double sum = 0.0;
        for (int jj = jlo; jj < w; ++jj) sum = fma(P[jj * W + dcol + di - jj], P[jj * W + dcol - jj], sum);
        Lb[c * W + di] -= sum;
      }
    }
    __syncthreads();
  }
  return true;
}

// Right-looking Cholesky of the assembled band in panels of NB columns, for
// bands narrow enough that the active window fits in LDS.  The window -
// columns j0 .. j0 + NB + W - 2 while the panel that starts at column j0 is
// factored - is a ring of R = NB + W - 1 columns of W entries (column c in
// slot c mod R).  Per panel:
//  * wave 0 takes the panel's columns into registers (lane l holds rows
//    j0 + l and j0 + 64 + l) and factors them there: each pivot and the
//    multipliers of the later panel columns come from the lanes that hold
//    them (readlane), so the panel needs no barrier.  It leaves the panel's
//    rows of L in LDS (Lp) and nothing else, to keep this serial part short;
//  * after one barrier waves 1-3 write the panel's columns of L to Lb, LbT
//    and invd while wave 0 moves the next NB columns of the assembled band,
//    loaded one panel earlier, into the panel's freed slots and issues the
//    loads for the panel after (its memory counter then holds only those
//    loads, so waiting for them never waits for the scattered stores); then
//    the workgroup subtracts L21 L21^T (L21: the rows of Lp below the panel)
//    from the trailing triangle (columns j0 + NB .. j0 + NB + W - 2):
//    thread (tx, ty) keeps its entries (row offset tx + 16 c, column offset
//    ty + 16 a) in registers over the panel's NB pivots.
// Every entry receives the same fused multiply-adds in the same pivot order as
// in a one-pivot-per-step right-looking factorization (an update from a pivot
// whose band does not reach the entry multiplies by an exact zero), so the
// factor is the same bit for bit; the trailing triangle makes one LDS round
// trip per NB pivots instead of one per pivot, with two barriers per panel.
// 256 threads; false in every thread on a pivot that is not positive and
// finite.
// BR > 0: L goes out in the layout of the blocked sweeps with blocks of BR rows
// (LbT the forward blocks, Lb - in place of the assembled band, whose columns of
// the block being written are all in the window by then - the backward ones).
template <int NB, int BR>
__device__ inline bool band_factor_panels(double* Lb, double* __restrict__ LbT, double* __restrict__ invd, int64_t p,
                                          int W, double* __restrict__ lds) {
  constexpr int LP = NB + 1;                   // Lp row stride, odd: 16 consecutive rows in distinct banks
  constexpr int NXT = (NB * kPanelMaxW + 63) / 64;  // entering band entries per lane of wave 0
  constexpr int kTB = 7;                       // 16-wide blocks of the trailing triangle (W - 1 <= 112)
  __shared__ int sh_bad;
  __shared__ double sh_inv[NB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tx = tid & 15, ty = tid >> 4;
  const int R = NB + W - 1;
  double* Lp = lds + R * W;  // rows j0 .. j0 + R - 1 of the panel's columns of L, LP apart
  const int64_t pw = p * (int64_t)W;
  {
    const int64_t n0 = (p < R ? p : (int64_t)R) * W;
    for (int64_t i = tid; i < n0; i += 256) lds[i] = Lb[i];
  }
  double nxt[NXT];
#pragma unroll
  for (int q = 0; q < NXT; ++q) {
    const int e = lane + 64 * q;
    const int64_t g = (int64_t)R * W + e;
    nxt[q] = (wave == 0 && e < NB * W && g < pw) ? Lb[g] : 0.0;
  }
  if (tid == 0) sh_bad = 0;
  int s0 = 0;  // ring slot of column j0
  for (int64_t j0 = 0; j0 < p; j0 += NB) {
    const int w = (p - j0) < (int64_t)NB ? (int)(p - j0) : NB;
    lds_barrier();
    if (wave == 0) {
      // the panel in registers.  Full panels (all but possibly the last) are
      // compiled without the per-column bounds; LDS reads are unconditional
      // at indices clamped into the column and selected afterwards (a
      // guarded read compiles to a branch), and ring positions wrap once at
      // R W: the slot of column j0 + jj starts at (s0 + jj) W mod R W.
      auto factor_panel = [&](auto full) {
        constexpr bool F = decltype(full)::value;
        const int ww = F ? NB : w;
        const int RW = R * W, base = s0 * W;
        double x0[NB], x1[NB];
#pragma unroll
        for (int jj = 0; jj < NB; ++jj) {
          const int k0 = lane - jj, k1 = lane + 64 - jj;  // entries of column j0 + jj in the lane's rows
          int a0 = base + jj * W + (k0 < 0 ? 0 : (k0 < W ? k0 : W - 1));
          int a1 = base + jj * W + (k1 < W ? k1 : W - 1);
          a0 = a0 >= RW ? a0 - RW : a0;
          a1 = a1 >= RW ? a1 - RW : a1;
          const double v0 = lds[a0], v1 = lds[a1];
          x0[jj] = ((F || jj < ww) && k0 >= 0 && k0 < W) ? v0 : 0.0;
          x1[jj] = ((F || jj < ww) && k1 < W) ? v1 : 0.0;
        }
        bool bad = false;
#pragma unroll
        for (int jj = 0; jj < NB; ++jj) {
          if (!F && jj >= ww) break;
          const double piv = readlane_f64(x0[jj], jj);
          if (!(piv > 0.0) || !isfinite(piv)) {
            bad = true;
            break;
          }
          const double ljj = sqrt(piv), rj = 1.0 / ljj;
          if (lane == 0) sh_inv[jj] = rj;
          const double l0 = lane > jj ? x0[jj] * rj : (lane == jj ? ljj : 0.0);
          const double l1 = x1[jj] * rj;
          x0[jj] = l0;
          x1[jj] = l1;
#pragma unroll
          for (int c = jj + 1; c < NB; ++c) {
            if (F || c < ww) {
              const double lc = readlane_f64(l0, c);
              x0[c] = fma(-l0, lc, x0[c]);
              x1[c] = fma(-l1, lc, x1[c]);
            }
          }
        }
        if (bad) {
          if (lane == 0) sh_bad = 1;
        } else {
#pragma unroll
          for (int jj = 0; jj < NB; ++jj) {
            if (lane < R) Lp[lane * LP + jj] = x0[jj];
            if (lane + 64 < R) Lp[(lane + 64) * LP + jj] = x1[jj];
          }
        }
      };
      if (w == NB)
        factor_panel(std::integral_constant<bool, true>());
      else
        factor_panel(std::integral_constant<bool, false>());
    }
    lds_barrier();
    if (sh_bad) return false;
    if (wave == 0) {
      // the panel's slots take the columns entering the window (entry e of
      // them at (s0 W + e) mod R W), then the loads for the next panel go out
      const int RW = R * W;
      const int64_t left = pw - (j0 + R) * W, left2 = left - (int64_t)NB * W;
      const int lim = left < (int64_t)NB * W ? (int)(left > 0 ? left : 0) : NB * W;
      const int lim2 = left2 < (int64_t)NB * W ? (int)(left2 > 0 ? left2 : 0) : NB * W;
#pragma unroll
      for (int q = 0; q < NXT; ++q) {
        const int e = lane + 64 * q, a = s0 * W + e;
        if (e < lim) lds[a >= RW ? a - RW : a] = nxt[q];
      }
      const double* src = Lb + (j0 + NB + R) * W;
#pragma unroll
      for (int q = 0; q < NXT; ++q) {
        const int e = lane + 64 * q;
        nxt[q] = e < lim2 ? src[e] : 0.0;
      }
    } else {
      // the panel's columns of L: Lb scaled by 1/L_jj below the diagonal,
      // LbT unscaled (the caller scales its rows), invd
      const int k = tid - 64;
      if constexpr (BR > 0) {
        // a thread per row i = j0 + k: eight neighbouring entries of the backward
        // block, and of the forward blocks lanes along the rows
        const int64_t i = j0 + k;
        if (k < R && i < p) {
          const int64_t bi = i / BR, bj = j0 / BR;  // the panel lies in one block (NB divides BR)
          const int ri = (int)(i - bi * BR), cj = (int)(j0 - bj * BR);
          const int ld = p - bi * BR < BR ? (int)(p - bi * BR) : BR;
          double* f = LbT + bi * BR * W + ri;
          if (bi == bj) {
            for (int jj = 0; jj < w; ++jj)
              if (k >= jj) f[(int64_t)(cj + jj ? cj + jj - 1 : W - 1) * ld] = Lp[k * LP + jj];
          } else {
            const int kk = (int)(j0 - bi * BR) + W - 1;
            double* g = Lb + bj * BR * W + (int64_t)(W - 2 - (int)(i - (bj + 1) * BR)) * BR + (BR - 1 - cj);
            for (int jj = 0; jj < w; ++jj) {
              if (k - jj < W) {
                const double v = Lp[k * LP + jj];
                f[(int64_t)(kk + jj) * ld] = v;
                g[-jj] = v;
              }
            }
          }
        }
      } else {
        for (int jj = 0; jj < w; ++jj) {
          const int64_t j = j0 + jj;
          if (k < W && j + k < p) {
            const double v = Lp[(jj + k) * LP + jj];
            Lb[j * W + k] = k ? v * sh_inv[jj] : v;
            LbT[(j + k) * W + k] = v;
          }
        }
      }
      if (k < w) invd[j0 + k] = sh_inv[k];
    }
    if (j0 + NB < p) {
      const int64_t rest = p - 1 - (j0 + NB);
      const int cmax = rest < (int64_t)(W - 2) ? (int)rest : W - 2;
      double t[kTB][kTB];
#pragma unroll
      for (int a = 0; a < kTB; ++a) {
        const int u = ty + 16 * a, uc = u < W - 2 ? u : W - 2;
        const int slot = s0 + NB + uc < R ? s0 + NB + uc : s0 + NB + uc - R;
#pragma unroll
        for (int c = a; c < kTB; ++c) {
          const int v = tx + 16 * c;
          t[a][c] = (u <= v && v <= cmax) ? lds[slot * W + (v - u)] : 0.0;
        }
      }
#pragma unroll 2
      for (int jj = 0; jj < NB; ++jj) {
        double lu[kTB], lv[kTB];
#pragma unroll
        for (int a = 0; a < kTB; ++a) {
          const int u = ty + 16 * a, v = tx + 16 * a;
          lu[a] = Lp[(NB + (u < W - 2 ? u : W - 2)) * LP + jj];
          lv[a] = Lp[(NB + (v < W - 2 ? v : W - 2)) * LP + jj];
        }
        // every tile entry is updated (entries outside the triangle hold
        // values that are never stored), so no per-entry selects
#pragma unroll
        for (int a = 0; a < kTB; ++a)
#pragma unroll
          for (int c = a; c < kTB; ++c) t[a][c] = fma(-lu[a], lv[c], t[a][c]);
      }
#pragma unroll
      for (int a = 0; a < kTB; ++a) {
        const int u = ty + 16 * a, uc = u < W - 2 ? u : W - 2;
        const int slot = s0 + NB + uc < R ? s0 + NB + uc : s0 + NB + uc - R;
#pragma unroll
        for (int c = a; c < kTB; ++c) {
          const int v = tx + 16 * c;
          if (u <= v && v <= cmax) lds[slot * W + (v - u)] = t[a][c];
        }
      }
    }
    s0 = s0 + NB < R ? s0 + NB : s0 + NB - R;
  }
  return true;
}

// ---------------------------------------------------------------------------
// Blocked sweeps.  A sweep solves L y = r (or, over reversed indexes, L^T z = y)
// in blocks of NB rows: t = r_b - (band part of L left of the block) y, then y_b
// = inv(L_bb) t.  In solve order v (v = j forward, p - 1 - j backward) a block
// that starts at v0 is stored as W columns of its NB rows (the last rows of the
// index range may form a shorter block; ld is its row count):
//   column kk < W - 1, rows i <= kk:  the coupling to element v0 - (W - 1) + kk,
//                      rows i > kk:   column kk + 1 of inv(L_bb),
//   column W - 1:                     column 0 of inv(L_bb):
// the corner that the band leaves empty holds the inverse, so the blocks take the
// band's own p W entries.  Inverting only the triangular diagonal blocks keeps
// the sweep a backward-stable substitution (L is an M-matrix factor: its entries
// off the diagonal are <= 0 and those of the inverse come out without
// cancellation).
// ---------------------------------------------------------------------------

// inv(L_bb) of every block, in place of L_bb in the forward blocks and into the
// backward ones.  One wave per block at a time: lane c substitutes column c with
// L_bb in LDS (packed rows, read as broadcasts), its values in registers.
template <int NB>
__device__ inline void band_invert_blocks(double* __restrict__ bwd, double* __restrict__ fwd,
                                          const double* __restrict__ invd, int64_t p, int W, double* lds) {
  constexpr int TRI = NB * (NB + 1) / 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* T = lds + wave * (TRI + NB);  // row r at r (r + 1) / 2, then 1 / L_rr
  double* D = T + TRI;
  const int64_t nblk = (p + NB - 1) / NB;
  for (int64_t b = wave; b < nblk; b += 4) {
    const int ld = p - b * NB < NB ? (int)(p - b * NB) : NB;
    double* f = fwd + b * NB * W;
    double* g = bwd + b * NB * W;
    for (int c = 0; c < ld; ++c)
      if (lane < ld && lane >= c) T[lane * (lane + 1) / 2 + c] = f[(int64_t)(c ? c - 1 : W - 1) * ld + lane];
    if (lane < ld) D[lane] = invd[b * NB + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double x[NB];
#pragma unroll
    for (int r = 0; r < NB; ++r) {
      double s0 = r == lane ? 1.0 : 0.0, s1 = 0.0;
#pragma unroll
      for (int k = 0; k < r; ++k) {
        if (k & 1)
          s1 = fma(-T[r * (r + 1) / 2 + k], x[k], s1);
        else
          s0 = fma(-T[r * (r + 1) / 2 + k], x[k], s0);
      }
      x[r] = r < ld ? (s0 + s1) * D[r] : 0.0;
    }
    if (lane < ld) {
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        if (r < ld && r >= lane) {  // inv(L_bb)[r][lane]
          f[(int64_t)(lane ? lane - 1 : W - 1) * ld + r] = x[r];
          const int c = ld - 1 - r;  // its column over reversed indexes
          g[(int64_t)(c ? c - 1 : W - 1) * ld + (ld - 1 - lane)] = x[r];
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __syncthreads();
}

// One blocked sweep by 256 threads: thread (i, stream) holds row i of every NS-th
// column of a block in registers, loaded ahead.  Per block two LDS
// barriers: after the band part (partial sums of the streams) and after the
// inverse (likewise); every stream forms t and y itself, and every wave keeps its
// own copy of the last solution values, twice in a row of 2 H so that a block
// reads them at fixed offsets.  Measured at W = 101, p = 10^4: two sweeps 0.61 ms
// for one column (1.09 with the row-by-row chain; 0.35 of it the arithmetic chain,
// 1.1 us per block, the rest the issue of the loads) and 0.91 ms with 256 columns
// (1.24; 4.1 GB, 4.5 TB/s: the loads bound it).
// U >= W / NS columns per stream; the ones past the band repeat column W - 1 and
// meet a zero.
template <int NB, int U, int WMIN>
__device__ __forceinline__ void band_sweep_blocks(const double* __restrict__ r, double* __restrict__ out,
                                                  const double* __restrict__ Z, int64_t p, int W, bool fwd,
                                                  double* __restrict__ lds) {
  constexpr int NS = kWG / NB;     // streams
  constexpr int UI = NB / NS;      // columns per stream with a part of the inverse
  constexpr int H = 256;           // history slots
  static_assert(NS * U + NB <= H && NB % NS == 0 && U >= UI, "history or stream split");
  const int tid = threadIdx.x, lane = tid & 63, i = tid % NB;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int st = NB == 64 ? wave : tid / NB;
  double* part = lds;                  // [NS][NB]
  double* part2 = lds + kWG;           // [NS][NB]
  double* hist = lds + 2 * kWG + wave * 2 * H;
  const int nfull = (int)(p / NB), tail = (int)(p - (int64_t)nfull * NB);
  for (int q = lane; q < 2 * H; q += 64) hist[q] = 0.0;
  int v0 = 0;  // elements solved
  // this thread's offset into a full block of its columns that may be past the band
  int clamped[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int kk = st + NS * u;
    clamped[u] = (kk < W ? kk : W - 1) * NB + i;
  }
  // block b (ld rows) into registers: its columns, column W - 1 and the right-hand side
  auto load = [&](int b, double (&v)[U], double& vl, double& rv) {
    const double* z = Z + (int64_t)b * NB * W;
    const double* zt = z + tid;  // column st, row i
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = NS * u + NS <= WMIN ? zt[NS * NB * u] : z[clamped[u]];
    vl = z[(W - 1) * NB + i];
    rv = r[(int64_t)b * NB + (fwd ? i : NB - 1 - i)];
  };
  auto load_tail = [&](double (&v)[U], double& vl, double& rv) {
    const double* z = Z + (int64_t)nfull * NB * W;
    const int ii = i < tail ? i : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = st + NS * u;
      v[u] = z[(kk < W ? kk : W - 1) * tail + ii];
    }
    vl = z[(W - 1) * tail + ii];
    rv = r[(int64_t)nfull * NB + (fwd ? ii : tail - 1 - ii)];
  };
  auto step = [&](int b, int ld, const double (&v)[U], double vl, double rv) {
    const double* h = hist + ((v0 - (W - 1)) & (H - 1)) + st;  // element v0 - (W - 1) + st
    double a0 = 0.0, a1 = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = st + NS * u;
      double y = h[NS * u];
      if (NS * u + NS >= WMIN) y = kk < W - 1 ? y : 0.0;
      if (u < UI) y = i > kk ? 0.0 : y;
      if (u & 1)
        a1 = fma(v[u], y, a1);
      else
        a0 = fma(v[u], y, a0);
    }
    part[st * NB + i] = a0 + a1;
    lds_barrier();
    double t = i < ld ? rv : 0.0;
#pragma unroll
    for (int q = 0; q < NS; ++q) t -= part[q * NB + i];
    if (i >= ld) t = 0.0;
    double c0 = st == 0 ? vl * (NB == 64 ? readlane_f64(t, 0) : __shfl(t, lane & ~(NB - 1), 64)) : 0.0, c1 = 0.0;
#pragma unroll
    for (int u = 0; u < UI; ++u) {
      const int kk = st + NS * u;
      const int c = kk + 1 < NB ? kk + 1 : 0;  // kk = NB - 1 holds no column of the inverse
      double tc = NB == 64 ? readlane_f64(t, c) : __shfl(t, (lane & ~(NB - 1)) + c, 64);
      tc = i > kk ? tc : 0.0;
      if (u & 1)
        c1 = fma(v[u], tc, c1);
      else
        c0 = fma(v[u], tc, c0);
    }
    part2[st * NB + i] = c0 + c1;
    lds_barrier();
    double y = 0.0;
#pragma unroll
    for (int q = 0; q < NS; ++q) y += part2[q * NB + i];
    if (i >= ld) y = 0.0;
    if (lane < NB) {
      const int s0 = (v0 + i) & (H - 1);
      hist[s0] = y;
      hist[s0 + H] = y;
    }
    if (tid < ld) out[(int64_t)b * NB + (fwd ? i : ld - 1 - i)] = y;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    v0 += ld;
  };
  double va[U], vb[U], la = 0.0, lb = 0.0, ra = 0.0, rb = 0.0;
  __syncthreads();
  if (!fwd && tail) {  // the short block is the first of the backward sweep and the last of the forward one
    load_tail(va, la, ra);
    step(nfull, tail, va, la, ra);
  }
  // blocks in two register sets, loaded a block ahead (two blocks ahead: the same)
  auto block = [&](int s) { return fwd ? s : nfull - 1 - s; };
  if (nfull > 0) load(block(0), va, la, ra);
  for (int s = 0; s < nfull; s += 2) {
    if (s + 1 < nfull) load(block(s + 1), vb, lb, rb);
    step(block(s), NB, va, la, ra);
    if (s + 1 < nfull) {
      if (s + 2 < nfull) load(block(s + 2), va, la, ra);
      step(block(s + 1), NB, vb, lb, rb);
    }
  }
  if (fwd && tail) {
    load_tail(va, la, ra);
    step(nfull, tail, va, la, ra);
  }
  __syncthreads();
}

// Both sweeps of the blocked form (fwd, bwd: the blocks; tmp: p doubles).
template <int NB, int U, int WMIN>
__device__ __forceinline__ void band_solve_blocks(const double* r, double* tmp, double* z, const double* fwd,
                                                  const double* bwd, int64_t p, int W, double* lds) {
  band_sweep_blocks<NB, U, WMIN>(r, tmp, fwd, p, W, true, lds);
  band_sweep_blocks<NB, U, WMIN>(tmp, z, bwd, p, W, false, lds);
}

// Cholesky factor of the assembled band: the register-panel factorization above
// when its window fits the band LDS (W <= 107), the blocked one with the trailing
// update in global memory otherwise.  256 threads; returns false in every thread
// when a pivot is not positive and finite.
__device__ inline bool band_factor(double* Lb, double* __restrict__ LbT, double* __restrict__ invd, int64_t p, int W,
                                   double* __restrict__ lds) {
  constexpr int NB = 8;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int br = band_blocks(W);
  if (br) {
    // the forward blocks that reach before the first element: zeros there
    const int64_t lead = (int64_t)((W - 2) / br + 1) * br;
    for (int64_t e = tid; e < (lead < p ? lead : p) * W; e += nt) LbT[e] = 0.0;
    const bool ok = br == 64   ? band_factor_panels<NB, 64>(Lb, LbT, invd, p, W, lds)
                    : br == 32 ? band_factor_panels<NB, 32>(Lb, LbT, invd, p, W, lds)
                               : band_factor_panels<NB, 16>(Lb, LbT, invd, p, W, lds);
    __syncthreads();  // the blocks' entries come from many threads (the panel loop's barriers order LDS only)
    if (ok) {
      if (br == 64)
        band_invert_blocks<64>(Lb, LbT, invd, p, W, lds);
      else if (br == 32)
        band_invert_blocks<32>(Lb, LbT, invd, p, W, lds);
      else
        band_invert_blocks<16>(Lb, LbT, invd, p, W, lds);
    }
    return ok;
  }
  const bool ok = W <= kPanelMaxW ? band_factor_panels<NB, 0>(Lb, LbT, invd, p, W, lds)
                                  : band_factor_blocked(Lb, LbT, invd, p, W, lds);
  // the rescale below reads invd (stored by lane 0) and LbT entries stored
  // by other threads: a full barrier orders those global stores (the panel
  // loop's barriers order LDS only)
  __syncthreads();
  if (ok) {  // rows of L scaled by their own 1/L_ii (the backward sweep's multipliers): a wave per row
    for (int64_t i = tid >> 6; i < p; i += nt >> 6) {
      const double s = invd[i];
      for (int k = 1 + (tid & 63); k < W; k += 64) LbT[i * W + k] *= s;
    }
    __syncthreads();
  }
  return ok;
}

// SC steps of the sweep by wave 0: elements t0 .. t0 + SC - 1, held in
// lanes lc0 .. lc0 + SC - 1 of ring register R0.  The staged multipliers
// already include 1/L_jj.  The dependent chain is one fma per step, on values
// every lane holds: bu = b_j (final), and the next element's final value
// b_{j+1} = pre - m b_j, where pre is b_{j+1} after the steps before j (read
// from its lane one step early) and m its multiplier at step j, which the
// lane of element j+1 already holds among the step's ring multipliers (a
// readlane, no LDS read on the chain).  The ring update - one fma per
// register - and those reads stay off that chain; the ring multipliers of a
// step are loaded DP steps ahead.  Elements j + 1, j + 2 live in register R0
// or, in the last two steps of a chunk, in the next ring register R1.
template <int NR, int SC, int R0>
__device__ __forceinline__ void band_steps(double (&reg)[NR], double& bu, double& pre, const double* __restrict__ buf,
                                           int lc0, int lane) {
  constexpr int R1 = (R0 + 1) % NR;
  constexpr int DP = SC < (NR <= 5 ? 4 : 2) ? SC : (NR <= 5 ? 4 : 2);  // steps of multipliers in flight
  double mq[DP][NR];
#pragma unroll
  for (int d = 0; d < DP; ++d)
#pragma unroll
    for (int r = 0; r < NR; ++r) mq[d][r] = buf[(d * NR + r) * 64 + lane];
#pragma unroll
  for (int l = 0; l < SC; ++l) {
    const int lc = lc0 + l;
    const int ln1 = (lc + 1) & 63, ln2 = (lc + 2) & 63;
    double(&mc)[NR] = mq[l % DP];
    const double m1 = readlane_f64(lc + 1 < 64 ? mc[R0] : mc[R1], ln1);
#pragma unroll
    for (int r = 0; r < NR; ++r) reg[r] = fma(-mc[r], bu, reg[r]);
    const double pre2 = readlane_f64(lc + 2 < 64 ? reg[R0] : reg[R1], ln2);
    bu = fma(-m1, bu, pre);
    pre = pre2;
    if (l + DP < SC) {
#pragma unroll
      for (int r = 0; r < NR; ++r) mc[r] = buf[((l + DP) * NR + r) * 64 + lane];
    }
  }
}

template <int NR, int SC, int R0>
__device__ __forceinline__ void band_steps_sw(int r0, double (&reg)[NR], double& bu, double& pre, const double* buf,
                                              int lc0, int lane) {
  if constexpr (R0 < NR) {
    if (r0 == R0)
      band_steps<NR, SC, R0>(reg, bu, pre, buf, lc0, lane);
    else
      band_steps_sw<NR, SC, R0 + 1>(r0, reg, bu, pre, buf, lc0, lane);
  }
}

// One triangular sweep: virtual step t handles element e(t) = t (forward,
// L y = b with the columns of L, Mul = Lb) or p - 1 - t (backward, L^T z = b
// with the rows of L, Mul = LbT); Mul[e(t)*W + k] (1 <= k < W) multiplies the
// element k steps ahead, which sits in ring slot (t + k) mod 64 NR.  Whole
// workgroup of 256 threads; stage: kBandLds doubles of LDS.  Ends with a
// barrier.
template <int NR, int SC>
__device__ __forceinline__ void band_sweep_t(const double* __restrict__ b, double* __restrict__ out, const double* __restrict__ Mul,
                             const double* __restrict__ invd, int64_t p, int W, bool fwd, double* __restrict__ stage) {
  constexpr int RS = 64 * NR;
  constexpr int BUF = SC * NR * 64;
  static_assert(2 * BUF <= kBandLds, "stage buffers exceed the LDS budget");
  static_assert(64 % SC == 0, "sub-chunks must tile a chunk");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t nsub = (p + SC - 1) / SC;
  auto elem = [&](int64_t t) { return fwd ? t : p - 1 - t; };
  // Waves 1..3 stage sub-chunk s: staging thread u owns the ring distances
  // k = u + NL c (c < KC) and, for each of the SC steps, loads the multiplier
  // at distance k (zero outside 1 <= k < W or past the end) and stores it into
  // the LDS row of that step at slot (t + k) mod RS.  Every slot of a row is
  // written, so stale values never survive.  All PER loads of a thread are
  // issued before any is written to LDS, one sub-chunk early (into pend), so
  // their latency hides behind wave 0's steps.
  constexpr int NL = kWG - 64;
  constexpr int KC = (RS + NL - 1) / NL;
  constexpr int PER = KC * SC;
  const int u = tid - 64;
  const int64_t rstep = fwd ? (int64_t)W : -(int64_t)W;
  double pend[PER];
  auto stage_load = [&](int64_t s) {
    const int64_t t0 = s * SC;
    const int64_t rem = p - t0;
    const int lim = rem < SC ? (int)rem : SC;
    const double* row = Mul + elem(t0) * (int64_t)W;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const int k = u + NL * c;
      const bool kin = k >= 1 && k < W;
#pragma unroll
      for (int l = 0; l < SC; ++l) pend[c * SC + l] = (kin && l < lim) ? row[l * rstep + k] : 0.0;
    }
  };
  auto stage_store = [&](double* buf, int64_t s) {
    const int rr0 = (int)((s * SC) % RS);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const int k = u + NL * c;
      if (k < RS) {
        int slot = rr0 + k;
        if (slot >= RS) slot -= RS;
#pragma unroll
        for (int l = 0; l < SC; ++l) {
          buf[l * RS + slot] = pend[c * SC + l];
          slot = slot + 1 == RS ? 0 : slot + 1;
        }
      }
    }
  };
  double reg[NR];
  double idv = 0.0, nb = 0.0, idv_nx = 0.0, nb_nx = 0.0;
  // 1/L_jj of a chunk's 64 steps and the 64 elements that enter the ring at
  // its end, loaded one chunk ahead
  auto load_chunk = [&](int64_t tc0, double& iv, double& nv) {
    const int64_t tc = tc0 + lane, tn = tc0 + RS + lane;
    iv = tc < p ? invd[elem(tc)] : 0.0;
    nv = tn < p ? b[elem(tn)] : 0.0;
  };
  double bu = 0.0, pre = 0.0;  // b of the current element (final) and of the next (before this step)
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int64_t t = r * 64 + lane;
      reg[r] = t < p ? b[elem(t)] : 0.0;
    }
    bu = readlane_f64(reg[0], 0);
    pre = readlane_f64(reg[0], 1);
    load_chunk(0, idv_nx, nb_nx);
  } else {
    stage_load(0);
    stage_store(stage, 0);
    if (nsub > 1) stage_load(1);
  }
  __syncthreads();
  for (int64_t s = 0; s < nsub; ++s) {
    double* cur = stage + (s & 1) * BUF;
    if (wave != 0) {
      if (s + 1 < nsub) stage_store(stage + ((s + 1) & 1) * BUF, s + 1);
      if (s + 2 < nsub) stage_load(s + 2);
    } else {
      const int64_t t0 = s * SC;
      const int r0 = (int)((t0 / 64) % NR);
      const int lc0 = (int)(t0 % 64);
      const int64_t tc0 = t0 - lc0;
      if (lc0 == 0) {
        idv = idv_nx;
        nb = nb_nx;
        load_chunk(tc0 + 64, idv_nx, nb_nx);
      }
      band_steps_sw<NR, SC, 0>(r0, reg, bu, pre, cur, lc0, lane);
      if (lc0 + SC == 64 || t0 + SC >= p) {
        // the chunk's slots hold their final right-hand sides: y = b / L_jj
        const int64_t tc = tc0 + lane;
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r == r0) {
            if (tc < p) out[elem(tc)] = reg[r] * idv;
            reg[r] = nb;
          }
      }
    }
    lds_barrier();  // the staging loads of the next sub-chunk stay in flight
  }
  __syncthreads();
}

template <int NR>
__device__ __forceinline__ void band_solve_nr(const double* r, double* tmp, double* z, const double* Lb,
                                              const double* LbT, const double* invd, int64_t p, int W, double* lds) {
  constexpr int SC = (2 * 32 * NR * 64 <= kBandLds) ? 32 : (2 * 16 * NR * 64 <= kBandLds) ? 16
                     : (2 * 8 * NR * 64 <= kBandLds) ? 8 : 4;
  band_sweep_t<NR, SC>(r, tmp, Lb, invd, p, W, true, lds);
  band_sweep_t<NR, SC>(tmp, z, LbT, invd, p, W, false, lds);
}

// z = M^-1 r = L^-T L^-1 r through tmp (p doubles).  Whole workgroup of 256
// threads; W <= kBandMaxW (checked on the host).  Ends with a barrier.
__device__ __forceinline__ void band_solve(const double* r, double* tmp, double* z, const double* Lb,
                                           const double* LbT, const double* invd, int64_t p, int W, double* lds) {
  switch (band_blocks(W)) {
    case 16: band_solve_blocks<16, 2, 16>(r, tmp, z, LbT, Lb, p, W, lds); return;
    case 32: band_solve_blocks<32, 8, 32>(r, tmp, z, LbT, Lb, p, W, lds); return;
    case 64:
      if (W <= 84)
        band_solve_blocks<64, 21, 64>(r, tmp, z, LbT, Lb, p, W, lds);
      else
        band_solve_blocks<64, 27, 84>(r, tmp, z, LbT, Lb, p, W, lds);
      return;
    default: break;
  }
  switch (band_nr(W)) {
    case 2: band_solve_nr<2>(r, tmp, z, Lb, LbT, invd, p, W, lds); break;
    case 3: band_solve_nr<3>(r, tmp, z, Lb, LbT, invd, p, W, lds); break;
    case 5: band_solve_nr<5>(r, tmp, z, Lb, LbT, invd, p, W, lds); break;
    case 8: band_solve_nr<8>(r, tmp, z, Lb, LbT, invd, p, W, lds); break;
    default: band_solve_nr<17>(r, tmp, z, Lb, LbT, invd, p, W, lds); break;
  }
}

}  // namespace flr

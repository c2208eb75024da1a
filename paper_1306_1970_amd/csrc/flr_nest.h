// M^-1 for graphs of index bandwidth bw >= 2 as a nested set of dense inverses
// (the exact preconditioner solve of Algorithm 2, section 3.1, for the single
// solves and the ragged batch).
//
// A banded triangular sweep is one dependent chain of p steps (57 ns each: 1.15
// ms per PCG step at p = 10^4, bw = 100, against 35 us for everything else).
// Here the index range is cut into S segments of m indexes with separators of
// bw indexes between them (segment s starts at s (m + bw)); no edge joins two
// segments, so with I the interiors and s the separators
//   z_s = T^-1 (r_s - W^T r_I),  T = M_ss - M_sI M_II^-1 M_Is,  W = M_II^-1 M_Is
//   z_I = M_II^-1 r_I - W z_s
// is three launches of matrix-vector products without any chain:
//   K1  M_II^-1 r_I and W^T r_I, segment by segment;  K2  T^-1 (..);  K3  z_I.
// S = 1 (no separators) leaves K1 alone.  The next A sums r^T z and r^T r.  S is
// chosen on the host by the bytes of one apply and the work of one factorization
// (nest_plan).
//
// The inverses come from the symmetric block sweep (Gauss-Jordan) with pivot
// blocks of 64 on the bordered segment matrices [M_II M_Is; M_sI 0], which
// turns them into [-M_II^-1 W; W^T -M_sI M_II^-1 M_Is], and then on T.  One
// launch per pivot block: every 64 x 64 tile of the lower triangle subtracts
// A_ik D A_jk^T (D = A_kk^-1) on v_mfma_f64_16x16x4f64; tiles of the next
// pivot column are also left in a panel buffer, and the workgroup of the next
// diagonal tile inverts it, so the next launch finds both ready.  The launches
// K1..K3 do one such stage each while the solve is in its factorization phase
// (PH_BANDMM), so the rotation needs no host decision.
//
// Accuracy: M is a symmetric M-matrix (positive diagonal, couplings -lambda2 w
// <= 0), and so is every Schur complement; off the diagonal the sweep only
// adds terms of one sign, so every entry of the inverses and of W has a
// relative error of a few ulp given the pivots, as in a Cholesky factorization,
// also where the weights reach 1/eps.  The products with the inverse are another
// matter: entries of its size ||M^-1|| hide its least eigenvalue 1 / ||M|| once the
// condition number comes near 2^53, where triangular solves still resolve it; such
// solves keep the band factor (nest_accurate in the engine).
//
// Measured (sweeps and factorization in one workgroup before -> here): the 100 x
// 100 lattice 1153 -> 26 us per PCG step and 10.2 -> 1.1 ms per factorization (the
// segment matrices are read once per step, 113 MB); 128 x 128
// 1875 -> 38 us and 76 -> 2.0 ms; 32 x 32 (S = 1) 114 -> 6 us and 0.95 -> 0.39 ms.
#pragma once
#include <utility>

#include "flr_device.h"

namespace flr {

constexpr int kNT = 512;          // threads of the K launches (8 wave64)
constexpr int kTile = 64;         // tile and pivot block
constexpr int kTE = kTile * kTile;
constexpr int kTLd = kTile + 4;   // LDS row stride of a tile (32-byte rows, 16 rows over distinct banks)
constexpr int kNestLds = 2 * kTile * kTLd;  // doubles: two tiles, 68 KiB, two workgroups per CU
constexpr int kTopCols = 16;      // columns of T^-1 per workgroup

typedef double nx4 __attribute__((ext_vector_type(4)));

// What the K launches read, in registers: taken field by field through the
// entry's pointer each use waits for its own scalar load (15 us more per round).
struct NestView {
  Nest nest;
  int64_t p;
  const int32_t* rowptr;
  const int32_t* col;
  const double* w;
  const double* d;
  const double* r;
  double* yv;
  double* btmp;
  unsigned* counter;
};
__host__ __device__ inline NestView nest_view(const Dims& D, const Bufs& B) {
  return {B.nest, D.p, B.rowptr, B.col, B.w, B.d, B.r, B.yv, B.btmp, B.counter};
}

__device__ __host__ inline int64_t nest_first(const Nest& Q, int s) { return (int64_t)s * (Q.m + Q.bw); }
__device__ __host__ inline int nest_rows(const Nest& Q, int64_t p, int s) {
  return s + 1 < Q.S ? Q.m : (int)(p - nest_first(Q, s));
}

// Local index of global index c in segment s's bordered matrix: interior, then
// the separator before it, then the one after it; -1 when it is in neither.
__device__ inline int nest_local(const Nest& Q, int64_t p, int s, int64_t c) {
  const int64_t o = c - nest_first(Q, s);
  if (o >= 0) {
    const int ms = nest_rows(Q, p, s);
    if (o < ms) return (int)o;
    return s + 1 < Q.S && o < Q.m + Q.bw ? Q.mt * kTile + Q.bw + (int)(o - Q.m) : -1;
  }
  return s > 0 && o >= -(int64_t)Q.bw ? Q.mt * kTile + (int)(o + Q.bw) : -1;
}
// Position of global index c among the separators, -1 for an interior index.
__device__ inline int nest_sep(const Nest& Q, int64_t c) {
  const int64_t s = c / (Q.m + Q.bw), o = c - s * (Q.m + Q.bw);
  return s + 1 < Q.S && o >= Q.m ? (int)(s * Q.bw + (o - Q.m)) : -1;
}
__device__ inline int64_t nest_sep_global(const Nest& Q, int a) {
  const int s = a / Q.bw;
  return nest_first(Q, s) + Q.m + (a - s * Q.bw);
}

// One pivot of the sweep of a 16 x 16 block held by one wave: lane l has row
// 4 (l & 3) + (l >> 2 & 3), columns 4 (l >> 4) .. + 3 (as the first operand of an
// FP64 MFMA).  The pivot row comes to every lane of its 16 by a row broadcast, the
// pivot column (by symmetry) from its lanes by permlane swaps: no LDS, no barrier.
template <int K>
__device__ __forceinline__ void nest_pivot(int lane, double (&x)[4], bool& ok) {
  constexpr int kg = K >> 2, kc = K & 3, at = 4 * kc + kg;  // the row's lane among 16
  double row[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) row[c] = dpp_f64<0x150 + at>(x[c]);  // row_newbcast
  const double piv = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x[kc]), 16 * kg + at),
                                      __builtin_amdgcn_readlane(__double2loint(x[kc]), 16 * kg + at));
  const auto l16 = __builtin_amdgcn_permlane16_swap(__double2loint(x[kc]), __double2loint(x[kc]), false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap(__double2hiint(x[kc]), __double2hiint(x[kc]), false, false);
  const auto l32 = __builtin_amdgcn_permlane32_swap(l16[kg & 1], l16[kg & 1], false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap(h16[kg & 1], h16[kg & 1], false, false);
  const double col = __hiloint2double((int)h32[kg >> 1], (int)l32[kg >> 1]);
  ok = ok && piv > 0.0 && isfinite(piv);
  const double d = 1.0 / piv;
  const bool mine = (lane & 15) == at;
  const double t = mine ? -d : col * d;
#pragma unroll
  for (int c = 0; c < 4; ++c) x[c] = fma(-t, row[c], mine ? 0.0 : x[c]);
  if ((lane >> 4) == kg) x[kc] = t;
}
template <int... K>
__device__ __forceinline__ void nest_sweep16(int lane, double (&x)[4], bool& ok, std::integer_sequence<int, K...>) {
  (nest_pivot<K>(lane, x, ok), ...);
}

// Inverse of the symmetric positive definite 64 x 64 tile in P (row stride kTLd;
// Q is a second such tile, both are overwritten), into out (row-major, ld 64): the
// sweep in pivot blocks of 16.  Wave 0 sweeps the diagonal block in its registers;
// then wave w forms blocks (w / 2, 2 (w & 1) + {0, 1}) of the result, A_ij - (A_ik D)
// A_kj, on the matrix cores, A_ik D as the transpose of D A_ki, whose layout is the
// second product's operand.  The chain of 64 pivots bounds it: with every pivot
// column published through LDS (a barrier and an LDS round trip each) 17 us, a stage
// of the 32 x 32 lattice 31, here 10 and 24; and the launches' registers, which that
// form set, went from 171 to 99 (K1 of the 100 x 100 lattice 16.5 -> 11.8 us).  *bad is set on a pivot that is not positive and finite.
__device__ inline void nest_invert(int tid, double* P, double* Q, double* __restrict__ out, unsigned* bad) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g4 = (lane >> 4) * 4, i16 = lane & 15, sig = 4 * (i16 & 3) + (i16 >> 2);
  const int i = wave >> 1;
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {
    const int kk = 16 * k * (kTLd + 1) + sig * kTLd + g4;  // this lane's part of the diagonal block
    if (wave == 0) {
      nx4 v = *reinterpret_cast<const nx4*>(P + kk);
      double x[4] = {v[0], v[1], v[2], v[3]};
      bool ok = true;
      nest_sweep16(lane, x, ok, std::make_integer_sequence<int, 16>());
      *reinterpret_cast<nx4*>(Q + kk) = nx4{x[0], x[1], x[2], x[3]};  // -D
      if (!ok && lane == 0) *bad = 1u;
    }
    __syncthreads();
    const nx4 d = *reinterpret_cast<const nx4*>(Q + kk);
    nx4 u = {0.0, 0.0, 0.0, 0.0};  // -(A_ik D)[i16][g4 ..]
    if (i != k) {
      const nx4 a = *reinterpret_cast<const nx4*>(P + (16 * i + i16) * kTLd + 16 * k + g4);
#pragma unroll
      for (int c = 0; c < 4; ++c) u = __builtin_amdgcn_mfma_f64_16x16x4f64(d[c], a[c], u, 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int j = 2 * (wave & 1) + b;
      if (i == k && j == k) continue;  // wave 0 has written it
      if (j == k) {
        *reinterpret_cast<nx4*>(Q + (16 * i + i16) * kTLd + 16 * k + g4) = -u;
        continue;
      }
      const nx4 a = *reinterpret_cast<const nx4*>(P + (16 * j + i16) * kTLd + 16 * k + g4);  // A_kj transposed
      if (i == k) {
        nx4 v = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < 4; ++c) v = __builtin_amdgcn_mfma_f64_16x16x4f64(d[c], a[c], v, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) Q[(16 * i + g4 + r) * kTLd + 16 * j + i16] = -v[r];
      } else {
        const int at = (16 * i + (lane >> 4)) * kTLd + 16 * j + i16;  // rows lane / 16 + 4 r
        nx4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = P[at + 4 * r * kTLd];
#pragma unroll
        for (int c = 0; c < 4; ++c) v = __builtin_amdgcn_mfma_f64_16x16x4f64(u[c], a[c], v, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) Q[at + 4 * r * kTLd] = v[r];
      }
    }
    __syncthreads();
    double* s = P;
    P = Q;
    Q = s;
  }
#pragma unroll
  for (int q = 0; q < kTE / kNT; ++q) {
    const int e = tid + kNT * q;
    out[e] = -P[(e >> 6) * kTLd + (e & 63)];
  }
}

// 64 x 64 product P[m][n] = sum_k A[m][k] Bm[n][k] of two LDS tiles: wave w
// owns rows 16 (w & 3) .., columns 32 (w >> 2) .. as two MFMA blocks; A rows are
// fed in the order 4 (i % 4) + i / 4, so that a lane ends up with four
// consecutive rows 4 (lane / 16) + r of column lane % 16 of each block.
__device__ inline void nest_product(int tid, const double* A, const double* Bm, nx4 (&acc)[2]) {
  const int lane = tid & 63, wave = tid >> 6;
  const int g4 = (lane >> 4) * 4, i16 = lane & 15, sig = 4 * (i16 & 3) + (i16 >> 2);
  const double* ar = A + ((wave & 3) * 16 + sig) * kTLd + g4;
  const double* b0 = Bm + ((wave >> 2) * 32 + i16) * kTLd + g4;
  const double* b1 = b0 + 16 * kTLd;
#pragma unroll 1  // unrolled, the operands of all four slices are loaded first and spill
  for (int h = 0; h < kTile / 16; ++h) {
    const nx4 av = *reinterpret_cast<const nx4*>(ar + 16 * h);
    const nx4 bv0 = *reinterpret_cast<const nx4*>(b0 + 16 * h), bv1 = *reinterpret_cast<const nx4*>(b1 + 16 * h);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[kk], bv0[kk], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[kk], bv1[kk], acc[1], 0, 0, 0);
    }
  }
}

// A contiguous 64 x 64 tile (ld 64) into registers, and from there into LDS.
__device__ inline void nest_load(int tid, const double* __restrict__ src, double2 (&v)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = reinterpret_cast<const double2*>(src)[(unsigned)tid + kNT * q];
}
__device__ inline void nest_put(int tid, double* dst, const double2 (&v)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = 2 * (tid + kNT * q);
    *reinterpret_cast<double2*>(dst + (e >> 6) * kTLd + (e & 63)) = v[q];
  }
}

// Tile (i, j) of segment s's bordered matrix from the weights, into LDS (zeroed
// here).  Every entry has an interior index on one side: the row for i < mt,
// the column for a border row; eight threads walk one such index's edges.
__device__ inline void nest_fill_seg(int tid, const NestView& B, double lam2, int s, int i, int j, double* A) {
  const Nest& Q = B.nest;
  for (int e = tid; e < kTile * kTLd; e += kNT) A[e] = 0.0;
  __syncthreads();
  if (j < Q.mt) {
    const bool border = i >= Q.mt;
    const int x = tid >> 3, lx = (border ? j : i) * kTile + x, ms = nest_rows(Q, B.p, s);
    if (lx < ms) {
      const int64_t g = nest_first(Q, s) + lx;
      for (int q = B.rowptr[g] + (tid & 7); q < B.rowptr[g + 1]; q += 8) {
        const int lc = nest_local(Q, B.p, s, B.col[q]);
        const int o = lc - (border ? i : j) * kTile;
        if (lc >= 0 && o >= 0 && o < kTile) A[border ? o * kTLd + x : x * kTLd + o] = -lam2 * B.w[q];
      }
      if (i == j && (tid & 7) == 0) A[x * kTLd + x] = B.d[g];
    } else if (i == j && (tid & 7) == 0) {
      A[x * kTLd + x] = 1.0;  // padding of the interior
    }
  }
  __syncthreads();
}

// Tile (i, j) of T = M_ss - M_sI M_II^-1 M_Is: the edges among separators plus
// the swept border blocks of the segments on either side.
__device__ inline void nest_fill_top(int tid, const NestView& B, double lam2, int i, int j, double* A) {
  const Nest& Q = B.nest;
  for (int e = tid; e < kTile * kTLd; e += kNT) A[e] = 0.0;
  __syncthreads();
  {
    const int x = tid >> 3, a = i * kTile + x;
    if (a < Q.nt) {
      const int64_t g = nest_sep_global(Q, a);
      for (int q = B.rowptr[g] + (tid & 7); q < B.rowptr[g + 1]; q += 8) {
        const int o = nest_sep(Q, B.col[q]) - j * kTile;  // -1 - 64 j < 0 for an interior index
        if (o >= 0 && o < kTile) A[x * kTLd + o] = -lam2 * B.w[q];
      }
      if (i == j && (tid & 7) == 0) A[x * kTLd + x] = B.d[g];
    } else if (i == j && (tid & 7) == 0) {
      A[x * kTLd + x] = 1.0;
    }
  }
  __syncthreads();
  // the border block of segment s, entry (x, y) of its 2 bw separator indexes
  auto border = [&](int s, int x, int y) {
    const int r = x >> 6 >= y >> 6 ? x : y, c = x >> 6 >= y >> 6 ? y : x;
    return B.nest.seg[((int64_t)s * Q.N + Q.mt * kTile + r) * Q.N + Q.mt * kTile + c];
  };
  for (int e = tid; e < kTE; e += kNT) {
    const int a = i * kTile + (e >> 6), b = j * kTile + (e & 63);
    if (a >= Q.nt || b >= Q.nt) continue;
    const int u = a / Q.bw, x = a - u * Q.bw, v = b / Q.bw, y = b - v * Q.bw;
    double add = 0.0;
    if (u == v)
      add = border(u, Q.bw + x, Q.bw + y) + border(u + 1, x, y);
    else if (u == v + 1)
      add = border(u, Q.bw + x, y);
    else if (v == u + 1)  // the upper half of a diagonal tile
      add = border(v, x, Q.bw + y);
    A[(e >> 6) * kTLd + (e & 63)] += add;
  }
  __syncthreads();
}

// One stage of the factorization: stage 0 assembles the segment matrices,
// 1 .. mt sweep their pivot blocks, then (S > 1) one assembles T and tt sweep
// it.  Workgroup wg of Q.wgs takes one tile of every Q.wgs; the next diagonal
// tiles, whose inversion is the longest item, come first, and every second round
// runs backwards, so that their workgroups get another tile last if at all (36
// tiles a side, 666 tiles: 40 us a stage with every round forwards, 31 so).
__device__ inline void nest_stage(const NestView& B, double lam2, int stage, int wg, double* lds) {
  const Nest& Q = B.nest;
  const bool top = stage > Q.mt;
  const int k = top ? stage - Q.mt - 2 : stage - 1;  // pivot block, -1: assembly
  const int nmat = top ? 1 : Q.S, nb = top ? Q.tt : Q.mt + Q.bt, np = top ? Q.tt : Q.mt;
  const int next = k + 1 < np ? k + 1 : -1;
  const unsigned ld = top ? Q.ntp : Q.N;
  const int ntile = nb * (nb + 1) / 2, nfirst = next >= 0 ? nmat : 0, rest = ntile - (next >= 0 ? 1 : 0);
  const double* pan0 = Q.pan + (int64_t)(k & 1) * Q.pans * kTE;
  double* pan1 = Q.pan + (int64_t)((k + 1) & 1) * Q.pans * kTE;
  const double* d0 = Q.dinv + (int64_t)(k & 1) * Q.S * kTE;
  double* d1 = Q.dinv + (int64_t)((k + 1) & 1) * Q.S * kTE;
  double *LA = lds, *LB = lds + kTile * kTLd;
  // whether block i of pivot column k can be nonzero (banded before it is swept)
  const int kb = (Q.bw + 63) / 64;
  auto reach = [&](int i) {
    if (top || i <= k) return true;
    if (i < Q.mt) return i - k <= kb;
    return (i - Q.mt) * kTile < Q.bw || k * kTile + 63 >= Q.m - Q.bw;
  };
  for (int round = 0;; ++round) {
    const int it = round * Q.wgs + (round & 1 ? Q.wgs - 1 - wg : wg);
    if (it >= nfirst + nmat * rest) break;
    // an opaque copy of the thread index: the addresses derived from it are formed
    // here and not kept for every case across the loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const unsigned lane = tid & 63, wave = tid >> 6;
    const unsigned m0 = (wave & 3) * 16 + (lane >> 4) * 4, n0 = (wave >> 2) * 32 + (lane & 15);
    int mat, i, j;
    if (it < nfirst) {
      mat = it;
      i = j = next;
    } else {
      mat = (it - nfirst) / rest;
      int t = (it - nfirst) - mat * rest;
      if (next >= 0 && t >= next * (next + 3) / 2) ++t;  // the next diagonal tile's own position
      i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
      while (i * (i + 1) / 2 > t) --i;
      while ((i + 1) * (i + 2) / 2 <= t) ++i;
      j = t - i * (i + 1) / 2;
    }
    // uniform (t went through floating point): bases in scalar registers
    mat = __builtin_amdgcn_readfirstlane(mat);
    i = __builtin_amdgcn_readfirstlane(i);
    j = __builtin_amdgcn_readfirstlane(j);
    double* A = (top ? Q.top : Q.seg + (int64_t)mat * Q.N * Q.N) + ((int64_t)i * kTile * ld + j * kTile);
    const double* pan = pan0 + (int64_t)mat * nb * kTE;
    const bool publish = next >= 0 && (i == next || j == next);
    const bool touched = k < 0 || next < 0 || (reach(i) && reach(j));
    if (!touched && !publish) continue;
    __syncthreads();  // the previous tile's LDS reads are done
    nx4 v[2];
    if (k < 0) {
      if (top)
        nest_fill_top(tid, B, lam2, i, j, LA);
      else
        nest_fill_seg(tid, B, lam2, mat, i, j, LA);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[b][r] = LA[(m0 + r) * kTLd + n0 + 16 * b];
      __syncthreads();
    } else if (i == k && j == k) {
      const double* d = d0 + (int64_t)mat * kTE;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[b][r] = -d[(m0 + r) * kTile + n0 + 16 * b];
    } else {
      if (i != k && j != k) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) v[b][r] = A[(m0 + r) * ld + n0 + 16 * b];
      }
      if (touched) {
        const double* d = d0 + (int64_t)mat * kTE;
        const double *pi = pan + (int64_t)i * kTE, *pj = pan + (int64_t)j * kTE;
        double2 ta[4], tb[4], tc[4];
        const bool two = i != k && j != k;
        nest_load(tid, i == k ? d : pi, ta);
        nest_load(tid, i == k ? pj : d, tb);
        nest_load(tid, pj, tc);
        nest_put(tid, LA, ta);
        nest_put(tid, LB, tb);
        __syncthreads();
        nx4 t[2] = {nx4{0.0, 0.0, 0.0, 0.0}, nx4{0.0, 0.0, 0.0, 0.0}};
        nest_product(tid, LA, LB, t);
        if (!two) {
          v[0] = t[0];
          v[1] = t[1];
        } else {
          __syncthreads();
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) LA[(m0 + r) * kTLd + n0 + 16 * b] = -t[b][r];
          nest_put(tid, LB, tc);
          __syncthreads();
          nest_product(tid, LA, LB, v);
        }
      }
    }
    if (touched) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) A[(m0 + r) * ld + n0 + 16 * b] = v[b][r];
        if (next < 0 && i > j && j < np) {  // the finished matrix is stored whole (column-wise products both ways)
          double* At = (top ? Q.top : Q.seg + (int64_t)mat * Q.N * Q.N) + ((int64_t)j * kTile * ld + i * kTile);
          *reinterpret_cast<nx4*>(At + ((n0 + 16 * b) * ld + m0)) = v[b];
        }
      }
    }
    if (publish) {
      double* pn = pan1 + (int64_t)mat * nb * kTE;
      if (i == j) {
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) LA[(m0 + r) * kTLd + n0 + 16 * b] = v[b][r];
        __syncthreads();
        nest_invert(tid, LA, LB, d1 + (int64_t)mat * kTE, B.counter + 32);
      } else if (j == next) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) (pn + (int64_t)i * kTE)[(m0 + r) * kTile + n0 + 16 * b] = v[b][r];
      } else {
#pragma unroll
        for (int b = 0; b < 2; ++b)
          *reinterpret_cast<nx4*>(pn + (int64_t)j * kTE + ((n0 + 16 * b) * kTile + m0)) = v[b];
      }
    }
  }
}

// sum_j A[j * ld + c] x[j], j < rows, for the CW columns that start at A: thread
// (c, stream) takes every (512 / CW)-th row, eight loads in flight; the streams'
// sums are added through LDS in order.  x is in LDS; the caller's barrier has
// made it visible.  The result is in threads 0 .. CW - 1.
template <int CW>
__device__ inline double nest_columns(const double* __restrict__ A, int ld, int rows, const double* x,
                                      double* red) {
  constexpr int NS = kNT / CW;
  const int c = threadIdx.x % CW, st = threadIdx.x / CW;
  unsigned a = st * (unsigned)ld + c;  // below 2^31 entries
  const unsigned step = NS * (unsigned)ld;
  double s0 = 0.0, s1 = 0.0;
  int j = st;
  for (; j + 7 * NS < rows; j += 8 * NS) {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = A[a + u * step];
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      s0 = fma(t[u], x[j + u * NS], s0);
      s1 = fma(t[u + 1], x[j + (u + 1) * NS], s1);
    }
    a += 8 * step;
  }
  {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = j + u * NS < rows ? A[a + u * step] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j + u * NS < rows) s0 = fma(t[u], x[j + u * NS], s0);
  }
  red[st * CW + c] = s0 + s1;
  __syncthreads();
  double v = 0.0;
  if (threadIdx.x < CW) {
#pragma unroll 8
    for (int q = 0; q < NS; ++q) v += red[q * CW + threadIdx.x];
  }
  return v;
}

// The item's share of r^T z and r^T r (threads 0 .. CW - 1 of wave 0 hold r, z).
__device__ inline void nest_partial(const Nest& Q, int at, double r, double z) {
  const double a = wave_sum(r * z), b = wave_sum(r * r);
  if (threadIdx.x == 0) {
    Q.part[2 * (int64_t)at] = a;
    Q.part[2 * (int64_t)at + 1] = b;
  }
}

template <int CW>
__device__ inline void nest_apply_segments(const NestView& B, int wg, double* lds) {
  const Nest& Q = B.nest;
  double *x = lds + kNT, *red = lds;
  const int per = Q.N / CW;
  for (int it = wg; it < Q.S * per; it += Q.wgs) {
    const int s = it / per, c0 = (it - s * per) * CW, ms = nest_rows(Q, B.p, s);
    const int64_t g0 = nest_first(Q, s);
    __syncthreads();
    for (int j = threadIdx.x; j < ms; j += kNT) x[j] = B.r[g0 + j];
    __syncthreads();
    const double v = nest_columns<CW>(Q.seg + (int64_t)s * Q.N * Q.N + c0, Q.N, ms, x, red);
    if (threadIdx.x < 64) {
      const int c = c0 + threadIdx.x;
      const bool mine = threadIdx.x < CW, in = mine && c < ms;
      if (Q.S == 1) {
        if (in) B.yv[c] = -v;
        nest_partial(Q, it, in ? x[c] : 0.0, in ? -v : 0.0);
      } else if (in) {
        B.btmp[g0 + c] = v;
      } else if (mine && c >= Q.mt * kTile) {
        Q.gpart[(int64_t)s * Q.bt * kTile + (c - Q.mt * kTile)] = v;
      }
    }
  }
}

__device__ inline void nest_apply_top(const NestView& B, int wg, double* lds) {
  const Nest& Q = B.nest;
  double *x = lds + kNT, *red = lds;
  if (wg >= Q.ntp / kTopCols) return;
  const int64_t bs = (int64_t)Q.bt * kTile;
  for (int a = threadIdx.x; a < Q.nt; a += kNT) {
    const int u = a / Q.bw, t = a - u * Q.bw;
    x[a] = B.r[nest_sep_global(Q, a)] - Q.gpart[u * bs + Q.bw + t] - Q.gpart[(u + 1) * bs + t];
  }
  __syncthreads();
  for (int it = wg; it < Q.ntp / kTopCols; it += Q.wgs) {
    const double v = nest_columns<kTopCols>(Q.top + it * kTopCols, Q.ntp, Q.nt, x, red);
    if (threadIdx.x < 64) {
      const int a = it * kTopCols + threadIdx.x;
      double r = 0.0, z = 0.0;
      if (threadIdx.x < kTopCols && a < Q.nt) {
        const int64_t g = nest_sep_global(Q, a);
        r = B.r[g];
        z = -v;
        B.yv[g] = z;
      }
      nest_partial(Q, it, r, z);
    }
    __syncthreads();
  }
}

template <int CW>
__device__ inline void nest_apply_back(const NestView& B, int wg, double* lds) {
  const Nest& Q = B.nest;
  double *x = lds + kNT, *red = lds;
  const int per = Q.mt * kTile / CW;
  for (int it = wg; it < Q.S * per; it += Q.wgs) {
    const int s = it / per, c0 = (it - s * per) * CW, ms = nest_rows(Q, B.p, s);
    const int64_t g0 = nest_first(Q, s);
    __syncthreads();
    for (int b = threadIdx.x; b < 2 * Q.bw; b += kNT) {  // the separators on either side (none at the ends)
      const bool left = b < Q.bw;
      const bool has = left ? s > 0 : s + 1 < Q.S;
      x[b] = has ? B.yv[left ? g0 - Q.bw + b : g0 + Q.m + (b - Q.bw)] : 0.0;
    }
    __syncthreads();
    const double v = nest_columns<CW>(Q.seg + ((int64_t)s * Q.N + Q.mt * kTile) * Q.N + c0, Q.N, 2 * Q.bw, x, red);
    if (threadIdx.x < 64) {
      const int c = c0 + threadIdx.x;
      double r = 0.0, z = 0.0;
      if (threadIdx.x < CW && c < ms) {
        r = B.r[g0 + c];
        z = -B.btmp[g0 + c] - v;
        B.yv[g0 + c] = z;
      }
      nest_partial(Q, Q.ntp / kTopCols + it, r, z);
    }
  }
}

}  // namespace flr

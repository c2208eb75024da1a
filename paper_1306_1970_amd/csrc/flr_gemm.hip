// FP64 matrix-core products of the lambda-grid solver (see flr_gemm.h).
//
// Tiling: a workgroup (4 wave64) owns a 64 x 64 output tile, each wave a
// 32 x 32 quarter computed as 2 x 2 blocks of v_mfma_f64_16x16x4f64 (WT = 2);
// where that leaves the chip idle, a 32 x 32 tile with one block per wave
// (WT = 1).  The reduction runs over K in tiles of 32 staged through LDS
// (double-buffered, one LDS barrier per tile); a tile's global loads are issued
// two tiles ahead, into two register sets, and stay in flight across the
// barriers.  The order of every output element's sum is the same in all of these.  Inside an MFMA the four reduction
// slots are fed by the four 16-lane groups of the wave; group g takes the
// reduction indices 4g .. 4g + 3 of a 16-wide slice over four consecutive
// instructions, so every lane reads its four operands as one contiguous
// 32-byte LDS load (A and B use the same assignment, so the sum is the same).
// X is widened to FP64 as it is staged, in its stored type.
//
// Workgroup ids are mapped to tiles so that the tiles of one row band of X
// (all column tiles of one split-K slice) land on the same XCD (dispatch is
// round-robin over the 8 XCDs by workgroup id), where they share X in L2.
// Each output element is a fixed-order sum that depends only on X and its own
// operand column, never on the batch size or on the column's slot.
#include <hip/hip_runtime.h>

#include "flr_device.h"
#include "flr_gemm.h"

namespace flr {

typedef double dx4 __attribute__((ext_vector_type(4)));

// E (8 or 4) consecutive stored elements widened to FP64 (16-byte loads, one of 8
// bytes for four bf16).
template <typename XT, int E>
__device__ inline void load_x(const XT* p, double (&v)[E]) {
  constexpr int V = XV<XT>::V;
  if constexpr (E >= V) {
#pragma unroll
    for (int q = 0; q < E / V; ++q) XV<XT>::cvt(load16(p + q * V), v + q * V);
  } else {
    const uint2 t = *reinterpret_cast<const uint2*>(p);
    v[0] = XV<XT>::lo(t.x);
    v[1] = XV<XT>::hi(t.x);
    v[2] = XV<XT>::lo(t.y);
    v[3] = XV<XT>::hi(t.y);
  }
}

template <int E>
__device__ inline void load_d(const double* p, double (&v)[E]) {
#pragma unroll
  for (int q = 0; q < E / 2; ++q) {
    const double2 t = *reinterpret_cast<const double2*>(p + 2 * q);
    v[2 * q] = t.x;
    v[2 * q + 1] = t.y;
  }
}

// TR = false: C (M = n) = X O, reduction over the columns of X, split over K
//             into nslice partial outputs.
// TR = true:  C (M = p_pad) = X^T U, reduction over the n rows of X.
// BX (with TR): the right operand is X as well, C = X^T X (the Gram matrix).
template <typename XT, bool TR, bool BX, int WT>
__global__ __launch_bounds__(256) void k_gemm_f64(GemmArgs g) {
  constexpr int MT = 32 * WT, NT = 32 * WT, KT = kGemmKT, LDK = KT + 2;
  constexpr int E = 4 * WT;  // elements of A and of B that a thread stages per tile
  __shared__ __align__(16) double As[2][MT * LDK];  // [m][k]
  __shared__ __align__(16) double Bs[2][NT * LDK];  // [n][k]
  const int T = g.tiles_m * g.tiles_n * g.nslice;
  const int per = (T + 7) / 8;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (t >= T) return;
  const int tn = t % g.tiles_n;
  const int rest = t / g.tiles_n;
  const int tm = rest % g.tiles_m;
  const int ts = rest / g.tiles_m;
  const int m0 = tm * MT, n0 = tn * NT;
  const int64_t kbase = (int64_t)ts * g.K;
  const XT* X = reinterpret_cast<const XT*>(g.X);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // staging: a thread loads E consecutive elements of A and of B per tile, along
  // K (rows of X, operand columns) or along M / N (eight threads per row of X)
  const int rk = tid / (KT / E), ck = (tid % (KT / E)) * E;  // row or column, first k
  const int kr = tid >> 3, cm = (tid & 7) * E;               // k, first m or n
  auto zero = [](double (&v)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = 0.0;
  };
  auto load_tile = [&](int kt, double (&ra)[E], double (&rb)[E]) {
    const int64_t k0 = kbase + (int64_t)kt * KT;
    if (!TR) {
      if (m0 + rk < g.M)
        load_x<XT, E>(X + (int64_t)(m0 + rk) * g.ldx + k0 + ck, ra);
      else
        zero(ra);
    } else {
      if (k0 + kr < g.K)
        load_x<XT, E>(X + (k0 + kr) * g.ldx + m0 + cm, ra);
      else
        zero(ra);
    }
    if (BX) {  // B(n, k) = X[k][n]
      if (k0 + kr < g.K)
        load_x<XT, E>(X + (k0 + kr) * g.ldx + n0 + cm, rb);
      else
        zero(rb);
    } else if (n0 + rk < g.N) {
      load_d<E>(g.Bm + (int64_t)(n0 + rk) * g.ldb + k0 + ck, rb);
    } else {
      zero(rb);
    }
  };
  auto store_tile = [&](int buf, const double (&ra)[E], const double (&rb)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) As[buf][TR ? (cm + e) * LDK + kr : rk * LDK + ck + e] = ra[e];
#pragma unroll
    for (int e = 0; e < E; ++e) Bs[buf][BX ? (cm + e) * LDK + kr : rk * LDK + ck + e] = rb[e];
  };

  const int wm = wave & 1, wn = wave >> 1;
  const int g4 = (lane >> 4) * 4, i16 = lane & 15;
  // The FP64 MFMA returns row i of its 16 x 16 block in lane group i % 4,
  // register i / 4.  Feeding A row sig(i) = 4 (i % 4) + i / 4 into MFMA row i
  // makes lane l hold the output rows 4 (l / 16) + r, r = 0..3: four
  // consecutive rows of one column, stored as one 32-byte write.
  const int sig = 4 * (i16 & 3) + (i16 >> 2);
  dx4 acc[WT][WT];
#pragma unroll
  for (int a = 0; a < WT; ++a)
#pragma unroll
    for (int b = 0; b < WT; ++b) acc[a][b] = dx4{0.0, 0.0, 0.0, 0.0};
  auto compute = [&](int buf) {
#pragma unroll
    for (int h = 0; h < KT / 16; ++h) {
      dx4 av[WT], bv[WT];
#pragma unroll
      for (int q = 0; q < WT; ++q) {
        av[q] = *reinterpret_cast<const dx4*>(&As[buf][((wm * WT + q) * 16 + sig) * LDK + h * 16 + g4]);
        bv[q] = *reinterpret_cast<const dx4*>(&Bs[buf][((wn * WT + q) * 16 + i16) * LDK + h * 16 + g4]);
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int a = 0; a < WT; ++a)
#pragma unroll
          for (int b = 0; b < WT; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a][kk], bv[b][kk], acc[a][b], 0, 0, 0);
    }
  };

  const int nk = (g.K + KT - 1) / KT;
  double ra0[E], rb0[E], ra1[E], rb1[E];
  load_tile(0, ra0, rb0);
  if (nk > 1) load_tile(1, ra1, rb1);
  store_tile(0, ra0, rb0);
  lds_barrier();
  for (int kt = 0; kt < nk; kt += 2) {
    if (kt + 2 < nk) load_tile(kt + 2, ra0, rb0);
    compute(0);
    if (kt + 1 < nk) store_tile(1, ra1, rb1);
    lds_barrier();
    if (kt + 1 >= nk) break;
    if (kt + 3 < nk) load_tile(kt + 3, ra1, rb1);
    compute(1);
    if (kt + 2 < nk) store_tile(0, ra0, rb0);
    lds_barrier();
  }
  // lane holds C[m = 4 (lane / 16) + r][n = lane % 16] of each 16 x 16 block (rows permuted above)
  double* Cs = g.C + (int64_t)ts * g.cslice;
#pragma unroll
  for (int a = 0; a < WT; ++a)
#pragma unroll
    for (int b = 0; b < WT; ++b) {
      const int n = n0 + (wn * WT + b) * 16 + i16;
      const int m = m0 + (wm * WT + a) * 16 + g4;
      if (n < g.N) *reinterpret_cast<dx4*>(Cs + (int64_t)n * g.ldc + m) = acc[a][b];
    }
}

template <typename XT, bool TR, bool BX, int WT>
static hipError_t launch_wt(GemmArgs g, hipStream_t st) {
  g.tiles_m = (g.M + 32 * WT - 1) / (32 * WT);
  g.tiles_n = (g.N + 32 * WT - 1) / (32 * WT);
  const int T = g.tiles_m * g.tiles_n * g.nslice;
  const int grid = 8 * ((T + 7) / 8);
  hipLaunchKernelGGL((k_gemm_f64<XT, TR, BX, WT>), dim3(grid), dim3(256), 0, st, g);
  return hipGetLastError();
}

// 64 x 64 tiles where there are at least as many as CUs; below that a K tile is
// bound by its latency, and a quarter of the work per workgroup on four times as
// many of them is faster (n = 601, p = 3001, 36 columns: X O and X^T U 37 and
// 35 us with 40 and 48 workgroups, 17 and 14 with 152 and 192).
template <typename XT, bool TR, bool BX = false>
static hipError_t launch_t(const GemmArgs& g, hipStream_t st) {
  const int64_t t64 = (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64) * g.nslice;
  return t64 >= 256 ? launch_wt<XT, TR, BX, 2>(g, st) : launch_wt<XT, TR, BX, 1>(g, st);
}

hipError_t launch_gram(int dtype, const GemmArgs& g, hipStream_t st) {
  switch (dtype) {
    case 0: return launch_t<double, true, true>(g, st);
    case 1: return launch_t<float, true, true>(g, st);
    default: return launch_t<uint16_t, true, true>(g, st);
  }
}

hipError_t launch_gemm_xo(int dtype, const GemmArgs& g, hipStream_t st) {
  switch (dtype) {
    case 0: return launch_t<double, false>(g, st);
    case 1: return launch_t<float, false>(g, st);
    default: return launch_t<uint16_t, false>(g, st);
  }
}

hipError_t launch_gemm_xtu(int dtype, const GemmArgs& g, hipStream_t st) {
  switch (dtype) {
    case 0: return launch_t<double, true>(g, st);
    case 1: return launch_t<float, true>(g, st);
    default: return launch_t<uint16_t, true>(g, st);
  }
}

}  // namespace flr

// X^T r on gfx950: h = X^T r (one or two right-hand sides) for column-major X
// stored FP32 / BF16 / FP64, accumulated in FP64.
//
// One wave per C adjacent columns streams the full column length: each lane
// loads 16 bytes of every column per step with non-temporal loads (X is read
// once per launch and should not displace the L2-resident right-hand side),
// one row step per lane in flight (a measured sweep over 1, 2, 4 steps on
// MI355X favoured 1), then a deterministic in-wave transpose reduction leaves
// column c's total in lane (64 / C) c.  With one right-hand side the stream
// runs best with as many waves as are resident at once (about 5 per SIMD):
// 4096 waves give 6.9 TB/s, 2048 5.9, and 8192 (1.6 rounds) 5.5-5.7, so C
// is the smallest of 2, 4, 8 that keeps p / C at or below 5120 (2 up to
// p = 10240; C = 2 beat 1, 4 and 8 on the 16384 x 8192 design).  With two,
// every wave re-reads both right-hand sides from L2 for its columns, and at
// small C that L2 traffic (at C = 2 twice the bytes of X) competes with X
// (logistic 32768 x 16384: 585 / 537 / 504 / 498 us per iteration at C = 2 /
// 4 / 8 / 16; 16 needs 254 VGPRs), while at large C small designs leave the
// grid short of waves (16384 x 8192: 5.6 TB/s at C = 8, 6.0 at C = 4): C is
// the smallest of 2, 4, 8 that keeps p / C at or below 2048 waves.  With
// all loads of a step issued together (below), C = 4 / 4096 waves and two
// row steps in flight stayed slower than C = 8, one step (345 / 325 vs 313
// us), and staging both right-hand sides in LDS per workgroup (one barrier
// per 1024-row tile) cost 380-440 us.
//
// Most designs with more columns than that (p > 10240 with one right-hand side,
// 4096 with two; gemv_lds_blocks has the rule) whose right-hand sides fit half of
// a compute unit's LDS run k_gemv_l instead: at most 512 workgroups of 8 waves,
// all resident, each with its own LDS copy of the right-hand sides, whose waves
// walk the columns two at a time.  The right-hand sides cost no L2 traffic, so two
// columns per wave suffice; a wave's start is paid once and not per eight columns,
// and the last round of workgroups, partly empty before, is gone.  A column's sum is formed in
// the same order, whatever C.  FP32, two right-hand sides: 2300 x 89989 134 ->
// 127 us (6.5 TB/s), 3000 x 20000 44.8 -> 38.4, 2000 x 8192 11.0 -> 9.9, 4460 x
// 4735 21.2 -> 19.0; one: 2300 x 89989 130 -> 124, BF16 10000 x 40000 148 -> 123.
// With C = 2 waves enough for one round (1000 x 4000) it is slower, 4.8 -> 5.2 us,
// and so it is with one right-hand side at p = 4735 (15.0 -> 16.4).
// Algorithmic bytes per launch: n*p*sizeof(X) + 8n per right-hand side + 8p
// per output.
#include <cstdlib>

#include "pr_device.h"

namespace pr {
namespace {
using namespace dev;

constexpr int kGemvWavesMax = 5120;  // waves of one resident round of the one-RHS kernel
constexpr int kGemvWaves2 = 2048;    // waves the two-RHS kernel aims for
// columns per wave, the smallest of 2, 4, 8 that keeps the grid within
// kGemvWavesMax waves (one right-hand side) or kGemvWaves2 (two)
inline int gemv_cols(int nrhs, int64_t p) {
  const int64_t wmax = nrhs == 1 ? kGemvWavesMax : kGemvWaves2;
  int c = 2;
  while (c < 8 && p > (int64_t)c * wmax) c *= 2;
  return c;
}

// Deterministic transpose reduction of C per-lane partial sums (one per
// column) over the 64 lanes: at each exchange over lane bit s (32, 16, ...)
// the lanes with that bit set keep the upper half of their columns and add
// their partner's, the others the lower half; once one column is left the
// plain butterfly finishes.  Column c's total ends in lane (64 / C) c.
template <int C>
__device__ __forceinline__ double reduce_cols(double (&v)[C]) {
  const int lane = lane_id();
  double cur[C];
#pragma unroll
  for (int i = 0; i < C; i++) cur[i] = v[i];
  int s = 32;
#pragma unroll
  for (int w = C; w > 1; w >>= 1, s >>= 1) {
    const bool hi = (lane & s) != 0;
#pragma unroll
    for (int i = 0; i < w / 2; i++) {
      const double send = hi ? cur[i] : cur[i + w / 2];
      const double keep = hi ? cur[i + w / 2] : cur[i];
      cur[i] = keep + __shfl_xor(send, s, 64);
    }
  }
#pragma unroll
  for (; s > 0; s >>= 1) cur[0] += __shfl_xor(cur[0], s, 64);
  return cur[0];
}

// g_N and the dom test of a node's iterate whose nonzeros (and only those)
// are listed in idx / val (ns entries, J1 and J0 entries flagged with
// kJ1Flag / kJ0Flag), for the node with parameters P, by one workgroup of NTH
// threads: theta = sum of the free |x_j|, the J1 sum of squares and the
// largest |x_j| off and on J0 in one block reduction (the dom test of the
// node step), then Algorithm 1 over the free magnitudes as the fixed point
// s <- (sum of the values <= s) / (kbar - #{q > s}) from s = theta / kbar,
// one block reduction per round (zeros of the free set change none of these
// sums).  Each pass loads eight entries per thread before using them.
// Writes S->gval and S->indom.  Runs as one extra workgroup of the X^T r
// product, which follows the column-list product of the same iterate and
// outlasts this evaluation.  The workgroup may have more threads than NTH: they
// take part in the barriers only, so the sums do not depend on its size.
template <int NTH>
__device__ void list_values(const NodeParams *__restrict__ P, const int32_t *__restrict__ idx,
                            const double *__restrict__ val, int ns, NodeState *S) {
  constexpr int NWS = NTH / 64;
  constexpr int U = 8;
  __shared__ double red[NWS * 4];
  const int kbar = P->kbar;
  const double M = P->M;
  const bool on = threadIdx.x < NTH;
  const int first = on ? (int)threadIdx.x : ns;
  double v[4] = {0.0, 0.0, 0.0, 0.0};  // theta, sum_{J1} x^2, max |x| off J0, max |x| on J0
  for (int t0 = first; t0 < ns; t0 += U * NTH) {
    int32_t it[U];
    double xv[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int t = t0 + u * NTH;
      it[u] = t < ns ? idx[t] : 0;
      xv[u] = t < ns ? val[t] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const double ax = fabs(xv[u]);
      if (it[u] & kJ0Flag) {
        v[3] = fmax(v[3], ax);
      } else {
        if (it[u] & kJ1Flag) v[1] += xv[u] * xv[u];
        else v[0] += ax;
        v[2] = fmax(v[2], ax);
      }
    }
  }
  v[0] = wave_sum(v[0]);
  v[1] = wave_sum(v[1]);
  v[2] = wave_max(v[2]);
  v[3] = wave_max(v[3]);
  if (on && lane_id() == 0) {
#pragma unroll
    for (int k = 0; k < 4; k++) red[wave_id() * 4 + k] = v[k];
  }
  __syncthreads();
  double theta = 0.0, sq = 0.0, gB = 0.0, g0 = 0.0;
  for (int w = 0; w < NWS; w++) {
    theta += red[w * 4];
    sq += red[w * 4 + 1];
    gB = fmax(gB, red[w * 4 + 2]);
    g0 = fmax(g0, red[w * 4 + 3]);
  }
  const double zt = 1e-9 * fmax(1.0, fmax(gB, g0));
  int ok = (g0 <= zt);
  if (isfinite(M) && gB > M * (1.0 + 1e-9)) ok = 0;
  if (kbar == 0) {
    if (theta > zt) ok = 0;
  } else if (isfinite(M) && theta > M * (double)kbar * (1.0 + 1e-9)) {
    ok = 0;
  }
  double a1 = 0.0;
  if (kbar > 0 && theta > 0.0) {
    const double K = (double)kbar;
    double sv = theta / K, prevK = 0.0;
    a1 = NAN;
    for (int round = 0; round <= kbar + 1; round++) {
      double r[3] = {0.0, 0.0, 0.0};  // #{q > s}, sum of q <= s, sum of q^2 over q > s
      for (int t0 = first; t0 < ns; t0 += U * NTH) {
        int32_t it[U];
        double xv[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          const int t = t0 + u * NTH;
          it[u] = t < ns ? idx[t] : kJ0Flag;  // past the list: skipped below
          xv[u] = t < ns ? val[t] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
          if (it[u] & (kJ1Flag | kJ0Flag)) continue;
          const double q = fabs(xv[u]);
          if (q > sv) {
            r[0] += 1.0;
            r[2] += q * q;
          } else {
            r[1] += q;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < 3; k++) r[k] = wave_sum(r[k]);
      __syncthreads();
      if (on && lane_id() == 0) {
#pragma unroll
        for (int k = 0; k < 3; k++) red[wave_id() * 3 + k] = r[k];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 3; k++) {
        double t = 0.0;
        for (int w = 0; w < NWS; w++) t += red[w * 3 + k];
        r[k] = t;
      }
      if (r[0] == prevK || r[0] >= K) {
        a1 = 0.5 * (r[2] + (K - r[0]) * sv * sv);
        break;
      }
      prevK = r[0];
      sv = fmin(sv, r[1] / (K - r[0]));
    }
  }
  if (threadIdx.x == 0) {
    S->gval = 0.5 * sq + a1;
    S->indom = ok;
  }
}


template <typename T, int NRHS, int C>
__global__ __launch_bounds__(kGemvThreads) void k_gemv_t(const T *__restrict__ X, int64_t n, int64_t p,
                                                         const double *__restrict__ r1,
                                                         const double *__restrict__ r2,
                                                         double *__restrict__ h1,
                                                         double *__restrict__ h2,
                                                         const int32_t *__restrict__ done,
                                                         const NodeParams *__restrict__ node, NodeState *S,
                                                         const int32_t *__restrict__ sidx,
                                                         const double *__restrict__ sval,
                                                         const int32_t *__restrict__ nlist,
                                                         const double *__restrict__ dsum, int nfin) {
  if (done && *done) return;
  // backtracking: a rejected trial needs no product (every wave takes the
  // node step's decision from the same sums)
  if (dsum && S->bt && S->iter > 0 && !bt_accept(bt_remainder(dsum, nfin), S->L, S->dxy, node->Lmax)) return;
  // with `node` the first workgroup (dispatched first) evaluates g_N of the
  // listed iterate; the product's workgroups follow it
  int bx = (int)blockIdx.x;
  if (node) {
    if (bx == 0) {
      list_values<kGemvThreads>(node, sidx, sval, *nlist, S);
      return;
    }
    bx--;
  }
  constexpr int VEC = XLoad<T>::VEC;
  const int lane = lane_id();
  const int64_t col0 = ((int64_t)bx * (kGemvThreads / 64) + wave_id()) * C;
  if (col0 >= p) return;
  const T *c[C];
#pragma unroll
  for (int q = 0; q < C; q++) {
    const int64_t cj = (col0 + q < p) ? col0 + q : p - 1;
    c[q] = X + cj * n;
  }
  double acc[NRHS][C];
#pragma unroll
  for (int h = 0; h < NRHS; h++)
#pragma unroll
    for (int q = 0; q < C; q++) acc[h][q] = 0.0;
  const int64_t step = 64 * VEC;
  int64_t i = (int64_t)lane * VEC;
  // With two right-hand sides every load of a step is issued before its first
  // use: the scheduling barrier keeps the compiler from sinking the
  // right-hand-side loads below the widening of the first X vector, which
  // made a step three dependent memory round trips (logistic 32768 x 16384:
  // 338 -> 312 us).  With one right-hand side the compiler's own order (X,
  // then the right-hand side once the first column has arrived) measured
  // faster: 316 vs 340 us on a 32768 x 16384 FP32 design, 89.8 vs 94.0 on
  // 16000 x 16000 BF16, equal on 16384 x 8192.
  // Of those loads the right-hand sides go first, fixed by a barrier of their own:
  // X first takes 3-6% longer in BF16 (1048576 x 128 1391 -> 1478 us, 16384 x 8192
  // 67.8 -> 71.3), 1% in FP32 with C < 8 (65536 x 1024 157 -> 160) and up to 8% in
  // FP64 (6000 x 40000 290 -> 312).  FP32 with C = 8 gains from X first where it
  // differs (6000 x 40000 178 -> 167, 8192 x 20000 128 -> 127).
  constexpr bool kRhsFirst = NRHS > 1 && !(C == 8 && std::is_same<T, float>::value);
  for (; i + VEC <= n; i += step) {
    typename XLoad<T>::raw_t xr[C];
    double rv[NRHS][VEC];
    if constexpr (kRhsFirst) {
      load_rhs<VEC>(r1, i, rv[0]);
      load_rhs<VEC>(r2, i, rv[NRHS - 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < C; q++) xr[q] = XLoad<T>::raw(c[q] + i);
    if constexpr (!kRhsFirst) {
      load_rhs<VEC>(r1, i, rv[0]);
      if (NRHS > 1) load_rhs<VEC>(r2, i, rv[NRHS - 1]);
    }
    if constexpr (NRHS > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < C; q++) {
      double xv[VEC];
      XLoad<T>::cvt(xr[q], xv);
#pragma unroll
      for (int h = 0; h < NRHS; h++)
#pragma unroll
        for (int e = 0; e < VEC; e++) acc[h][q] = fma(xv[e], rv[h][e], acc[h][q]);
    }
  }
  constexpr int LPC = 64 / C;  // lanes per column after the reduction
  const int64_t col = col0 + lane / LPC;
  const bool writer = (lane % LPC) == 0 && col < p;
  {
    double t = reduce_cols(acc[0]);
    if (writer) h1[col] = t;
  }
  if (NRHS > 1) {
    double t = reduce_cols(acc[NRHS - 1]);
    if (writer) h2[col] = t;
  }
}

// The same product for many columns and right-hand sides of at most
// kGemvLdsRows entries together (see the head of this file).
constexpr int kGemvLThreads = 512;
constexpr int kGemvLBlocks = 512;   // two workgroups per compute unit
constexpr int kGemvLdsRows = 10176; // 79.5 KB: two workgroups with list_values' sums share 160 KB

template <typename T, int NRHS>
__global__ __launch_bounds__(kGemvLThreads) void k_gemv_l(const T *__restrict__ X, int64_t n, int64_t p,
                                                          const double *__restrict__ r1,
                                                          const double *__restrict__ r2,
                                                          double *__restrict__ h1,
                                                          double *__restrict__ h2,
                                                          const int32_t *__restrict__ done,
                                                          const NodeParams *__restrict__ node, NodeState *S,
                                                          const int32_t *__restrict__ sidx,
                                                          const double *__restrict__ sval,
                                                          const int32_t *__restrict__ nlist,
                                                          const double *__restrict__ dsum, int nfin) {
  constexpr int VEC = XLoad<T>::VEC, C = 2, NWG = kGemvLThreads / 64;
  __shared__ __align__(16) double rl[kGemvLdsRows];
  if (done && *done) return;
  if (dsum && S->bt && S->iter > 0 && !bt_accept(bt_remainder(dsum, nfin), S->L, S->dxy, node->Lmax)) return;
  int bx = (int)blockIdx.x, nb = (int)gridDim.x;
  if (node) {
    if (bx == 0) {
      list_values<kGemvThreads>(node, sidx, sval, *nlist, S);
      return;
    }
    bx--;
    nb--;
  }
  for (int i = 2 * (int)threadIdx.x; i < (int)n; i += 2 * kGemvLThreads) {
    *reinterpret_cast<d2_t *>(rl + i) = *reinterpret_cast<const d2_t *>(r1 + i);
    if (NRHS > 1) *reinterpret_cast<d2_t *>(rl + n + i) = *reinterpret_cast<const d2_t *>(r2 + i);
  }
  __syncthreads();
  const int lane = lane_id();
  const int64_t step = 64 * VEC;
  for (int64_t col0 = ((int64_t)bx * NWG + wave_id()) * C; col0 < p; col0 += (int64_t)nb * NWG * C) {
    const T *c[C];
#pragma unroll
    for (int q = 0; q < C; q++) c[q] = X + ((col0 + q < p) ? col0 + q : p - 1) * n;
    double acc[NRHS][C];
#pragma unroll
    for (int h = 0; h < NRHS; h++)
#pragma unroll
      for (int q = 0; q < C; q++) acc[h][q] = 0.0;
    for (int64_t i = (int64_t)lane * VEC; i + VEC <= n; i += step) {
      typename XLoad<T>::raw_t xr[C];
      double rv[NRHS][VEC];
#pragma unroll
      for (int q = 0; q < C; q++) xr[q] = XLoad<T>::raw(c[q] + i);
      load_rhs<VEC>(rl, i, rv[0]);
      if (NRHS > 1) load_rhs<VEC>(rl + n, i, rv[NRHS - 1]);
#pragma unroll
      for (int q = 0; q < C; q++) {
        double xv[VEC];
        XLoad<T>::cvt(xr[q], xv);
#pragma unroll
        for (int h = 0; h < NRHS; h++)
#pragma unroll
          for (int e = 0; e < VEC; e++) acc[h][q] = fma(xv[e], rv[h][e], acc[h][q]);
      }
    }
    const int64_t col = col0 + (lane >> 5);
    const bool writer = (lane & 31) == 0 && col < p;
    {
      const double t = reduce_cols(acc[0]);
      if (writer) h1[col] = t;
    }
    if (NRHS > 1) {
      const double t = reduce_cols(acc[NRHS - 1]);
      if (writer) h2[col] = t;
    }
  }
}

// Workgroups of k_gemv_l (at most cap, the number resident at once), or 0 where
// k_gemv_t is the faster one.  A workgroup takes 16 columns a round; `fit` is the
// part of its rounds that the whole grid fills.  Measured as k_gemv_t -> k_gemv_l in
// us, one or two right-hand sides:
// - Columns of fewer than four row steps of a wave (1 KiB each) do not repay the
//   start of a resident workgroup while C = 4 gives k_gemv_t enough waves: one, FP32
//   256 x 16385 4.6 -> 5.5, BF16 256 x 10241 3.8 -> 4.7; two, FP32 256 x 8192 3.7 -> 4.0.
//   With four (FP32 n = 1024) it is 13.8 -> 12.1 at p = 16384, 6.7 -> 6.4 at 5000.
// - With one right-hand side two steps, and in FP64 at least that many, repay it on
//   rounds that are filled: FP32 960 x 14000 (fit 0.85) 10.6 -> 9.2, FP64 1024 x 14000
//   20.9 -> 18.0, but 896 x 18000 (0.73) 19.3 -> 19.7, BF16 1024 x 20480 (0.83) 8.7 -> 9.0.
// - With C = 8, one right-hand side always gains (FP32 2048 x 65536 93.7 -> 79.6).
//   Two do on full rounds (FP32 2048 x 18000 34.9 -> 24.8), but not on half-empty
//   ones (FP32 1024 x 8193, fit 0.5: 8.7 -> 9.5, 5088 x 8193 29.4 -> 32.9; so is p =
//   8192 where the list has a workgroup: iterations of 5040 x 8192 in FP64 +5%).
// - A grid of equal rounds leaves compute units idle there.  Columns of few steps, and
//   BF16, whose bound is not the memory, run faster on all of them with rounds of
//   unequal length: BF16 512 x 16385 8.1 -> 9.1 with equal rounds, 7.0 so, 5088 x
//   16385 35.0 -> 37.4 and 29.0; FP64 2048 x 10241 36.2 -> 31.8 and 37.3.
// - Columns 32 KiB apart lie on the same memory channels, and waves that start
//   together walk them together (k_gemv_t's waves do not): one, FP32 8192 x 16384
//   96 -> 116, 8192 x 12000 80 -> 88; two, FP64 4096 x 16384 99 -> 111.  16 KiB apart
//   it is 3% on average with C = 4 (one, FP32 4096 x 12000 47.3 -> 50.1) and a gain with
//   C = 8; 4 KiB apart 3% in FP32 from p = 65536 on with two.  48 and 64 KiB are no
//   worse than others.
unsigned gemv_lds_blocks(int32_t xdt, bool two, int64_t n, int64_t p, int cols, int64_t cap) {
  if (cols <= 2 || n * (two ? 2 : 1) > kGemvLdsRows) return 0;
  const int64_t size = xdt == kF64 ? 8 : (xdt == kF32 ? 4 : 2), step = 1024 / size, stride = n * size;
  if (stride == 32768 || (!two && xdt == kF32 && llabs(stride - 32768) <= 512)) return 0;
  if ((stride == 16384 && cols == 4) || (two && xdt == kF32 && stride == 4096 && p >= 65536)) return 0;
  const bool few = n < 4 * step;
  const int64_t need = (p + 15) / 16, rounds = (need + cap - 1) / cap;
  const double fit = (double)need / (double)(rounds * cap);
  const bool filled = !two && n >= 2 * step && fit >= 0.84;
  if (cols == 4 && (few || (!two && xdt == kF64)) && !filled) return 0;
  if (two && (few || xdt == kBF16)) return (unsigned)(need < cap ? need : cap);
  if (two && rounds > 1 && fit < 0.6) return 0;
  return (unsigned)((need + rounds - 1) / rounds);
}

}  // namespace

hipError_t launch_gemv_t(const Problem &P, const double *r1, const double *r2, double *h1, double *h2,
                         const int32_t *done, hipStream_t s, const NodeParams *node, NodeState *S,
                         const int32_t *sidx, const double *sval, const int32_t *nlist, const double *dsum,
                         int32_t nfin) {
  if (node && (!S || !sidx || !sval || !nlist)) return hipErrorInvalidValue;
  if (dsum && !node) return hipErrorInvalidValue;
  const bool two = (r2 != nullptr);
  const int cols = gemv_cols(two ? 2 : 1, P.p);
  // the list's workgroup is one of those resident at once
  if (const unsigned wgs = gemv_lds_blocks(P.xdt, two, P.n, P.p, cols, kGemvLBlocks - (node ? 1 : 0))) {
    const unsigned lgrid = wgs + (node ? 1u : 0u);
#define PR_GEMVL(T, R)                                                                                              \
  k_gemv_l<T, R><<<lgrid, kGemvLThreads, 0, s>>>((const T *)P.X, P.n, P.p, r1, r2, h1, h2, done, node, S, sidx, sval, \
                                                 nlist, dsum, nfin)
    switch (P.xdt) {
      case kF32:
        if (two) PR_GEMVL(float, 2);
        else PR_GEMVL(float, 1);
        break;
      case kF64:
        if (two) PR_GEMVL(double, 2);
        else PR_GEMVL(double, 1);
        break;
      default:
        if (two) PR_GEMVL(uint16_t, 2);
        else PR_GEMVL(uint16_t, 1);
        break;
    }
#undef PR_GEMVL
    return hipGetLastError();
  }
  const int cols_per_block = (kGemvThreads / 64) * cols;
  dim3 grid((unsigned)((P.p + cols_per_block - 1) / cols_per_block) + (node ? 1u : 0u));
  dim3 block(kGemvThreads);
#define PR_GEMVT(T, R, C)                                                                                \
  k_gemv_t<T, R, C><<<grid, block, 0, s>>>((const T *)P.X, P.n, P.p, r1, r2, h1, h2, done, node, S, sidx, sval, \
                                           nlist, dsum, nfin)
#define PR_GEMVT1(T, R)                \
  switch (cols) {                      \
    case 2: PR_GEMVT(T, R, 2); break;  \
    case 4: PR_GEMVT(T, R, 4); break;  \
    default: PR_GEMVT(T, R, 8); break; \
  }
  switch (P.xdt) {
    case kF32:
      if (two) PR_GEMVT1(float, 2)
      else PR_GEMVT1(float, 1)
      break;
    case kF64:
      if (two) PR_GEMVT1(double, 2)
      else PR_GEMVT1(double, 1)
      break;
    default:
      if (two) PR_GEMVT1(uint16_t, 2)
      else PR_GEMVT1(uint16_t, 1)
      break;
  }
#undef PR_GEMVT1
#undef PR_GEMVT
  return hipGetLastError();
}

}  // namespace pr

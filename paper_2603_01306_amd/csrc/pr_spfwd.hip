// Column-list GEMV on gfx950: u = sum_t X[:, idx[t]] val[t] over the support
// of the iterate (or all columns), FP64 accumulation, followed by the loss
// epilogue of the solver.  Two kernels:
//
// k_spfwd_part  grid = row blocks x column chunks.  The list entries of a
//               chunk are wave-uniform, so column bases live in scalar
//               registers and every lane keeps 16 independent 16-byte
//               non-temporal loads in flight (2 to 8 rows per lane),
//               converted to FP64 at the FMA; the chunk's last columns form
//               one masked round of 4, 8 or 16.  Writes its partial sums to
//               part[chunk][n].
// k_spfwd_final grid over rows: sums the chunk partials in chunk order (so the
//               result does not depend on scheduling) and runs the epilogue:
//   least squares: r = y - u, F = ||r||^2, -F*(-zeta) = 2 r^T y - ||r||^2;
//   logistic:      zeta = y sigma(-y u), F, binary entropies, and the gradient
//                  at the momentum point (1+m)u - m u_prev;
//   Gram (least squares with X^T X held in memory): the "matrix" is G = X^T X
//                  and y holds b = X^T y, so the kernel writes h = b - G x.
// Bytes per launch pair: |list| * n * sizeof(X) + 16 * nch * n (partials)
// + the epilogue vectors.
#include "pr_device.h"

namespace pr {
namespace {
using namespace dev;

constexpr int kSpInFlight = 16;   // columns in flight per lane
constexpr int kFinThreads = 128;  // 2 waves: twice the workgroups of 256, more CUs on the partial planes
constexpr int kFinRows = 2;       // rows per thread in the finalize kernel

// 16 raw bytes of X and their FP64 value e (exact upcast)
template <typename T>
struct XRaw;
template <>
struct XRaw<float> {
  static constexpr int VEC = 4;
  __device__ __forceinline__ static double at(const u4_t &r, int e) { return (double)__uint_as_float(r[e]); }
};
template <>
struct XRaw<double> {
  static constexpr int VEC = 2;
  __device__ __forceinline__ static double at(const u4_t &r, int e) {
    return __hiloint2double((int)r[2 * e + 1], (int)r[2 * e]);
  }
};
template <>
struct XRaw<uint16_t> {
  static constexpr int VEC = 8;
  __device__ __forceinline__ static double at(const u4_t &r, int e) {
    const unsigned int w = r[e >> 1];
    return (double)__uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};

// The chunk's last, partial round: list entries t .. t1 - 1, at most U columns
// (16 bytes per lane each) loaded together; the slots at or past t1 re-read the
// chunk's last column and are weighted by zero.  A sparse iterate leaves few
// columns per chunk, so the rounds come in three sizes (16 slots for one column:
// 1% slower on a 4460 x 4735 child and on the 500 x 200 root; 24 or 32 columns in
// flight 1-3% slower on both and on the 16384 x 8192 root).
template <typename T, int U>
__device__ __forceinline__ void sp_tail(double (&acc)[XRaw<T>::VEC], const T *__restrict__ X, int64_t n, int64_t row0,
                                        const int32_t *__restrict__ idx, const double *__restrict__ val, int t, int t1) {
  u4_t raw[U];
#pragma unroll
  for (int c = 0; c < U; c++) {
    const int tc = (t + c < t1) ? t + c : t1 - 1;
    const T *col = X + (int64_t)(idx[tc] & kIdxMask) * n;   // wave-uniform column base
    raw[c] = __builtin_nontemporal_load(reinterpret_cast<const u4_t *>(col + row0));
  }
#pragma unroll
  for (int c = 0; c < U; c++) {
    const double w = (t + c < t1) ? val[t + c < t1 ? t + c : t1 - 1] : 0.0;
#pragma unroll
    for (int e = 0; e < XRaw<T>::VEC; e++) acc[e] = fma(XRaw<T>::at(raw[c], e), w, acc[e]);
  }
}

template <typename T>
__device__ __forceinline__ void sp_use_r(const u4_t (&raw)[kSpInFlight], double (&acc)[XRaw<T>::VEC],
                                         const double *__restrict__ val, int t) {
#pragma unroll
  for (int c = 0; c < kSpInFlight; c++) {
    const double w = val[t + c];
#pragma unroll
    for (int e = 0; e < XRaw<T>::VEC; e++) acc[e] = fma(XRaw<T>::at(raw[c], e), w, acc[e]);
  }
}

template <typename T>
__global__ __launch_bounds__(kSpThreads) void k_spfwd_part(const T *__restrict__ X, int64_t n, ProbBufs B,
                                                           const int32_t *__restrict__ idx,
                                                           const double *__restrict__ val,
                                                           const int32_t *__restrict__ nlist,
                                                           const NodeState *S) {
  constexpr int VEC = XRaw<T>::VEC;
  // both loads issued before the stop test waits
  const int done = S ? S->done : 0;
  const int ns = *nlist;
  if (done) return;
  const int rb = blockIdx.x, ch = blockIdx.y;
  const int cs = (ns + B.nch - 1) / B.nch;
  const int t0 = ch * cs;
  const int t1 = (t0 + cs < ns) ? t0 + cs : ns;
  const int64_t row0 = (int64_t)rb * B.rows + (int64_t)threadIdx.x * VEC;
  if (row0 >= n) return;
  double acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; e++) acc[e] = 0.0;
  // full rounds of kSpInFlight columns, then the chunk's remaining columns as
  // one masked round (all its loads in flight together)
  int t = t0;
  if (t + kSpInFlight <= t1) {
    // the next round's column indices are loaded while this round's columns
    // stream, so a round does not start with a wait on its own indices
    // (root solves 0.7-0.9% faster; issuing the next round's column loads
    // ahead of this round's arithmetic from two load buffers gained nothing)
    int32_t ci[kSpInFlight];
#pragma unroll
    for (int c = 0; c < kSpInFlight; c++) ci[c] = idx[t + c];
    for (;;) {
      u4_t raw[kSpInFlight];
#pragma unroll
      for (int c = 0; c < kSpInFlight; c++)
        raw[c] = __builtin_nontemporal_load(
            reinterpret_cast<const u4_t *>(X + (int64_t)(ci[c] & kIdxMask) * n + row0));
      const int tn = t + kSpInFlight;
      const bool more = tn + kSpInFlight <= t1;
      if (more) {
#pragma unroll
        for (int c = 0; c < kSpInFlight; c++) ci[c] = idx[tn + c];
      }
      sp_use_r<T>(raw, acc, val, t);
      t = tn;
      if (!more) break;
    }
  }
  if (t1 - t > 8) sp_tail<T, kSpInFlight>(acc, X, n, row0, idx, val, t, t1);
  else if (t1 - t > 4) sp_tail<T, 8>(acc, X, n, row0, idx, val, t, t1);
  else if (t < t1) sp_tail<T, 4>(acc, X, n, row0, idx, val, t, t1);
  double *part = B.part + (int64_t)ch * n + row0;
#pragma unroll
  for (int e = 0; e < VEC; e += 2) *reinterpret_cast<d2_t *>(part + e) = d2_t{acc[e], acc[e + 1]};
}

// U planes from c0 on of two rows, every load in flight together; those past
// the end re-read the last plane (add_planes leaves them out).
template <int U>
__device__ __forceinline__ void load_planes(d2_t (&pv)[U], const double *__restrict__ part, int c0, int nch, int64_t n) {
  static_assert(kFinRows == 2, "one 16-byte load per plane");
#pragma unroll
  for (int q = 0; q < U; q++) {
    const int c = c0 + q < nch ? c0 + q : nch - 1;
    pv[q] = *reinterpret_cast<const d2_t *>(part + (int64_t)c * n);
  }
}
template <int U>
__device__ __forceinline__ void add_planes(const d2_t (&pv)[U], int c0, int nch, double (&u)[kFinRows]) {
#pragma unroll
  for (int q = 0; q < U; q++) {
    if (c0 + q < nch) {
      u[0] += pv[q].x;
      u[1] += pv[q].y;
    }
  }
}

// Bound by latency (a few dozen workgroups, one dependent chain each): the
// node state, the first PL planes and the rows' vectors are loaded together
// before the stop test is waited for, and the planes are added in chunk order.
// PL = 32 where there are more than 16 chunks.  (Loads behind the stop test and
// the state, 8 planes at a time and the remainder one by one took 6.6 us on the
// 52 planes of a 4460 x 4735 design, this 5.6; 16 planes 5.75.)
template <int PL>
__global__ __launch_bounds__(kFinThreads) void k_spfwd_final(int64_t n, const double *__restrict__ y, ProbBufs B,
                                                             int32_t mode, const NodeState *S, double *u_out) {
  constexpr int VEC = kFinRows;
  __shared__ double red[(kFinThreads / 64) * 4];
  const int fb = blockIdx.x;
  const int64_t row0 = ((int64_t)fb * kFinThreads + threadIdx.x) * VEC;
  const bool active = row0 < n;
  const int64_t rowc = active ? row0 : 0;
  int done = 0, improved = 0, bt = 0, acc = 0;
  double mp = 0.0, t = 1.0;
  if (S) {
    done = S->done;
    improved = S->improved;
    bt = S->bt;
    acc = S->bt_acc;
    mp = S->mom;
    t = S->t;
  }
  const double *part = B.part + rowc;
  const int nch = B.nch;
  d2_t pv[PL];
  load_planes<PL>(pv, part, 0, nch, n);
  const bool loss = mode == kSpLogistic || mode == kSpLsq;
  double yv[VEC], ro[VEC], uo[VEC], up[VEC], uyo[VEC];
#pragma unroll
  for (int e = 0; e < VEC; e++) {
    yv[e] = mode != kSpPlain ? y[rowc + e] : 0.0;
    ro[e] = loss ? B.r[rowc + e] : 0.0;
    uo[e] = loss ? B.ucur[rowc + e] : 0.0;
    up[e] = loss ? B.uprev[rowc + e] : 0.0;
    uyo[e] = loss ? B.uy[rowc + e] : 0.0;
  }
  __builtin_amdgcn_sched_barrier(0);
  if (done) return;
  double u[VEC];
#pragma unroll
  for (int e = 0; e < VEC; e++) u[e] = 0.0;
  add_planes<PL>(pv, 0, nch, u);
  for (int c = PL; c < nch; c += PL) {
    load_planes<PL>(pv, part, c, nch, n);
    add_planes<PL>(pv, c, nch, u);
  }
  double sums[3] = {0.0, 0.0, 0.0};
  if (mode == kSpPlain) {
    if (active)
#pragma unroll
      for (int e = 0; e < VEC; e++) u_out[row0 + e] = u[e];
    return;
  }
  if (mode == kSpGram) {
    // the product is G x over the Gram matrix and y holds b = X^T y: h = b - G x
    if (active)
#pragma unroll
      for (int e = 0; e < VEC; e++) B.h1[row0 + e] = yv[e] - u[e];
    return;
  }
  if (mode == kSpLsq) {
    // backtracking: X y of the pending trial as in the logistic branch below,
    // and its model-test remainder ||X x - X y||^2 row by row
    if (active) {
#pragma unroll
      for (int e = 0; e < VEC; e++) {
        const int64_t i = row0 + e;
        if (improved) B.zbest[i] = 2.0 * ro[e];
        const double yi = yv[e];
        const double ri = yi - u[e];
        B.r[i] = ri;
        sums[0] += ri * ri;
        sums[1] += 2.0 * ri * yi - ri * ri;
        if (bt) {
          double uyv = uyo[e];
          if (acc) {
            uyv = (1.0 + mp) * uo[e] - mp * up[e];
            B.uy[i] = uyv;
            B.uprev[i] = uo[e];
          }
          B.ucur[i] = u[e];
          const double du = u[e] - uyv;
          sums[2] += du * du;
        }
      }
    }
  } else {
    const double mt = (t - 1.0) / fista_next_t(t);
    // backtracking: uprev holds X x of the last accepted iterate; when the
    // previous evaluation was accepted it moves there and the momentum point
    // y of the pending trial, X y = (1 + m) X x_k - m X x_{k-1} (m the step's
    // momentum, 0 after a restart), is kept in uy until the trial is decided
    if (active) {
#pragma unroll
      for (int e = 0; e < VEC; e++) {
        const int64_t i = row0 + e;
        double upv = uo[e], uyv = uyo[e];
        if (bt) {
          upv = up[e];
          if (acc) {
            uyv = (1.0 + mp) * uo[e] - mp * upv;
            B.uy[i] = uyv;
            upv = uo[e];
            B.uprev[i] = upv;
          }
        } else {
          B.uprev[i] = uo[e];
        }
        B.ucur[i] = u[e];
        if (improved) B.zbest[i] = ro[e];
        const double yi = yv[e];
        const double z = yi * u[e];
        const double a = 1.0 / (1.0 + exp(z));
        B.r[i] = yi * a;
        sums[0] += softplus(-z);
        sums[1] += a * softplus(z) + (1.0 - a) * softplus(-z);
        if (bt) {
          // F(X x) - F(X y) - <grad F(X y), X x - X y> of this row, with
          // a = -y_i (X y)_i and d = -y_i (X x - X y)_i: log1p(s expm1(d)) - s d,
          // s = 1 / (1 + exp(-a))
          const double aa = -yi * uyv, dd = -yi * (u[e] - uyv);
          const double sg = 1.0 / (1.0 + exp(-aa));
          sums[2] += log1p(sg * expm1(dd)) - sg * dd;
        }
        const double sm = (1.0 + mt) * u[e] - mt * upv;
        B.gm[i] = -yi / (1.0 + exp(yi * sm));
      }
    }
  }
  block_sum<kFinThreads, 3>(sums, red);
  if (threadIdx.x == 0) {
    B.rbsum[2 * fb] = sums[0];
    B.rbsum[2 * fb + 1] = sums[1];
    if (B.dsum) B.dsum[fb] = sums[2];
  }
}

}  // namespace

hipError_t launch_spfwd(const Problem &P, const ProbBufs &B, const int32_t *idx, const double *val,
                        const int32_t *nlist, int32_t mode, const NodeState *S, double *u_out,
                        hipStream_t s) {
  dim3 grid((unsigned)B.rb, (unsigned)B.nch);
  dim3 block(kSpThreads);
  switch (P.xdt) {
    case kF32:
      k_spfwd_part<float><<<grid, block, 0, s>>>((const float *)P.X, P.n, B, idx, val, nlist, S);
      break;
    case kF64:
      k_spfwd_part<double><<<grid, block, 0, s>>>((const double *)P.X, P.n, B, idx, val, nlist, S);
      break;
    default:
      k_spfwd_part<uint16_t><<<grid, block, 0, s>>>((const uint16_t *)P.X, P.n, B, idx, val, nlist, S);
      break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (B.nch <= 16) k_spfwd_final<16><<<(unsigned)B.nfin, kFinThreads, 0, s>>>(P.n, P.y, B, mode, S, u_out);
  else k_spfwd_final<32><<<(unsigned)B.nfin, kFinThreads, 0, s>>>(P.n, P.y, B, mode, S, u_out);
  return hipGetLastError();
}

int spfwd_final_blocks(int64_t n) { return (int)((n + kFinThreads * kFinRows - 1) / (kFinThreads * kFinRows)); }

}  // namespace pr

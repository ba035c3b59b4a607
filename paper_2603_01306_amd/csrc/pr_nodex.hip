// Per-node kernels whose vector is spread over several workgroups (gfx950).
//
// A node's vector lives in registers: workgroup w of W owns the EPT * 512
// consecutive coordinates from w * EPT * 512, thread t of it the coordinates
// t + e * 512 of that range.  The node step is a chain of small reductions
// (dual sums, threshold evaluations of the prox, support counts, Algorithm 1)
// over elementwise work.  One workgroup pays the elementwise work of the whole
// vector on one compute unit between any two of them, from L2 when the vector
// does not fit its registers: 512 us per step on average at p = 89989 (n =
// 2300, logistic), up to 1.18 ms while the iterates are dense.  W workgroups
// pay a W-th of it, and each reduction becomes an exchange between them
// (pr_xwg.h, 1.2-2 us): 300 such iterations took 228 ms before and 53 now, of
// which the X^T pass takes 38.  The chain is kept short: the
// top-kbar window's candidates travel with the dual sums, the prox statistics
// with the first threshold evaluation at the previous tau, the sums of the
// dom test with the support counts, and every workgroup takes the scalar
// decisions itself from the same totals.
#include "pr_xwg.h"

namespace pr {
namespace {
using namespace dev;
using xwg::Group;

constexpr int64_t kXMin = 16384;  // vectors up to here: one workgroup

// The status codes (2 bits) of the EPT coordinates of this thread from the
// packed layout of NodeParams::stp.
template <int EPT>
struct Codes {
  uint32_t w;
  __device__ __forceinline__ int operator()(int e) const { return (int)((w >> (2 * e)) & 3u); }
  __device__ __forceinline__ void load_packed(const uint32_t *__restrict__ stp, int wg) {
    static_assert(EPT <= 16 && (EPT & (EPT - 1)) == 0, "a thread's codes lie in one packed word");
    const int b = wg * EPT;
    w = stp[(b >> 4) * NT + (int)threadIdx.x] >> (2 * (b & 15));
  }
  // from the status vector; `bad` counts the codes outside {free, J0, J1}
  __device__ __forceinline__ void load(const int8_t *__restrict__ st, int64_t j0, int64_t p, int &bad) {
    w = 0u;
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      const int64_t j = j0 + (int64_t)e * NT;
      const int c = j < p ? (int)st[j] : 3;
      if (j < p && (c < 0 || c > 2)) bad++;
      w |= ((uint32_t)c & 3u) << (2 * e);
    }
  }
};

struct NodeXLds {
  xwg::Lds x;
  int cnt[16 * NW];      // support entries per (e, wave) group
  int ngat, nwin;
  double gat[kXwgMax];   // window candidates of this workgroup
  double win[kXwgMax];   // ... of all of them
  double srt[kXwgMax];
  double bc[2];
};
static_assert(kXwgMax == 64, "one wave reads a slot per workgroup and ranks a window");

// The mm-th largest (1-based) of L.win[0 .. cw), cw <= 64, and the sum of H_M
// over the mm largest: ranks by counting (ties by position), one wave.
__device__ __forceinline__ void rank_window(NodeXLds &L, int cw, int mm, double M, double *kth, double *hsum) {
  const int lane = lane_id();
  const double v = lane < cw ? L.win[lane] : -1.0;
  int rank = 0;
  for (int j = 0; j < cw; j++) {
    const double o = L.win[j];
    rank += (o > v || (o == v && j < lane)) ? 1 : 0;
  }
  if (lane < cw) L.srt[rank] = v;
  __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  const double sv = lane < cw ? L.srt[lane] : -1.0;
  *kth = __shfl(sv, mm - 1, 64);
  *hsum = wave_sum(lane < mm ? huber(sv, M) : 0.0);
}

// Exact k-th largest of the entries aval(e) >= 0 over all workgroups, 1 <= k
// <= their number.  A bracket of IEEE bit patterns (monotone for non-negative
// doubles) that holds the value shrinks by the counts at 15 inner points per
// exchange, until it is a single pattern or holds at most 64 entries, which
// every workgroup then gathers and ranks.  [lo, hi) with nlo entries >= lo
// (at least k) and nhi >= hi (fewer than k) is the starting bracket.  The k-th
// of the largest values lies near the upper end, so the first points are a
// quarter of a binary order apart below it, the second's four orders, and only
// then do they divide the bracket evenly.
template <int EPT, class F>
__device__ double select_x(F aval, int k, uint64_t lo, uint64_t hi, double nlo, double nhi, NodeXLds &L, Group &X) {
  uint64_t key[EPT];
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const double a = aval(e);
    key[e] = a >= 0.0 ? (uint64_t)__double_as_longlong(a) + 1u : 0u;  // 0: ignored
  }
  const int lane = lane_id();
  int width = 50;  // log2 of the spacing below hi
  while (hi - lo > 1 && nlo - nhi > (double)xwg::kGat) {
    uint64_t step = (hi - lo + 15u) >> 4;
    if (width < 58 && step > (1ull << width)) step = 1ull << width;
    width += 4;
    const uint64_t first = hi - lo > 16 * step ? hi - 15 * step : lo + step;
    int c = 0;
#pragma unroll 1
    for (int i = 0; i < 15; i++) {
      const uint64_t pv = first + step * (uint64_t)i;
      int n = 0;
#pragma unroll
      for (int e = 0; e < EPT; e++) n += __popcll(__ballot(key[e] > pv));  // entries whose pattern is >= pv
      if (lane == i) c = n;
    }
    const double tot = X.counts<15>((double)c);
    if (X.failed) return 0.0;
    const uint64_t mine = first + step * (uint64_t)lane;
    const bool in = lane < 15 && mine < hi;
    const unsigned long long up = __ballot(in && tot >= (double)k), dn = __ballot(in && !(tot >= (double)k));
    if (up) {
      const int i = 63 - __clzll((long long)up);
      lo = first + step * (uint64_t)i;
      nlo = __shfl(tot, i, 64);
    }
    if (dn) {
      const int i = __ffsll((long long)dn) - 1;
      hi = first + step * (uint64_t)i;
      nhi = __shfl(tot, i, 64);
    }
  }
  if (hi - lo <= 1) return __longlong_as_double((long long)lo);
  // gather the bracket's entries (at most 64 over all workgroups)
  lds_barrier();
  if (threadIdx.x == 0) L.ngat = L.nwin = 0;
  lds_barrier();
#pragma unroll
  for (int e = 0; e < EPT; e++)
    if (key[e] > lo && key[e] <= hi) {
      const int at = atomicAdd(&L.ngat, 1);
      if (at < xwg::kGat) L.gat[at] = __longlong_as_double((long long)(key[e] - 1u));
    }
  double one[1] = {0.0};
  auto pub = [&] {
    const int t = threadIdx.x;
    if (t < xwg::kGat) X.put_f64(X.gat_slot(X.w, t, xwg::kGat), t < L.ngat ? L.gat[t] : -1.0);
  };
  auto take = [&] {
    for (int v = wave_id(); v < X.W; v += NW) {
      const double x = X.poll(X.gat_slot(v, lane_id(), xwg::kGat), true);
      if (x >= 0.0) {
        const int at = atomicAdd(&L.nwin, 1);
        if (at < xwg::kGat) L.win[at] = x;
      }
    }
  };
  X.run<1, 0, false>(one, nullptr, nullptr, pub, take);
  if (X.failed) return 0.0;
  if (wave_id() == 0) {
    double kth, hs;
    rank_window(L, L.nwin < xwg::kGat ? L.nwin : xwg::kGat, k - (int)nhi, INFINITY, &kth, &hs);
    if (lane_id() == 0) L.bc[0] = kth;
  }
  lds_barrier();
  return L.bc[0];
}

// Per-thread part of one evaluation of the prox threshold's S(tau): {head
// count, count, block sum} over the magnitudes aval(e).
template <int EPT, class F>
__device__ __forceinline__ void tau_sums(F aval, double rho, double M, double tau, double *v) {
  const double top = tau + (isfinite(M) ? fmin(tau / rho, M) : tau / rho);
  v[0] = v[1] = v[2] = 0.0;
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const double x = aval(e);
    if (x > tau) {
      v[1] += 1.0;
      if (x > top) v[0] += 1.0;
      else v[2] += x;
    }
  }
}

// The prox threshold tau (the search of solve_tau, pr_regularizer.h) over the
// register-resident magnitudes aval(e).  s: the totals {evaluation at warm
// (used when warm lies inside the bracket), number and sum of the positive
// magnitudes}, amax their largest.
template <int EPT, class F>
__device__ __forceinline__ double solve_tau_x(F aval, int kbar, double rho, double M, double warm, const double *s,
                                              double amax, Group &X, int *evals) {
  const bool finM = isfinite(M);
  auto Dof = [&](double t) { return finM ? fmin(t / rho, M) : t / rho; };
  *evals = 0;
  if (kbar <= 0) return INFINITY;
  const double K = (double)kbar;
  if (s[3] <= K) return 0.0;
  auto froot = [&](double h, double nb, double sB) -> double {
    if (nb <= 0.0) return NAN;
    if (finM) {
      const double Sf = h + (sB - nb * rho * M) / M;
      if (Sf >= K) return (sB - M * (K - h)) / nb;
    }
    return rho * sB / (K - h + rho * nb);
  };
  double lo = 0.0, hi = amax;
  bool have = warm > lo && warm < hi;  // the evaluation at tau is at hand
  double tau = have ? warm : froot(0.0, s[3], s[4]);
  if (!(tau > lo && tau < hi)) tau = 0.5 * (lo + hi);
  bool from_root = false;
  double ph = -1.0, pb = -1.0;
  int nsteps = 0;
  double wref = hi - lo;
  for (int it = 0; it < 200; it++) {
    const double D = Dof(tau);
    double v[3] = {s[0], s[1], s[2]};
    if (!have) {
      tau_sums<EPT>(aval, rho, M, tau, v);
      X.sum(v);
      if (X.failed) return 0.0;
    }
    have = false;
    *evals = it + 1;
    if (from_root && v[0] == ph && v[1] == pb) return tau;
    const double S = v[0] + (v[2] - (v[1] - v[0]) * tau) / D;
    if (S > K) lo = tau;
    else if (S < K) hi = tau;
    else return tau;
    double c = froot(v[0], v[1] - v[0], v[2]);
    if (c == tau) return tau;
    if (nsteps >= 2 && hi - lo > 0.5 * wref) {
      nsteps = 0;
      wref = hi - lo;
      c = NAN;
    }
    if (c > lo && c < hi) {
      from_root = true;
      nsteps++;
    } else {
      c = 0.5 * (lo + hi);
      from_root = false;
      nsteps = 0;
      wref = hi - lo;
    }
    ph = v[0];
    pb = v[1];
    if (!(c > lo && c < hi)) return c;
    tau = c;
  }
  return tau;
}

// Algorithm 1 (alg1_free, pr_regularizer.h) over the free magnitudes aval(e).
template <int EPT, class F>
__device__ __forceinline__ double alg1_x(F aval, int kbar, double theta, Group &X) {
  if (kbar <= 0 || !(theta > 0.0)) return 0.0;
  const double K = (double)kbar;
  double s = theta / K;
  double prevK = 0.0;
  for (int it = 0; it <= kbar + 1; it++) {
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      const double x = aval(e);
      if (x >= 0.0) {
        if (x > s) {
          v[0] += 1.0;
          v[2] += x * x;
        } else {
          v[1] += x;
        }
      }
    }
    X.sum(v);
    if (X.failed) return 0.0;
    if (v[0] == prevK || v[0] >= K) return 0.5 * (v[2] + (K - v[0]) * s * s);
    prevK = v[0];
    s = fmin(s, v[1] / (K - v[0]));
  }
  return NAN;
}

// Sums and maxima of an iterate for the dom test and Algorithm 1.
struct XStats {
  double theta, sq1, amax, j0max, boxmax;
};
template <int EPT>
__device__ __forceinline__ XStats local_stats(const double (&x)[EPT], const Codes<EPT> &sv) {
  XStats t{0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int s = sv(e);
    const double ax = fabs(x[e]);
    if (s != 3) {
      t.amax = fmax(t.amax, ax);
      if (s == kZero) t.j0max = fmax(t.j0max, ax);
      else t.boxmax = fmax(t.boxmax, ax);
      if (s == kFree) t.theta += ax;
      else if (s == kOne) t.sq1 += x[e] * x[e];
    }
  }
  return t;
}
// dom g_N with relative slack 1e-9 (the node kernels' test)
__device__ __forceinline__ int in_domain(const XStats &t, int kbar, double M) {
  const double zt = 1e-9 * fmax(1.0, t.amax);
  int ok = (t.j0max <= zt);
  if (isfinite(M) && t.boxmax > M * (1.0 + 1e-9)) ok = 0;
  if (kbar == 0) {
    if (t.theta > zt) ok = 0;
  } else if (isfinite(M) && t.theta > M * (double)kbar * (1.0 + 1e-9)) {
    ok = 0;
  }
  return ok;
}

// Support list of the iterate (ascending j; J1 / J0 entries flagged) and, in
// the same exchange, the totals of the statistics t.  Returns the list length.
template <int EPT>
__device__ __forceinline__ int support_list_x(const double (&x)[EPT], const Codes<EPT> &sv, int64_t j0,
                                              int32_t *__restrict__ sidx, double *__restrict__ sval, NodeXLds &L,
                                              Group &X, XStats &t) {
  const int lane = lane_id(), w = wave_id();
  const unsigned long long below = (1ull << lane) - 1ull;
  double s[3] = {0.0, t.theta, t.sq1}, m[3] = {t.amax, t.j0max, t.boxmax};
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int c = __popcll(__ballot(sv(e) != 3 && x[e] != 0.0));
    if (lane == 0) {
      L.cnt[e * NW + w] = c;
      s[0] += (double)c;
    }
  }
  double pre = 0.0;
  X.run<3, 3, true>(s, m, &pre, [] {}, [] {});
  if (X.failed) return 0;
  t = XStats{s[1], s[2], m[0], m[1], m[2]};
  // exclusive prefix of the groups (e, wave) in j order, in every wave
  int off[EPT];
  int run = (int)pre;
  constexpr int NO = EPT * NW;
#pragma unroll
  for (int q0 = 0; q0 < NO; q0 += 64) {
    const int c = (q0 + lane < NO) ? L.cnt[q0 + lane] : 0;
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
#pragma unroll
    for (int e = 0; e < EPT; e++)
      if ((e * NW) / 64 == q0 / 64) off[e] = run + __shfl(incl - c, (e * NW + w) & 63, 64);
    run += __shfl(incl, 63, 64);
  }
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const bool nz = sv(e) != 3 && x[e] != 0.0;
    const unsigned long long mk = __ballot(nz);
    if (nz) {
      const int pos = off[e] + __popcll(mk & below);
      sidx[pos] = (int32_t)(j0 + (int64_t)e * NT) | (sv(e) == kOne ? kJ1Flag : (sv(e) == kZero ? kJ0Flag : 0));
      sval[pos] = x[e];
    }
  }
  return (int)s[0];
}

// A step whose workgroups lost each other ends the solve: the host finds
// *XBuf::lost written, whatever the state says.
__device__ __forceinline__ void give_up(NodeState *S, const Group &X, const XBuf &xb) {
  if (threadIdx.x == 0) S->done = 1;
  X.finish(xb);
}

template <int EPT>
__global__ __launch_bounds__(NT) void k_node_init_x(const NodeParams *__restrict__ prm, NodeState *S, NodeBufs nb,
                                                    const double *__restrict__ beta0, double L, XBuf xb) {
  __shared__ NodeXLds lds;
  Group X;
  X.init(xb, &lds.x);
  const int64_t p = prm->p;
  const int64_t j0 = (int64_t)X.w * (EPT * NT) + threadIdx.x;
  Codes<EPT> sv;
  sv.load_packed(prm->stp, X.w);
  double x[EPT];
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int64_t j = j0 + (int64_t)e * NT;
    x[e] = 0.0;
    if (j < p) {
      const double b = beta0 ? beta0[j] : 0.0;
      x[e] = b;
      nb.x0[j] = b;
      nb.xbest[j] = b;
      nb.x1[j] = 0.0;
      nb.hprev[j] = 0.0;
    }
  }
  const int kbar = prm->kbar;
  const double M = prm->M;
  XStats t = local_stats<EPT>(x, sv);
  const int ns = support_list_x<EPT>(x, sv, j0, nb.sidx, nb.sval, lds, X, t);
  auto aval = [&](int e) { return sv(e) == kFree ? fabs(x[e]) : -1.0; };
  const double gv = 0.5 * t.sq1 + alg1_x<EPT>(aval, kbar, t.theta, X);
  if (X.w == 0 && threadIdx.x == 0) {
    NodeState s{};
    s.L = L;
    s.t = 1.0;
    s.gap_ref = INFINITY;
    s.lb = -INFINITY;
    s.ub = INFINITY;
    s.phi = INFINITY;
    s.psi = -INFINITY;
    s.rel_gap = INFINITY;
    s.gval = gv;
    s.tau = -1.0;
    s.tk = -1.0;
    s.tkw = 0.25;
    s.status = kMaxIter;
    s.nsupp = ns;
    s.indom = in_domain(t, kbar, M);
    s.bt = is_bt(prm->method) ? 1 : 0;
    s.done = X.failed ? 1 : 0;
    *S = s;
  }
  X.finish(xb);
}

// The node step of k_node_step (pr_node.hip) over W workgroups: the same
// quantities and decisions from the same products, sums associated per
// workgroup.
template <int EPT>
__global__ __launch_bounds__(NT) void k_node_step_x(const NodeParams *__restrict__ prm, NodeState *S, NodeBufs nb,
                                                    ProbBufs B, StepArgs A, XBuf xb) {
  __shared__ NodeXLds lds;
  const int tid = threadIdx.x;
  const NodeState s0 = *S;
  if (s0.done) return;
  Group X;
  X.init(xb, &lds.x);
  if (tid == 0) lds.ngat = lds.nwin = 0;
  const int64_t p = A.p;
  const int64_t j0 = (int64_t)X.w * (EPT * NT) + tid;
  const int parity = A.parity;
  const int kbar = prm->kbar, loss = prm->loss;
  const double lam2 = prm->lambda2, M = prm->M, L = s0.L;
  const double *__restrict__ xc = parity ? nb.x1 : nb.x0;
  double *__restrict__ xn = parity ? nb.x0 : nb.x1;  // holds x^{k-1}, receives x^{k+1}
  const double *__restrict__ gp = (loss == kLsq) ? nb.hprev : B.h2;
  Codes<EPT> sv;
  sv.load_packed(A.stp, X.w);
  double x[EPT], xk[EPT], xq[EPT], g2[EPT];
  double r1[4] = {0.0, 0.0, 0.0, 0.0};  // sum_{J1} H_M(w), #{w > wb}, #{w >= wa}, sum_{w > wb} H_M(w)
  double wmax[1] = {0.0};               // the largest free |w|
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int64_t j = j0 + (int64_t)e * NT;
    const bool in = j < p;
    x[e] = in ? B.h1[j] : 0.0;
    xk[e] = in ? xc[j] : 0.0;
    xq[e] = in ? xn[j] : 0.0;
    g2[e] = in ? gp[j] : 0.0;
  }
  double Fk = 0.0, negconj = 0.0;
  for (int i = lane_id(); i < B.nfin; i += 64) {
    Fk += B.rbsum[2 * i];
    negconj += B.rbsum[2 * i + 1];
  }
  Fk = wave_sum(Fk);
  negconj = wave_sum(negconj);
  const bool lead = X.w == 0 && tid == 0;
  // the LDS counters are cleared, and this workgroup has read all it needs of
  // the state before it publishes anything (workgroup 0 then updates it)
  __syncthreads();

  // dual sums; the window around the previous kbar-th value and its candidates
  const double wscale = (loss == kLsq) ? 1.0 / lam2 : 0.5 / lam2;
  const double tkp = s0.tk, dlt = s0.tkw;
  const bool wv = tkp > 0.0 && kbar > 0;
  const double wa = wv ? tkp * (1.0 - dlt) : INFINITY, wb = wv ? tkp * (1.0 + dlt) : INFINITY;
  auto wabs = [&](int e) { return sv(e) == kFree ? fabs(x[e] * wscale) : -1.0; };
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int s = sv(e);
    if (s == 3) continue;
    const double w = x[e] * wscale;
    if (s == kOne) r1[0] += huber(w, M);
    if (s == kFree) {
      const double aw = fabs(w);
      wmax[0] = fmax(wmax[0], aw);
      if (aw > wb) {
        r1[1] += 1.0;
        r1[3] += huber(aw, M);
      } else if (wv && aw >= wa) {
        const int at = atomicAdd(&lds.ngat, 1);
        if (at < xwg::kWin) lds.gat[at] = aw;
      }
      if (aw >= wa) r1[2] += 1.0;
    }
  }
  {
    auto pub = [&] {
      const int t = tid;
      if (t < xwg::kWin) {
        const int ng = lds.ngat;
        // a workgroup with more than kWin entries says so in its first slot
        const double v = ng > xwg::kWin ? (t == 0 ? INFINITY : -1.0) : (t < ng ? lds.gat[t] : -1.0);
        X.put_f64(X.gat_slot(X.w, t, xwg::kWin), v);
      }
    };
    auto take = [&] {
      constexpr int per = 64 / xwg::kWin;  // workgroups read by one wave at once
      for (int v0 = wave_id() * per; v0 < X.W; v0 += NW * per) {
        const int v = v0 + lane_id() / xwg::kWin;
        const double c = X.poll(X.gat_slot(v, lane_id() % xwg::kWin, xwg::kWin), v < X.W);
        if (v < X.W && c >= 0.0) {
          const int at = atomicAdd(&lds.nwin, c == INFINITY ? 2 * kXwgMax : 1);
          if (at < kXwgMax) lds.win[at] = c;
        }
      }
    };
    X.run<4, 1, false>(r1, wmax, nullptr, pub, take);
  }
  if (X.failed) {
    give_up(S, X, xb);
    return;
  }
  const double cgt = r1[1], cge = r1[2];
  const int cw = (int)(cge - cgt);
  const bool fast = wv && cgt < (double)kbar && (double)kbar <= cge && cge - cgt <= (double)kXwgMax && lds.nwin == cw;
  double topsum = 0.0, tkn = -1.0;
  if (kbar > 0 && fast) {
    if (wave_id() == 0) {
      double kth, hs;
      rank_window(lds, cw, kbar - (int)cgt, M, &kth, &hs);
      if (lane_id() == 0) {
        lds.bc[0] = kth;
        lds.bc[1] = r1[3] + hs;
      }
    }
    lds_barrier();
    tkn = lds.bc[0];
    topsum = lds.bc[1];
  } else if (kbar > 0) {
    // the bracket the window counts leave (all patterns up to the largest without)
    uint64_t lo = 0ull, hi = (uint64_t)__double_as_longlong(wmax[0]) + 1u;
    double nlo = (double)p, nhi = 0.0;
    if (wv) {
      const uint64_t ka = (uint64_t)__double_as_longlong(wa), kb = (uint64_t)__double_as_longlong(wb) + 1u;
      if (cgt >= (double)kbar) {
        lo = kb;
        nlo = cgt;
      } else if (cge >= (double)kbar) {
        lo = ka;
        nlo = cge;
        hi = kb;
        nhi = cgt;
      } else {
        hi = ka;
        nhi = cge;
      }
    }
    tkn = select_x<EPT>(wabs, kbar, lo, hi, nlo, nhi, lds, X);
    const double Ht = huber(tkn, M);
    double v1[1] = {0.0};
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      const double aw = wabs(e);
      if (aw >= 0.0) v1[0] += fmax(huber(aw, M) - Ht, 0.0);
    }
    X.sum(v1);
    if (X.failed) {
      give_up(S, X, xb);
      return;
    }
    topsum = (double)kbar * Ht + v1[0];
  }

  // bounds, stopping test, restart and momentum: the same in every thread
  const double psi = negconj - 2.0 * lam2 * (r1[0] + topsum);
  const double phi = s0.indom ? Fk + 2.0 * lam2 * s0.gval : INFINITY;
  const int it = s0.iter;
  const double gap = phi - psi;
  double lb = s0.lb, ub = s0.ub;
  int improved = 0, ub_improved = 0;
  if (psi > lb) {
    lb = psi;
    improved = 1;
  }
  if (phi < ub) {
    ub = phi;
    ub_improved = 1;
  }
  const double rel = (ub - lb) / fmax(fabs(ub), 1e-300);
  int done = 0, status = kMaxIter;
  if (rel <= prm->tol) {
    done = 1;
    status = kConverged;
  } else if (!isnan(prm->cutoff) && lb >= prm->cutoff) {
    done = 1;
    status = kCutoffPrune;
  } else if (!isnan(prm->cutoff) && ub <= prm->cutoff) {
    done = 1;
    status = kCutoffBranch;
  } else if (it >= prm->max_iter) {
    done = 1;
    status = kMaxIter;
  }
  double m = 0.0, t = s0.t, gap_ref = s0.gap_ref;
  int restart = 0, restarts = s0.restarts;
  if (!done) {
    restart = decide_restart(prm, it, gap, phi, s0.phi, gap_ref, restarts);
    if (restart) {
      t = 1.0;
    } else {
      const double tn = fista_next_t(t);
      m = (t - 1.0) / tn;
      t = tn;
    }
  }
  if (lead) {
    if (prm->trace && it <= prm->max_iter) {
      prm->trace[2 * it] = phi;
      prm->trace[2 * it + 1] = psi;
    }
    double tw = 0.25;
    if (wv && tkn > 0.0) tw = fmin(0.25, fmax(1e-12, 2.0 * fabs(tkn - tkp) / tkn));
    if (wv && !fast && cgt < (double)kbar && (double)kbar <= cge) tw = fmin(tw, 0.25 * dlt);
    S->phi = phi;
    S->psi = psi;
    S->lb = lb;
    S->ub = ub;
    S->rel_gap = rel;
    S->improved = improved;
    S->status = status;
    S->t = t;
    S->gap_ref = gap_ref;
    S->restarts = restarts;
    S->mom = m;
    S->tk = tkn;
    S->tkw = tw;
    if (done) S->done = 1;
  }
  if (ub_improved) {
#pragma unroll
    for (int e = 0; e < EPT; e++)
      if (sv(e) != 3) nb.xbest[j0 + (int64_t)e * NT] = xk[e];
  }
  if (done) {
    X.finish(xb);
    return;
  }
  // gradient step at the momentum point, x[] <- v
  const double invL = 1.0 / L;
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const double h = x[e];
    const double yj = xk[e] + m * (xk[e] - xq[e]);
    double gj;
    if (loss == kLsq) gj = -2.0 * ((1.0 + m) * h - m * g2[e]);
    else gj = restart ? -h : g2[e];
    x[e] = sv(e) != 3 ? yj - gj * invL : 0.0;
    if (loss == kLsq && sv(e) != 3) nb.hprev[j0 + (int64_t)e * NT] = h;
  }
  // x[] <- prox_{(2 lambda2 / L) g_N}(v)
  const double rho = 2.0 * lam2 * invL;
  int evals = 0;
  auto vabs = [&](int e) { return sv(e) == kFree ? fabs(x[e]) : -1.0; };
  double sv5[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, mx[1] = {0.0};
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const double a = vabs(e);
    if (a > 0.0) {
      sv5[3] += 1.0;
      sv5[4] += a;
      mx[0] = fmax(mx[0], a);
    }
  }
  if (s0.tau > 0.0) tau_sums<EPT>(vabs, rho, M, s0.tau, sv5);
  X.summax(sv5, mx);
  const double tau = solve_tau_x<EPT>(vabs, kbar, rho, M, s0.tau, sv5, mx[0], X, &evals);
  if (X.failed) {
    give_up(S, X, xb);
    return;
  }
  const double inv1p = 1.0 / (1.0 + rho);
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int s = sv(e);
    double xv = 0.0;
    if (s != 3) {
      if (s != kZero) {
        const double av = fabs(x[e]);
        double r = fmin(av * inv1p, M);
        if (s == kFree) r = fmin(r, fmax(av - tau, 0.0));
        xv = (r == 0.0) ? 0.0 : copysign(r, x[e]);
      }
      xn[j0 + (int64_t)e * NT] = xv;
    }
    x[e] = xv;
  }
  XStats ts = local_stats<EPT>(x, sv);
  const int ns = support_list_x<EPT>(x, sv, j0, nb.sidx, nb.sval, lds, X, ts);
  auto xabs = [&](int e) { return sv(e) == kFree ? fabs(x[e]) : -1.0; };
  const double gval = 0.5 * ts.sq1 + alg1_x<EPT>(xabs, kbar, ts.theta, X);
  if (X.failed) {
    give_up(S, X, xb);
    return;
  }
  if (lead) {
    S->gval = gval;
    S->indom = in_domain(ts, kbar, M);
    S->nsupp = ns;
    S->tau = tau;
    S->tau_iters = evals;
    S->parity = parity ^ 1;
    S->iter = it + 1;
  }
  X.finish(xb);
}

// Standalone prox_{rho g_N}(v) (Algorithm 2 + Moreau, pooled-threshold form).
// |J1| and |J_f| are counted here, kbar = min(k - |J1|, |J_f|).  out is not
// written where XResult::flag is not 0.
template <int EPT>
__global__ __launch_bounds__(NT) void k_prox_x(const double *v, double *out, int64_t p, double rho, int k, double M,
                                               const int8_t *__restrict__ st, XResult *res, XBuf xb) {
  __shared__ xwg::Lds lds;
  Group X;
  X.init(xb, &lds);
  const int64_t j0 = (int64_t)X.w * (EPT * NT) + threadIdx.x;
  double x[EPT];
  double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, mx[1] = {0.0};  // bad codes, |J1|, |J_f|, #, sum of a > 0
  Codes<EPT> sv;
  int bad = 0;
  sv.load(st, j0, p, bad);
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int64_t j = j0 + (int64_t)e * NT;
    x[e] = j < p ? v[j] : 0.0;
    const int c = sv(e);
    s[1] += c == kOne ? 1.0 : 0.0;
    s[2] += c == kFree ? 1.0 : 0.0;
    const double a = c == kFree ? fabs(x[e]) : 0.0;
    if (a > 0.0) {
      s[3] += 1.0;
      s[4] += a;
      mx[0] = fmax(mx[0], a);
    }
  }
  s[0] = (double)bad;
  X.summax(s, mx);
  const bool lead = X.w == 0 && threadIdx.x == 0;
  int err = X.failed ? 3 : (s[0] > 0.0 ? 1 : (s[1] > (double)k ? 2 : 0));
  if (err == 0) {
    const int kbar = (int)fmin((double)k - s[1], s[2]);
    auto vabs = [&](int e) { return sv(e) == kFree ? fabs(x[e]) : -1.0; };
    int evals;
    const double tau = solve_tau_x<EPT>(vabs, kbar, rho, M, -1.0, s, mx[0], X, &evals);
    const double inv1p = 1.0 / (1.0 + rho);
    if (X.failed) {
      err = 3;
    } else {
#pragma unroll
      for (int e = 0; e < EPT; e++) {
        const int c = sv(e);
        if (c == 3) continue;
        double xv = 0.0;
        if (c != kZero) {
          const double av = fabs(x[e]);
          double r = fmin(av * inv1p, M);
          if (c == kFree) r = fmin(r, fmax(av - tau, 0.0));
          xv = (r == 0.0) ? 0.0 : copysign(r, x[e]);
        }
        out[j0 + (int64_t)e * NT] = xv;
      }
    }
  }
  if (lead && res) {
    res->flag = err;
    res->tag = X.tag();
  }
  X.finish(xb);
}

// g_N(beta) (Algorithm 1, +inf off its domain) into out[0], g_N*(ascale alpha)
// into out[1] (each if its input is given; NaN where the workgroups lost each
// other); counts and flag as in k_prox_x.
template <int EPT>
__global__ __launch_bounds__(NT) void k_regularizer_x(const double *__restrict__ beta,
                                                      const double *__restrict__ alpha, double ascale, int64_t p,
                                                      int k, double M, const int8_t *__restrict__ st, double *out,
                                                      XResult *res, XBuf xb) {
  __shared__ NodeXLds lds;
  Group X;
  X.init(xb, &lds.x);
  const int64_t j0 = (int64_t)X.w * (EPT * NT) + threadIdx.x;
  Codes<EPT> sv;
  int bad = 0;
  sv.load(st, j0, p, bad);
  double x[EPT], a[EPT];
  // bad codes, |J1|, |J_f|, theta, sum_{J1} beta^2, sum_{J1} H_M(alpha); maxima of |beta|, of free |alpha|
  double s[6] = {(double)bad, 0.0, 0.0, 0.0, 0.0, 0.0}, m[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int64_t j = j0 + (int64_t)e * NT;
    x[e] = (beta && j < p) ? beta[j] : 0.0;
    a[e] = (alpha && j < p) ? ascale * alpha[j] : 0.0;
    const int c = sv(e);
    s[1] += c == kOne ? 1.0 : 0.0;
    s[2] += c == kFree ? 1.0 : 0.0;
    if (c == kOne) s[5] += huber(a[e], M);
    if (c == kFree) m[3] = fmax(m[3], fabs(a[e]));
  }
  {
    const XStats t = local_stats<EPT>(x, sv);
    s[3] = t.theta;
    s[4] = t.sq1;
    m[0] = t.amax;
    m[1] = t.j0max;
    m[2] = t.boxmax;
  }
  X.summax(s, m);
  const bool lead = X.w == 0 && threadIdx.x == 0;
  int err = X.failed ? 3 : (s[0] > 0.0 ? 1 : (s[1] > (double)k ? 2 : 0));
  if (err == 0) {
    const int kbar = (int)fmin((double)k - s[1], s[2]);
    if (beta) {
      const XStats t{s[3], s[4], m[0], m[1], m[2]};
      auto xabs = [&](int e) { return sv(e) == kFree ? fabs(x[e]) : -1.0; };
      const double g = 0.5 * t.sq1 + alg1_x<EPT>(xabs, kbar, t.theta, X);
      if (lead) out[0] = in_domain(t, kbar, M) ? g : INFINITY;
    }
    if (alpha) {
      auto aabs = [&](int e) { return sv(e) == kFree ? fabs(a[e]) : -1.0; };
      double top = 0.0;
      if (kbar > 0) {
        const double t = select_x<EPT>(aabs, kbar, 0ull, (uint64_t)__double_as_longlong(m[3]) + 1u, s[2], 0.0, lds, X);
        const double Ht = huber(t, M);
        double v[1] = {0.0};
#pragma unroll
        for (int e = 0; e < EPT; e++) {
          const double w = aabs(e);
          if (w >= 0.0) v[0] += fmax(huber(w, M) - Ht, 0.0);
        }
        X.sum(v);
        top = (double)kbar * Ht + v[0];
      }
      if (lead) out[1] = s[5] + top;
    }
    if (X.failed) err = 3;
  }
  if (lead && err == 3) out[0] = out[1] = NAN;
  if (lead && res) {
    res->flag = err;
    res->tag = X.tag();
  }
  X.finish(xb);
}

}  // namespace

// Workgroups (at most cap) and entries per thread for a vector of p; {0, 0} where
// one workgroup takes the step (pr_node.hip): up to 16384 entries its registers
// hold the vector, and past cap * 16 * 512 (524288 with kXwgMax) the vector is
// too long for this kernel's.  Between, few entries per thread are worth more workgroups:
// p = 89989, 300 iterations, 56.5 ms with 4 (44 workgroups), 57.3 with 8, 59.6
// with 16.
XShape node_xshape(int64_t p, int cap) {
  if (p <= kXMin) return XShape{0, 0};
  for (int e = 4; e <= 16; e *= 2) {
    const int64_t w = (p + (int64_t)e * NT - 1) / ((int64_t)e * NT);
    if (w <= cap) return XShape{(int)w, e};
  }
  return XShape{0, 0};
}

hipError_t launch_node_init_x(const NodeParams *prm, NodeState *S, NodeBufs nb, const double *beta0, double L,
                              XShape g, const XBuf &xb, hipStream_t s) {
  switch (g.ept) {
    case 4: k_node_init_x<4><<<g.wgs, NT, 0, s>>>(prm, S, nb, beta0, L, xb); break;
    case 8: k_node_init_x<8><<<g.wgs, NT, 0, s>>>(prm, S, nb, beta0, L, xb); break;
    case 16: k_node_init_x<16><<<g.wgs, NT, 0, s>>>(prm, S, nb, beta0, L, xb); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_node_step_x(const NodeParams *prm, NodeState *S, NodeBufs nb, const ProbBufs &B, const StepArgs &a,
                              XShape g, const XBuf &xb, hipStream_t s) {
  if (a.gb || a.bt) return hipErrorInvalidValue;  // both end at 16384 entries
  switch (g.ept) {
    case 4: k_node_step_x<4><<<g.wgs, NT, 0, s>>>(prm, S, nb, B, a, xb); break;
    case 8: k_node_step_x<8><<<g.wgs, NT, 0, s>>>(prm, S, nb, B, a, xb); break;
    case 16: k_node_step_x<16><<<g.wgs, NT, 0, s>>>(prm, S, nb, B, a, xb); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Shape of the standalone kernels: one workgroup up to kXOne entries (its
// reductions stay in LDS), then few entries per thread and the same limits as above.
constexpr int64_t kXOne = 4096;
int reg_x_cap(int64_t p, hipStream_t s) { return p <= kXOne ? 1 : xwg_cap(s); }
XShape reg_xshape(int64_t p, int cap) {
  for (int e = 1; e <= 16; e *= 2) {
    const int64_t w = (p + (int64_t)e * NT - 1) / ((int64_t)e * NT);
    if (w == 1 && p <= kXOne) return XShape{1, e};
    if (p > kXOne && e >= 4 && w <= cap) return XShape{(int)w, e};
  }
  return XShape{0, 0};
}

#define PR_REGX(CALL)        \
  switch (g.ept) {           \
    case 1: CALL(1); break;  \
    case 2: CALL(2); break;  \
    case 4: CALL(4); break;  \
    case 8: CALL(8); break;  \
    case 16: CALL(16); break; \
    default: return hipErrorInvalidValue; \
  }
hipError_t launch_prox_x(const double *v, double *out, int64_t p, double rho, int32_t k, double M, const int8_t *st,
                         XResult *res, const XBuf &xb, hipStream_t s) {
  const XShape g = reg_xshape(p, xb.cap);
#define PR_CALL(E) k_prox_x<E><<<g.wgs, NT, 0, s>>>(v, out, p, rho, k, M, st, res, xb)
  PR_REGX(PR_CALL)
#undef PR_CALL
  return hipGetLastError();
}

hipError_t launch_regularizer_x(const double *beta, const double *alpha, double ascale, int64_t p, int32_t k,
                                double M, const int8_t *st, double *out2, XResult *res, const XBuf &xb, hipStream_t s) {
  const XShape g = reg_xshape(p, xb.cap);
#define PR_CALL(E) k_regularizer_x<E><<<g.wgs, NT, 0, s>>>(beta, alpha, ascale, p, k, M, st, out2, res, xb)
  PR_REGX(PR_CALL)
#undef PR_CALL
  return hipGetLastError();
}
#undef PR_REGX

}  // namespace pr

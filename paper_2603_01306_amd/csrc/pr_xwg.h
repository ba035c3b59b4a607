// Reductions over several workgroups of one launch (gfx950): a handful of
// workgroups that share one per-node computation exchange small vectors of
// FP64 partials through device memory without a kernel boundary.
//
// Every FP64 value travels as two 64-bit words, each a 32-bit half of the value
// under a 32-bit round number, written and read with relaxed device-scope
// accesses.  A reader polls until both words carry the current round, so the
// data is its own flag: no fence, no counter to reset, one store and one load
// round trip per exchange.  Rounds alternate between two slot sets; a
// workgroup publishes round i + 1 only after it has read all of round i, so
// nobody overwrites a slot that is still being read (round i + 2 starts after
// every workgroup published i + 1).  Every workgroup reads the same words and
// combines them in the same order, so all of them hold bit-identical results,
// and a repeated run repeats them.  Measured on MI355X over all XCDs (512
// threads, up to 8 values, the reduction inside the workgroups included): 1.25
// us per exchange with 8 workgroups, 1.37 with 16, 1.6 with 32, 2.1 with 64.
//
// All workgroups of the launch must be resident together (xwg_cap).  A wait of
// more than kXwgTicks (pr_wait.h) ends with `failed` set instead of a hang, and
// the workgroup reports it in *XBuf::lost: what such a launch wrote is not to be
// used.  A test switch in the area's head lets the last workgroup give up the
// first exchange of every launch and the others after kLostTicks.
#pragma once
#include "pr_device.h"
#include "pr_wait.h"

namespace pr {
namespace {
namespace xwg {
using namespace dev;

constexpr int kQ = 16;         // values per reduction at most
constexpr int kWin = 16;       // values per workgroup in a small gather
constexpr int kGat = 64;       // ... and in a large one
constexpr long long kXwgTicks = 2000000000ll;  // 20 s of the 100 MHz clock
constexpr long long kLostTicks = 200000ll;     // 2 ms

__device__ __forceinline__ void put(uint64_t *w, uint32_t round, uint32_t half) {
  __hip_atomic_store(w, ((uint64_t)round << 32) | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Lds {
  double red[2][NW * kQ];
  double res[2][kQ + 1];
  int bad;          // a wait of this workgroup was given up
  long long ticks;  // limit of a wait
};

struct Group {
  uint64_t *slots;  // [2][kQ][kXwgMax][2] reductions, then [2][kXwgMax][kGat][2] gathers
  uint32_t round, round0;  // current, at the start of the launch
  int W, w;         // workgroups, this one
  Lds *L;
  int ph;
  bool failed;

  // Call once per workgroup, before any exchange (followed by a barrier inside).
  __device__ __forceinline__ void init(const XBuf &xb, Lds *lds) {
    slots = xb.slots;
    round = round0 = xb.head[0];
    W = (int)gridDim.x;
    w = (int)blockIdx.x;
    L = lds;
    ph = 0;
    failed = false;
    if (threadIdx.x == 0) {
      const bool lose = xb.head[1] != 0;
      lds->bad = lose && w > 0 && w == W - 1;
      lds->ticks = lose ? kLostTicks : kXwgTicks;
    }
  }

  __device__ __forceinline__ uint64_t *red_slot(int q, int v) const {
    return slots + ((((size_t)(round & 1) * kQ + q) * kXwgMax + v) << 1);
  }
  __device__ __forceinline__ uint64_t *gat_slot(int v, int c, int cap) const {
    return slots + ((((size_t)2 * kQ + (size_t)(round & 1) * kGat) * kXwgMax + (size_t)v * cap + c) << 1);
  }

  __device__ __forceinline__ void put_f64(uint64_t *s, double x) const {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    put(s, round, (uint32_t)b);
    put(s + 1, round, (uint32_t)(b >> 32));
  }

  // Value of the slot pair s in every lane with `want`, polled by the whole wave.
  __device__ __forceinline__ double poll(const uint64_t *s, bool want) {
    uint64_t a = 0, b = 0;
    bool ok = !want;
    int spin = 0;
    WaitClock t;
    for (;;) {
      if (!ok) {
        a = __hip_atomic_load(s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        b = __hip_atomic_load(s + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = (uint32_t)(a >> 32) == round && (uint32_t)(b >> 32) == round;
      }
      if (__all(ok)) break;
      if ((++spin & 1023) == 0 &&
          t.expired((long long)__builtin_amdgcn_s_memrealtime(), L->ticks)) {
        if (lane_id() == 0) L->bad = 1;
        break;
      }
    }
    return __longlong_as_double((long long)((a & 0xffffffffull) | (b << 32)));
  }

  __device__ __forceinline__ void begin() {
    if (++round == 0) round = 2;  // 0 is the tag of memory never written; the parity alternates
  }

  // One exchange of the K values (sums q < KS, then maxima) whose per-wave
  // partials are in L->red[ph][q * NW + wave]: totals in L->res[ph][q] after
  // it.  `pub` runs in every thread once the workgroup's partials are complete,
  // `take` before the final barrier (the gathers use them); PREFIX: res[kQ] is
  // the sum of value 0 over the workgroups before this one.
  template <int K, int KS, bool PREFIX, class PUB, class TAKE>
  __device__ __forceinline__ void exchange(PUB pub, TAKE take) {
    const int lane = lane_id(), wv = wave_id();
    const double *r = L->red[ph];
    double *res = L->res[ph];
    lds_barrier();
    pub();
    // wave q carries value q (and q + NW): combine the waves' partials,
    // publish, read everybody's, combine
#pragma unroll
    for (int q0 = 0; q0 < K; q0 += NW) {
      const int q = q0 + wv;
      if (q < K) {
        const bool mx = q >= KS;
        double v = r[q * NW + (lane & (NW - 1))];
        // total of the eight partials in every lane (pairs, quads, half rows)
        auto op = [&](double a, double b) { return mx ? fmax(a, b) : a + b; };
        v = op(v, dpp_f64<0xb1, 0xf>(v, 0ll));
        v = op(v, dpp_f64<0x4e, 0xf>(v, 0ll));
        v = op(v, dpp_f64<0x141, 0xf>(v, 0ll));
        double x = v, t = v, pv = 0.0;
        if (W > 1) {
          uint64_t *mine = red_slot(q, w);
          const uint64_t b = (uint64_t)__double_as_longlong(v);
          if (lane < 2) put(mine + lane, round, lane ? (uint32_t)(b >> 32) : (uint32_t)b);
          x = poll(red_slot(q, lane), lane < W);
          const double y = lane < W ? x : (mx ? -INFINITY : 0.0);
          t = mx ? wave_max(y) : wave_sum(y);
          if (PREFIX && q == 0) pv = wave_sum(lane < w ? x : 0.0);
        }
        if (lane == 0) {
          res[q] = t;
          if (PREFIX && q == 0) res[kQ] = pv;
        }
      }
    }
    take();
    lds_barrier();
    failed = L->bad != 0;
    ph ^= 1;
  }

  // Sums s[0..KS) and maxima m[0..KM) over all workgroups, per-thread partials
  // in, totals out (in every thread); PREFIX: *pre receives the sum of s[0]
  // over the workgroups before this one.
  template <int KS, int KM, bool PREFIX, class PUB, class TAKE>
  __device__ __forceinline__ void run(double *s, double *m, double *pre, PUB pub, TAKE take) {
    constexpr int K = KS + KM;
    static_assert(K >= 1 && K <= kQ, "at most kQ values per exchange");
    if (failed) return;
    begin();
    const int lane = lane_id(), wv = wave_id();
    double *r = L->red[ph];
    const double *res = L->res[ph];
#pragma unroll
    for (int k = 0; k < KS; k++) {
      const double v = wave_sum(s[k]);
      if (lane == 0) r[k * NW + wv] = v;
    }
#pragma unroll
    for (int k = 0; k < KM; k++) {
      const double v = wave_max(m[k]);
      if (lane == 0) r[(KS + k) * NW + wv] = v;
    }
    exchange<K, KS, PREFIX>(pub, take);
#pragma unroll
    for (int k = 0; k < KS; k++) s[k] = res[k];
#pragma unroll
    for (int k = 0; k < KM; k++) m[k] = res[KS + k];
    if (PREFIX) *pre = res[kQ];
  }

  // Lane i < K of every wave holds a count of its wave; returns in lane i the
  // total over all waves of all workgroups.
  template <int K>
  __device__ __forceinline__ double counts(double c) {
    if (failed) return 0.0;
    begin();
    const int lane = lane_id();
    if (lane < K) L->red[ph][lane * NW + wave_id()] = c;
    const double *res = L->res[ph];
    exchange<K, K, false>([] {}, [] {});
    return lane < K ? res[lane] : 0.0;
  }

  template <int KS>
  __device__ __forceinline__ void sum(double (&s)[KS]) {
    run<KS, 0, false>(s, nullptr, nullptr, [] {}, [] {});
  }
  template <int KS, int KM>
  __device__ __forceinline__ void summax(double (&s)[KS], double (&m)[KM]) {
    run<KS, KM, false>(s, m, nullptr, [] {}, [] {});
  }

  __device__ __forceinline__ uint64_t tag() const { return (1ull << 32) | round0; }

  // Last exchange done: the next launch continues after this one's rounds (a
  // launch that gave up skips far past any round its peers may have reached).
  __device__ __forceinline__ void finish(const XBuf &xb) const {
    if (threadIdx.x != 0) return;
    if (failed) __hip_atomic_store(xb.lost, tag(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (w == 0) *xb.head = round + (failed ? 1u << 24 : 0u);
  }
};

}  // namespace xwg
}  // namespace
}  // namespace pr

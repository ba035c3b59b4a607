// Learned warm start for child nodes: per-coordinate features, and the MLP
// 8 -> 64 -> 64 -> 1 (ReLU) on gfx950 BF16 MFMA (v_mfma_f32_32x32x16_bf16)
// with FP32 master parameters.  Not part of the paper's method: its output is
// only a candidate starting point that the FP64 duality gap accepts or rejects.
//
// Layout.  A wave takes 32 rows (coordinates) at a time and keeps every layer
// transposed, units x rows: Z1^T = W1 F^T, Z2^T = W2 A1^T, so the weights are
// the A operands (converted once per block) and the activations stay in the MFMA
// C layout, where register v of lane l holds unit 8(v/4) + 4(l/32) + v%4 of row
// l%32.  Turning a C tile into the B operand of the next product (lane l needs
// 8 consecutive units of row l%32) takes one exchange of 4 values between
// lanes l and l^32 per 16-unit step.  The weight gradients are products over
// rows (dW2 = dZ2^T A1, dW1 = dZ1^T F); their operands go through LDS tiles of
// the block's 128 rows and come back by transposing reads.  The bias gradient
// of layer 1 rides on a column of ones next to the 8 features in the dW1
// product.
#include "pr_device.h"
#include "pr_internal.h"

namespace pr {
namespace {

constexpr int kH = 64, kNF = 8;
constexpr int OW1 = 0, OB1 = 512, OW2 = 576, OB2 = 4672, OW3 = 4736, OB3 = 4800;
constexpr int kNP = 4801;
constexpr int kWaves = 4;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// FP32 -> BF16, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ unsigned short f2bf(float f) { return __builtin_bit_cast(unsigned short, (__bf16)f); }
__device__ __forceinline__ bf16x8_t as_bf(u16x8_t u) { return __builtin_bit_cast(bf16x8_t, u); }
__device__ __forceinline__ f32x16_t mma(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// unit (tile row) held in C register v by the lanes of half hh
__device__ __forceinline__ int crow(int v, int hh) { return 8 * (v >> 2) + 4 * hh + (v & 3); }

// B operand of the next product from a C-layout tile: units 16*S .. 16*S+15
// of the tile as the reduction index, the lane's row as the column.  Lane
// l < 32 holds units 16S + 0..3 (registers 8S + i) and 16S + 8..11 (8S + 4 + i)
// and needs 16S + 0..7; lane l + 32 holds 16S + 4..7 and 16S + 12..15 and
// needs 16S + 8..15.  After the conversion a register holds two units, so two
// v_permlane32_swap exchange the upper half of the wave in one register with
// the lower half in the other.
template <int S>
__device__ __forceinline__ bf16x8_t b_from_c(const f32x16_t &c) {
  u32x4_t r;
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const bf16x2_t lo = {(__bf16)c[8 * S + 2 * i], (__bf16)c[8 * S + 2 * i + 1]};
    const bf16x2_t up = {(__bf16)c[8 * S + 4 + 2 * i], (__bf16)c[8 * S + 5 + 2 * i]};
    const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, lo),
                                                     __builtin_bit_cast(unsigned, up), false, false);
    r[i] = sw[0];
    r[2 + i] = sw[1];
  }
  return __builtin_bit_cast(bf16x8_t, r);
}

__device__ __forceinline__ bf16x8_t lds8(const unsigned short *p) {
  return as_bf(*reinterpret_cast<const u16x8_t *>(p));
}

// Values of one 32-unit tile in the C layout's order, from LDS (broadcast reads)
__device__ __forceinline__ f32x16_t units(const float *sp, int hh) {
  f32x16_t r;
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const f32x4_t t = *reinterpret_cast<const f32x4_t *>(sp + 8 * g + 4 * hh);
#pragma unroll
    for (int e = 0; e < 4; e++) r[4 * g + e] = t[e];
  }
  return r;
}

// Weights as MFMA operands (lane: unit, eight consecutive reduction indices),
// BF16.  Layer 1 has 8 inputs and the product 16 reduction indices: the upper
// eight are zero.
__device__ __forceinline__ void load_w1(const float *sp, int lr, int hh, bf16x8_t (&w1)[2]) {
#pragma unroll
  for (int u = 0; u < 2; u++) {
    u16x8_t t;
#pragma unroll
    for (int e = 0; e < 8; e++) t[e] = hh ? (unsigned short)0 : f2bf(sp[OW1 + (32 * u + lr) * kNF + e]);
    w1[u] = as_bf(t);
  }
}
// Layer 2: units 32o .., reduction indices 16s ..; of W2, or of W2^T
__device__ __forceinline__ bf16x8_t load_w2(const float *sp, int lr, int hh, int o, int s, bool transposed) {
  const int k = 16 * s + 8 * hh, u = 32 * o + lr;
  u16x8_t t;
#pragma unroll
  for (int e = 0; e < 8; e++) t[e] = f2bf(sp[OW2 + (transposed ? (k + e) * kH + u : u * kH + k + e)]);
  return as_bf(t);
}

// Forward of the wave's 32 rows (feature operand fb): the activations of layer
// 1 as operands b (lane: row, eight consecutive units), layer 2 after its ReLU
// in a2 (units x rows), and the row's output in every lane.  Starting the
// products from the bias saves nothing: the maximum of an MFMA result with zero
// costs a second instruction, that of a sum does not.  w2(o, s): operand of
// layer 2.
template <class W2>
__device__ __forceinline__ float forward_rows(const bf16x8_t (&w1)[2], const W2 &w2, const float *b1, const float *b2, const float *w3, float b3,
                                              bf16x8_t fb, int hh, bf16x8_t (&b)[4], f32x16_t (&a2)[2]) {
  const f32x16_t zero = {};
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const f32x16_t bias = units(b1 + 32 * u, hh);
    f32x16_t a1 = mma(w1[u], fb, zero);
#pragma unroll
    for (int v = 0; v < 16; v++) a1[v] = fmaxf(a1[v] + bias[v], 0.f);
    b[2 * u] = b_from_c<0>(a1);
    b[2 * u + 1] = b_from_c<1>(a1);
  }
  float po = 0.f;
#pragma unroll
  for (int o = 0; o < 2; o++) {
    const f32x16_t bias = units(b2 + 32 * o, hh), wo = units(w3 + 32 * o, hh);
    a2[o] = zero;
#pragma unroll
    for (int s = 0; s < 4; s++) a2[o] = mma(w2(o, s), b[s], a2[o]);
#pragma unroll
    for (int v = 0; v < 16; v++) {
      a2[o][v] = fmaxf(a2[o][v] + bias[v], 0.f);
      po += wo[v] * a2[o][v];
    }
  }
  return po + __shfl_xor(po, 32) + b3;
}

// out[row] = network output.  Block = 4 waves; block b takes row chunks
// (b * cpb + it) * 4 + wave.
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ P, const uint16_t *__restrict__ F,
                                                     int64_t rows, int cpb, float *__restrict__ out) {
  __shared__ __align__(16) float sp[kNP];
  for (int i = threadIdx.x; i < kNP; i += blockDim.x) sp[i] = P[i];
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, hh = lane >> 5, lr = lane & 31;
  bf16x8_t w1[2], w2[2][4];
  load_w1(sp, lr, hh, w1);
#pragma unroll
  for (int o = 0; o < 2; o++)
#pragma unroll
    for (int s = 0; s < 4; s++) w2[o][s] = load_w2(sp, lr, hh, o, s, false);
  for (int it = 0; it < cpb; it++) {
    const int64_t row = (((int64_t)blockIdx.x * cpb + it) * kWaves + w) * 32 + lr;
    const bool valid = row < rows;
    u16x8_t fu = {0, 0, 0, 0, 0, 0, 0, 0};
    if (valid && hh == 0) fu = *reinterpret_cast<const u16x8_t *>(F + row * kNF);
    bf16x8_t b[4];
    f32x16_t a2[2];
    const float orow = forward_rows(w1, [&](int o, int s) { return w2[o][s]; }, sp + OB1, sp + OB2, sp + OW3, sp[OB3],
                                    as_bf(fu), hh, b, a2);
    if (valid && hh == 0) out[row] = orow;
  }
}

// LDS tiles of the training kernel: kRows rows x 32 units, BF16, rows of 64 B
// whose four 16 B chunks are permuted by bits 2-3 of the row, so that the eight
// rows of a 16 B store and the four rows of a transposing read each cover all
// banks once.
constexpr int kRows = 32 * kWaves;
struct Tile {
  unsigned short v[kRows * 32];
  // units 8c .. 8c+7 of one row
  __device__ __forceinline__ void put(int row, int c, bf16x8_t x) {
    *reinterpret_cast<bf16x8_t *>(&v[row * 32 + ((c ^ ((row >> 2) & 3)) << 3)]) = x;
  }
};
// MFMA operand over rows: lane = unit, rows 16ks + 8hh .. + 7.  A transposing
// read hands lane i of 16 the i-th of 16 units over four rows; the lane's own
// address is that of four units in row i / 4 of them.
__device__ __forceinline__ bf16x8_t rows8(const unsigned short *lo, const unsigned short *up) {
  typedef __attribute__((address_space(3))) s16x4_t lds_t;
  const s16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t *)lo);
  const s16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t *)up);
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// x where the packed activation a (>= 0) is not zero, else 0: two packed 16-bit
// instructions per pair.  (With a constant one the compiler takes the product
// apart into compares and selects of single halves, five per pair.)
__device__ __forceinline__ bf16x8_t relu_mask(bf16x8_t x, bf16x8_t a, unsigned one) {
  const u32x4_t ones = {one, one, one, one};
  return as_bf(__builtin_bit_cast(u16x8_t, x) *
               __builtin_elementwise_min(__builtin_bit_cast(u16x8_t, a), __builtin_bit_cast(u16x8_t, ones)));
}

// Sum of x[v] over the 32 rows of each half of the wave, for all 16 registers
// in 16 exchanges: every step halves the registers a lane is responsible for.
// The lane ends with the sum for register (lane & 15), lane bit 4 apart.
__device__ __forceinline__ float sum_rows(const float (&x)[16], int lane) {
  float t[8];
#pragma unroll
  for (int s = 3; s >= 0; s--) {
    const bool upper = (lane >> s) & 1;
#pragma unroll
    for (int v = 0; v < (1 << s); v++) {
      const float a = s == 3 ? x[v] : t[v], c = s == 3 ? x[v + 8] : t[v + (1 << s)];
      t[v] = (upper ? c : a) + __shfl_xor(upper ? a : c, 1 << s);
    }
  }
  return t[0] + __shfl_xor(t[0], 16);
}

// Forward + backward: block partial sums of the gradient of
// inv_n * sum_rows (out - T)^2 and of sum_rows (out - T)^2 into part[block].
//
// Bound by LDS and vector instructions together: per 128 rows the four waves
// issue about 2600 cycles of LDS accesses and 2000 of vector instructions per
// SIMD beside 960 of MFMA.  The weight gradients are products over rows, so
// their operands are needed transposed: the packed operands of the forward and
// backward products go to LDS as they are (16 B stores) and come back through
// transposing reads.  The waves share the tiles, and each accumulates one
// 32 x 32 quarter of dW2 and, over half the rows, one 32 x 9 half of dW1: 32
// accumulator registers instead of 96, which with layer 2's operands in LDS
// leaves room for two waves per SIMD, and dW2 needs no sum over waves.
// 1M rows 171 -> 71 us, one row 25 -> 13 us, both with the reduction kernel
// (before: 2-byte transposing stores, one wave per SIMD, all accumulators in
// every wave).  Recomputing the transposed operands by MFMAs with their factors
// swapped, without LDS tiles, took 120 us.
__global__ __launch_bounds__(256, 2) void k_mlp_grad(const float *__restrict__ P, const uint16_t *__restrict__ F,
                                                     const float *__restrict__ T, int64_t rows, int cpb, float inv_n,
                                                     float *__restrict__ part) {
  struct Tiles {
    Tile z2[2], a1[2], z1[2];
  };
  __shared__ __align__(16) union {
    Tiles t;
    float sp[kNP];
  } u;
  __shared__ __align__(16) unsigned short t_f[kRows * 16];      // 8 features, a one (bias of layer 1), zeros
  __shared__ __align__(16) unsigned short w2f[16][64 * 8];   // operands of W2, then of W2^T
  __shared__ __align__(16) float s_b1[kH], s_b2[kH], s_w3[kH];
  __shared__ float red[2][kWaves][kH];
  __shared__ float lred[2][kWaves];
  for (int i = threadIdx.x; i < kNP; i += blockDim.x) u.sp[i] = P[i];
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, hh = lane >> 5, lr = lane & 31;
  bf16x8_t w1[2];
  load_w1(u.sp, lr, hh, w1);
  for (int f = w; f < 16; f += kWaves)
    *reinterpret_cast<bf16x8_t *>(&w2f[f][8 * lane]) = load_w2(u.sp, lr, hh, (f >> 2) & 1, f & 3, f >= 8);
  if (threadIdx.x < kH) {
    s_b1[threadIdx.x] = u.sp[OB1 + threadIdx.x];
    s_b2[threadIdx.x] = u.sp[OB2 + threadIdx.x];
    s_w3[threadIdx.x] = u.sp[OW3 + threadIdx.x];
  }
  const float b3 = u.sp[OB3];
  const int lrow = 32 * w + lr;  // the lane's row of the block's 128
  if (hh) *reinterpret_cast<u16x8_t *>(&t_f[lrow * 16 + 8]) = u16x8_t{0x3f80, 0, 0, 0, 0, 0, 0, 0};
  __syncthreads();

  // the lane's addresses in transposing reads, rows 8hh + (0..3) and + 4
  const int i16 = lane & 15, tr = 8 * hh + (i16 >> 2), tc = 2 * ((lane >> 4) & 1) + ((i16 & 3) >> 1);
  const int off0 = tr * 32 + ((tc ^ (2 * hh)) << 3) + 4 * (i16 & 1);
  const int off1 = (tr + 4) * 32 + ((tc ^ (2 * hh + 1)) << 3) + 4 * (i16 & 1);
  const int offf = tr * 16 + 4 * (i16 & 3);  // features: both groups of 16 lanes read the 16 columns

  const int qo = w & 1, qi = w >> 1;  // the wave's quarter of dW2; for dW1: half qo of the units, rows 64 qi ..
  unsigned one = 0x00010001u;
  __asm__("" : "+v"(one));
  const f32x16_t zero = {};
  f32x16_t gW2 = zero, gW1 = zero;
  float gb2[2][16], gw3[2][16], gb3 = 0.f, lsum = 0.f;
#pragma unroll
  for (int o = 0; o < 2; o++)
#pragma unroll
    for (int v = 0; v < 16; v++) gb2[o][v] = gw3[o][v] = 0.f;

  const int64_t row0 = (int64_t)blockIdx.x * cpb * kRows + lrow;
  u16x8_t fu = {0, 0, 0, 0, 0, 0, 0, 0};
  if (row0 < rows && hh == 0) fu = *reinterpret_cast<const u16x8_t *>(F + row0 * kNF);
  float tv = row0 < rows ? T[row0] : 0.f;
  for (int it = 0; it < cpb; it++) {
    const int64_t row = row0 + (int64_t)it * kRows, next = row + kRows;
    const bool valid = row < rows;
    // the next rows' inputs are on their way during this iteration
    u16x8_t fn = {0, 0, 0, 0, 0, 0, 0, 0};
    float tn = 0.f;
    if (it + 1 < cpb && next < rows) {
      if (hh == 0) fn = *reinterpret_cast<const u16x8_t *>(F + next * kNF);
      tn = T[next];
    }

    bf16x8_t b[4], bd[4];
    f32x16_t a2[2];
    const float orow = forward_rows(w1, [&](int o, int s) { return lds8(&w2f[4 * o + s][8 * lane]); }, s_b1,
                                    s_b2, s_w3, b3, as_bf(fu), hh, b, a2);
#pragma unroll
    for (int s = 0; s < 4; s++) u.t.a1[s >> 1].put(lrow, 2 * (s & 1) + hh, b[s]);
    const float d = valid ? orow - tv : 0.f;
    const float dout = 2.f * d * inv_n;
    if (hh == 0) {
      lsum += d * d;
      gb3 += dout;
      *reinterpret_cast<u16x8_t *>(&t_f[lrow * 16]) = fu;
    }
#pragma unroll
    for (int o = 0; o < 2; o++) {
      const f32x16_t wo = units(s_w3 + 32 * o, hh);
#pragma unroll
      for (int v = 0; v < 16; v++) {
        gw3[o][v] += a2[o][v] * dout;
        const float g = wo[v] * dout;
        a2[o][v] = a2[o][v] > 0.f ? g : 0.f;
        gb2[o][v] += a2[o][v];
      }
      bd[2 * o] = b_from_c<0>(a2[o]);
      bd[2 * o + 1] = b_from_c<1>(a2[o]);
    }
#pragma unroll
    for (int s = 0; s < 4; s++) u.t.z2[s >> 1].put(lrow, 2 * (s & 1) + hh, bd[s]);
    // dA1^T = W2^T dZ2^T, then the ReLU mask of layer 1: where its packed activation is not zero
#pragma unroll
    for (int i = 0; i < 2; i++) {
      f32x16_t z = zero;
#pragma unroll
      for (int s = 0; s < 4; s++) z = mma(lds8(&w2f[8 + 4 * i + s][8 * lane]), bd[s], z);
      u.t.z1[i].put(lrow, hh, relu_mask(b_from_c<0>(z), b[2 * i], one));
      u.t.z1[i].put(lrow, 2 + hh, relu_mask(b_from_c<1>(z), b[2 * i + 1], one));
    }
    dev::lds_barrier();
#pragma unroll
    for (int ks = 0; ks < kRows / 16; ks++) {
      const unsigned short *zp = u.t.z2[qo].v + 512 * ks, *ap = u.t.a1[qi].v + 512 * ks;
      gW2 = mma(rows8(zp + off0, zp + off1), rows8(ap + off0, ap + off1), gW2);
      if (ks & 1) {
        const int kf = 4 * qi + (ks >> 1);
        const unsigned short *yp = u.t.z1[qo].v + 512 * kf, *fp = t_f + 256 * kf + offf;
        gW1 = mma(rows8(yp + off0, yp + off1), rows8(fp, fp + 64), gW1);
      }
    }
    dev::lds_barrier();
    fu = fn;
    tv = tn;
  }

  // sums over the block's waves, each in a fixed order
  float *dst = part + (int64_t)blockIdx.x * kMlpPartStride;
#pragma unroll
  for (int v = 0; v < 16; v++) dst[OW2 + (32 * qo + crow(v, hh)) * kH + 32 * qi + lr] = gW2[v];
#pragma unroll
  for (int o = 0; o < 2; o++) {
    const float x = sum_rows(gb2[o], lane), y = sum_rows(gw3[o], lane);
    if ((lane & 16) == 0) {
      red[0][w][32 * o + crow(lane & 15, hh)] = x;
      red[1][w][32 * o + crow(lane & 15, hh)] = y;
    }
  }
#pragma unroll
  for (int m = 1; m < 32; m <<= 1) {
    lsum += __shfl_xor(lsum, m);
    gb3 += __shfl_xor(gb3, m);
  }
  if (lane == 0) {
    lred[0][w] = lsum;
    lred[1][w] = gb3;
  }
  if (qi == 1 && lr <= kNF) {
#pragma unroll
    for (int v = 0; v < 16; v++) u.sp[(32 * qo + crow(v, hh)) * (kNF + 1) + lr] = gW1[v];
  }
  __syncthreads();
  if (qi == 0 && lr <= kNF) {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int un = 32 * qo + crow(v, hh);
      dst[lr < kNF ? OW1 + un * kNF + lr : OB1 + un] = gW1[v] + u.sp[un * (kNF + 1) + lr];
    }
  }
  if (threadIdx.x < 2 * kH) {
    const int q = threadIdx.x / kH, un = threadIdx.x % kH;
    dst[(q ? OW3 : OB2) + un] = ((red[q][0][un] + red[q][1][un]) + red[q][2][un]) + red[q][3][un];
  }
  if (threadIdx.x < 2) {
    const float *l = lred[threadIdx.x];
    dst[threadIdx.x ? OB3 : kNP] = ((l[0] + l[1]) + l[2]) + l[3];
  }
}

// grad[i] = sum over blocks of part[b][i]; grad[kNP] = loss.  A workgroup
// owns 64 consecutive entries (one per lane) and its kRedWaves waves split
// the blocks into contiguous ranges: each wave adds its range in block order
// with the loads of 16 blocks issued together, then lane i of the first wave
// adds the wave totals in wave order, so the sum is fixed and reproducible.
// (One thread per entry walking all blocks left 76 waves on the chip, each
// waiting on nblk / 16 dependent memory round trips.)
constexpr int kRedWaves = 16;
__global__ __launch_bounds__(64 * kRedWaves) void k_mlp_reduce(const float *__restrict__ part, int nblk, float inv_n,
                                                               float *__restrict__ grad) {
  __shared__ float red[kRedWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const int b0 = (int)((int64_t)nblk * w / kRedWaves), b1 = (int)((int64_t)nblk * (w + 1) / kRedWaves);
  constexpr int kBatch = 16;
  float s = 0.f;
  if (i <= kNP) {
    int b = b0;
    for (; b + kBatch <= b1; b += kBatch) {
      float v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; u++) v[u] = part[(int64_t)(b + u) * kMlpPartStride + i];
#pragma unroll
      for (int u = 0; u < kBatch; u++) s += v[u];
    }
    for (; b < b1; b++) s += part[(int64_t)b * kMlpPartStride + i];
  }
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && i <= kNP) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kRedWaves; k++) t += red[k][lane];
    grad[i] = i == kNP ? t * inv_n : t;
  }
}

__global__ __launch_bounds__(256) void k_mlp_adam(float *__restrict__ P, const float *__restrict__ g,
                                                  float *__restrict__ m1, float *__restrict__ m2, float lr,
                                                  float beta1, float beta2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kNP) return;
  const float gi = g[i];
  const float m = beta1 * m1[i] + (1.f - beta1) * gi;
  const float v = beta2 * m2[i] + (1.f - beta2) * gi * gi;
  m1[i] = m;
  m2[i] = v;
  P[i] -= lr * (m * c1) / (sqrtf(v * c2) + eps);
}

// Feature kernels, grid.y (or grid.x of the prologue) = node; every vector of
// node q starts at q * p.
//
// Prologue, one workgroup per node: fs[q] = {max |w|, nnz} and the nonzero
// magnitudes of beta compacted into nzv with their coordinates in nzi (in
// thread order: ranks only count).  Two passes of coalesced loads, eight in
// flight; a pass in index order, three barriers per 512 entries, took 16 us at
// p = 8192.
__global__ __launch_bounds__(dev::NT) void k_feat_prep(const double *__restrict__ beta, const double *__restrict__ w,
                                                       int64_t p, double *__restrict__ nzv, int32_t *__restrict__ nzi,
                                                       double *__restrict__ fs) {
  using namespace dev;
  __shared__ double red[NW];
  __shared__ int scan[NW];
  const int64_t o = (int64_t)blockIdx.x * p;
  beta += o;
  w += o;
  double hm = 0.0;
  int c = 0;
#pragma unroll 8
  for (int64_t j = threadIdx.x; j < p; j += NT) {
    hm = fmax(hm, fabs(w[j]));
    c += beta[j] != 0.0;
  }
  int tot;
  int at = block_excl_scan<NT>(c, scan, &tot);
#pragma unroll 8
  for (int64_t j = threadIdx.x; j < p; j += NT) {
    const double b = beta[j];
    if (b != 0.0) {
      nzv[o + at] = fabs(b);
      nzi[o + at] = (int32_t)j;
      at++;
    }
  }
  hm = block_max<NT>(hm, red);
  if (threadIdx.x == 0) {
    fs[2 * blockIdx.x] = hm;
    fs[2 * blockIdx.x + 1] = (double)tot;
  }
}

// rank[q][j] = #{i : |beta_i| > |beta_j|} of every nonzero beta_j.  Bound by the
// compares of one wave after another: a workgroup takes 64 entries of the node's
// compacted list, one per lane, its four waves each compare them with a quarter
// of every LDS tile of the list, and the counts are added.  The list is as long as
// the support, so only its entries pay for it (with the loop in the kernel that
// writes the rows, the few lanes with a nonzero coordinate kept their whole wave
// for nnz dependent loads: 87 us per node at p = 8192, nnz = 1200; 32 such nodes
// took 28.5 us with 256 entries per workgroup and the whole list per wave, 11.4 so).
constexpr int kRankTile = 1024;
__global__ __launch_bounds__(256) void k_feat_rank(const double *__restrict__ nzv, const int32_t *__restrict__ nzi,
                                                   const double *__restrict__ fs, int64_t p,
                                                   int32_t *__restrict__ rank) {
  __shared__ __align__(16) double tile[kRankTile];
  __shared__ int cnt[kWaves][64];
  const int64_t o = (int64_t)blockIdx.y * p;
  const int nnz = (int)fs[2 * blockIdx.y + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int i0 = (int)blockIdx.x * 64; i0 < nnz; i0 += (int)gridDim.x * 64) {
    const int i = i0 + lane;
    const double a = i < nnz ? nzv[o + i] : INFINITY;
    int r = 0;
    for (int t0 = 0; t0 < nnz; t0 += kRankTile) {
      __syncthreads();
      for (int t = threadIdx.x; t < kRankTile; t += 256) tile[t] = t0 + t < nnz ? nzv[o + t0 + t] : 0.0;
      __syncthreads();
      // a quarter of the entries left, in eights (zeros pad the last tile)
      const int left = nnz - t0 < kRankTile ? nnz - t0 : kRankTile;
      const int q = ((left + kWaves - 1) / kWaves + 7) & ~7;
      const int e = (w + 1) * q < kRankTile ? (w + 1) * q : kRankTile;
#pragma unroll 8
      for (int t = w * q; t < e; t++) r += tile[t] > a;
    }
    cnt[w][lane] = r;
    __syncthreads();
    if (w == 0 && i < nnz) rank[o + nzi[o + i]] = ((cnt[0][lane] + cnt[1][lane]) + cnt[2][lane]) + cnt[3][lane];
  }
}

// The rows.  With RANK the ranks are counted here, every lane's against LDS tiles
// of the whole list, and there is no launch of k_feat_rank.
template <bool RANK>
__global__ __launch_bounds__(256) void k_feat_rows(const double *__restrict__ beta, const double *__restrict__ w,
                                                   const int8_t *__restrict__ st, int64_t p,
                                                   const double *__restrict__ nzv, const int32_t *__restrict__ rank,
                                                   const double *__restrict__ fs,
                                                   const FeatScalars *__restrict__ scs, FeatScalars one,
                                                   const double *__restrict__ beta_child, uint16_t *__restrict__ F,
                                                   float *__restrict__ T) {
  const int64_t jj = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t j = (int64_t)blockIdx.y * p + jj;
  const double hm = fs[2 * blockIdx.y], nnz = fs[2 * blockIdx.y + 1];
  const FeatScalars sc = scs ? scs[blockIdx.y] : one;
  const double b = jj < p ? beta[j] : 0.0;
  int r = 0;
  if constexpr (RANK) {
    __shared__ __align__(16) double tile[kRankTile];
    const double *list = nzv + (int64_t)blockIdx.y * p;
    const int len = (int)nnz;
    const double a = fabs(b);
    const bool any = __any(b != 0.0);
    for (int t0 = 0; t0 < len; t0 += kRankTile) {
      __syncthreads();
      for (int t = threadIdx.x; t < kRankTile; t += 256) tile[t] = t0 + t < len ? list[t0 + t] : 0.0;
      __syncthreads();
      const int e = any ? ((len - t0 < kRankTile ? len - t0 : kRankTile) + 7) & ~7 : 0;
#pragma unroll 8
      for (int t = 0; t < e; t++) r += tile[t] > a;
    }
  }
  if (jj >= p) return;
  if constexpr (!RANK) r = b != 0.0 ? rank[j] : 0;
  const int s = st[j];
  double f[kNF];
  f[0] = b;
  f[1] = hm > 0.0 ? w[j] / hm : 0.0;
  f[2] = (b != 0.0 ? (double)r : nnz) / (double)p;
  f[3] = s == kZero ? -1.0 : (s == kOne ? 1.0 : 0.0);
  f[4] = sc.lambda2;
  f[5] = (double)sc.n1 / sc.k;
  f[6] = (double)sc.n0 / sc.k;
  f[7] = (double)sc.kbar / sc.k;
  u16x8_t u;
#pragma unroll
  for (int e = 0; e < kNF; e++) u[e] = f2bf((float)f[e]);
  *reinterpret_cast<u16x8_t *>(F + j * kNF) = u;
  if (T && beta_child) T[j] = (float)(beta_child[j] - b);
}

// vhat = beta + out (the network's proposal before the prox step)
__global__ void k_mlp_propose(const double *__restrict__ beta, const float *__restrict__ out, int64_t p,
                              double *__restrict__ vhat) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < p; j += (int64_t)gridDim.x * blockDim.x)
    vhat[j] = beta[j] + (double)out[j];
}

}  // namespace

int mlp_grid(int64_t rows, int *cpb) {
  const int64_t per = 32 * kWaves;
  int64_t c = (rows + per * 512 - 1) / (per * 512);
  if (c < 1) c = 1;
  *cpb = (int)c;
  return (int)((rows + per * c - 1) / (per * c));
}

hipError_t launch_mlp_forward(const float *P, const uint16_t *F, int64_t rows, float *out, hipStream_t s) {
  int cpb;
  const int blocks = mlp_grid(rows, &cpb);
  k_mlp_forward<<<blocks, 256, 0, s>>>(P, F, rows, cpb, out);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const float *P, const uint16_t *F, const float *T, int64_t rows, float *part,
                           float *grad, hipStream_t s) {
  int cpb;
  const int blocks = mlp_grid(rows, &cpb);
  const float inv_n = 1.0f / (float)rows;
  k_mlp_grad<<<blocks, 256, 0, s>>>(P, F, T, rows, cpb, inv_n, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_mlp_reduce<<<(kNP + 1 + 63) / 64, 64 * kRedWaves, 0, s>>>(part, blocks, inv_n, grad);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float *P, const float *g, float *m1, float *m2, float lr, float beta1, float beta2,
                           float eps, float c1, float c2, hipStream_t s) {
  k_mlp_adam<<<(kNP + 255) / 256, 256, 0, s>>>(P, g, m1, m2, lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError();
}

// A single node of p <= 4096 has its ranks counted by the kernel that writes its
// rows: the launch of k_feat_rank was the eighth operation of a one-node call, and
// from the eighth on the runtime's wait takes some 20 us longer (512 x 512: 40-44 us
// with neither it nor a second upload, 67 with the launch, 41 so; 256 x 1152 54,
// 68, 43; 512 x 4096 94, 67, 53).  At 8192 both take 70 us, at 16384 (a seventh of
// the entries nonzero) 91 with the launch and 100 without.
constexpr int64_t kRankRows = 4096;
hipError_t launch_features(const double *beta, const double *w, const int8_t *st, int64_t p, int m,
                           const FeatBufs &fb, const FeatScalars *one, const double *beta_child, uint16_t *F, float *T,
                           hipStream_t s) {
  if (m < 1 || m > kFeatNodes || (one && m != 1)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((p + 255) / 256), (unsigned)m);
  k_feat_prep<<<(unsigned)m, dev::NT, 0, s>>>(beta, w, p, fb.nzv, fb.nzi, fb.fs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (one && p <= kRankRows) {
    k_feat_rows<true><<<grid, 256, 0, s>>>(beta, w, st, p, fb.nzv, nullptr, fb.fs, nullptr, *one, beta_child, F, T);
    return hipGetLastError();
  }
  k_feat_rank<<<grid, 256, 0, s>>>(fb.nzv, fb.nzi, fb.fs, p, fb.rank);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_feat_rows<false><<<grid, 256, 0, s>>>(beta, w, st, p, fb.nzv, fb.rank, fb.fs, one ? nullptr : fb.sc,
                                          one ? *one : FeatScalars{}, beta_child, F, T);
  return hipGetLastError();
}

hipError_t launch_mlp_propose(const double *beta, const float *out, int64_t p, double *vhat, hipStream_t s) {
  k_mlp_propose<<<(unsigned)((p + 255) / 256 < 1024 ? (p + 255) / 256 : 1024), 256, 0, s>>>(beta, out, p, vhat);
  return hipGetLastError();
}

}  // namespace pr

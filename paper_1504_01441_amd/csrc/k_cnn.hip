// k_cnn.hip -- the learned displacement proposal (an extension beyond the
// paper: a small CNN predicts each level-0 tile's displacement so that the
// Sec. 2.2 search only scans a window around it). Inference and training run
// on the matrix cores: every convolution is an implicit GEMM on
// v_mfma_f32_16x16x16_bf16 (bf16 operands, fp32 accumulation).
//
// Network (per tile): x [16][16][4] -> conv3x3 s1 -> 32 ch [16][16] -> conv s2
// -> [8][8] -> conv s1 -> [8][8] -> conv s2 -> [4][4] -> linear 512 -> 3,
// ReLU after every convolution, activations rounded to bf16; outputs
// (dx / 8, dy / 8, confidence logit). On the device, activations are NHWC
// (32 channels innermost) so that an MFMA operand is one 8-byte load.
//
// MFMA 16x16x16 operand layout (lane l, r = l % 16, g = l / 16, j = 0..3):
//   A[r][4g + j],  B[4g + j][r],  D[4g + j][r].
//
//  k_cnn_set      loads fp32 master parameters: clears the AdamW moments and
//                 writes the bf16 weight layouts for the kernels
//  k_cnn_input    tile pairs -> network input: the tiles' 2x2 sums and the
//                 64 x 64 windows' 4x4 sums (bf16), for listed tiles
//  k_cnn_fwd      one or four samples per workgroup at a time, four waves per
//                 sample (each a quarter of every layer's output tiles),
//                 weights shared in LDS;
//                 inference writes the proposal (window centre, fallback
//                 flag), training writes the activations and outputs
//  k_cnn_bwd      loss, output gradient and back-propagation through the ReLUs
//                 and the transposed convolutions (activation gradients), one
//                 sample per workgroup at a time
//  k_cnn_wgrad    weight and bias gradients of every layer, per block of samples
//  k_cnn_adamw    sums the per-block gradients, applies AdamW (fp32) and
//                 refreshes the bf16 layouts
#include "lnr_device.h"
#include "lnr_internal.h"

namespace lnr {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int CH = 32;
constexpr int kWave = 64;
constexpr int kFwdGroupWaves = 4;  // forward: waves per sample
// the forward workgroup holds four samples at a time; one where the samples
// would leave CUs without a workgroup (training forward of 256 samples: 16 us
// on 256 workgroups, with 16-byte activation stores; 48 us on 64, 2-byte)
constexpr int kFwdMany = 4;

constexpr int C1 = 4;              // input channels
constexpr int kIn = C1 * 256;       // input values per sample

// flat parameter vector: W1[32][4][3][3] b1 W2[32][32][3][3] b2 W3 b3 W4 b4
// Wh[3][512] bh[3]
constexpr int kOffW[4] = {0, 1184, 10432, 19680};
constexpr int kOffB[4] = {1152, 10400, 19648, 28896};
constexpr int kOffWh = 28928, kOffBh = 30464, kNParam = 30467;

// packed bf16 weights: W1p[32 co][48 k] (k = tap * 4 + ci, zero from 36),
// Wp[l][32 co][9 tap][32 ci] and the transposes WT[l][32 ci][9 tap][32 co]
constexpr int kK1 = 48;
constexpr int kW1p = CH * kK1;
constexpr int kWp = CH * 9 * CH;
constexpr int kPacked = kW1p + 3 * kWp + 3 * kWp;

// per-sample stored activations (bf16, NHWC): x, a1, a2, a3, a4
constexpr int kActX = 0, kActA1 = kIn, kActA2 = kActA1 + 8192, kActA3 = kActA2 + 2048,
              kActA4 = kActA3 + 2048, kActN = kActA4 + 512;
// per-sample activation gradients after the ReLU (bf16, channel-major [c][p])
constexpr int kDz1 = 0, kDz2 = 8192, kDz3 = kDz2 + 2048, kDz4 = kDz3 + 2048,
              kDzN = kDz4 + 512;

__device__ inline uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ inline f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
// relu(v + bias) of four channels as bf16 (hardware conversion, the rounding of
// f2bf; no NaN is left after the maximum), one 8-byte store
__device__ inline void st4_relu(uint16_t* p, const f32x4& v, const f32x4& bias) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 h2 __attribute__((ext_vector_type(2)));
  const f32x2 lo = {fmaxf(v[0] + bias[0], 0.f), fmaxf(v[1] + bias[1], 0.f)};
  const f32x2 hi = {fmaxf(v[2] + bias[2], 0.f), fmaxf(v[3] + bias[3], 0.f)};
  const h2 a = __builtin_convertvector(lo, h2), b = __builtin_convertvector(hi, h2);
  *reinterpret_cast<uint2*>(p) =
      make_uint2(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b));
}
__device__ inline bf16x4 ld4(const uint16_t* p) { return *reinterpret_cast<const bf16x4*>(p); }

// Parameter i's place(s) in the packed layouts (none for biases and the head).
__device__ inline void pack_param(int i, float v, uint16_t* __restrict__ pk) {
  if (i < kOffB[0]) {
    const int co = i / (9 * C1), ci = i / 9 % C1, tap = i % 9;
    pk[co * kK1 + tap * C1 + ci] = f2bf(v);
    return;
  }
#pragma unroll
  for (int l = 1; l < 4; ++l) {
    const int e = i - kOffW[l];
    if (e >= 0 && i < kOffB[l]) {
      const int co = e / (9 * CH), ci = e / 9 % CH, tap = e % 9;
      const uint16_t h = f2bf(v);
      uint16_t* w = pk + kW1p + (l - 1) * kWp;
      w[(co * 9 + tap) * CH + ci] = h;
      w[3 * kWp + (ci * 9 + tap) * CH + co] = h;
    }
  }
}

// Master parameters P[0, kNParam) from src (null: P already holds them), the
// moments after them cleared with `fresh`, and the packed layouts.
__global__ __launch_bounds__(256) void k_cnn_set(const float* __restrict__ src,
                                                 float* __restrict__ P, int fresh,
                                                 uint16_t* __restrict__ pk) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < CH * (kK1 - 9 * C1))  // W1's zero columns
    pk[i / (kK1 - 9 * C1) * kK1 + 9 * C1 + i % (kK1 - 9 * C1)] = 0;
  if (i >= kNParam) return;
  const float v = src ? src[i] : P[i];
  if (src) P[i] = v;
  if (fresh) P[kNParam + i] = P[2 * kNParam + i] = 0.f;
  pack_param(i, v, pk);
}

// Network inputs: sample i is tile tiles[i] (tile i without a list), i below
// *count (or n). The 64 x 64 windows of both images around the tile (16 px
// on every side; rows and columns outside the image repeat the edge) are
// staged in workgroup memory; channels 0, 1 are the 2x2 sums of the central
// 32 x 32 tile, channels 2, 3 the 4x4 sums of the window, each value
// bf16((s - mid) / scale), exact before the one rounding. Bound by latency: 16
// us for a 5 MP pair with a dword's loads per turn of a loop, 12 with a thread's
// eight in flight together.
__global__ __launch_bounds__(256) void k_cnn_input(const uint8_t* __restrict__ ref,
                                                   const uint8_t* __restrict__ wrp, int w, int h,
                                                   int ntx, const int32_t* __restrict__ tiles,
                                                   const int* __restrict__ count, int n,
                                                   uint16_t* __restrict__ x) {
  __shared__ uint32_t win[2][64][16];
  const int i = blockIdx.x;
  const int m = count ? *count : n;
  if (i >= m) return;
  const int t = tiles ? tiles[i] : i;
  const int x0 = (t % ntx) * 32 - 16, y0 = (t / ntx) * 32 - 16;
  // a thread's eight dwords (column d of rows 16 apart, both images) all in
  // flight before the first is stored; the branch is the tile's column's
  const int d = threadIdx.x & 15, xs = x0 + 4 * d;
  uint32_t v[8];
  const uint8_t* rows[8];
#pragma unroll
  for (int q = 0; q < 8; ++q)
    rows[q] = (q >> 2 ? wrp : ref) +
              (size_t)min(max(y0 + (q & 3) * 16 + (int)(threadIdx.x >> 4), 0), h - 1) * w;
  if (xs >= 0 && xs + 4 <= w) {
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = reinterpret_cast<const UnalignedU32*>(rows[q] + xs)->v;
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      v[q] = 0;
      for (int b = 0; b < 4; ++b)
        v[q] |= (uint32_t)rows[q][min(max(xs + b, 0), w - 1)] << (8 * b);
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) win[q >> 2][(q & 3) * 16 + (threadIdx.x >> 4)][d] = v[q];
  __syncthreads();
  uint16_t* xo = x + (size_t)i * kIn;
  const uint8_t* wb = reinterpret_cast<const uint8_t*>(win);
  for (int k = threadIdx.x; k < kIn; k += 256) {
    const int c = k >> 8, yi = (k >> 4) & 15, xj = k & 15;
    const int img = c & 1;
    float v;
    if (c < 2) {
      const uint8_t* p0 = wb + (img * 64 + 16 + 2 * yi) * 64 + 16 + 2 * xj;
      const int s = p0[0] + p0[1] + p0[64] + p0[65];
      v = (float)(s - 510) * (1.f / 512.f);
    } else {
      uint32_t s = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        s = __builtin_amdgcn_udot4(win[img][4 * yi + u][xj], 0x01010101u, s, false);
      v = (float)((int)s - 2040) * (1.f / 2048.f);
    }
    xo[k] = f2bf(v);
  }
}

// The forward layers, each computed by the four waves of a sample (part):
// conv1 (2 -> 32, stride 1; K = 18 (tap, ci) padded to 32) four of its 16
// position tiles per wave, the 32 -> 32 layers (3x3, pad 1, stride S, NHWC
// bf16 in / out, W [co][tap][ci]) one position tile per wave, and the last
// layer's two channel halves on parts 0 and 1. Every output element sums its
// MFMA products in (tap, channel half) order. The weights are the products'
// left operand: a lane then receives four neighbouring channels of a position,
// which are converted in pairs and stored in 8 bytes (with the activations on
// the left it holds one channel of four positions, 2-byte stores).
// (Their LDS layouts: act_at below.)
//
// The backward's LDS: a position's 32 channels take kPS elements (80 bytes)
// and a weight row kWS (592 bytes), which spreads the 16 rows of an operand
// over half of the bank pairs (unpadded: one or two of them).
constexpr int kPS = 40;
constexpr int kWS = 9 * CH + 8;

// `rows` rows of N elements into rows of STRIDE elements in LDS, 16 bytes per
// thread, all of a thread's loads (up to eight) in flight before its stores
template <int N, int STRIDE>
__device__ inline void load_rows(const uint16_t* __restrict__ src, uint16_t* dst, int rows,
                                 int tid, int nt) {
  static_assert(N % 8 == 0 && STRIDE % 8 == 0, "16-byte rows");
  const int total = rows * (N / 8);
  for (int i0 = tid; i0 < total; i0 += 8 * nt) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = reinterpret_cast<const uint4*>(src)[min(i0 + u * nt, total - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * nt;
      if (i < total) *reinterpret_cast<uint4*>(dst + i / (N / 8) * STRIDE + i % (N / 8) * 8) = v[u];
    }
  }
}

// The forward's LDS layouts. An operand read takes the 8-byte units of one
// channel group from 16 rows (positions, or output channels), 16 lanes at a
// time; unpadded rows of 64 or 576 bytes would put them in one or two of the
// 16 pairs of banks. So unit c (channels 4c .. 4c + 3) of a row is held at c
// XOR a number that counts through the rows of an operand, and where a layer's
// operand takes every other position, neighbouring positions change places on
// every other of its image rows: no conflicts on any operand. (Rows padded to
// 80 and 592 bytes: half of the LDS cycles were conflicts.)
// Element offset of unit c at position pos of the activations of layer A (0:
// a4, not read as an operand; 1: a1, 16 x 16, stride 2; 2: a2, 8 x 8, stride 1;
// 3: a3, 8 x 8, stride 2):
template <int A>
__device__ inline int act_at(int pos, int c) {
  if constexpr (A == 1) return (((pos ^ ((pos >> 5) & 1)) << 3) + (c ^ ((pos >> 1) & 7))) * 4;
  if constexpr (A == 2) return ((pos << 3) + (c ^ ((pos >> 1) & 7))) * 4;
  if constexpr (A == 3)
    return (((pos ^ ((pos >> 5) & 1)) << 3) + (c ^ (((pos >> 1) & 3) | ((pos >> 2) & 4)))) * 4;
  return ((pos << 3) + c) * 4;
}
constexpr int kK1S = kK1 + 4;  // W1's rows: an odd number of units

// W2 .. W4, `rows` rows [co][9 tap][32 ci], into LDS: unit c of a tap at c XOR
// (co / 2) % 8
__device__ inline void load_weights(const uint16_t* __restrict__ src, uint16_t* dst, int rows,
                                    int tid, int nt) {
  constexpr int N = 9 * CH / 8;  // 16-byte loads (two units) per row
  const int total = rows * N;
  for (int i0 = tid; i0 < total; i0 += 8 * nt) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = reinterpret_cast<const uint4*>(src)[min(i0 + u * nt, total - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * nt;
      if (i >= total) break;
      const int row = i / N, c = 2 * (i % N), sw = (row >> 1) & 7;
      uint2* d = reinterpret_cast<uint2*>(dst + row * 9 * CH);
      d[c ^ sw] = make_uint2(v[u].x, v[u].y);
      d[(c + 1) ^ sw] = make_uint2(v[u].z, v[u].w);
    }
  }
}

// Lane constants of a wave's operand reads, as byte offsets into the
// workgroup's memory, formed once: with the bounds tests and the layouts'
// arithmetic in every product's read, the vector ALU, not the matrix cores or
// the LDS, took most of the time. Positions outside a layer read zeros.
struct FwdOffsets {
  int c1[3];                 // conv1: the tap of step ks, in the wave's first row
  int c2[9], c3[9];          // unit g of each tap; the other half's is at XOR 32
  int wt;                    // unit g of weight row r; the other half's at XOR 32
};

template <int HIN, int HOUT, int S, int A>
__device__ inline void tap_offsets(int (&o)[9], int base, int zero, int m, int g) {
  const int oy = m / HOUT, ox = m % HOUT;
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    const int iy = oy * S + tap / 3 - 1, ix = ox * S + tap % 3 - 1;
    const bool ok = iy >= 0 && iy < HIN && ix >= 0 && ix < HIN;
    o[tap] = ok ? base + 2 * act_at<A>(iy * HIN + ix, g) : zero;
    asm volatile("" : "+v"(o[tap]));  // (held, not formed again for every sample)
  }
}

__device__ inline bf16x4 lds4(const uint8_t* sm, int off) {
  return *reinterpret_cast<const bf16x4*>(sm + off);
}

// x in LDS: 18 x 18 positions of 4 channels, zeros around the 16 x 16
constexpr int kXW = 18, kXElems = kXW * kXW * C1;

__device__ inline void conv1_fwd_part(const uint8_t* sm, const FwdOffsets& f, const uint16_t* W1p,
                                      const float* bias, uint16_t* out, int lane, int part) {
  // K = (tap, ci) = tap * 4 + ci over three steps of 16: step ks covers taps
  // 4 ks .. 4 ks + 3, lane group g one tap's four channels (one 8-byte load)
  const int r = lane & 15, g = lane >> 4;
  f32x4 acc[4][2];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u][0] = acc[u][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < 3; ++ks) {
    const bf16x4 b0 = ld4(W1p + r * kK1S + ks * 16 + g * 4);
    const bf16x4 b1 = ld4(W1p + (16 + r) * kK1S + ks * 16 + g * 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bf16x4 a = lds4(sm, f.c1[ks] + u * kXW * C1 * 2);
      acc[u][0] = mfma(b0, a, acc[u][0]);
      acc[u][1] = mfma(b1, a, acc[u][1]);
    }
    __builtin_amdgcn_sched_barrier(0);  // (all steps' operands at once: spills)
  }
  const f32x4 c0 = *reinterpret_cast<const f32x4*>(bias + 4 * g);
  const f32x4 c1 = *reinterpret_cast<const f32x4*>(bias + 16 + 4 * g);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    // act_at<1> of position (4 part + u) 16 + r: u decides the exchange
    const int p = r ^ (u >> 1), at = ((p << 3) + (g ^ (r >> 1))) * 4;
    uint16_t* o = out + (4 * part + u) * 16 * CH;
    st4_relu(o + at, acc[u][0], c0);
    st4_relu(o + (at ^ 16), acc[u][1], c1);
  }
}

// MT == 4: position tile `part`, both channel halves; MT == 1: channel half
// `part` of the single position tile (parts 2, 3 idle). o: the taps' offsets;
// wt: the layer's first weight row's.
template <int MT, int B>
__device__ inline void conv_fwd_part(const uint8_t* sm, const int (&o)[9], int wt,
                                     const float* bias, uint16_t* out, int lane, int part) {
  const int r = lane & 15, g = lane >> 4;
  constexpr int NT = MT == 4 ? 2 : 1;
  if (MT == 1 && part >= 2) return;
  const int n0 = MT == 4 ? 0 : part;
  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int w = wt + n0 * 16 * 9 * CH * 2;
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const bf16x4 a = lds4(sm, o[tap] ^ (32 * half));
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[nt] = mfma(lds4(sm, (w ^ (32 * half)) + (nt * 16 * 9 + tap) * CH * 2), a, acc[nt]);
    }
    if (tap % 3 == 2) __builtin_amdgcn_sched_barrier(0);  // (all taps' operands at once: spills)
  }
  const int m = (MT == 4 ? part : 0) * 16 + r;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    st4_relu(out + act_at<B>(m, (n0 + nt) * 4 + g), acc[nt],
             *reinterpret_cast<const f32x4*>(bias + (n0 + nt) * 16 + 4 * g));
}

struct ProposalOut {
  int32_t* centre;    // [ntiles][2] window centre (null: not wanted)
  uint8_t* fallback;  // [ntiles] 1: exhaustive search
  int clampc;         // |centre| <= clampc
  float conf_logit;   // window search when the logit is >= this
  const int32_t* tiles;  // sample -> tile (null: sample s is tile s)
  const int* count;      // samples (device; null: the launch's n)
  int* lists;            // window tiles [0, ntiles), fallback tiles [ntiles, 2 ntiles)
  int* counts;           // [2] entries of the two lists
  int ntiles;
};

// LDS: packed weights (W1p with padded rows, then W2..W4) and biases, shared
// by the workgroup's waves; then per sample in flight a 256-position and a
// 64-position activation buffer (x -> a1 -> a2 -> a3 -> a4 ping-pong). The
// head's weights are read from global memory.
constexpr int kFwdLdsWeights = (CH * kK1S + 3 * kWp) * 2 + 4 * CH * 4;
constexpr int kFwdBufA = 256 * CH, kFwdBufB = 64 * CH;  // elements
constexpr int kFwdLdsSample = (kFwdBufA + kFwdBufB) * 2;
constexpr int kFwdZero = 512;  // bytes of zeros, read for positions outside a layer
constexpr int fwd_lds(int spb) { return kFwdLdsWeights + spb * kFwdLdsSample + kFwdZero; }
static_assert(kFwdLdsWeights % 64 == 0 && kFwdLdsSample % 64 == 0 && kFwdBufA % 32 == 0,
              "XOR 32 stays in a position's 64 bytes");
static_assert(3 * kXW * C1 * 2 + 40 <= kFwdZero, "conv1 reads its four rows of zeros");
static_assert(fwd_lds(kFwdMany) <= 160 * 1024, "forward workgroup LDS");

// a1 .. a4 as stored for training: position * 32 + channel, 8 channels (one
// 16-byte store) at a time
template <int A>
__device__ inline void store_acts(const uint16_t* buf, uint16_t* __restrict__ out, int npos,
                                  int gt, int nt) {
  for (int i = gt; i < npos * 4; i += nt) {
    const uint2 lo = *reinterpret_cast<const uint2*>(buf + act_at<A>(i >> 2, 2 * (i & 3)));
    const uint2 hi = *reinterpret_cast<const uint2*>(buf + act_at<A>(i >> 2, 2 * (i & 3) + 1));
    reinterpret_cast<uint4*>(out)[i] = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
}

// Bound by the LDS reads (an activation and two weight operands for two matrix
// products: 18 us for 4860 samples; the products alone 13) and by the waits
// between the layers, whose waves run in step. 4860 samples take 35 us; 55
// with seven barriers per sample, the input staged and the head run by
// themselves, 2-byte activation stores and conflicts on half of the LDS cycles.
// (Traced, step by step: 61 us; stores, input and head 48; layouts 42; lane
// constants 41.)
template <bool TRAIN, int SPB>
__global__ __launch_bounds__(SPB * kFwdGroupWaves * kWave) void k_cnn_fwd(
    const uint16_t* __restrict__ pk, const float* __restrict__ P, const uint16_t* __restrict__ x,
    int n, float* __restrict__ out, uint16_t* __restrict__ acts, ProposalOut po) {
  extern __shared__ __align__(16) uint8_t sm[];
  if (po.count) n = *po.count;
  uint16_t* sW1 = reinterpret_cast<uint16_t*>(sm);
  uint16_t* sW = sW1 + CH * kK1S;  // [3][32 co][9 tap][32 ci]
  float* sb = reinterpret_cast<float*>(sW + 3 * kWp);  // [4][32]
  const int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // a group's parts are rotated, so that the parts that are idle in the last
  // layer or run the head are on different SIMDs
  const int grp = wave / kFwdGroupWaves, part = (wave + grp) % kFwdGroupWaves;
  const int gt = part * kWave + lane;  // thread index within the sample's group
  constexpr int GT = kFwdGroupWaves * kWave;
  {
    for (int i = tid; i < CH * kK1 / 4; i += SPB * GT)
      reinterpret_cast<uint2*>(sW1)[i / (kK1 / 4) * (kK1S / 4) + i % (kK1 / 4)] =
          reinterpret_cast<const uint2*>(pk)[i];
    load_weights(pk + kW1p, sW, 3 * CH, tid, SPB * GT);
    for (int i = tid; i < 4 * CH; i += blockDim.x) sb[i] = P[kOffB[i / CH] + i % CH];
  }
  uint16_t* bufA = reinterpret_cast<uint16_t*>(sm + kFwdLdsWeights + grp * kFwdLdsSample);
  uint16_t* bufB = bufA + kFwdBufA;
  uint16_t* bufX = bufB + kXElems;  // a4, past the network input in bufB
  static_assert(kXElems + 16 * CH <= kFwdBufB, "a4 beside x");
  const int oA = kFwdLdsWeights + grp * kFwdLdsSample, oB = oA + kFwdBufA * 2;
  const int oZ = kFwdLdsWeights + SPB * kFwdLdsSample;
  if (tid < kFwdZero / 4) reinterpret_cast<uint32_t*>(sm + oZ)[tid] = 0u;
  FwdOffsets fo;
  {
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      const int tap = 4 * ks + g;
      fo.c1[ks] = tap < 9 ? oB + ((4 * part + tap / 3) * kXW + r + tap % 3) * C1 * 2 : oZ;
      asm volatile("" : "+v"(fo.c1[ks]));
    }
    tap_offsets<16, 8, 2, 1>(fo.c2, oA, oZ, part * 16 + r, g);
    tap_offsets<8, 8, 1, 2>(fo.c3, oB, oZ, part * 16 + r, g);
    fo.wt = CH * kK1S * 2 + (r * 9 * CH + 4 * (g ^ ((r >> 1) & 7))) * 2;
    static_assert(CH * kK1S * 2 % 64 == 0, "XOR 32 stays in a tap's 64 bytes");
  }
  // x: NCHW [4][16][16] -> NHWC in bufB with its border, two positions per
  // thread of parts 2 and 3 (x may be aligned to its elements only)
  const int xq = 2 * (gt - GT / 2);
  auto fetch = [&](int s, uint32_t (&v)[C1]) {
#pragma unroll
    for (int c = 0; c < C1; ++c)
      v[c] = part >= 2 && s < n
                 ? reinterpret_cast<const UnalignedU32*>(x + (size_t)s * kIn + c * 256 + xq)->v
                 : 0u;
  };
  auto put = [&](const uint32_t (&v)[C1]) {
    if (part < 2) return;
    uint2* d = reinterpret_cast<uint2*>(bufB);  // one position each
    const int q = (xq / 16 + 1) * kXW + xq % 16 + 1;
    d[q] = make_uint2((v[0] & 0xffffu) | (v[1] << 16), (v[2] & 0xffffu) | (v[3] << 16));
    d[q + 1] = make_uint2((v[0] >> 16) | (v[1] & 0xffff0000u), (v[2] >> 16) | (v[3] & 0xffff0000u));
    // the border (the second layer's output lay there): rows 0 and 17, then
    // both sides of the rows between
    const int e = xq / 2;
    if (e < 2 * kXW) d[e < kXW ? e : (kXW - 1) * kXW + e - kXW] = make_uint2(0u, 0u);
    else if (e < 2 * kXW + 32)
      d[((e - 2 * kXW) / 2 + 1) * kXW + ((e & 1) ? kXW - 1 : 0)] = make_uint2(0u, 0u);
  };
  // the head of sample s, whose a4 is complete, by the wave of part 0
  auto head = [&](int s) {
    if (TRAIN) store_acts<0>(bufX, acts + (size_t)s * kActN + kActA4, 16, gt, GT);
    if (part != 0) return;
    // head (fp32): f = p * 32 + c, eight features per lane
    float o[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int f = lane * 8 + k;
      const float a = bf2f(bufX[f]);
#pragma unroll
      for (int j = 0; j < 3; ++j) o[j] += P[kOffWh + j * 512 + f] * a;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) o[j] += __shfl_xor(o[j], off);
    if (lane != 0) return;
    const float o0 = o[0] + P[kOffBh], o1 = o[1] + P[kOffBh + 1], o2 = o[2] + P[kOffBh + 2];
    if (out) {
      out[(size_t)s * 3] = o0;
      out[(size_t)s * 3 + 1] = o1;
      out[(size_t)s * 3 + 2] = o2;
    }
    if (po.centre) {
      // window centre: prediction rounded half up, kept inside the search range
      int cx = (int)floorf(8.f * o0 + 0.5f), cy = (int)floorf(8.f * o1 + 0.5f);
      cx = min(max(cx, -po.clampc), po.clampc);
      cy = min(max(cy, -po.clampc), po.clampc);
      const int t = po.tiles ? po.tiles[s] : s;
      const int fb = o2 >= po.conf_logit ? 0 : 1;
      po.centre[2 * t] = cx;
      po.centre[2 * t + 1] = cy;
      po.fallback[t] = (uint8_t)fb;
      if (po.lists) po.lists[fb * po.ntiles + atomicAdd(&po.counts[fb], 1)] = t;
    }
  };
  // every group runs the same number of rounds (the barriers are block-wide);
  // a group past the last sample idles through its round. The next sample's
  // input is fetched during a round and written beside the last layer, and the
  // head runs beside the next sample's first layer: four barriers per round.
  const int step = gridDim.x * SPB;
  int s = blockIdx.x * SPB + grp;
  uint32_t xv[C1];
  fetch(s, xv);
  put(xv);
  int prev = -1;  // the sample whose head is due
  for (int s0 = blockIdx.x * SPB; s0 < n; s0 += step, s += step) {
    const bool act = s < n;
    asm volatile("" : "+v"(lane));  // (the stores' and the head's addresses: formed again)
    uint16_t* as = acts + (size_t)s * kActN;
    __syncthreads();  // weights and x in place, the previous round's a4 too
    if (prev >= 0) head(prev);
    if (act) {
      if (TRAIN)
        for (int i = gt; i < kIn; i += GT)
          as[kActX + i] = bufB[((i >> 6) * kXW + kXW + 1) * C1 + (i & 63)];
      conv1_fwd_part(sm, fo, sW1, sb, bufA, lane, part);  // a1 -> bufA
    }
    fetch(s + step, xv);
    __syncthreads();
    if (act) {
      if (TRAIN) store_acts<1>(bufA, as + kActA1, 256, gt, GT);
      conv_fwd_part<4, 2>(sm, fo.c2, fo.wt, sb + CH, bufB, lane, part);  // a2 -> bufB
    }
    __syncthreads();
    if (act) {
      if (TRAIN) store_acts<2>(bufB, as + kActA2, 64, gt, GT);
      conv_fwd_part<4, 3>(sm, fo.c3, fo.wt + 2 * kWp, sb + 2 * CH, bufA, lane, part);  // a3 -> bufA
    }
    __syncthreads();
    if (act) {
      if (TRAIN) store_acts<3>(bufA, as + kActA3, 64, gt, GT);
      int c4[9];  // (formed here: kept too, they would spill)
      tap_offsets<8, 4, 2, 3>(c4, oA, oZ, lane & 15, lane >> 4);
      conv_fwd_part<1, 0>(sm, c4, fo.wt + 4 * kWp, sb + 3 * CH, bufX, lane, part);  // a4
    }
    put(xv);
    prev = act ? s : -1;
  }
  __syncthreads();
  if (prev >= 0) head(prev);
}

// da_in = transposed conv of dz (LDS, [HOUT^2] rows of kPS) with W (WT, ci
// rows of kWS: [tap][co]); dz_in = bf16(da_in where a_in > 0), to LDS (unless
// null) and global ([ci][q]). The workgroup's waves take the (position tile,
// channel half) units in turn; a unit's sums run in (tap, channel half) order.
template <int HIN, int HOUT, int S>
__device__ void conv_bwd_data(const uint16_t* dz, const uint16_t* WT,
                              const uint16_t* __restrict__ a_in /*global NHWC*/,
                              uint16_t* dz_in, uint16_t* __restrict__ dz_in_g, int lane,
                              int wave, int nwaves) {
  const int r = lane & 15, g = lane >> 4;
  constexpr int MT = HIN * HIN / 16;
  const bf16x4 zero = {0, 0, 0, 0};
  for (int unit = wave; unit < 2 * MT; unit += nwaves) {
    const int mt = unit >> 1, ci = (unit & 1) * 16 + r;
    const int q = mt * 16 + r, qy = q / HIN, qx = q % HIN;
    const int p0 = mt * 16 + g * 4;
    uint16_t av[4];  // in flight with the products
#pragma unroll
    for (int j = 0; j < 4; ++j) av[j] = a_in[(p0 + j) * CH + ci];
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int ty = qy + 1 - tap / 3, tx = qx + 1 - tap % 3;
      const int oy = ty / S, ox = tx / S;
      const bool ok = ty >= 0 && tx >= 0 && ty % S == 0 && tx % S == 0 && oy < HOUT && ox < HOUT;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int co = half * 16 + g * 4;
        const bf16x4 a = ok ? ld4(dz + (oy * HOUT + ox) * kPS + co) : zero;
        acc = mfma(a, ld4(WT + ci * kWS + tap * CH + co), acc);
      }
    }
    bf16x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = av[j] != 0 && bf2f(av[j]) > 0.f ? (short)f2bf(acc[j]) : (short)0;
      if (dz_in) dz_in[(p0 + j) * kPS + ci] = (uint16_t)v[j];
    }
    *reinterpret_cast<bf16x4*>(dz_in_g + ci * HIN * HIN + p0) = v;
  }
}

constexpr int kBwdWaves = 8;
constexpr int kBwdLdsWeights = 3 * CH * kWS * 2 + 3 * 512 * 4;
constexpr int kBwdLds = kBwdLdsWeights + 2 * 64 * kPS * 2;
static_assert(2 * kBwdLds <= 160 * 1024, "two backward workgroups per CU");

// Loss and output gradient (the soft target is held constant) of sample s,
// then its activation gradients. One sample per workgroup at a time, its
// position tiles spread over eight waves: the chain of four layers is bound
// by latency, and a training batch of 256 gives every CU a sample (one wave
// per sample on 64 workgroups: 82 us at 256 samples, this form 14 us).
__global__ __launch_bounds__(kBwdWaves * kWave) void k_cnn_bwd(
    const uint16_t* __restrict__ pk, const float* __restrict__ P,
    const uint16_t* __restrict__ acts, const float* __restrict__ o,
    const int32_t* __restrict__ lab, int n, float* __restrict__ dO, float* __restrict__ loss,
    uint16_t* __restrict__ dzs) {
  extern __shared__ __align__(16) uint8_t sm[];
  uint16_t* sWT = reinterpret_cast<uint16_t*>(sm);  // [3][32 ci][kWS]: [9][32 co] + padding
  float* sWh = reinterpret_cast<float*>(sWT + 3 * CH * kWS);
  uint16_t* bufB = reinterpret_cast<uint16_t*>(sm + kBwdLdsWeights);
  uint16_t* bufC = bufB + 64 * kPS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  load_rows<9 * CH, kWS>(pk + kW1p + 3 * kWp, sWT, 3 * CH, tid, kBwdWaves * kWave);
  for (int i = tid; i < 3 * 512; i += kBwdWaves * kWave) sWh[i] = P[kOffWh + i];
  const float inv = 1.f / (float)n;
  for (int s = blockIdx.x; s < n; s += gridDim.x) {
    __syncthreads();  // weights loaded / the previous sample's buffers free
    const uint16_t* a = acts + (size_t)s * kActN;
    uint16_t* dz = dzs + (size_t)s * kDzN;
    const float ex = 8.f * o[3 * s] - (float)lab[2 * s];
    const float ey = 8.f * o[3 * s + 1] - (float)lab[2 * s + 1];
    const float z = o[3 * s + 2];
    const float q = 1.f / (1.f + expf(-4.f * (2.5f - fmaxf(fabsf(ex), fabsf(ey)))));
    const float d0 = 8.f * fminf(fmaxf(ex, -1.f), 1.f) * inv;
    const float d1 = 8.f * fminf(fmaxf(ey, -1.f), 1.f) * inv;
    const float d2 = (1.f / (1.f + expf(-z)) - q) * inv;
    if (tid == 0) {
      dO[3 * s] = d0;
      dO[3 * s + 1] = d1;
      dO[3 * s + 2] = d2;
      if (loss) {
        auto hub = [](float e) { return fabsf(e) <= 1.f ? 0.5f * e * e : fabsf(e) - 0.5f; };
        loss[s] = hub(ex) + hub(ey) + fmaxf(z, 0.f) - q * z + log1pf(expf(-fabsf(z)));
      }
    }
    // through the head and the last ReLU: dz4 (LDS rows, [c][p] global)
    for (int f = tid; f < 512; f += kBwdWaves * kWave) {
      const float da = sWh[f] * d0 + sWh[512 + f] * d1 + sWh[1024 + f] * d2;
      const uint16_t av = a[kActA4 + f];
      const uint16_t v = av != 0 && bf2f(av) > 0.f ? f2bf(da) : 0;
      bufB[(f >> 5) * kPS + (f & 31)] = v;
      dz[kDz4 + (f % CH) * 16 + f / CH] = v;
    }
    __syncthreads();
    conv_bwd_data<8, 4, 2>(bufB, sWT + 2 * CH * kWS, a + kActA3, bufC, dz + kDz3, lane, wave,
                           kBwdWaves);
    __syncthreads();
    conv_bwd_data<8, 8, 1>(bufC, sWT + CH * kWS, a + kActA2, bufB, dz + kDz2, lane, wave,
                           kBwdWaves);
    __syncthreads();
    conv_bwd_data<16, 8, 2>(bufB, sWT, a + kActA1, nullptr, dz + kDz1, lane, wave, kBwdWaves);
  }
}

// Weight and bias gradients of layer L (1..4) over samples [s0, s1):
// dW[co][tap][ci] = sum_{s,p} dz[s][co][p] a_in[s][in(p, tap)][ci]
// (M = co, N = (tap, ci) and one column of ones for the bias, K = (s, p)),
// written to out in the master layout. A sample's input activations are
// staged channel-major, once for each of a tap row's three columns, shifted
// and subsampled so that output position ox reads element ox: an operand's
// four positions are one aligned 8-byte read, whatever the tap and stride.
// The next sample's activations are loaded during the current one's products.
template <int L>
struct WgradGeom {
  static constexpr int CIN = L == 1 ? C1 : CH;
  static constexpr int HIN = L <= 2 ? 16 : 8;
  static constexpr int HOUT = L == 1 ? 16 : (L == 4 ? 4 : 8);
  static constexpr int S = (L == 2 || L == 4) ? 2 : 1;
  static constexpr int ROWS = S == 2 ? HIN + 1 : HIN + 2;  // row -1 first
  // elements per (column, channel) plane; the padding spreads the 16 planes
  // of an operand over the banks
  static constexpr int PL = ROWS * HOUT + (S == 2 ? 0 : 8);
  static constexpr int LDS = 3 * CIN * PL;  // elements
};
constexpr int kWgradLds = WgradGeom<2>::LDS;
static_assert(kWgradLds >= WgradGeom<1>::LDS && kWgradLds >= WgradGeom<3>::LDS &&
              kWgradLds >= WgradGeom<4>::LDS, "the largest layer's staging");

template <int L>
__device__ void wgrad_layer(const uint16_t* __restrict__ acts, const uint16_t* __restrict__ dzs,
                            int s0, int s1, uint16_t* sa, float* __restrict__ out) {
  using G = WgradGeom<L>;
  constexpr int CIN = G::CIN, HIN = G::HIN, HOUT = G::HOUT, S = G::S, PL = G::PL;
  constexpr int NP = HOUT * HOUT;
  constexpr int NN = 9 * CIN;               // 36 or 288; column NN: the bias
  constexpr int NT = (NN + 1 + 15) / 16;     // N tiles
  constexpr int NTW = (NT + 3) / 4;          // per wave
  constexpr int AIN = L == 1 ? kActX : (L == 2 ? kActA1 : (L == 3 ? kActA2 : kActA3));
  constexpr int DZ = L == 1 ? kDz1 : (L == 2 ? kDz2 : (L == 3 ? kDz3 : kDz4));
  constexpr int EV = CIN == CH ? 8 : 4;      // channels per staging load
  constexpr int NV = HIN * HIN * CIN / EV / 256;
  static_assert(HIN * HIN * CIN % (EV * 256) == 0, "whole staging rounds");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  for (int i = tid; i < G::LDS / 2; i += 256) reinterpret_cast<uint32_t*>(sa)[i] = 0u;
  // this wave's operand columns: LDS element offset of position 0, -1: ones,
  // -2: none
  int boff[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int nn = (wave + 4 * t) * 16 + r, tap = nn / CIN, ci = nn % CIN;
    boff[t] = nn < NN ? (tap % 3 * CIN + ci) * PL + tap / 3 * HOUT : (nn == NN ? -1 : -2);
  }
  f32x4 acc[2][NTW];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < NTW; ++t) acc[m][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  typedef uint16_t vec __attribute__((ext_vector_type(EV)));
  vec st[NV];
  auto fetch = [&](int s) {
    const vec* a = reinterpret_cast<const vec*>(acts + (size_t)s * kActN + AIN);
#pragma unroll
    for (int u = 0; u < NV; ++u) st[u] = a[tid + 256 * u];
  };
  if (s0 < s1) fetch(s0);
  for (int s = s0; s < s1; ++s) {
    __syncthreads();  // cleared / the previous sample's products done
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int i = tid + 256 * u, p = i / (CIN / EV), c0 = i % (CIN / EV) * EV;
      const int iy = p / HIN, ix = p % HIN;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int t = ix + 1 - dx;
        if (t < 0 || t % S != 0 || t / S >= HOUT) continue;
        uint16_t* d = sa + (dx * CIN + c0) * PL + (iy + 1) * HOUT + t / S;
#pragma unroll
        for (int e = 0; e < EV; ++e) d[e * PL] = st[u][e];
      }
    }
    __syncthreads();
    if (s + 1 < s1) fetch(s + 1);
    const uint16_t* dz = dzs + (size_t)s * kDzN + DZ;
#pragma unroll 4
    for (int k0 = 0; k0 < NP; k0 += 16) {
      const int p0 = k0 + g * 4;
      const bf16x4 a0 = ld4(dz + r * NP + p0);
      const bf16x4 a1 = ld4(dz + (16 + r) * NP + p0);
      const int po = p0 / HOUT * S * HOUT + p0 % HOUT;
#pragma unroll
      for (int t = 0; t < NTW; ++t) {
        if (wave + 4 * t >= NT) continue;
        const short one = boff[t] == -1 ? (short)0x3f80 : (short)0;
        bf16x4 b = {one, one, one, one};
        if (boff[t] >= 0) b = ld4(sa + boff[t] + po);
        acc[0][t] = mfma(a0, b, acc[0][t]);
        acc[1][t] = mfma(a1, b, acc[1][t]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int nn = (wave + 4 * t) * 16 + r, tap = nn / CIN, ci = nn % CIN;
    if (nn > NN) continue;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int co = m * 16 + g * 4 + j;
        if (nn < NN) out[kOffW[L - 1] + (co * CIN + ci) * 9 + tap] = acc[m][t][j];
        else out[kOffB[L - 1] + co] = acc[m][t][j];
      }
  }
}

// head gradients over samples [s0, s1)
__device__ void wgrad_head(const uint16_t* __restrict__ acts, const float* __restrict__ dO,
                           int s0, int s1, float* __restrict__ out) {
  const int tid = threadIdx.x;
  for (int f = tid; f < 512; f += 256) {
    float g0 = 0.f, g1 = 0.f, g2 = 0.f;
    for (int s = s0; s < s1; ++s) {
      const float a = bf2f(acts[(size_t)s * kActN + kActA4 + f]);
      g0 += dO[3 * s] * a;
      g1 += dO[3 * s + 1] * a;
      g2 += dO[3 * s + 2] * a;
    }
    out[kOffWh + f] = g0;
    out[kOffWh + 512 + f] = g1;
    out[kOffWh + 1024 + f] = g2;
  }
  if (tid < 3) {
    float b = 0.f;
    for (int s = s0; s < s1; ++s) b += dO[3 * s + tid];
    out[kOffBh + tid] = b;
  }
}

// Block (x, y): layer y + 1 (4: the head) over block x's samples, into
// part[x]. Bound by the staging's latency per sample, so a block takes few
// samples (cnn_grad_blocks): at a training batch of 256, 64 blocks per layer
// of 4 samples, all layers in one launch, take 21 us; one launch per layer
// with 4 blocks of 64 samples, reading the operands element by element from
// global memory, took 2210 us.
__global__ __launch_bounds__(256) void k_cnn_wgrad(const uint16_t* __restrict__ acts,
                                                   const uint16_t* __restrict__ dzs,
                                                   const float* __restrict__ dO, int n,
                                                   int per_block, float* __restrict__ part) {
  __shared__ __align__(16) uint16_t sa[kWgradLds];
  const int s0 = min(n, (int)blockIdx.x * per_block), s1 = min(n, s0 + per_block);
  float* out = part + (size_t)blockIdx.x * kNParam;
  switch (blockIdx.y) {
    case 0: wgrad_layer<1>(acts, dzs, s0, s1, sa, out); break;
    case 1: wgrad_layer<2>(acts, dzs, s0, s1, sa, out); break;
    case 2: wgrad_layer<3>(acts, dzs, s0, s1, sa, out); break;
    case 3: wgrad_layer<4>(acts, dzs, s0, s1, sa, out); break;
    default: wgrad_head(acts, dO, s0, s1, out); break;
  }
}

struct AdamArgs {
  float lr, b1, b2, eps, wd, c1, c2;  // c1 = 1 - b1^t, c2 = 1 - b2^t
};

__global__ __launch_bounds__(256) void k_cnn_adamw(const float* __restrict__ part, int nblk,
                                                   float* __restrict__ P, float* __restrict__ m,
                                                   float* __restrict__ v, AdamArgs a,
                                                   float* __restrict__ grad_out,
                                                   uint16_t* __restrict__ pk) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= kNParam) return;
  float g = 0.f;
#pragma unroll 16
  for (int b = 0; b < nblk; ++b) g += part[(size_t)b * kNParam + i];
  if (grad_out) grad_out[i] = g;
  if (a.lr == 0.f && a.wd == 0.f) return;  // gradient only
  const float mi = a.b1 * m[i] + (1.f - a.b1) * g;
  const float vi = a.b2 * v[i] + (1.f - a.b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / a.c1, vh = vi / a.c2;
  const float p = P[i] - a.lr * (mh / (sqrtf(vh) + a.eps) + a.wd * P[i]);
  P[i] = p;
  pack_param(i, p, pk);
}

}  // namespace

int cnn_param_count() { return kNParam; }
size_t cnn_packed_elems() { return kPacked; }
size_t cnn_act_elems() { return kActN; }
size_t cnn_dz_elems() { return kDzN; }
size_t cnn_input_elems() { return kIn; }

hipError_t launch_cnn_set(const float* src, float* params, bool fresh, uint16_t* packed,
                          hipStream_t st) {
  LNR_LAUNCH(k_cnn_set, dim3((kNParam + 255) / 256), dim3(256), 0, st, src, params, fresh ? 1 : 0,
             packed);
  return hipGetLastError();
}

hipError_t launch_cnn_input(const uint8_t* ref, const uint8_t* warped, int w, int h, int ntx,
                            int nty, const int32_t* tiles, const int* count, uint16_t* x,
                            hipStream_t st) {
  if (ntx * nty == 0) return hipSuccess;
  LNR_LAUNCH(k_cnn_input, dim3(ntx * nty), dim3(256), 0, st, ref, warped, w, h, ntx, tiles,
             count, ntx * nty, x);
  return hipGetLastError();
}

// at most one forward workgroup per CU (each loads the weights once), looping
// over the samples spb at a time
template <bool TRAIN, int SPB>
static hipError_t launch_fwd(const uint16_t* packed, const float* params, const uint16_t* x, int n,
                             float* out, uint16_t* acts, const ProposalOut& po, hipStream_t st) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cnn_fwd<TRAIN, SPB>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, fwd_lds(SPB));
  if (e != hipSuccess) return e;
  const int blocks = (n + SPB - 1) / SPB;
  LNR_LAUNCH((k_cnn_fwd<TRAIN, SPB>), dim3(blocks < 256 ? blocks : 256),
             dim3(SPB * kFwdGroupWaves * kWave), fwd_lds(SPB), st, packed, params, x, n, out, acts,
             po);
  return hipGetLastError();
}

hipError_t launch_cnn_forward(const uint16_t* packed, const float* params, const uint16_t* x,
                              int n, float* out, uint16_t* acts, int32_t* centre,
                              uint8_t* fallback, int clampc, float conf_logit, hipStream_t st,
                              const int32_t* tiles, const int* count, int* lists, int* counts) {
  if (n <= 0) return hipSuccess;
  ProposalOut po{centre, fallback, clampc, conf_logit, tiles, count, lists, counts, n};
  const bool few = n <= 256;
  if (acts)
    return few ? launch_fwd<true, 1>(packed, params, x, n, out, acts, po, st)
               : launch_fwd<true, kFwdMany>(packed, params, x, n, out, acts, po, st);
  return few ? launch_fwd<false, 1>(packed, params, x, n, out, acts, po, st)
             : launch_fwd<false, kFwdMany>(packed, params, x, n, out, acts, po, st);
}

// Samples per gradient block: the batch over 64 blocks per layer (320 in
// all, a little over one per CU) down to one sample a block, over at most
// 256 for large batches (their partial gradients are summed once more).
int cnn_grad_blocks(int n, int* per_block) {
  const int pb = n <= 256 ? (n + 63) / 64 : (n + 255) / 256 < 4 ? 4 : (n + 255) / 256;
  *per_block = pb;
  return (n + pb - 1) / pb;
}

hipError_t launch_cnn_backward(const uint16_t* packed, const float* params,
                               const uint16_t* acts, const float* out, const int32_t* labels,
                               int n, float* dO, float* loss, uint16_t* dzs, float* part,
                               hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cnn_bwd),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBwdLds);
  if (e != hipSuccess) return e;
  LNR_LAUNCH(k_cnn_bwd, dim3(n < 512 ? n : 512), dim3(kBwdWaves * kWave), kBwdLds, st, packed,
             params, acts, out, labels, n, dO, loss, dzs);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int pb = 0;
  const int nb = cnn_grad_blocks(n, &pb);
  LNR_LAUNCH(k_cnn_wgrad, dim3(nb, 5), dim3(256), 0, st, acts, dzs, dO, n, pb, part);
  return hipGetLastError();
}

hipError_t launch_cnn_adamw(const float* part, int nblk, float* params, float* m, float* v,
                            float lr, float wd, int step, float* grad_out, uint16_t* packed,
                            hipStream_t st) {
  AdamArgs a;
  a.lr = lr;
  a.b1 = 0.9f;
  a.b2 = 0.999f;
  a.eps = 1e-8f;
  a.wd = wd;
  a.c1 = (float)(1.0 - pow(0.9, step));
  a.c2 = (float)(1.0 - pow(0.999, step));
  LNR_LAUNCH(k_cnn_adamw, dim3((kNParam + 255) / 256), dim3(256), 0, st, part, nblk, params, m,
             v, a, grad_out, packed);
  return hipGetLastError();
}

}  // namespace lnr

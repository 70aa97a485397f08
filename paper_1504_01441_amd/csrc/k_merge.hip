// k_merge.hip -- error-tolerant exposure fusion (paper Sec. 2.5): Mertens et
// al.'s contrast, saturation and well-exposedness weights, times the SSIM
// between the equalised reference and each warped frame (Wang et al.:
// Gaussian window, five filterings), blended with Laplacian pyramids.
//
//  k_ssim:    4 output rows x (256 - 2r) columns per block: the vertical
//             Gaussian sums of each input column are built in registers, the
//             horizontal ones from LDS, two output columns per thread. The
//             sums (x, y, xy, x^2 + y^2) are double precision: SSIM divides
//             covariance errors by sx^2 + sy^2 + C2 (~1e-3 in flat regions)
//             and the fusion weights amplify them again.
//  k_weights: per pixel, every frame's C * S * E (* max(SSIM, 0)) + 1e-12,
//             normalised over the frames; threads walk down columns so that
//             the Laplacian's rows are read once, and take the left and right
//             neighbours from the adjacent lanes.
//  k_reduce:  REDUCE ([1 4 6 4 1]/16 separable, clamped, even samples) of
//             every weight and image plane of one level, in registers.
//  k_blend:   from the top level down, R_l = sum_k W_k,l (G_k,l - E(G_k,l+1))
//             + E(R_l+1), E the EXPAND rule, on 64x32 tiles whose coarse
//             neighbourhoods are staged in LDS; level 0 goes to the output. Small
//             levels use k_blend_px instead (one thread per pixel and channel,
//             samples read directly).
#include "lnr_device.h"
#include "lnr_internal.h"

namespace lnr {
namespace {

struct FramePtrs {
  const float* img[16];
  const float* ssim[16];
  float* wout[16];
};

constexpr int kMaxMaps = 64;
constexpr int kSsimMaxR = 8, kSsimTH = 4;

// normalised Gaussian window taps g[0 .. 2r]
struct SsimWin {
  double g[2 * kSsimMaxR + 1];
};

// the warped frames' planes and their maps, one frame per blockIdx.z
struct SsimMaps {
  const float* b[16];
  float* out[16];
};

// One block: kSsimTH output rows by 256 - 2R output columns. SSIM needs the
// Gaussian sums of x, y, xy and of x^2 + y^2 (only the sum of the two
// variances enters it), accumulated in double precision: SSIM divides
// covariance errors by sx^2 + sy^2 + C2 (~1e-3 in flat regions) and the
// fusion weights amplify them again near SSIM = 0, so float sums of
// E[x^2] - E[x]^2 are not accurate enough there.
//  1. vertical: thread t owns input column ox - R + t (clamped) and reads its
//     kSsimTH + 2R rows straight from global memory (a wave reads 64
//     consecutive floats per row); each row's values and products are
//     scattered into the kSsimTH outputs they belong to, all in registers;
//  2. the vertical sums go to LDS; thread t takes output columns 2t and 2t+1
//     of half the tile's rows, reading the shared window as aligned pairs of
//     doubles (16-byte LDS reads, half the reads of one column per thread).
// Bound by the double-precision units (about 140 instructions per pixel) and
// the LDS reads beside them; a 5 MP map took 51 us with separate multiplies
// and adds, takes 32 with fused ones and 32-bit load offsets; two 1 MP maps,
// which are one launch, 34 -> 20.
template <int R>
__global__ __launch_bounds__(256) void k_ssim(const float* __restrict__ a, SsimMaps maps, int W,
                                              int H, SsimWin win, double c1, double c2) {
  const float* __restrict__ b = maps.b[blockIdx.z];
  float* __restrict__ out = maps.out[blockIdx.z];
  constexpr int TW = 256 - 2 * R, NR = kSsimTH + 2 * R, NS = 4;
  static_assert(kSsimTH % 2 == 0, "two row halves");
  __shared__ double2 vs[NS][kSsimTH][128];  // column pairs of the vertical sums
  int bx, by;
  xcd_block(gridDim.x, gridDim.y, bx, by);
  const int tid = threadIdx.x;
  const int ox = bx * TW, oy = by * kSsimTH;
  {
    const int gx = min(max(ox - R + tid, 0), W - 1);
    float pa[NR], pb[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {  // every load in flight before the sums
      // (32-bit byte offsets, since a plane has at most 2^26 pixels: 64-bit
      // addresses of all the loads would cost a block per CU)
      const uint32_t o =
          4u * ((uint32_t)min(max(oy - R + i, 0), H - 1) * (uint32_t)W + (uint32_t)gx);
      pa[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a) + o);
      pb[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(b) + o);
    }
    double acc[kSsimTH][NS];
#pragma unroll
    for (int o = 0; o < kSsimTH; ++o)
#pragma unroll
      for (int t = 0; t < NS; ++t) acc[o][t] = 0.0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const double p = pa[i], q = pb[i];
      const double ss = fma(p, p, q * q), pq = p * q;
#pragma unroll
      for (int o = 0; o < kSsimTH; ++o) {
        const int k = i - o;  // tap of input row oy - R + i for output row oy + o
        if (k < 0 || k > 2 * R) continue;
        const double wd = win.g[k];
        acc[o][0] = fma(wd, p, acc[o][0]);
        acc[o][1] = fma(wd, q, acc[o][1]);
        acc[o][2] = fma(wd, ss, acc[o][2]);
        acc[o][3] = fma(wd, pq, acc[o][3]);
      }
    }
    double* vd = reinterpret_cast<double*>(vs);
#pragma unroll
    for (int o = 0; o < kSsimTH; ++o)
#pragma unroll
      for (int t = 0; t < NS; ++t) vd[(t * kSsimTH + o) * 256 + tid] = acc[o][t];
  }
  __syncthreads();
  const int pr = tid & 127, half = tid >> 7;  // column pair, row half
  const int gx = ox + 2 * pr;
  if (2 * pr >= TW || gx >= W) return;
  const bool two = 2 * pr + 1 < TW && gx + 1 < W;
#pragma unroll
  for (int oo = 0; oo < kSsimTH / 2; ++oo) {
    const int o = half * (kSsimTH / 2) + oo;
    const int gy = oy + o;
    if (gy >= H) break;
    double s0[NS] = {0.0, 0.0, 0.0, 0.0}, s1[NS] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int m = 0; m <= R; ++m) {  // inputs 2pr + 2m and 2pr + 2m + 1
      const double wl = win.g[2 * m];
      const double wr = 2 * m + 1 <= 2 * R ? win.g[2 * m + 1] : 0.0;
      const double wp = m > 0 ? win.g[2 * m - 1] : 0.0;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const double2 v = vs[t][o][pr + m];
        // output 2pr takes taps 2m (v.x) and 2m + 1 (v.y); output 2pr + 1
        // takes taps 2m - 1 (v.x) and 2m (v.y)
        s0[t] = fma(wl, v.x, s0[t]);
        if (2 * m + 1 <= 2 * R) s0[t] = fma(wr, v.y, s0[t]);
        if (m > 0) s1[t] = fma(wp, v.x, s1[t]);
        s1[t] = fma(wl, v.y, s1[t]);
      }
    }
    // (else the second column's sums are put off past the branch below and the
    // window's values held for them: 106 registers, not 60, a block per CU less)
    asm volatile("" : "+v"(s1[0]), "+v"(s1[1]), "+v"(s1[2]), "+v"(s1[3]));
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (c == 1 && !two) break;
      const double* sv = c ? s1 : s0;
      const double m1 = sv[0], m2 = sv[1];
      const double vxy = sv[2] - m1 * m1 - m2 * m2, cxy = sv[3] - m1 * m2;
      out[(size_t)gy * W + gx + c] = (float)(((2.0 * m1 * m2 + c1) * (2.0 * cxy + c2)) /
                                             ((m1 * m1 + m2 * m2 + c1) * (vxy + c2)));
    }
  }
}

__device__ inline double grey_of(int ch, float r, float g, float b) {
  return ch == 3 ? (0.299 * (double)r + 0.587 * (double)g) + 0.114 * (double)b : (double)r;
}

// C * S * E (* max(SSIM, 0)) of one frame at one pixel, from the grey values
// of the pixel (gc) and its four neighbours, and the pixel's colour. Contrast
// and saturation are differences of nearly equal values in flat regions, and
// the normalised weights divide by their sum, which can be ~1e-12 there: they
// are evaluated in double precision.
__device__ inline double raw_weight(int ch, double gu, double gl, double gr, double gd,
                                    double gc, float R, float G, float B, bool warped,
                                    float ssim, float two_se2) {
  const double C = fabs(gu + gl + gr + gd - 4.0 * gc);
  double S = 1.0;
  float e;
  if (ch == 3) {
    const double r = R, g = G, b = B;
    const double mu = (r + g + b) * (1.0 / 3.0);
    const double var = ((r - mu) * (r - mu) + (g - mu) * (g - mu) + (b - mu) * (b - mu)) * (1.0 / 3.0);
    S = (double)sqrtf((float)var);  // the cancelling differences are in double
    e = (float)((r - 0.5) * (r - 0.5) + (g - 0.5) * (g - 0.5) + (b - 0.5) * (b - 0.5));
  } else {
    e = (float)(((double)R - 0.5) * ((double)R - 0.5));
  }
  double wt = C * S * (double)expf(-e / two_se2);
  if (warped) wt *= fmax((double)ssim, 0.0);
  return wt + 1e-12;
}

// the value of the lane before (kWaveShr1) or after, on the vector ALU; the
// wave's first or last lane gets 0
constexpr int kWaveShr1 = 0x138, kWaveShl1 = 0x130;
template <int CTRL>
__device__ inline double from_lane(double v) {
  return __hiloint2double(
      __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false),
      __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false));
}

template <int CTRL>
__device__ inline float from_lane(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

constexpr int kWeightRows = 8;
constexpr int kWeightCols = 62;  // output columns per wave (lanes 1..62)

// Each thread walks down kWeightRows rows of one column: the grey values of
// the rows above, at and below the pixel stay in registers, so every colour
// sample is fetched from memory once. A wave covers 62 columns and two halo
// lanes (0 and 63, clamped at the image border like the pixels' own
// neighbours); the left and right neighbours' grey values come from the
// adjacent lanes by shuffle. The samples of the next row are loaded before
// the current row's weights are formed and stored, so one row's loads are
// always in flight. Bound by its instructions (295 per wave and row, 40 of the
// 48 us of two 5 MP frames); 52 us with the neighbours' grey values through
// the LDS unit and a division per weight.
template <int NMAX>
__global__ __launch_bounds__(256) void k_weights(FramePtrs f, int n, int ch, int W, int H,
                                                 int ref, float two_se2) {
  int bx, by;
  xcd_block(gridDim.x, gridDim.y, bx, by);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x = (bx * 4 + wave) * kWeightCols + lane - 1;
  const int xc = min(max(x, 0), W - 1);
  const bool writes = lane >= 1 && lane <= kWeightCols && x < W;
  const int y0 = by * kWeightRows, y1 = min(y0 + kWeightRows, H);
  const size_t plane = (size_t)W * H;
  auto ld = [&](const float* I, size_t o, float& r, float& g, float& b) {
    r = I[o];
    g = ch == 3 ? I[plane + o] : 0.f;
    b = ch == 3 ? I[2 * plane + o] : 0.f;
  };
  // samples of row y: d* the row below, s the SSIM
  float dr[NMAX], dg[NMAX], db[NMAX], sv[NMAX];
  auto fetch = [&](int y) {  // y < H
    const size_t od = (size_t)min(y + 1, H - 1) * W + xc;
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
      if (k >= n) continue;
      ld(f.img[k], od, dr[k], dg[k], db[k]);
      sv[k] = k != ref ? f.ssim[k][(size_t)y * W + xc] : 0.f;
    }
  };
  double gu[NMAX], gc[NMAX];
  float cr[NMAX], cg[NMAX], cb[NMAX];
#pragma unroll
  for (int k = 0; k < NMAX; ++k) {
    if (k >= n) continue;
    float r, g, b;
    ld(f.img[k], (size_t)max(y0 - 1, 0) * W + xc, r, g, b);
    gu[k] = grey_of(ch, r, g, b);
    ld(f.img[k], (size_t)y0 * W + xc, cr[k], cg[k], cb[k]);
    gc[k] = grey_of(ch, cr[k], cg[k], cb[k]);
  }
  // stacks of up to 4 frames keep the next row's samples in flight; larger
  // ones (whose samples would not fit the registers) load each frame's
  // samples where they are used
  constexpr bool kAhead = NMAX <= 4;
  if constexpr (kAhead) fetch(y0);
  for (int y = y0; y < y1; ++y) {
    const size_t o = (size_t)y * W + xc;
    float Dr[NMAX], Dg[NMAX], Db[NMAX], S[NMAX];
    if constexpr (kAhead) {
#pragma unroll
      for (int k = 0; k < NMAX; ++k) {
        Dr[k] = dr[k]; Dg[k] = dg[k]; Db[k] = db[k];
        S[k] = sv[k];
      }
      if (y + 1 < y1) fetch(y + 1);
    }
    // the raw weights keep 24-bit relative precision as floats once the
    // cancelling differences inside them were taken in double precision
    float wk[NMAX];
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
      if (k >= n) continue;
      if constexpr (!kAhead) {
        ld(f.img[k], (size_t)min(y + 1, H - 1) * W + xc, Dr[k], Dg[k], Db[k]);
        S[k] = k != ref ? f.ssim[k][o] : 0.f;
      }
      const bool warped = k != ref;
      const double gd = grey_of(ch, Dr[k], Dg[k], Db[k]);
      const double gl = from_lane<kWaveShr1>(gc[k]), gr = from_lane<kWaveShl1>(gc[k]);
      wk[k] = (float)raw_weight(ch, gu[k], gl, gr, gd, gc[k], cr[k], cg[k], cb[k], warped, S[k],
                                two_se2);
      sum += (double)wk[k];
      gu[k] = gc[k];
      gc[k] = gd;
      cr[k] = Dr[k]; cg[k] = Dg[k]; cb[k] = Db[k];
    }
    if (writes) {
#pragma unroll
      for (int k = 0; k < NMAX; k += 2) {  // two at a time share the reciprocal
        if (k >= n) continue;
        double q0, q1;
        recip_quotients((double)wk[k], k + 1 < n ? (double)wk[k + 1] : 0.0, sum, q0, q1);
        f.wout[k][o] = (float)q0;
        if (k + 1 < n) f.wout[k + 1][o] = (float)q1;
      }
    }
  }
}

// Irradiance map of the registered frames, one pixel per thread and every
// channel: each frame's value over its relative exposure, averaged with the
// hat weight min(v, 1 - v) (0 at black and saturation), non-reference
// frames' weights times max(SSIM, 0); the reference's value where every
// weight is 0.
struct IrrPtrs {
  const float* img[16];
  const float* ssim[16];
  float rel[16];  // exposure relative to the reference
};

__device__ inline float hat_weight(float v) {
  const float a = v < 1.f - v ? v : 1.f - v;
  return a > 0.f ? a : 0.f;
}

template <int NMAX>
__global__ __launch_bounds__(256) void k_irradiance(IrrPtrs f, int n, int ch, int ref,
                                                    long long npix, float* __restrict__ out) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= npix) return;
  float s[NMAX];
#pragma unroll
  for (int k = 0; k < NMAX; ++k) {
    s[k] = 1.f;
    if (k < n && k != ref) {
      const float q = f.ssim[k][i];
      s[k] = q > 0.f ? q : 0.f;
    }
  }
  for (int c = 0; c < ch; ++c) {
    const long long o = (long long)c * npix + i;
    float v[NMAX];
#pragma unroll
    for (int k = 0; k < NMAX; ++k) v[k] = k < n ? f.img[k][o] : 0.f;  // all loads in flight
    float sw = 0.f, se = 0.f;
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
      if (k >= n) continue;
      const float wk = hat_weight(v[k]) * s[k];
      sw += wk;
      se += wk * (v[k] / f.rel[k]);
    }
    out[o] = sw > 0.f ? se / sw : f.img[ref][o];
  }
}

struct MapPtrs {
  const float* in[kMaxMaps];
  float* out[kMaxMaps];
};

constexpr int kRedCols = 62;  // output columns per wave (lanes 1..62)

// A wave forms ROWS output rows of 62 columns of one plane: a lane loads the
// two source columns of its output in every source row, all of them in flight
// before the first sum, and takes the neighbours' from the adjacent lanes.
// Bound by memory at level 0 of a large frame. The staged tile this replaces
// spent 38 of its 40 us (eight planes of two 5 MP frames) on instructions, 150
// per output, most of them index arithmetic; with two rows in flight at a time
// instead of all it was as slow, by latency. 40 -> 38 us at
// that level, 14.2 -> 12.3 at the next, 6.3 -> 5.5.
template <int ROWS>
__global__ __launch_bounds__(256) void k_reduce(MapPtrs m, int w, int h, int w2, int h2) {
  const float* __restrict__ in = m.in[blockIdx.z];
  float* __restrict__ out = m.out[blockIdx.z];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int X0 = blockIdx.x * kRedCols - 1, X = X0 + lane;
  const int oy0 = (blockIdx.y * 4 + wave) * ROWS;
  if (oy0 >= h2) return;
  constexpr int N = 2 * ROWS + 3;
  float a[N], b[N];
  // (32-bit byte offsets: a plane has at most 2^26 pixels)
  const char* p = reinterpret_cast<const char*>(in);
  auto row_at = [&](int i) {
    return 4u * ((uint32_t)min(max(2 * oy0 - 2 + i, 0), h - 1) * (uint32_t)w);
  };
  if (X0 >= 0 && 2 * (X0 + 63) + 1 < w) {
    struct __attribute__((packed, aligned(4))) Pair {
      float a, b;
    };
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const Pair v = *reinterpret_cast<const Pair*>(p + (row_at(i) + 8u * (uint32_t)X));
      a[i] = v.a;
      b[i] = v.b;
    }
  } else {
    const uint32_t c0 = 4u * (uint32_t)min(max(2 * X, 0), w - 1);
    const uint32_t c1 = 4u * (uint32_t)min(max(2 * X + 1, 0), w - 1);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      a[i] = *reinterpret_cast<const float*>(p + (row_at(i) + c0));
      b[i] = *reinterpret_cast<const float*>(p + (row_at(i) + c1));
    }
  }
  // [1 4 6 4 1] / 16 in that order (every product but the middle one is exact)
  auto taps = [](float v0, float v1, float v2, float v3, float v4) {
    float s = fmaf(0.25f, v1, 0.0625f * v0);
    s += 0.375f * v2;
    return fmaf(0.0625f, v4, fmaf(0.25f, v3, s));
  };
#pragma unroll
  for (int i = 0; i < N; ++i)
    a[i] = taps(from_lane<kWaveShr1>(a[i]), from_lane<kWaveShr1>(b[i]), a[i], b[i],
                from_lane<kWaveShl1>(a[i]));
  if (lane < 1 || lane > kRedCols || X >= w2) return;
#pragma unroll
  for (int j = 0; j < ROWS; ++j)
    if (oy0 + j < h2)
      out[(uint32_t)(oy0 + j) * (uint32_t)w2 + (uint32_t)X] =
          taps(a[2 * j], a[2 * j + 1], a[2 * j + 2], a[2 * j + 3], a[2 * j + 4]);
}

struct BlendPtrs {
  const float* w[16];        // normalised weights at level l
  const float* g[16][3];     // image planes at level l
  const float* gc[16][3];    // image planes at level l + 1
  const float* rc[3];        // collapsed result at level l + 1
  float* out[3];             // collapsed result at level l
};

constexpr int kBW = 64, kBH = 32;                 // fine output tile
constexpr size_t kBlendPxMax = 1 << 18;           // levels up to this size: k_blend_px
constexpr int kCW = kBW / 2 + 2, kCH = kBH / 2 + 2;  // coarse tile with its EXPAND halo
constexpr int kCT = kCW * kCH;

// EXPAND (clamped coarse indices, rows first, then columns): even samples 2i
// (c[i-1] + 6 c[i] + c[i+1]) / 8, odd ones 2i + 1 (c[i] + c[i+1]) / 2.
__device__ inline float ex_even(float a, float m, float p) {
  return fmaf(0.75f, m, 0.125f * (a + p));
}
__device__ inline float ex_odd(float m, float p) { return 0.5f * (m + p); }

// the four fine columns from the even one of staged column i + 1 on (row + i
// is 8-byte aligned)
__device__ inline float4 ex_row4(const float* row) {
  const float2 u = *reinterpret_cast<const float2*>(row);
  const float2 v = *reinterpret_cast<const float2*>(row + 2);
  return make_float4(ex_even(u.x, u.y, v.x), ex_odd(u.y, v.x), ex_even(u.y, v.x, v.y),
                     ex_odd(v.x, v.y));
}

// two fine rows of four columns: t at the coarse row and column before
__device__ inline void expand_tile8(const float* t, float4& e, float4& o) {
  const float4 a = ex_row4(t), m = ex_row4(t + kCW), p = ex_row4(t + 2 * kCW);
  e = make_float4(ex_even(a.x, m.x, p.x), ex_even(a.y, m.y, p.y), ex_even(a.z, m.z, p.z),
                  ex_even(a.w, m.w, p.w));
  o = make_float4(ex_odd(m.x, p.x), ex_odd(m.y, p.y), ex_odd(m.z, p.z), ex_odd(m.w, p.w));
}

// four floats of a row that is aligned to its elements only
struct __attribute__((packed, aligned(4))) Float4 {
  float x, y, z, w;
};
__device__ inline float4 load4(const float* p, int valid) {  // the first `valid` of them
  if (valid >= 4) {
    const Float4 v = *reinterpret_cast<const Float4*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
  }
  return make_float4(p[0], valid > 1 ? p[1] : 0.f, valid > 2 ? p[2] : 0.f, 0.f);
}
__device__ inline void store4(float* p, const float4& v, int valid) {
  if (valid >= 4) {
    *reinterpret_cast<Float4*>(p) = Float4{v.x, v.y, v.z, v.w};
    return;
  }
  p[0] = v.x;
  if (valid > 1) p[1] = v.y;
  if (valid > 2) p[2] = v.z;
}
__device__ inline void blend4(float4& acc, const float4& w, const float4& g, const float4& e) {
  acc.x = fmaf(w.x, g.x - e.x, acc.x);
  acc.y = fmaf(w.y, g.y - e.y, acc.y);
  acc.z = fmaf(w.z, g.z - e.z, acc.z);
  acc.w = fmaf(w.w, g.w - e.w, acc.w);
}

// One 64 x 32 tile of a level below the top, channels [c0, c0 + cg):
//   R_l = sum_k W_k (G_k - E(G_k,l+1)) + E(R_l+1).
// EXPAND reads the coarse planes from LDS tiles (kCH x kCW, clamped at load)
// loaded once per block, a thread's places in them found once; a thread owns
// two rows of four pixels, which share their expanded coarse rows, and reads
// each weight once. With one row per thread and the staging's places found
// for every plane by divisions the kernel was bound by its instructions, 345
// per pixel (44 of the 51 us of two 5 MP frames' level 0);
// now 46 us there, by memory, 17.7 -> 14 at the next level.
__global__ __launch_bounds__(256) void k_blend(BlendPtrs b, int n, int c0, int cg, int w, int h,
                                               int cw, int chh) {
  extern __shared__ __align__(16) float sm[];  // plane m = cc (n + 1) + k, k = n: R
  const int tid = threadIdx.x;
  int bx, by;
  xcd_block(gridDim.x, gridDim.y, bx, by);
  const int ox = bx * kBW, oy = by * kBH;
  {
    constexpr int U = (kCT + 255) / 256;
    uint32_t off[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = tid + 256 * u, r = i / kCW, q = i % kCW;
      const int gy = min(max((oy >> 1) - 1 + r, 0), chh - 1);
      const int gx = min(max((ox >> 1) - 1 + q, 0), cw - 1);
      off[u] = (uint32_t)gy * (uint32_t)cw + (uint32_t)gx;  // (in bounds past the tile too)
    }
    for (int cc = 0; cc < cg; ++cc)
      for (int k0 = 0; k0 <= n; k0 += 4) {  // four planes' loads in flight
        float v[4][U];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = k0 + j;
          if (k > n) break;
          const float* __restrict__ src = k < n ? b.gc[k][c0 + cc] : b.rc[c0 + cc];
#pragma unroll
          for (int u = 0; u < U; ++u) v[j][u] = src[off[u]];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (k0 + j > n) break;
          float* ct = sm + (cc * (n + 1) + k0 + j) * kCT;
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (tid + 256 * u < kCT) ct[tid + 256 * u] = v[j][u];
        }
      }
    __syncthreads();
  }
  const int xq = 4 * (tid & 15), yq = 2 * (tid >> 4);
  const int x = ox + xq, y = oy + yq;
  if (x >= w || y >= h) return;
  const int valid = w - x;
  const uint32_t o0 = (uint32_t)y * (uint32_t)w + (uint32_t)x;
  const uint32_t o1 = y + 1 < h ? o0 + (uint32_t)w : o0;  // (the last row again, not stored)
  const float* t = sm + (yq >> 1) * kCW + (xq >> 1);
  float4 acc[3][2];
#pragma unroll
  for (int cc = 0; cc < 3; ++cc) acc[cc][0] = acc[cc][1] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k = 0; k < n; ++k) {
    const float4 w0 = load4(b.w[k] + o0, valid), w1 = load4(b.w[k] + o1, valid);
    float4 g0[3], g1[3];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      if (cc >= cg) break;
      g0[cc] = load4(b.g[k][c0 + cc] + o0, valid);
      g1[cc] = load4(b.g[k][c0 + cc] + o1, valid);
    }
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      if (cc >= cg) break;
      float4 e0, e1;
      expand_tile8(t + (cc * (n + 1) + k) * kCT, e0, e1);
      blend4(acc[cc][0], w0, g0[cc], e0);
      blend4(acc[cc][1], w1, g1[cc], e1);
    }
  }
#pragma unroll
  for (int cc = 0; cc < 3; ++cc) {
    if (cc >= cg) break;
    float4 e0, e1;
    expand_tile8(t + (cc * (n + 1) + n) * kCT, e0, e1);
    const float4 u = acc[cc][0], v = acc[cc][1];
    float* out = b.out[c0 + cc];
    store4(out + o0, make_float4(u.x + e0.x, u.y + e0.y, u.z + e0.z, u.w + e0.w), valid);
    if (y + 1 < h)
      store4(out + o1, make_float4(v.x + e1.x, v.y + e1.y, v.z + e1.z, v.w + e1.w), valid);
  }
}

// A pixel of EXPAND(c) at (x, y) of the finer level: rows of the coarse plane
// (cw x chh, clamped indices) expanded along x first, then along y, as k_blend
// does from its staged tiles.
__device__ inline float expand_px(const float* __restrict__ c, int cw, int chh, int x, int y) {
  const int i = x >> 1, j = y >> 1;
  const int xa = max(i - 1, 0), xm = min(i, cw - 1), xp = min(i + 1, cw - 1);
  float rv[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const float* row = c + (size_t)min(max(j - 1 + q, 0), chh - 1) * cw;
    const float a = row[xa], m = row[xm], p = row[xp];
    rv[q] = (x & 1) == 0 ? ex_even(a, m, p) : ex_odd(m, p);
  }
  return (y & 1) == 0 ? ex_even(rv[0], rv[1], rv[2]) : ex_odd(rv[1], rv[2]);
}

// Small levels: one thread per pixel and channel (blockIdx.y), every sample
// read straight from memory (all in flight together) instead of staged
// tiles, which leave too few workgroups to hide their latency.
__global__ __launch_bounds__(256) void k_blend_px(BlendPtrs b, int n, int w, int h, int cw,
                                                  int chh, int top) {
  const int pix = blockIdx.x * 256 + threadIdx.x, c = blockIdx.y;
  if (pix >= w * h) return;
  const int x = pix % w, y = pix / w;
  float acc = 0.f;
  for (int k = 0; k < n; ++k) {
    const float wv = b.w[k][pix], gv = b.g[k][c][pix];
    const float e = top ? 0.f : expand_px(b.gc[k][c], cw, chh, x, y);
    acc += wv * (gv - e);
  }
  if (!top) acc += expand_px(b.rc[c], cw, chh, x, y);
  b.out[c][pix] = acc;
}

}  // namespace

int merge_levels(int W, int H) {
  const int m = W < H ? W : H;
  int k = 0;
  while ((8ll << (k + 1)) <= m) ++k;
  return 1 + k;
}

// elements of one plane's pyramid levels 1..L-1
size_t merge_pyr_elems(int W, int H, int levels) {
  size_t tot = 0;
  int w = W, h = H;
  for (int l = 1; l < levels; ++l) {
    w = (w + 1) / 2;
    h = (h + 1) / 2;
    tot += (size_t)w * h;
  }
  return tot;
}

// SSIM of every frame but the reference against the reference, into
// ssim + k * W * H
hipError_t launch_ssim_maps(int n, int W, int H, const float* const* yeqs, int ref_index,
                            const lnr_params& p, float* ssim, hipStream_t st) {
  const size_t N = (size_t)W * H;
  const int r = p.ssim_radius;
  SsimWin win;
  double gs = 0.0;
  for (int j = -r; j <= r; ++j) {
    win.g[j + r] = exp(-(double)(j * j) / (2.0 * p.ssim_sigma * p.ssim_sigma));
    gs += win.g[j + r];
  }
  for (int j = 0; j <= 2 * r; ++j) win.g[j] /= gs;
  SsimMaps maps;
  int m = 0;
  for (int k = 0; k < n; ++k) {
    if (k == ref_index) continue;
    maps.b[m] = yeqs[k];
    maps.out[m++] = ssim + (size_t)k * N;
  }
  if (m == 0) return hipSuccess;
  const int tw = 256 - 2 * r;
  const dim3 g((W + tw - 1) / tw, (H + kSsimTH - 1) / kSsimTH, m);
  const float* ya = yeqs[ref_index];
  switch (r) {
#define SSIM_CASE(R_)                                                                           \
  case R_:                                                                                      \
    LNR_LAUNCH(k_ssim<R_>, g, dim3(256), 0, st, ya, maps, W, H, win, p.ssim_c1, p.ssim_c2);     \
    break;
    SSIM_CASE(1) SSIM_CASE(2) SSIM_CASE(3) SSIM_CASE(4)
    SSIM_CASE(5) SSIM_CASE(6) SSIM_CASE(7) SSIM_CASE(8)
#undef SSIM_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_merge(int n, int ch, int W, int H, const float* const* imgs,
                        const float* const* yeqs, int ref_index, const lnr_params& p,
                        const MergeBufs& bufs, float* out, hipStream_t st) {
  const int L = merge_levels(W, H);
  const size_t N = (size_t)W * H;
  const size_t tot = merge_pyr_elems(W, H, L);
  int lw[32], lh[32];
  size_t loff[33];
  lw[0] = W; lh[0] = H; loff[0] = 0; loff[1] = 0;
  for (int l = 1; l < L; ++l) {
    lw[l] = (lw[l - 1] + 1) / 2;
    lh[l] = (lh[l - 1] + 1) / 2;
    loff[l + 1] = loff[l] + (size_t)lw[l] * lh[l];
  }
  hipError_t e;
  FramePtrs fp;
  for (int k = 0; k < n; ++k) {
    fp.img[k] = imgs[k];
    fp.ssim[k] = bufs.ssim + (size_t)k * N;
    fp.wout[k] = bufs.w0 + (size_t)k * N;
  }
  if ((e = launch_ssim_maps(n, W, H, yeqs, ref_index, p, bufs.ssim, st)) != hipSuccess) return e;
  {
    const dim3 g((W + 4 * kWeightCols - 1) / (4 * kWeightCols),
                 (H + kWeightRows - 1) / kWeightRows);
    const float two_se2 = (float)(2.0 * p.sigma_e * p.sigma_e);
    if (n <= 2)
      LNR_LAUNCH(k_weights<2>, g, dim3(256), 0, st, fp, n, ch, W, H, ref_index, two_se2);
    else if (n <= 4)
      LNR_LAUNCH(k_weights<4>, g, dim3(256), 0, st, fp, n, ch, W, H, ref_index, two_se2);
    else if (n <= 8)
      LNR_LAUNCH(k_weights<8>, g, dim3(256), 0, st, fp, n, ch, W, H, ref_index, two_se2);
    else
      LNR_LAUNCH(k_weights<16>, g, dim3(256), 0, st, fp, n, ch, W, H, ref_index, two_se2);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // Gaussian pyramids of every weight and image plane
  const int maps = n * (ch + 1);
  auto plane_ptr = [&](int z, int l) -> float* {
    const int k = z / (ch + 1), q = z % (ch + 1);
    if (l == 0)
      return q == 0 ? bufs.w0 + (size_t)k * N : const_cast<float*>(imgs[k]) + (size_t)(q - 1) * N;
    return bufs.pyr + (size_t)z * tot + loff[l];
  };
  for (int l = 1; l < L; ++l) {
    MapPtrs mp;
    for (int z = 0; z < maps; ++z) {
      mp.in[z] = plane_ptr(z, l - 1);
      mp.out[z] = plane_ptr(z, l);
    }
    // eight rows per wave read 19 source rows; two (7 rows) where the level would
    // leave the chip idle
    const bool tall = (size_t)lw[l] * lh[l] * maps >= (1u << 20);
    const int rows = tall ? 8 : 2;
    const dim3 g((lw[l] + kRedCols - 1) / kRedCols, (lh[l] + 4 * rows - 1) / (4 * rows), maps);
    if (tall)
      LNR_LAUNCH(k_reduce<8>, g, dim3(256), 0, st, mp, lw[l - 1], lh[l - 1], lw[l], lh[l]);
    else
      LNR_LAUNCH(k_reduce<2>, g, dim3(256), 0, st, mp, lw[l - 1], lh[l - 1], lw[l], lh[l]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // blend + collapse, top level first
  for (int l = L - 1; l >= 0; --l) {
    BlendPtrs bp;
    for (int k = 0; k < n; ++k) {
      bp.w[k] = plane_ptr(k * (ch + 1), l);
      for (int c = 0; c < ch; ++c) {
        bp.g[k][c] = plane_ptr(k * (ch + 1) + 1 + c, l);
        bp.gc[k][c] = l + 1 < L ? plane_ptr(k * (ch + 1) + 1 + c, l + 1) : nullptr;
      }
    }
    for (int c = 0; c < ch; ++c) {
      bp.rc[c] = l + 1 < L ? bufs.acc + (size_t)c * tot + loff[l + 1] : nullptr;
      bp.out[c] = l == 0 ? out + (size_t)c * N : bufs.acc + (size_t)c * tot + loff[l];
    }
    const int cw = l + 1 < L ? lw[l + 1] : 1, chh = l + 1 < L ? lh[l + 1] : 1;
    const int top = l + 1 == L ? 1 : 0;
    const size_t per_plane = (size_t)kCH * kCW * sizeof(float);
    int cg = ch;  // channels per launch, so that the coarse tiles fit in 64 KB of LDS
    while (cg > 1 && (size_t)(n + 1) * cg * per_plane > 64 * 1024) --cg;
    if ((size_t)lw[l] * lh[l] <= kBlendPxMax) {
      LNR_LAUNCH(k_blend_px, dim3((lw[l] * lh[l] + 255) / 256, ch), dim3(256), 0, st, bp, n,
                 lw[l], lh[l], cw, chh, top);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      continue;
    }
    for (int c0 = 0; c0 < ch; c0 += cg) {  // (a top level is below kBlendPxMax)
      const int g = min(cg, ch - c0);
      LNR_LAUNCH(k_blend, dim3((lw[l] + kBW - 1) / kBW, (lh[l] + kBH - 1) / kBH), dim3(256),
                 (size_t)(n + 1) * g * per_plane, st, bp, n, c0, g, lw[l], lh[l], cw, chh);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

hipError_t launch_irradiance(int n, int ch, int W, int H, const float* const* imgs,
                             const float* const* yeqs, const float* rel, int ref_index,
                             const lnr_params& p, float* ssim, float* out, hipStream_t st) {
  hipError_t e;
  if ((e = launch_ssim_maps(n, W, H, yeqs, ref_index, p, ssim, st)) != hipSuccess) return e;
  const long long N = (long long)W * H;
  IrrPtrs f;
  for (int k = 0; k < 16; ++k) {
    f.img[k] = k < n ? imgs[k] : nullptr;
    f.ssim[k] = k < n && k != ref_index ? ssim + (size_t)k * N : nullptr;
    f.rel[k] = k < n ? rel[k] : 1.f;
  }
  const dim3 g((unsigned)((N + 255) / 256));
  if (n <= 2)
    LNR_LAUNCH(k_irradiance<2>, g, dim3(256), 0, st, f, n, ch, ref_index, N, out);
  else if (n <= 4)
    LNR_LAUNCH(k_irradiance<4>, g, dim3(256), 0, st, f, n, ch, ref_index, N, out);
  else if (n <= 8)
    LNR_LAUNCH(k_irradiance<8>, g, dim3(256), 0, st, f, n, ch, ref_index, N, out);
  else
    LNR_LAUNCH(k_irradiance<16>, g, dim3(256), 0, st, f, n, ch, ref_index, N, out);
  return hipGetLastError();
}

}  // namespace lnr

// k_warp.hip -- backward warp of the source to the reference (paper Sec. 2.1:
// the goal is to warp the source to the reference; Sec. 2.4: the dense flow).
// The sample position m(x) = Hp1(x + F(x)) is computed in double precision (a
// 5 MP frame needs position errors well below 1e-4 px), the samples are FP32
// bilinear with clamp to edge. I420 chroma is upsampled by pixel repetition
// and converted with BT.601 full-range coefficients; outputs are planar FP32
// in [0, 1] plus the warped equalised luma (for the SSIM weight of Sec. 2.5).
#include <algorithm>

#include "lnr_device.h"
#include "lnr_internal.h"

namespace lnr {
namespace {

__device__ inline float bil(float p00, float p10, float p01, float p11, float ax, float ay) {
  const float bx = 1.f - ax;
  return fmaf(ay, fmaf(ax, p11, bx * p01), (1.f - ay) * fmaf(ax, p10, bx * p00));
}

// a / 255, correctly rounded: the quotient by the reciprocal, corrected by its
// exact residual (checked against the division for every significand)
__device__ inline float over_255(float a) {
  const float r = 1.f / 255.f, q = a * r;
  return fmaf(fmaf(-255.f, q, a), r, q);
}

__device__ inline void yuv_rgb(float Y, float U, float V, float& r, float& g, float& b) {
  const float up = U - 128.f, vp = V - 128.f;
  r = over_255(Y + 1.402f * vp);
  g = over_255(Y - 0.344136f * up - 0.714136f * vp);
  b = over_255(Y + 1.772f * up);
}

// Bilinear sample from two rows' byte pairs a and c: the left and right taps
// at bits s0 and s1.
__device__ inline float bil_pairs(uint32_t a, uint32_t c, int s0, int s1, float ax, float ay) {
  return bil((float)((a >> s0) & 255u), (float)((a >> s1) & 255u), (float)((c >> s0) & 255u),
             (float)((c >> s1) & 255u), ax, ay);
}

// The source and flow planes and the size, with offsets of type OFF: 32 bits
// where every plane is below 4 GiB.
struct WarpSrc {
  const uint8_t* y;
  const uint8_t* u;
  const uint8_t* v;
  const uint8_t* yeq;
  int sy, su, sv, cs, W, H;
};

// A column of `rows` output pixels per thread. Bound by instructions: with
// byte gathers, separate divisions and 64-bit offsets about 330 per pixel, 51
// us for a 5 MP I420 frame and 64 for NV12. So the two taps of a row are one
// load, the divisions share a reciprocal, the offsets are 32 bits and the
// bilinear steps fused: 39 and 37 us, in 62 registers. (The next row's flow
// loaded ahead gains nothing.)
template <typename OFF>
__global__ __launch_bounds__(256) void k_bwarp(WarpSrc s, const double* __restrict__ Hn,
                                               const float* __restrict__ flow, int rows,
                                               float* __restrict__ img, float* __restrict__ yw) {
  int bx, by;
  xcd_block(gridDim.x, gridDim.y, bx, by);  // neighbouring rows gather from shared source rows
  const int px = bx * blockDim.x + threadIdx.x;
  const int W = s.W, H = s.H;
  if (px >= W) return;
  const size_t plane = (size_t)W * H;
  double hp[9];  // formed per thread (uniform, no barrier)
  pixel_homography_sparse(Hn, W, H, hp);
  const bool mod = moderate(hp);
  const int p0 = by * rows, p1 = min(p0 + rows, H);
#pragma unroll 1
  for (int py = p0; py < p1; ++py) {
    const OFF o = (OFF)py * (OFF)W + (OFF)px;
    const double X = (double)px + (double)flow[o];
    const double Y = (double)py + (double)(flow + plane)[o];
    const double den = (hp[6] * X + hp[7] * Y) + hp[8];
    // (a flow far outside any image would leave the moderate range)
    const bool fast = mod && fabs(X) < 0x1p100 && fabs(Y) < 0x1p100;
    double sx, sy2;
    div2((hp[0] * X + hp[1] * Y) + hp[2], (hp[3] * X + hp[4] * Y) + hp[5], den, fast, sx, sy2);
    if (!(sx >= -1.0)) sx = -1.0;
    if (sx > (double)W) sx = (double)W;
    if (!(sy2 >= -1.0)) sy2 = -1.0;
    if (sy2 > (double)H) sy2 = (double)H;
    const double fx0 = floor(sx), fy0 = floor(sy2);
    const float ax = (float)(sx - fx0), ay = (float)(sy2 - fy0);
    const int ix = (int)fx0, iy = (int)fy0;
    const int x0 = min(max(ix, 0), W - 1), x1 = min(max(ix + 1, 0), W - 1);
    const int y0 = min(max(iy, 0), H - 1), y1 = min(max(iy + 1, 0), H - 1);
    float Yv;
    if (W >= 2) {
      const uint32_t b = pair_base(x0, W);
      const int s0 = x0 == (int)b ? 0 : 8, s1 = x1 == (int)b ? 0 : 8;
      const uint32_t ya = load_pair(s.y + ((OFF)y0 * (OFF)s.sy + b));
      const uint32_t yc = load_pair(s.y + ((OFF)y1 * (OFF)s.sy + b));
      const uint32_t ea = load_pair(s.yeq + ((OFF)y0 * (OFF)W + b));
      const uint32_t ec = load_pair(s.yeq + ((OFF)y1 * (OFF)W + b));
      Yv = bil_pairs(ya, yc, s0, s1, ax, ay);
      yw[o] = over_255(bil_pairs(ea, ec, s0, s1, ax, ay));
    } else {  // a column: both taps are its byte
      Yv = bil_pairs(s.y[(OFF)y0 * (OFF)s.sy], s.y[(OFF)y1 * (OFF)s.sy], 0, 0, ax, ay);
      yw[o] = over_255(bil_pairs(s.yeq[y0], s.yeq[y1], 0, 0, ax, ay));
    }
    if (!s.u) {
      img[o] = over_255(Yv);
      continue;
    }
    // chroma sample x >> 1 of the half-size planes (even W): again both taps of
    // a row within two neighbouring samples, of which a 2-pixel wide frame has one
    const OFF ca = (OFF)(y0 >> 1), cc = (OFF)(y1 >> 1);
    const int c0 = x0 >> 1, c1 = x1 >> 1;
    float Uv, Vv;
    if (W < 4) {
      const OFF ua = ca * (OFF)s.su, uc = cc * (OFF)s.su, va = ca * (OFF)s.sv, vc = cc * (OFF)s.sv;
      Uv = bil_pairs(s.u[ua], s.u[uc], 0, 0, ax, ay);
      Vv = bil_pairs(s.v[va], s.v[vc], 0, 0, ax, ay);
    } else if (s.cs == 1) {
      const uint32_t b = pair_base(c0, W >> 1);
      const int s0 = c0 == (int)b ? 0 : 8, s1 = c1 == (int)b ? 0 : 8;
      const uint32_t ua = load_pair(s.u + (ca * (OFF)s.su + b));
      const uint32_t uc = load_pair(s.u + (cc * (OFF)s.su + b));
      const uint32_t va = load_pair(s.v + (ca * (OFF)s.sv + b));
      const uint32_t vc = load_pair(s.v + (cc * (OFF)s.sv + b));
      Uv = bil_pairs(ua, uc, s0, s1, ax, ay);
      Vv = bil_pairs(va, vc, s0, s1, ax, ay);
    } else {  // interleaved: U, V of both samples are four bytes
      const uint32_t b = pair_base(c0, W >> 1);
      const int s0 = c0 == (int)b ? 0 : 16, s1 = c1 == (int)b ? 0 : 16;
      const uint32_t a = reinterpret_cast<const UnalignedU32*>(s.u + (ca * (OFF)s.su + 2 * b))->v;
      const uint32_t c = reinterpret_cast<const UnalignedU32*>(s.u + (cc * (OFF)s.su + 2 * b))->v;
      Uv = bil_pairs(a, c, s0, s1, ax, ay);
      Vv = bil_pairs(a >> 8, c >> 8, s0, s1, ax, ay);
    }
    float r, g, bl;
    yuv_rgb(Yv, Uv, Vv, r, g, bl);
    img[o] = r;
    (img + plane)[o] = g;
    (img + 2 * plane)[o] = bl;
  }
}

// Four consecutive pixels per thread: 32-bit luma loads and 128-bit stores
// where the row allows; with yin, the 8-bit plane yin is also mapped to
// [0, 1] into yout (the merge's equalised reference luma).
__global__ __launch_bounds__(256) void k_frame_rgb4(const uint8_t* __restrict__ y, int sy,
                                                    const uint8_t* __restrict__ u, int su,
                                                    const uint8_t* __restrict__ v, int sv, int cs,
                                                    int W,
                                                    int H, float* __restrict__ img,
                                                    const uint8_t* __restrict__ yin,
                                                    float* __restrict__ yout) {
  int bx, py;
  xcd_block(gridDim.x, gridDim.y, bx, py);
  const int px = 4 * (bx * blockDim.x + threadIdx.x);
  if (px >= W) return;
  const size_t plane = (size_t)W * H, o = (size_t)py * W + px;
  const uint8_t* yr = y + (size_t)py * sy + px;
  const bool full = px + 4 <= W;
  const bool vin = full && ((reinterpret_cast<uintptr_t>(yr) & 3u) == 0);
  const bool vout = full && ((reinterpret_cast<uintptr_t>(img + o) & 15u) == 0);
  float Yv[4], r[4], g[4], b[4];
  if (vin) {
    const uint32_t w4 = *reinterpret_cast<const uint32_t*>(yr);
#pragma unroll
    for (int k = 0; k < 4; ++k) Yv[k] = (float)((w4 >> (8 * k)) & 255u);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) Yv[k] = px + k < W ? (float)yr[k] : 0.f;
  }
  if (u) {
    const uint8_t* ur = u + (size_t)(py >> 1) * su + (size_t)(px >> 1) * cs;
    const uint8_t* vr = v + (size_t)(py >> 1) * sv + (size_t)(px >> 1) * cs;
    const int nc = full ? 2 : (W - px + 1) / 2;  // chroma samples of these pixels
    float U[2] = {128.f, 128.f}, V[2] = {128.f, 128.f};
    for (int c = 0; c < nc; ++c) {
      U[c] = ur[c * cs];
      V[c] = vr[c * cs];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) yuv_rgb(Yv[k], U[k >> 1], V[k >> 1], r[k], g[k], b[k]);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = Yv[k] / 255.f;
  }
  if (vout) {
    *reinterpret_cast<float4*>(img + o) = make_float4(r[0], r[1], r[2], r[3]);
    if (u) {
      *reinterpret_cast<float4*>(img + plane + o) = make_float4(g[0], g[1], g[2], g[3]);
      *reinterpret_cast<float4*>(img + 2 * plane + o) = make_float4(b[0], b[1], b[2], b[3]);
    }
  } else {
    for (int k = 0; k < 4 && px + k < W; ++k) {
      img[o + k] = r[k];
      if (u) {
        img[plane + o + k] = g[k];
        img[2 * plane + o + k] = b[k];
      }
    }
  }
  if (yin) {
    const uint8_t* q = yin + o;
    if (vout && ((reinterpret_cast<uintptr_t>(q) & 3u) == 0) &&
        ((reinterpret_cast<uintptr_t>(yout + o) & 15u) == 0)) {
      const uint32_t w4 = *reinterpret_cast<const uint32_t*>(q);
      *reinterpret_cast<float4*>(yout + o) =
          make_float4((float)(w4 & 255u) / 255.f, (float)((w4 >> 8) & 255u) / 255.f,
                      (float)((w4 >> 16) & 255u) / 255.f, (float)(w4 >> 24) / 255.f);
    } else {
      for (int k = 0; k < 4 && px + k < W; ++k) yout[o + k] = q[k] / 255.f;
    }
  }
}

}  // namespace

hipError_t launch_backward_warp(const uint8_t* y, int sy, const Chroma& c, const uint8_t* yeq,
                                int W, int H, const double* Hn, const float* flow, float* image,
                                float* yeq_w, hipStream_t st) {
  const WarpSrc s{y, c.u, c.v, yeq, sy, c.su, c.sv, c.cs, W, H};
  // four rows share a thread's set-up (41 -> 39 us at 5 MP) where that leaves
  // enough blocks (VGA: 4.8 us with one row, 6.4 with four)
  const int rows = (long long)W * H >= (2 << 20) ? 4 : 1;
  const dim3 grid((W + 255) / 256, (H + rows - 1) / rows);
  const long long pitch = std::max({(long long)sy, (long long)c.su, (long long)c.sv, 4ll * W});
  if (pitch * H <= 0xffffffffll)
    LNR_LAUNCH(k_bwarp<uint32_t>, grid, dim3(256), 0, st, s, Hn, flow, rows, image, yeq_w);
  else
    LNR_LAUNCH(k_bwarp<size_t>, grid, dim3(256), 0, st, s, Hn, flow, rows, image, yeq_w);
  return hipGetLastError();
}

hipError_t launch_frame_rgb_unit(const uint8_t* y, int sy, const Chroma& c, int W, int H,
                                 float* image, const uint8_t* yin, float* yout, hipStream_t st) {
  dim3 grid((W + 1023) / 1024, H);
  LNR_LAUNCH(k_frame_rgb4, grid, dim3(256), 0, st, y, sy, c.u, c.su, c.v, c.sv, c.cs, W, H,
             image, yin, yout);
  return hipGetLastError();
}

}  // namespace lnr

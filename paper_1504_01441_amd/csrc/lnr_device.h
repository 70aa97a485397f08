// lnr_device.h -- double-precision helpers shared by the GPU kernels. Every
// operation is written in a fixed order (compiled without FMA contraction) so
// results whose rounding decides an integer are reproducible.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lnr {

// nx / den and ny / den from one reciprocal: two Newton steps from the
// hardware's approximation, then each quotient corrected by its exact
// residual -- the steps a compiled double division takes for operands that
// need no scaling, so the quotients are the same correctly rounded ones
// wherever operands and quotients stay clear of the ends of the exponent
// range (and den of 0).
__device__ inline void recip_quotients(double nx, double ny, double den, double& qx, double& qy) {
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  r = fma(fma(-den, r, 1.0), r, r);
  const double x = nx * r, y = ny * r;
  qx = fma(fma(-den, x, nx), r, x);
  qy = fma(fma(-den, y, ny), r, y);
}

// out = a b for row-major 3x3 matrices; each entry sums left to right.
__device__ inline void mat3_mul(const double* a, const double* b, double* out) {
  double t[9];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double s = a[3 * i + 0] * b[0 + j];
      s = s + a[3 * i + 1] * b[3 + j];
      s = s + a[3 * i + 2] * b[6 + j];
      t[3 * i + j] = s;
    }
  for (int i = 0; i < 9; ++i) out[i] = t[i];
}

// Normalised frame of paper Sec. 2.2 (origin at the image centre, x in [-1, 1],
// y in [-h/w, h/w]): xn ~ C x with C = [[2,0,-(w-1)],[0,2,-(h-1)],[0,0,w]] and
// x ~ B xn with B = [[w,0,w-1],[0,w,h-1],[0,0,2]] (B C = 2w I), so the level
// pixel homography is Hp = B (H C).
__device__ inline void pixel_homography(const double* H, int w, int h, double* Hp) {
  const double B[9] = {(double)w, 0, (double)(w - 1), 0, (double)w, (double)(h - 1), 0, 0, 2};
  const double C[9] = {2, 0, (double)(-(w - 1)), 0, 2, (double)(-(h - 1)), 0, 0, (double)w};
  double T[9];
  mat3_mul(H, C, T);
  mat3_mul(B, T, Hp);
}

// pixel_homography with the products written out without the terms that
// multiply by 0 (they add nothing to a finite sum); a homography that is not
// finite takes the full products. For the warps, where every thread forms it
// (the search's kernels, short of registers, are slower with it).
__device__ inline void pixel_homography_sparse(const double* H, int w, int h, double* Hp) {
  double all = 0.0;
#pragma unroll
  for (int i = 0; i < 9; ++i) all += fabs(H[i]);
  if (!(all < 0x1p1000)) {
    pixel_homography(H, w, h, Hp);
    return;
  }
  const double W = (double)w, cx = (double)(w - 1), cy = (double)(h - 1);
  double T[9];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    T[3 * i] = H[3 * i] * 2.0;
    T[3 * i + 1] = H[3 * i + 1] * 2.0;
    T[3 * i + 2] = (H[3 * i] * -cx + H[3 * i + 1] * -cy) + H[3 * i + 2] * W;
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    Hp[j] = W * T[j] + cx * T[6 + j];
    Hp[3 + j] = W * T[3 + j] + cy * T[6 + j];
    Hp[6 + j] = 2.0 * T[6 + j];
  }
}

// Whether the products of these coefficients and pixel coordinates stay clear
// of the exponent range's upper end (not so for NaN), for recip_quotients.
__device__ inline bool moderate(const double* hp) {
  bool ok = true;
#pragma unroll
  for (int i = 0; i < 9; ++i) ok = ok && fabs(hp[i]) < 0x1p400;
  return ok;
}

// nx / den and ny / den; fast: the operands' upper ends are known to be
// moderate. A den near 0 (or NaN) is divided plainly.
__device__ inline void div2(double nx, double ny, double den, bool fast, double& qx, double& qy) {
  if (fast && fabs(den) > 0x1p-400) {
    recip_quotients(nx, ny, den, qx, qy);
  } else {
    qx = nx / den;
    qy = ny / den;
  }
}

struct __attribute__((packed)) UnalignedU16 {
  uint16_t v;
};
struct __attribute__((packed)) UnalignedU32 {
  uint32_t v;
};

// The bytes at x0 and x1 of a row of at least two: both lie in the two bytes
// from b on, one load.
__device__ inline uint32_t pair_base(int x0, int n) { return (uint32_t)min(x0, n - 2); }
__device__ inline uint32_t load_pair(const uint8_t* p) {
  return reinterpret_cast<const UnalignedU16*>(p)->v;
}

// inclusive sums over the wave's lanes
__device__ inline int wave_scan_i32(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast 15, 31
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// F(v, v of an earlier lane) folded over the wave on the vector ALU; the
// total in every lane (0 is F's neutral value)
template <typename F>
__device__ inline unsigned long long wave_fold_u64(unsigned long long v, F&& f) {
#define LNR_FOLD(CTRL, ROWS)                                                                    \
  v = f(v, ((unsigned long long)(uint32_t)__builtin_amdgcn_update_dpp(                          \
                0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, false)                            \
            << 32) |                                                                            \
               (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, false))
  LNR_FOLD(0x111, 0xf);  // row_shr 1, 2, 4, 8
  LNR_FOLD(0x112, 0xf);
  LNR_FOLD(0x114, 0xf);
  LNR_FOLD(0x118, 0xf);
  LNR_FOLD(0x142, 0xa);  // row_bcast 15, 31
  LNR_FOLD(0x143, 0xc);
#undef LNR_FOLD
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ inline unsigned long long wave_max_u64(unsigned long long v) {
  return wave_fold_u64(v, [](unsigned long long p, unsigned long long q) { return q > p ? q : p; });
}

}  // namespace lnr

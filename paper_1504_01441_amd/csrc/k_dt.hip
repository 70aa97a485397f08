// k_dt.hip -- sparse-to-dense flow (paper Sec. 2.4, Eq. 6-7): the sparse maps
// P_u, P_v (match displacement at each kept corner) and N (1 there) are
// cross-bilateral filtered with the domain transform's recursive filter
// (Gastal & Oliveira 2011), guided by the equalised reference; F = P~ / N~.
//
// Each recursive pass  J[x] = J[x] + c_x (J[x-1] - J[x])  is a chain of affine
// maps z -> c_x z + (1 - c_x) v_x, so it is split into segments whose composed
// maps are combined with a parallel scan, then re-run with the exact carry.
// The step coefficient c = a_i^(1 + sigma_s/sigma_r |dI|) depends only on the
// 8-bit guide difference, so each iteration uses a 256-entry table.
// The recursions run in double precision (the maps are stored as float between
// passes): with c close to 1 (sigma_s = 400) a float recursion amplifies
// rounding by ~1/(1 - c), which would move the flow by ~1e-4 px.
//
// Between passes a pixel is one 12-byte record of the three maps, so that a
// column pass reads whole 24-96 byte runs of neighbouring columns rather than
// 8-32 byte pieces of three planes; the column pass takes the guide from a
// column-major copy (a segment's rows are one aligned load).
//
//  k_dt_row: one workgroup per row; the row's records are loaded straight into
//          LDS, each of the 256 or 512 threads keeps a segment in registers, and
//          lane exchanges on the vector ALU + LDS combine the segment maps. The first pass writes
//          the sparse maps itself from the tile list (no zero-fill pass); a
//          row that holds no sample stays exactly zero through it, so that
//          pass writes only a row flag for it, and the first column pass
//          reads the records of flagged rows only (the rest are zeros).
//  k_dt_col: one workgroup per strip of 2 to 8 columns over the full height, as
//          128 or 256 segments per column held in registers; the records are read
//          and written once per pass. The last pass writes F (and N~) instead.
#include <algorithm>

#include "lnr_device.h"
#include "lnr_internal.h"

namespace lnr {
namespace {

struct DtArgs {
  int iters;
  double sigma_s, ratio;  // ratio = sigma_s / sigma_r
};

// c_i[k] = a_i ^ (1 + ratio * k / 255),  a_i = exp(-sqrt(2) / sigma_i),
// sigma_i = sigma_s sqrt(3) 2^(n - i) / sqrt(4^n - 1)  (i = 1..n)
// Block 0 also clears zero[0, nzero) and zero64[0, nzero64) and sets ident to
// the identity (the registration's first launch does this set-up with the
// tables: histograms, the top level's weeding bits).
__device__ inline void dt_coef(const DtArgs& a, double* __restrict__ coef,
                               uint32_t* __restrict__ zero, int nzero,
                               double* __restrict__ ident,
                               unsigned long long* __restrict__ zero64, int nzero64) {
  const int i = blockIdx.x + 1, k = threadIdx.x;
  if (blockIdx.x == 0) {
    for (int j = k; j < nzero; j += 256) zero[j] = 0u;
    for (int j = k; j < nzero64; j += 256) zero64[j] = 0ull;
    if (ident && k < 9) ident[k] = (k % 4 == 0) ? 1.0 : 0.0;
  }
  const double sig = a.sigma_s * sqrt(3.0) * pow(2.0, (double)(a.iters - i)) /
                     sqrt(pow(4.0, (double)a.iters) - 1.0);
  const double ai = exp(-sqrt(2.0) / sig);
  coef[blockIdx.x * 256 + k] = pow(ai, 1.0 + a.ratio * ((double)k / 255.0));
}

__global__ __launch_bounds__(256) void k_dt_coef(DtArgs a, double* __restrict__ coef,
                                                 uint32_t* __restrict__ zero, int nzero,
                                                 double* __restrict__ ident,
                                                 unsigned long long* __restrict__ zero64,
                                                 int nzero64) {
  dt_coef(a, coef, zero, nzero, ident, zero64, nzero64);
}

// every pair of a batch, one per blockIdx.y
__global__ __launch_bounds__(256) void k_dt_coef_jobs(DtArgs a, const SetupJob* __restrict__ jobs) {
  const SetupJob& J = jobs[blockIdx.y];
  dt_coef(a, J.coef, J.hist, 512, J.ident, J.vb, J.nvb);
}

struct Rec {  // one pixel of the three maps between passes
  float m0, m1, m2;
};

struct Aff {  // z -> A z + B (three channels share A)
  double A, B0, B1, B2;
};

// later o earlier
__device__ inline Aff compose(const Aff& later, const Aff& earlier) {
  Aff r;
  r.A = later.A * earlier.A;
  r.B0 = fma(later.A, earlier.B0, later.B0);
  r.B1 = fma(later.A, earlier.B1, later.B1);
  r.B2 = fma(later.A, earlier.B2, later.B2);
  return r;
}

// Lane exchange on the vector ALU; lanes without a source get `none`.
template <int CTRL, int ROWS>
__device__ inline double dpp_or(double v, double none) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(none), __double2loint(v), CTRL, ROWS,
                                             0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(none), __double2hiint(v), CTRL, ROWS,
                                             0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL, int ROWS>
__device__ inline Aff dpp_aff(const Aff& v) {  // (the identity without a source)
  return Aff{dpp_or<CTRL, ROWS>(v.A, 1.0), dpp_or<CTRL, ROWS>(v.B0, 0.0),
             dpp_or<CTRL, ROWS>(v.B1, 0.0), dpp_or<CTRL, ROWS>(v.B2, 0.0)};
}
__device__ inline Aff shfl_aff(const Aff& v, int src) {
  return Aff{__shfl(v.A, src), __shfl(v.B0, src), __shfl(v.B1, src), __shfl(v.B2, src)};
}

constexpr int kRowShl = 0x100, kRowShr = 0x110;  // + the distance, within 16 lanes
constexpr int kWaveShl1 = 0x130, kWaveShr1 = 0x138;
constexpr int kBcast15 = 0x142, kBcast31 = 0x143;

// Inclusive composition over the segments of one line in a wave, segment
// i on lanes i STRIDE + (line): forward, everything up to a lane's segment;
// backward, everything from it on. Within 16 lanes on the vector ALU, then
// across the four groups of 16.
template <int STRIDE, bool FWD>
__device__ inline Aff wave_scan(Aff inc) {
  constexpr int dir = FWD ? kRowShr : kRowShl;
  if constexpr (STRIDE <= 1) inc = compose(inc, dpp_aff<dir + 1, 0xf>(inc));
  if constexpr (STRIDE <= 2) inc = compose(inc, dpp_aff<dir + 2, 0xf>(inc));
  if constexpr (STRIDE <= 4) inc = compose(inc, dpp_aff<dir + 4, 0xf>(inc));
  inc = compose(inc, dpp_aff<dir + 8, 0xf>(inc));
  if constexpr (STRIDE == 1 && FWD) {
    inc = compose(inc, dpp_aff<kBcast15, 0xa>(inc));
    inc = compose(inc, dpp_aff<kBcast31, 0xc>(inc));
  } else {
    const int lane = threadIdx.x & 63, l = lane % STRIDE;
    const Aff a = shfl_aff(inc, FWD ? (lane & 32) | (16 - STRIDE + l) : (lane & 32) | (16 + l));
    if (FWD ? (lane & 16) != 0 : (lane & 16) == 0) inc = compose(inc, a);
    const Aff b = shfl_aff(inc, FWD ? 32 - STRIDE + l : 32 + l);
    if (FWD ? lane >= 32 : lane < 32) inc = compose(inc, b);
  }
  return inc;
}

// Carry into each segment of a block of NW waves: the composition of every
// earlier segment of its line (forward: lower lanes and waves; backward:
// higher ones), applied to 0. wt: NW * STRIDE entries of LDS.
template <int STRIDE, int NW, bool FWD>
__device__ inline void line_carry(const Aff& v, Aff* wt, double& c0, double& c1, double& c2) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l = lane % STRIDE;
  const Aff inc = wave_scan<STRIDE, FWD>(v);
  if (FWD ? lane >= 64 - STRIDE : lane < STRIDE) wt[wave * STRIDE + l] = inc;
  Aff prev;  // the wave's earlier segments
  if constexpr (STRIDE == 1) {
    prev = dpp_aff<FWD ? kWaveShr1 : kWaveShl1, 0xf>(inc);
  } else {
    prev = shfl_aff(inc, FWD ? lane - STRIDE : lane + STRIDE);
    if (FWD ? lane < STRIDE : lane >= 64 - STRIDE) prev = Aff{1.0, 0.0, 0.0, 0.0};
  }
  __syncthreads();
  double z0 = 0.0, z1 = 0.0, z2 = 0.0;  // carry into this wave
#pragma unroll 2
  for (int i = 0; i < (FWD ? wave : NW - 1 - wave); ++i) {
    const Aff t = wt[(FWD ? i : NW - 1 - i) * STRIDE + l];
    z0 = fma(t.A, z0, t.B0);
    z1 = fma(t.A, z1, t.B1);
    z2 = fma(t.A, z2, t.B2);
  }
  c0 = fma(prev.A, z0, prev.B0);
  c1 = fma(prev.A, z1, prev.B1);
  c2 = fma(prev.A, z2, prev.B2);
  __syncthreads();
}

// Pins a value to a register of its own type at this point: without it the
// segments' double values of one sweep are kept for the next (twice the
// registers), and the addresses of the loads for the stores.
template <typename T>
__device__ inline void hold(T& v) {
  asm volatile("" : "+v"(v));
}

// The three sweeps over a segment. A causal step is p = u + c (p - u); the
// first sweep composes the segment's causal steps. The second applies them
// and composes the anti-causal ones (z -> c z + (1 - c) p, c towards the next
// pixel) from the left as it goes, the third applies those. A pixel past the
// line's end has value 0 and c 0 on both sides, so it needs no test.
__device__ inline void causal_sum(Aff& t, double c, double u0, double u1, double u2) {
  t.B0 = fma(c, t.B0 - u0, u0);
  t.B1 = fma(c, t.B1 - u1, u1);
  t.B2 = fma(c, t.B2 - u2, u2);
  t.A *= c;
}
__device__ inline void step(double& p, double c, float& u) {
  const double v = u;
  p = fma(c, p - v, v);
  u = (float)p;
  hold(u);
}
__device__ inline void anticausal_sum(Aff& t, double c, double p0, double p1, double p2) {
  const double n = t.A * c, d = t.A - n;  // A (1 - c)
  t.B0 = fma(d, p0, t.B0);
  t.B1 = fma(d, p1, t.B1);
  t.B2 = fma(d, p2, t.B2);
  t.A = n;
}


// Every fourth step of a sweep: the coefficients of later steps are not
// fetched (nor values converted) before these are done with their registers.
__device__ inline void pace(int j) {
  if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
}

// 4 or 16 bytes per lane from g straight into LDS, lane after lane from l
// (the wave's base) on; the wave must wait for its memory counter before it or
// another wave reads them. (12 bytes per lane would land 16 apart.)
__device__ inline void to_lds4(const float* g, float* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 4, 0, 0);
}
__device__ inline void to_lds16(const float* g, float* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------------------
// Horizontal pass: one block per row. The row's records are staged in LDS as
// they are (12 bytes, loaded straight into it), each thread keeps a segment
// of SEG consecutive pixels in registers (a segment's records are whole
// 16-byte reads that cover the banks evenly), the results go back the same
// way.
// A pass moves its 24 bytes per pixel through the last-level cache in about
// 15 us at 5 MP; the rest of its time is the sweeps' double-precision work and
// the two carries, a few blocks per CU overlapping each other's. Of 37 us at
// 5 MP, fused multiply-adds, the anti-causal composition folded into the
// causal sweep, scans without LDS round trips and the staging without
// registers leave 26 (8 MP at an odd width, staged by dwords: 80 -> 44).
template <int SEG, int NT, bool FIRST>
__device__ __forceinline__ void row_pass_of(int y, Rec* __restrict__ maps,
                                            const uint8_t* __restrict__ guide, int W, int H,
                                            const double* cf, Aff* wt, float* sm,
                                            const int32_t* __restrict__ cxy,
                                            const int32_t* __restrict__ disp,
                                            const uint8_t* __restrict__ flags, int ntx, int nty,
                                            int tile, uint8_t* __restrict__ rowflag) {
  Rec* row = reinterpret_cast<Rec*>(sm);
  const int tid = threadIdx.x;
  const size_t ro = (size_t)y * W;
  if (FIRST) {
    // the row's samples (kept level-0 matches whose corner lies on it)
    int has = 0;
    const int ty = y / tile;
    if (ty < nty)
      for (int tx = tid; tx < ntx; tx += NT) {
        const int t = ty * ntx + tx;
        has |= (flags[t] & 4) && cxy[2 * t + 1] == y;
      }
    has = __syncthreads_or(has);
    if (tid == 0) rowflag[y] = (uint8_t)(has != 0);
    if (!has) return;  // all zeros: the column pass does not read this row
    for (int x = tid; x < W; x += NT) row[x] = Rec{0.f, 0.f, 0.f};
  } else {
    const float* src = reinterpret_cast<const float*>(maps + ro);
    if ((W & 3) == 0) {  // every row is whole 16-byte words
#pragma unroll
      for (int u = 0; u < (3 * SEG + 3) / 4; ++u) {
        const int i = u * NT + tid;
        if (4 * i < 3 * W) to_lds16(src + 4 * i, sm + 4 * (u * NT + (tid & ~63)));
      }
    } else {
#pragma unroll
      for (int u = 0; u < 3 * SEG; ++u) {
        const int i = u * NT + tid;
        if (i < 3 * W) to_lds4(src + i, sm + (u * NT + (tid & ~63)));
      }
    }
  }
  // guide bytes of pixels xb - 1 .. xb + SEG as unaligned dwords, where those
  // stay inside the image, else one by one
  const int xb = tid * SEG;
  constexpr int ND = (SEG + 2 + 3) / 4;
  uint32_t gw[ND];
#pragma unroll
  for (int q = 0; q < ND; ++q) gw[q] = 0u;
  if (xb < W) {
    const long long g0 = (long long)ro + xb - 1;
    if (g0 >= 0 && g0 + 4 * ND <= (long long)W * H) {
#pragma unroll
      for (int q = 0; q < ND; ++q)
        gw[q] = reinterpret_cast<const UnalignedU32*>(guide + g0 + 4 * q)->v;
    } else {
#pragma unroll
      for (int k = 0; k < SEG + 2; ++k)
        if (xb - 1 + k >= 0 && xb - 1 + k < W) gw[k >> 2] |= (uint32_t)guide[g0 + k] << (8 * (k & 3));
    }
  }
  if (FIRST) {
    __syncthreads();
    const int ty = y / tile;
    if (ty < nty)
      for (int tx = tid; tx < ntx; tx += NT) {
        const int t = ty * ntx + tx;
        if ((flags[t] & 4) && cxy[2 * t + 1] == y)
          row[cxy[2 * t]] = Rec{(float)disp[2 * t], (float)disp[2 * t + 1], 1.f};
      }
  } else {
    wait_loads();
  }
  __syncthreads();
  // the segment is held as float (as stored between passes); every recursion
  // step and carry is computed in double precision
  float a[3 * SEG];
  constexpr int VW = SEG % 4 == 0 ? 4 : 2;  // floats per LDS access
  typedef float fv __attribute__((ext_vector_type(VW)));
  fv* seg = reinterpret_cast<fv*>(row + xb);
#pragma unroll
  for (int q = 0; q < 3 * SEG / VW; ++q) {
    fv v = 0.f;
    if (xb < W) v = seg[q];
#pragma unroll
    for (int k = 0; k < VW; ++k) a[VW * q + k] = v[k];
  }
  if (xb < W && xb + SEG > W) {
#pragma unroll
    for (int j = 0; j < SEG; ++j)
      if (xb + j >= W) a[3 * j] = a[3 * j + 1] = a[3 * j + 2] = 0.f;
  }
  double cc[SEG + 1];  // cc[j]: between xb + j - 1 and xb + j, 0 at the ends
#pragma unroll
  for (int j = 0; j <= SEG; ++j) {
    const int g0 = (int)(gw[j >> 2] >> (8 * (j & 3))) & 255;
    const int g1 = (int)(gw[(j + 1) >> 2] >> (8 * ((j + 1) & 3))) & 255;
    const int x = xb + j;
    cc[j] = x > 0 && x < W ? cf[abs(g1 - g0)] : 0.0;
  }
  Aff t{1.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < SEG; ++j) causal_sum(t, cc[j], a[3 * j], a[3 * j + 1], a[3 * j + 2]);
  double p0, p1, p2;
  line_carry<1, NT / 64, true>(t, wt, p0, p1, p2);
  t = Aff{1.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < SEG; ++j) {
    hold(a[3 * j]);
    hold(a[3 * j + 1]);
    hold(a[3 * j + 2]);
    step(p0, cc[j], a[3 * j]);
    step(p1, cc[j], a[3 * j + 1]);
    step(p2, cc[j], a[3 * j + 2]);
    anticausal_sum(t, cc[j + 1], p0, p1, p2);
  }
  line_carry<1, NT / 64, false>(t, wt, p0, p1, p2);
#pragma unroll
  for (int j = SEG - 1; j >= 0; --j) {
    step(p0, cc[j + 1], a[3 * j]);
    step(p1, cc[j + 1], a[3 * j + 1]);
    step(p2, cc[j + 1], a[3 * j + 2]);
  }
  if (xb < W) {
#pragma unroll
    for (int q = 0; q < 3 * SEG / VW; ++q) {
      fv v;
#pragma unroll
      for (int k = 0; k < VW; ++k) v[k] = a[VW * q + k];
      seg[q] = v;
    }
  }
  __syncthreads();
#pragma unroll 4
  for (int x = tid; x < W; x += NT) maps[ro + x] = row[x];
}

template <int SEG, int NT, bool FIRST>
__global__ __launch_bounds__(NT) void k_dt_row(Rec* __restrict__ maps,
                                                const uint8_t* __restrict__ guide, int W, int H,
                                                const double* __restrict__ coef,
                                                const int32_t* __restrict__ cxy,
                                                const int32_t* __restrict__ disp,
                                                const uint8_t* __restrict__ flags, int ntx,
                                                int nty, int tile,
                                                uint8_t* __restrict__ rowflag) {
  extern __shared__ __align__(16) float sm[];
  __shared__ double cf[256];
  __shared__ Aff wt[NT / 64];
  if (threadIdx.x < 256) cf[threadIdx.x] = coef[threadIdx.x];
  if (FIRST) {
    // several rows per block: most hold no sample and end at once. The rows
    // are dealt by their place within the tiles first, since the corners lie
    // on the few rows around the tiles' centres.
    const int nr = (H + tile - 1) / tile;
    for (int i = blockIdx.x; i < nr * tile; i += gridDim.x) {
      const int y = i % nr * tile + i / nr;
      if (y < H)
        row_pass_of<SEG, NT, true>(y, maps, guide, W, H, cf, wt, sm, cxy, disp, flags, ntx, nty,
                                   tile, rowflag);
    }
  } else {
    row_pass_of<SEG, NT, false>(blockIdx.x, maps, guide, W, H, cf, wt, sm, cxy, disp, flags, ntx,
                                nty, tile, rowflag);
  }
}

// ---------------------------------------------------------------------------
// Vertical pass: a block covers NCOL adjacent columns over the full height as
// NSEG segments of L rows (512 or 1024 threads); each thread keeps its
// segment of one column in registers, so the maps are read and written once.
// Segments of a column sit NCOL lanes apart. The segments' registers bound the
// blocks in flight (two per CU at L = 16), so the sweeps are written not to
// keep their double values: 42 -> 35 us per pass at 5 MP, the last 52 -> 41.
// Runs of 48 bytes per row cost more than the recursion: a copy with this
// access takes 34 us, with runs of 192 bytes 21, but a block of 16 such
// columns would not fit a CU's registers.
template <int NCOL, int NSEG, bool FWD>
__device__ inline void seg_carry(const Aff& v, Aff* wt, double& c0, double& c1, double& c2) {
  line_carry<NCOL, NSEG * NCOL / 64, FWD>(v, wt, c0, c1, c2);
}

template <int L, int NCOL, int NSEG, bool LAST>
__global__ __launch_bounds__(NCOL * NSEG, 4) void k_dt_col(Rec* __restrict__ maps,
                                                        const uint8_t* __restrict__ gt, int hp,
                                                        int W, int H,
                                                        const double* __restrict__ coef,
                                                        float* __restrict__ flow,
                                                        float* __restrict__ ntilde, double nmin,
                                                        const uint8_t* __restrict__ rowflag) {
  __shared__ double cf[257];  // [256]: 0, past the ends
  __shared__ Aff wt[NSEG * NCOL / 64 * NCOL];
  const int tid = threadIdx.x, cl = tid % NCOL, sg = tid / NCOL;
  // XCD-aware strip order: consecutive blocks run on different XCDs, so
  // neighbouring strips (which share cache lines) are given to one XCD
  const int nb = gridDim.x, b = blockIdx.x, full = nb / 8 * 8;
  const int strip = b < full ? (b % 8) * (nb / 8) + b / 8 : b;
  const int col = strip * NCOL + cl;
  const bool act = col < W;
  const int r0 = sg * L;
  const size_t plane = (size_t)W * H;
  for (int i = tid; i < 257; i += NCOL * NSEG) cf[i] = i < 256 ? coef[i] : 0.0;
  __syncthreads();
  // guide bytes of rows r0 .. r0+L-1, four per register, as one aligned load
  // from the column-major copy (r0 is a multiple of L, a multiple of 4, and
  // the copy's rows run past r0 + L), plus the rows r0-1 and r0+L
  static_assert(L % 4 == 0, "segments are whole 4-byte guide words");
  constexpr int NG = L / 4;
  uint32_t gpk[NG];
  uint32_t gup = 0u, gdn = 0u;
  const bool seg_in = act && r0 < H;
  const uint8_t* gcol = gt + (size_t)col * hp;
  if (seg_in) {
    const uint32_t* gw = reinterpret_cast<const uint32_t*>(gcol + r0);
#pragma unroll
    for (int q = 0; q < NG; ++q) gpk[q] = gw[q];
    if (r0 > 0) gup = gcol[r0 - 1];
    if (r0 + L < H) gdn = gcol[r0 + L];
  } else {
#pragma unroll
    for (int q = 0; q < NG; ++q) gpk[q] = 0u;
  }
  // first pass: the rows the row pass left at zero are not read (their
  // flags, as for the guide, aligned loads; the flag buffer runs past the
  // last row)
  uint32_t rf[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) rf[q] = 0x01010101u;
  if (rowflag) {
    const uint32_t* rw = reinterpret_cast<const uint32_t*>(rowflag + r0);
#pragma unroll
    for (int q = 0; q < NG; ++q) rf[q] = seg_in ? rw[q] : 0u;
  }
  // the segment is held as float (as stored between passes); every recursion
  // step and carry is computed in double precision
  float a0[L], a1[L], a2[L];
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const int y = r0 + j;
    const bool in = act && y < H && ((rf[j >> 2] >> (8 * (j & 3))) & 255u);
    const Rec r = in ? maps[(size_t)y * W + col] : Rec{0.f, 0.f, 0.f};
    a0[j] = r.m0;
    a1[j] = r.m1;
    a2[j] = r.m2;
  }
#pragma unroll
  for (int j = 0; j < L; ++j) {
    hold(a0[j]);
    hold(a1[j]);
    hold(a2[j]);
  }
  // |g[j] - g[j - 1]| of rows j = 0 .. L as a byte offset into the table, in
  // 16 bits each (12 used); rows past the ends (and the image's) take the 0
  // behind it
#define GB(j)                                                              \
  ((j) < 0 ? (int)gup                                                      \
   : (j) >= L ? (int)gdn                                                   \
              : (int)((gpk[((j) >= 0 && (j) < L ? (j) : 0) >> 2] >> (8 * ((j) & 3))) & 255u))
  uint32_t dpk[(L + 2) / 2];
#pragma unroll
  for (int j = 0; j <= L; ++j) {
    const uint32_t d = r0 + j > 0 && r0 + j < H ? (uint32_t)abs(GB(j) - GB(j - 1)) : 256u;
    if (j & 1) dpk[j >> 1] |= d << 19;
    else dpk[j >> 1] = d << 3;
  }
#undef GB
  const char* cfb = reinterpret_cast<const char*>(cf);
#define CC(j) \
  (*reinterpret_cast<const double*>(cfb + ((j) & 1 ? dpk[(j) >> 1] >> 16 : dpk[(j) >> 1] & 0xffffu)))
  Aff t{1.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < L; ++j) {
    causal_sum(t, CC(j), a0[j], a1[j], a2[j]);
    pace(j);
  }
  double p0, p1, p2;
  seg_carry<NCOL, NSEG, true>(t, wt, p0, p1, p2);
  t = Aff{1.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < L; ++j) {
    hold(a0[j]);
    hold(a1[j]);
    hold(a2[j]);
    const double c = CC(j);
    step(p0, c, a0[j]);
    step(p1, c, a1[j]);
    step(p2, c, a2[j]);
    anticausal_sum(t, CC(j + 1), p0, p1, p2);
    pace(j);
  }
  seg_carry<NCOL, NSEG, false>(t, wt, p0, p1, p2);
#pragma unroll
  for (int j = L - 1; j >= 0; --j) {
    const double c = CC(j + 1);
    step(p0, c, a0[j]);
    step(p1, c, a1[j]);
    step(p2, c, a2[j]);
    pace(L - 1 - j);
  }
#undef CC
  if (!act) return;
  int rs = r0;
  hold(rs);
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const int y = rs + j;
    if (y >= H) break;
    const size_t o = (size_t)y * W + col;
    if (LAST) {
      const bool ok = (double)a2[j] > nmin;
      double fu, fv;  // (float operands: far from the double range's ends)
      recip_quotients((double)a0[j], (double)a1[j], (double)a2[j], fu, fv);
      flow[o] = ok ? (float)fu : 0.f;
      flow[plane + o] = ok ? (float)fv : 0.f;
      if (ntilde) ntilde[o] = a2[j];
    } else {
      maps[o] = Rec{a0[j], a1[j], a2[j]};
    }
  }
  if (LAST && nmin < 0.0) {  // N~ = 0 counts, which the reciprocal does not take
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const int y = rs + j;
      if (y >= H) break;
      const size_t o = (size_t)y * W + col;
      if (a2[j] == 0.f) {
        flow[o] = a0[j] / a2[j];
        flow[plane + o] = a1[j] / a2[j];
      }
    }
  }
}

// The guide's column-major copy for the column pass, one 64 x 64 tile per
// block (used when the equalisation did not write it).
__global__ __launch_bounds__(256) void k_guide_columns(const uint8_t* __restrict__ guide, int W,
                                                       int H, int hp, uint8_t* __restrict__ gt) {
  __shared__ uint8_t tile[64 * 64];
  const int bx = blockIdx.x * 64, by = blockIdx.y * 64;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int i = threadIdx.x + 256 * u, r = i >> 6, c = i & 63;
    tile[i] = (by + r < H && bx + c < W) ? guide[(size_t)(by + r) * W + bx + c] : 0;
  }
  __syncthreads();
  store_tile_columns(tile, bx, by, W, hp, gt);
}

template <int SEG, int NT>
hipError_t launch_row(bool first, Rec* maps, const uint8_t* guide, int W, int H,
                      const double* cf, const int32_t* cxy, const int32_t* disp,
                      const uint8_t* flags, int ntx, int nty, int tile, uint8_t* rowflag,
                      hipStream_t st) {
  const size_t lds = (size_t)((W + SEG - 1) / SEG) * SEG * sizeof(Rec);
  if (lds > 64 * 1024) {  // rows wider than ~5000 px need more than the default LDS
    hipError_t e = hipFuncSetAttribute(
        reinterpret_cast<const void*>(first ? &k_dt_row<SEG, NT, true> : &k_dt_row<SEG, NT, false>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  // first pass: as many rows per block as leave every block resident at once
  // (16 waves per CU, which the registers of every shape allow, and the LDS);
  // one row per block took two rounds at 5 MP: 23 us against 15
  const int per_cu = (int)std::min<size_t>(1024 / NT, 160 * 1024 / (lds + 3072));
  const int resident = 256 * std::max(per_cu, 1), turns = (H + resident - 1) / resident;
  if (first)
    LNR_LAUNCH((k_dt_row<SEG, NT, true>), dim3((H + turns - 1) / turns), dim3(NT), lds, st, maps, guide, W, H, cf, cxy,
               disp, flags, ntx, nty, tile, rowflag);
  else
    LNR_LAUNCH((k_dt_row<SEG, NT, false>), dim3(H), dim3(NT), lds, st, maps, guide, W, H, cf, cxy,
               disp, flags, ntx, nty, tile, nullptr);
  return hipGetLastError();
}

template <int L, int NCOL, int NSEG>
hipError_t launch_col(bool last, Rec* maps, const uint8_t* gt, int W, int H,
                      const double* cf, float* flow, float* ntilde, double nmin,
                      const uint8_t* rowflag, hipStream_t st) {
  const dim3 grid((W + NCOL - 1) / NCOL);
  const int hp = dt_guide_stride(H);
  if (last)
    LNR_LAUNCH((k_dt_col<L, NCOL, NSEG, true>), grid, dim3(NCOL * NSEG), 0, st, maps, gt, hp, W,
               H, cf, flow, ntilde, nmin, rowflag);
  else
    LNR_LAUNCH((k_dt_col<L, NCOL, NSEG, false>), grid, dim3(NCOL * NSEG), 0, st, maps, gt, hp, W,
               H, cf, flow, ntilde, nmin, rowflag);
  return hipGetLastError();
}

}  // namespace

namespace {
const DtShape kRowShapes[] = {{4, 256, 0, 0, 0}, {8, 256, 0, 0, 0}, {12, 256, 0, 0, 0},
                              {4, 512, 0, 0, 0}, {6, 512, 0, 0, 0}, {8, 512, 0, 0, 0},
                              {12, 512, 0, 0, 0}};
const DtShape kColShapes[] = {{0, 0, 8, 8, 128},  {0, 0, 8, 4, 128},  {0, 0, 16, 4, 128},
                              {0, 0, 8, 2, 256},  {0, 0, 24, 4, 128}, {0, 0, 16, 2, 256},
                              {0, 0, 24, 2, 256}};

hipError_t row_pass(const DtShape& s, bool first, Rec* maps, const uint8_t* guide, int W, int H,
                    const double* cf, const int32_t* cxy, const int32_t* disp,
                    const uint8_t* flags, int ntx, int nty, int tile, uint8_t* rowflag,
                    hipStream_t st) {
#define ROW(SEG, NT)                                                                           \
  if (s.seg == SEG && s.nt == NT)                                                              \
    return launch_row<SEG, NT>(first, maps, guide, W, H, cf, cxy, disp, flags, ntx, nty, tile, \
                               rowflag, st);
  ROW(4, 256) ROW(8, 256) ROW(12, 256) ROW(4, 512) ROW(6, 512) ROW(8, 512) ROW(12, 512)
#undef ROW
  return hipErrorInvalidValue;
}

hipError_t col_pass(const DtShape& s, bool last, Rec* maps, const uint8_t* gt, int W, int H,
                    const double* cf, float* flow, float* ntilde, double nmin,
                    const uint8_t* rowflag, hipStream_t st) {
#define COL(L, NC, NS)                                                                       \
  if (s.l == L && s.ncol == NC && s.nseg == NS)                                               \
    return launch_col<L, NC, NS>(last, maps, gt, W, H, cf, flow, ntilde, nmin, rowflag, st);
  // the listed shapes
  COL(8, 8, 128) COL(8, 4, 128) COL(16, 4, 128) COL(8, 2, 256) COL(24, 4, 128)
  COL(16, 2, 256) COL(24, 2, 256)
  // the others of the fewest rows
  COL(4, 8, 128) COL(4, 4, 128) COL(12, 4, 128) COL(20, 4, 128)
  COL(4, 4, 256) COL(8, 4, 256) COL(12, 4, 256) COL(16, 4, 256) COL(20, 4, 256) COL(24, 4, 256)
#undef COL
  return hipErrorInvalidValue;
}

bool same_col(const DtShape& a, const DtShape& b) {
  return a.l == b.l && a.ncol == b.ncol && a.nseg == b.nseg;
}

bool listed_col(const DtShape& s) {
  for (const DtShape& c : kColShapes)
    if (same_col(c, s)) return true;
  return false;
}

// The column shapes of a height: the fewest rows per segment (whole guide
// words) that cover it, which leaves no segment idle (1440 rows would fill 90
// of 128 segments of 16: of 12, all 120), in blocks of eight columns (up to 8
// rows) or four by 128 segments, or of four by 256.
struct ColForm {
  int ncol, nseg, most;
};
constexpr ColForm kColForms[] = {{8, 128, 8}, {4, 128, 24}, {4, 256, 24}};

DtShape fewest_rows(const ColForm& f, int H) {
  return DtShape{0, 0, ((H + f.nseg - 1) / f.nseg + 3) / 4 * 4, f.ncol, f.nseg};
}
}  // namespace

// A listed row shape with a listed column shape or with one of the height's.
bool dt_shape_valid(const DtShape& s, int W, int H) {
  bool row = false, col = listed_col(s);
  for (const DtShape& r : kRowShapes) row |= r.seg == s.seg && r.nt == s.nt;
  for (const ColForm& f : kColForms) col |= s.l <= f.most && same_col(s, fewest_rows(f, H));
  return row && col && W <= s.seg * s.nt && H <= s.l * s.nseg;
}

// Every listed (row, column) pair that covers W x H; for the tuner, the row
// shapes with the height's column shapes instead. Of 28 sizes none was faster
// with a listed column shape of more rows or of two columns, and 4000 x 3000
// takes 12 rows by 256 segments (a registration 897 us, against 922 with the
// fastest listed one).
int dt_shape_candidates(int W, int H, DtShape* out, int max, bool tuner) {
  int n = 0;
  auto add = [&](const DtShape& r, const DtShape& c) {
    const DtShape s{r.seg, r.nt, c.l, c.ncol, c.nseg};
    if (dt_shape_valid(s, W, H) && n < max) out[n++] = s;
  };
  for (const DtShape& r : kRowShapes) {
    if (tuner)
      for (const ColForm& f : kColForms) add(r, fewest_rows(f, H));
    else
      for (const DtShape& c : kColShapes) add(r, c);
  }
  return n;
}

// The default: the fewest pixels per thread that cover a row, and one of the
// height's column shapes. Heights of more than 128 segments of 24 rows take
// 256 of them in blocks of four columns, not two: runs of 48 bytes per row
// instead of 24 (3000 x 4000: 85 -> 72 us, last 139 -> 103). The column
// kernels' launch bound holds them to 128 registers, which segments of 24 rows
// exceed by 24 to 28 bytes of scratch per lane.
DtShape dt_default_shape(int W, int H) {
  DtShape s;
  if (W <= 1024) { s.seg = 4; s.nt = 256; }
  else if (W <= 2048) { s.seg = 8; s.nt = 256; }
  else if (W <= 3072) { s.seg = 12; s.nt = 256; }
  else if (W <= 4096) { s.seg = 8; s.nt = 512; }
  else { s.seg = 12; s.nt = 512; }
  const DtShape c = fewest_rows(kColForms[H <= 1024 ? 0 : H <= 3072 ? 1 : 2], H);
  return DtShape{s.seg, s.nt, c.l, c.ncol, c.nseg};
}

static DtArgs dt_args(const lnr_params& p) {
  DtArgs a;
  a.iters = p.dt_iters;
  a.sigma_s = p.sigma_s;
  a.ratio = p.sigma_s / p.sigma_r;
  return a;
}

hipError_t launch_dt_coef(const lnr_params& p, double* coef, uint32_t* zero, int nzero,
                          double* ident, hipStream_t st, unsigned long long* zero64,
                          int nzero64) {
  LNR_LAUNCH(k_dt_coef, dim3(p.dt_iters), dim3(256), 0, st, dt_args(p), coef, zero, nzero, ident,
             zero64, zero64 ? nzero64 : 0);
  return hipGetLastError();
}

hipError_t launch_dt_coef_jobs(const lnr_params& p, const SetupJob* jobs, int njobs,
                               hipStream_t st) {
  LNR_LAUNCH(k_dt_coef_jobs, dim3(p.dt_iters, njobs), dim3(256), 0, st, dt_args(p), jobs);
  return hipGetLastError();
}

hipError_t launch_flow(const int32_t* corner_xy, const int32_t* disp, const uint8_t* flags,
                       int ntx, int nty, int tile, const uint8_t* guide, uint8_t* guide_t,
                       int W, int H, const lnr_params& p, void* maps_v, double* coef,
                       float* flow, float* ntilde, hipStream_t st, const DtShape* shape,
                       bool coef_ready, bool guide_t_ready) {
  Rec* maps = static_cast<Rec*>(maps_v);
  uint8_t* rowflag = static_cast<uint8_t*>(maps_v) + dt_rowflag_offset(W, H);
  if (!guide_t_ready) {
    LNR_LAUNCH(k_guide_columns, dim3((W + 63) / 64, (H + 63) / 64), dim3(256), 0, st, guide, W, H,
               dt_guide_stride(H), guide_t);
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
  }
  DtArgs a;
  a.iters = p.dt_iters;
  const DtShape sh = shape && dt_shape_valid(*shape, W, H) ? *shape : dt_default_shape(W, H);
  hipError_t e;
  if (!coef_ready && (e = launch_dt_coef(p, coef, nullptr, 0, nullptr, st)) != hipSuccess) return e;
  const double nmin = p.n_min;
  for (int i = 0; i < a.iters; ++i) {
    const double* cf = coef + 256 * i;
    const bool first = i == 0, last = i + 1 == a.iters;
    e = row_pass(sh, first, maps, guide, W, H, cf, corner_xy, disp, flags, ntx, nty, tile,
                 rowflag, st);
    if (e != hipSuccess) return e;
    e = col_pass(sh, last, maps, guide_t, W, H, cf, flow, ntilde, nmin,
                 first ? rowflag : nullptr, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lnr

// k_weed.hip -- match weeding (paper Sec. 2.3, Eq. 5) and the level
// homography (Sec. 2.2) on the GPU, with no host round trip. Matches are the
// valid tiles of the level, indexed in tile order (centred level coordinates:
// source side p + d - c, reference side p - c).
//
// k_valid: the valid-match bits of the tiles, one 64-bit word per 64 tiles
//         (a wave ballot each). In a registration the level's warp clears
//         them and its search sets the bits instead.
// k_hyp:  a block draws and solves a group of hypotheses and tests every tile
//         against them. Its first wave prefix-sums the words' popcounts,
//         draws four distinct match indices per hypothesis from the
//         counter-based SplitMix64 stream, maps them to tiles with a
//         rank-select over the words and solves the 8x8 systems in double
//         precision, a row per lane; wave ballots over the tiles give each
//         hypothesis' count and inlier bits, so that the block knows by
//         itself which of its hypotheses are accepted (count above delta),
//         the union of their inliers and its best hypothesis. A few
//         iterations over many tiles: a block per chunk of the tiles as well,
//         which leaves every hypothesis' inlier bits and its chunk's count.
// k_fit:  M, the union of the blocks' unions (any split of the iterations
//         gives the same M, as the paper notes), and the best consensus of
//         all blocks (most inliers, lowest iteration), whose inliers are
//         tested once more; writes the tiles' flags and sums the
//         least-squares normal equations of G: p -> p + d over those inliers
//         exactly in int64 (order-free), solves them (the solver of k_hyp)
//         and composes H_l = H_{l+1} o G. One block up to kFitWords words;
//         larger levels spread the tiles over blocks and k_solve finishes.
// The kernels are ordered by the stream; no block waits for another.
#include <algorithm>

#include "lnr_device.h"
#include "lnr_internal.h"

namespace lnr {
namespace {

__device__ inline unsigned long long splitmix64(unsigned long long x) {
  unsigned long long z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Lane exchanges within groups of eight lanes, on the vector ALU.
template <int CTRL>
__device__ inline int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)dpp_i32<CTRL>((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)dpp_i32<CTRL>((int)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror8 = 0x141;  // quad_perm, row_half_mirror

// 8x8 solve of augmented systems, one per group of eight lanes: lane r of a
// group holds row r (9 values). Gaussian elimination with partial pivoting:
// of the rows not yet used, the largest |pivot|, the first on ties in the
// order that swapping rows would leave them in (pos; rows stay in their
// lanes); |pivot| < 1e-12 or NaN fails. Every value is computed with the
// operations, in the order, of the one-lane elimination, so the solution
// does not depend on the layout; a column's row updates and divisions run
// side by side instead of one after another. Every lane keeps the pivot rows
// (broadcast once per column) and substitutes back by itself. All 64 lanes
// take part; a failed group goes on with meaningless values.
// Quotients are formed as div2 does, from one reciprocal per pivot: the
// values of a system of integer coordinates stay far from the ends of the
// exponent range, where that differs from a plain division.
__device__ inline bool solve8_rows(double (&a)[9], double (&x)[8]) {
  const int lane = threadIdx.x & 63, group = lane & 56;
  int pos = lane & 7;
  bool ok = true;
  double U[8][9], r[8];  // pivot rows and the pivots' reciprocals
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    // the largest high word decides unless two rows share it
    const double v = fabs(a[c]);
    const int hw = pos >= c ? __double2hiint(v) : -1;
    int top = max(hw, dpp_i32<kXor1>(hw));
    top = max(top, dpp_i32<kXor2>(top));
    top = max(top, dpp_i32<kMirror8>(top));
    double rc = __builtin_amdgcn_rcp(a[c]);  // every row's, while the search goes on
    rc = fma(fma(-a[c], rc, 1.0), rc, rc);
    rc = fma(fma(-a[c], rc, 1.0), rc, rc);
    int at = (int)(__ballot(hw == top) >> group) & 255;
    if (__any((at & (at - 1)) != 0)) {
      const double w = pos >= c ? v : -1.0;
      double best = fmax(w, dpp_f64<kXor1>(w));
      best = fmax(best, dpp_f64<kXor2>(best));
      best = fmax(best, dpp_f64<kMirror8>(best));
      int first = w == best ? pos : 99;
      first = min(first, dpp_i32<kXor1>(first));
      first = min(first, dpp_i32<kXor2>(first));
      first = min(first, dpp_i32<kMirror8>(first));
      at = (int)(__ballot(pos == first) >> group) & 255;
    }
    const int src = group | ((__ffs(at) - 1) & 7);
#pragma unroll
    for (int j = c; j < 9; ++j) U[c][j] = __shfl(a[j], src);
    r[c] = __shfl(rc, src);
    const int was = __shfl(pos, src);
    ok = ok && fabs(U[c][c]) >= 1e-12;
    if (lane == src) pos = c;
    else if (pos == c) pos = was;
    const double q = a[c] * r[c];
    const double f = fma(fma(-U[c][c], q, a[c]), r[c], q);  // a[c] / pivot
    if (pos > c) {
#pragma unroll
      for (int j = c + 1; j < 9; ++j) a[j] = a[j] - f * U[c][j];
    }
  }
#pragma unroll
  for (int c = 7; c >= 0; --c) {
    double t = U[c][8];
#pragma unroll
    for (int j = c + 1; j < 8; ++j) t = t - U[c][j] * x[j];
    const double q = t * r[c];
    x[c] = fma(fma(-U[c][c], q, t), r[c], q);  // t / pivot
  }
  return ok;
}

// inlier test |G(s) - t|^2 < eps^2, fixed operation order. Without a plain
// division (PLAIN false) the quotients come straight from div2's reciprocal,
// with no branch, so that the tests of several hypotheses overlap: the same
// decisions for coefficients below kPlainG, since the products of
// coefficients and integer coordinates then stay in range, and the
// denominator g6 x + g7 y + 1 is 0 (both forms reject) or at least 2^-54.
constexpr double kPlainG = 0x1p400;

template <bool PLAIN>
__device__ inline bool is_inlier(const double* g, int4 m, double eps2) {
  const double sx = (double)m.x, sy = (double)m.y;
  const double den = (g[6] * sx + g[7] * sy) + 1.0;
  const double nx = (g[0] * sx + g[1] * sy) + g[2], ny = (g[3] * sx + g[4] * sy) + g[5];
  double gx, gy;
  if constexpr (PLAIN) {
    gx = nx / den;
    gy = ny / den;
  } else {
    recip_quotients(nx, ny, den, gx, gy);
  }
  const double ex = gx - (double)m.z, ey = gy - (double)m.w;
  const double e2 = ex * ex + ey * ey;
  return e2 < eps2;
}

// whether the tests of hypothesis g need plain divisions (NaN included)
__device__ inline bool needs_plain(const double* g) {
  bool small = true;
#pragma unroll
  for (int i = 0; i < 8; ++i) small = small && fabs(g[i]) < kPlainG;
  return !small;
}

__device__ inline int4 tile_match(const int32_t* __restrict__ cxy,
                                  const int32_t* __restrict__ disp, int t, int ox, int oy) {
  const int px = cxy[2 * t], py = cxy[2 * t + 1];
  return make_int4(px + disp[2 * t] - ox, py + disp[2 * t + 1] - oy, px - ox, py - oy);
}

struct WeedArgs {
  int iters, level, delta_min, delta_pct;
  double eps2;
  unsigned long long seed;
};

__device__ inline int weed_delta(int N, const WeedArgs& a) {
  const int d = (N * a.delta_pct + 99) / 100;
  return d > a.delta_min ? d : a.delta_min;
}

// position of the k-th (0-based) set bit of m (k < popcount(m))
__device__ inline int select_bit(unsigned long long m, int k) {
  int pos = 0;
#pragma unroll
  for (int half = 32; half >= 1; half >>= 1) {
    const unsigned long long lo = m & ((1ull << half) - 1ull);
    const int c = __popcll(lo);
    if (k >= c) {
      k -= c;
      m >>= half;
      pos += half;
    } else {
      m = lo;
    }
  }
  return pos;
}

constexpr int kValidThreads = 256;
constexpr int kFitThreads = 512;
constexpr int kFitOne = 32;       // levels of up to this many words: one k_fit block
constexpr int kMaxIters = 65536;  // the parameter check's bound on weed_iters
constexpr int kMaxWords = 2304;   // tile bitmask words: (6144 / 16)^2 tiles

// word wi of vb = valid-match bits of tiles 64 wi .. 64 wi + 63
__global__ __launch_bounds__(kValidThreads) void k_valid(const uint8_t* __restrict__ flags,
                                                         int ntiles, int nwords,
                                                         unsigned long long* __restrict__ vb) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wi = blockIdx.x * (kValidThreads / 64) + (tid >> 6);
  if (wi >= nwords) return;  // whole waves
  const int t = wi * 64 + lane;
  const unsigned long long m = __ballot(t < ntiles && (flags[t] & 2));
  if (lane == 0) vb[wi] = m;
}

// Orders the LDS accesses of one wave's lanes (they execute in order).
__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ inline unsigned long long wave_or_u64(unsigned long long v) {
  return wave_fold_u64(v, [](unsigned long long p, unsigned long long q) { return p | q; });
}

// dynamic LDS of k_hyp: the words, the union and the inlier bits of ipb
// hypotheses (8 bytes a word each), the prefix counts; where more than ipb are
// solved together, their coefficients and usability
constexpr size_t hyp_lds(int words, int ipb, int per) {
  return (size_t)words * 8 * (2 + ipb) + ((size_t)words + 1) * 4 +
         (per > ipb ? (size_t)per * (64 + 4) : 0);
}
// what a workgroup can take, less k_hyp's own shared variables
constexpr size_t kHypLdsMax = 160 * 1024 - 1024;
static_assert(hyp_lds(kMaxWords, 4, 64) <= kHypLdsMax, "the wide form takes every level");

// The kernels below take one level of one pair (JOBS false: the job is the
// kernel argument) or a table of jobs, one per blockIdx.z (batches).

// How k_hyp splits a level's iterations: hypotheses that a block tests
// together (ipb) and its threads, hypotheses that it solves together (per) and
// blocks. A pair's levels of more than 256 tiles test four per 512 threads
// (every CU a block at the default 1024 iterations, half the tests per wave);
// the smallest levels, and batches, whose jobs fill the chip anyway, eight (a
// full wave of eight-lane solves) per 256, unless the inlier words of eight do
// not fit a workgroup's memory (more than 1938 words: 124,032 tiles). More
// iterations than the blocks take so are solved by as many of a block's waves
// as it needs, eight hypotheses each, before they are tested: with every solve
// on the first wave 65,536 iterations took 274 us at 300 tiles and 735 at
// 4860 (all of a level's weeding), so 130 and 586. Iterations that leave half of
// the CUs without a block are tested by several blocks per group, each on a
// chunk of the tiles, where the level is large enough for that to pay for the
// chunks' counts: from 49 words on, above 256 hypotheses from 129 on (one
// iteration over 46,500 tiles 98 us in one block, 28 in chunks; 256 over 3136
// tiles 28.0 and 25.6; 512 over 4860 tiles 31 and 34, over 11,625 44 and 38).
struct HypForm {
  bool wide;
  int per, blocks, chunks;
};
inline HypForm hyp_form(int iters, int ntiles, int words, int njobs) {
  HypForm f;
  const int groups = (iters + 3) / 4;
  f.chunks = 1;
  if (iters <= kSplitIters && words > (iters <= kWeedBlocks ? 48 : 128) && groups * njobs <= 128)
    f.chunks = std::min({256 / (groups * njobs), words / kSplitWords, kSplitChunks});
  if (f.chunks > 1) {
    f.wide = true;
    f.per = 4;
    f.blocks = groups;
    return f;
  }
  const int share = (iters + kWeedBlocks - 1) / kWeedBlocks;
  const int narrow = std::min(std::max((share + 7) / 8 * 8, 8), 32);
  f.wide = (ntiles > 256 && njobs < 4) || hyp_lds(words, 8, narrow) > kHypLdsMax;
  f.per = f.wide ? std::min((share + 3) / 4 * 4, 64) : narrow;
  f.blocks = weed_blocks(iters, f.per);
  return f;
}

// A coarse level (15 to 1200 tiles) is bound by the first wave's instruction
// count, one every four or five cycles: eight-lane solves, draws in parallel,
// tests without branches. 8.0 us at 300 tiles and 9 at 15; one system per
// lane and a launch of its own for the tests took 8.6 + 4.2 us. At 4860
// tiles the tests are the work: 17 us against 9.2 + 12.8.
// kManyHyp: `solved` hypotheses are solved together, else IPB (a kernel of its
// own: the usual one takes 0.3 us less without the turns). kSplitHyp: the tiles
// of chunk blockIdx.y only.
enum HypMode { kUsualHyp, kManyHyp, kSplitHyp };
template <bool JOBS, int IPB, int NT, HypMode MODE>
__global__ __launch_bounds__(NT, NT == 256 ? 3 : 2) void k_hyp(WeedJob one,
                                                               const WeedJob* __restrict__ jobs,
                                                               WeedArgs a, int solved) {
  constexpr bool MANY = MODE == kManyHyp, SPLIT = MODE == kSplitHyp;
  const int per = MANY ? solved : IPB;
  const WeedJob J = JOBS ? jobs[blockIdx.z] : one;
  const unsigned long long* __restrict__ vbg = J.b.vb;
  const int32_t* __restrict__ cxy = J.cxy;
  const int32_t* __restrict__ disp = J.disp;
  const int nwords = J.words, ntiles = J.ntiles;
  const int ox = J.w / 2, oy = J.h / 2;
  constexpr int NW = NT / 64;
  extern __shared__ __align__(16) unsigned long long dyn[];
  __shared__ __align__(16) double few_gs[MANY ? 1 : IPB][8];
  __shared__ int few_usable[MANY ? 1 : IPB];
  double (*gs)[8] = MANY ? reinterpret_cast<double (*)[8]>(dyn) : few_gs;  // [per]
  unsigned long long* vb = dyn + (MANY ? 8 * per : 0);  // valid-tile bits, tile order
  unsigned long long* uni = vb + nwords;           // union of the accepted inliers
  unsigned long long* inl = uni + nwords;          // [nwords][IPB] inlier bits
  // valid tiles before a word
  int* wpre = reinterpret_cast<int*>(inl + (SPLIT ? 0 : (size_t)nwords * IPB));
  // [per] 0: not usable, 1: usable, 2: usable, tested with plain divisions
  int* usable = MANY ? wpre + nwords + 1 : few_usable;
  __shared__ int wc[IPB][NW];
  __shared__ int matches;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the tested words
  const int wpc = SPLIT ? split_words(nwords, gridDim.y) : nwords;
  const int w0 = SPLIT ? blockIdx.y * wpc : 0, w1 = SPLIT ? min(nwords, w0 + wpc) : nwords;
  if (SPLIT && w0 >= nwords) return;  // (a level has at least one word)
  // this thread's first tile, in flight with the words
  int4 mine = make_int4(0, 0, 0, 0);
  if (ntiles > 0) mine = tile_match(cxy, disp, min(w0 * 64 + tid, ntiles - 1), ox, oy);
  // The first wave prepares, solves (up to eight hypotheses) and counts by
  // itself; the others only test, between the two barriers of a group.
  int N = 0, delta = 0;           // (N: the solving waves; delta: the first)
  unsigned long long best = 0ull;  // this block's best key (first wave)
  double bg = 0.0;                 // its coefficient `lane` (lanes 0..7)
  const unsigned long long seed = a.seed ^ ((unsigned long long)(uint32_t)a.level << 56);
  if (wave == 0) {
    // exclusive prefix of the words' popcounts
    int incl;
    if (nwords <= 64) {
      const unsigned long long v = lane < nwords ? vbg[lane] : 0ull;
      const int c = __popcll(v);
      incl = wave_scan_i32(c);
      if (lane < nwords) {
        vb[lane] = v;
        uni[lane] = 0ull;
        wpre[lane] = incl - c;
      }
    } else {
      for (int q0 = 0; q0 < nwords; q0 += 8 * 64) {
        unsigned long long r[8];  // eight loads in flight per lane
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = vbg[min(q0 + u * 64 + lane, nwords - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int wi = q0 + u * 64 + lane;
          if (wi < nwords) {
            vb[wi] = r[u];
            uni[wi] = 0ull;
          }
        }
      }
      wave_lds_order();
      const int K = (nwords + 63) / 64;  // lane owns a run of K words
      int c = 0;
      for (int j = 0; j < K; ++j) {
        const int wi = lane * K + j;
        if (wi < nwords) c += __popcll(vb[wi]);
      }
      incl = wave_scan_i32(c);
      int run = incl - c;
      for (int j = 0; j < K; ++j) {
        const int wi = lane * K + j;
        if (wi < nwords) {
          wpre[wi] = run;
          run += __popcll(vb[wi]);
        }
      }
    }
    wave_lds_order();
    N = __builtin_amdgcn_readlane(incl, 63);
    delta = weed_delta(N, a);
    if (blockIdx.x == 0 && w0 == 0 && lane == 0) *J.b.nmatch = N;
    if (MANY && lane == 0) matches = N;
  }
  if (MANY) {  // more waves solve: the words are theirs too
    __syncthreads();
    N = matches;
  }
  // (one turn but for kManyHyp; a straight line compiles to tests unrolled
  // further, 0.5 us per launch of a batch's)
  const int turn = (int)gridDim.x * per;
  for (int r0 = blockIdx.x * per; r0 < a.iters; r0 += turn) {
    if (MANY ? 8 * wave < per : wave == 0) {
      // eight lanes per hypothesis: each draws one index of the first eight
      // and sets up row (lane & 7) of the system, the x or y equation of
      // match row / 2
      const int q0 = MANY ? 8 * wave : 0;
      const int q = min(q0 + (lane >> 3), per - 1), row = lane & 7;
      const int it = r0 + q;
      const unsigned long long base = seed + (unsigned long long)it * 16ull;
      auto draw = [&](int t) {
        return (int)__umulhi((uint32_t)(splitmix64(base + (unsigned long long)t) >> 32),
                             (uint32_t)N);
      };
      const int own = draw(row);
      int pk[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) pk[t] = __shfl(own, (lane & 56) + t);
      int np = 4;
      if (__any(pk[1] == pk[0] || pk[2] == pk[0] || pk[2] == pk[1] || pk[3] == pk[0] ||
                pk[3] == pk[1] || pk[3] == pk[2])) {
        // a repeat is drawn again: the first four distinct of sixteen draws
        pk[0] = pk[1] = pk[2] = pk[3] = -1;
        np = 0;
        for (int t = 0; t < 16; ++t) {
          const int id = t < 8 ? __shfl(own, (lane & 56) + t) : draw(t);
          const bool take = np < 4 && id != pk[0] && id != pk[1] && id != pk[2];
          if (take && np == 0) pk[0] = id;
          if (take && np == 1) pk[1] = id;
          if (take && np == 2) pk[2] = id;
          if (take && np == 3) pk[3] = id;
          np += take;
          if (t >= 7 && __all(np == 4)) break;
        }
      }
      bool good = N >= 4 && np == 4 && it < a.iters;
      // match index -> tile: last word with wpre <= id, then the bit within it
      const int m = row >> 1;
      const int id = max(m == 0 ? pk[0] : m == 1 ? pk[1] : m == 2 ? pk[2] : pk[3], 0);
      int lo = 0, hi = nwords - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (wpre[mid] <= id) lo = mid;
        else hi = mid - 1;
      }
      const int tq = max(min(lo * 64 + select_bit(vb[lo], id - wpre[lo]), ntiles - 1), 0);
      int4 mt = make_int4(0, 0, 0, 0);
      if (ntiles > 0) mt = tile_match(cxy, disp, tq, ox, oy);
      const double sx = (double)mt.x, sy = (double)mt.y;
      const bool yrow = row & 1;
      const double tt = yrow ? (double)mt.w : (double)mt.z;
      double A[9] = {yrow ? 0.0 : sx, yrow ? 0.0 : sy, yrow ? 0.0 : 1.0,
                     yrow ? sx : 0.0, yrow ? sy : 0.0, yrow ? 1.0 : 0.0,
                     -(sx * tt),      -(sy * tt),      tt};
      double g[8];
      const bool solved = solve8_rows(A, g);
      good = good && solved;
      if (row == 0 && q0 + (lane >> 3) < per) {
        // not usable: too few matches, degenerate draw or fit
        usable[q] = good ? (needs_plain(g) ? 2 : 1) : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) gs[q][i] = g[i];
      }
    }
    __syncthreads();
    for (int it0 = r0;; it0 += IPB) {
      // every tile against the next IPB hypotheses
      const double (*g)[8] = MANY ? gs + (it0 - r0) : gs;
      const int* use = MANY ? usable + (it0 - r0) : usable;
      bool plain = false;
#pragma unroll
      for (int q = 0; q < IPB; ++q) plain = plain || use[q] == 2;
      // four hypotheses of many stay in registers over the tiles (read again for
      // every tile they keep the LDS unit busier than the tests the vector ALU)
      constexpr bool HELD = MANY && IPB == 4;
      double r[4][8];
      if constexpr (HELD)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < 8; ++i) r[q][i] = g[q][i];
      int cnt = 0;  // lane q: hypothesis q
      for (int t0 = w0 * 64; t0 < w1 * 64; t0 += NT) {
        const int t = t0 + tid, word = t >> 6;
        if (word >= w1) break;  // whole waves
        const bool valid = (vb[word] >> lane) & 1ull;
        const int4 m = t0 == w0 * 64 ? mine : tile_match(cxy, disp, min(t, ntiles - 1), ox, oy);
        unsigned long long keep = 0ull;
#pragma unroll 4
        for (int q = 0; q < IPB; ++q) {
          const unsigned long long b =
              __ballot(valid && is_inlier<false>(HELD ? r[q & 3] : g[q], m, a.eps2));
          if (lane == q) keep = b;
        }
        if (plain)
          for (int q = 0; q < IPB; ++q) {
            if (use[q] != 2) continue;
            const unsigned long long b = __ballot(valid && is_inlier<true>(g[q], m, a.eps2));
            if (lane == q) keep = b;
          }
        cnt += __popcll(keep);
        if constexpr (SPLIT) {
          if (lane < IPB && it0 + lane < a.iters)
            J.b.part[(size_t)word * a.iters + it0 + lane] = keep;
        } else {
          if (lane < IPB) inl[(size_t)word * IPB + lane] = keep;
        }
      }
      if (lane < IPB) wc[lane][wave] = cnt;
      __syncthreads();
      if (wave == 0) {
        // lane q counts hypothesis q
        int c = 0;
        unsigned long long key = 0ull;
        if (lane < IPB && use[lane]) {
#pragma unroll
          for (int w = 0; w < NW; ++w) c += wc[lane][w];
          key = ((unsigned long long)(uint32_t)c << 32) |
                (unsigned long long)(~(uint32_t)(it0 + lane));
        }
        if constexpr (SPLIT) {  // k_fit adds up the chunks' counts
          if (lane < IPB && it0 + lane < a.iters)
            J.b.key[(size_t)blockIdx.y * a.iters + it0 + lane] = key;
          if (w0 == 0 && lane < IPB * 8 && it0 + (lane >> 3) < a.iters)
            J.b.G[(size_t)it0 * 8 + lane] = g[lane >> 3][lane & 7];
          return;
        }
        const unsigned int acc = (unsigned int)__ballot(c > delta);  // accepted
        const unsigned long long top = wave_max_u64(key);
        if (top > best) {
          best = top;
          const int q = (int)(~(uint32_t)top) - it0;
          if (lane < 8) bg = g[q][lane];
        }
        if (acc)
          for (int w = lane; w < nwords; w += 64) {
            unsigned long long v = uni[w];
            for (unsigned int r = acc; r; r &= r - 1)
              v |= inl[(size_t)w * IPB + __builtin_ctz(r)];
            uni[w] = v;
          }
      }
      // (the first wave is done with the counts, the bits and the hypotheses
      // before they are written again)
      if (!MANY) break;
      const bool more = it0 + IPB < min(r0 + per, a.iters);
      if (more || r0 + turn < a.iters) __syncthreads();
      if (!more) break;
    }
  }
  if (wave != 0 || SPLIT) return;
  if (lane < 8) J.b.G[(size_t)blockIdx.x * 8 + lane] = bg;
  if (lane == 0) J.b.key[blockIdx.x] = best;
  if ((int)(best >> 32) > delta)  // an accepted hypothesis: k_fit reads them
    for (int w = lane; w < nwords; w += 64)
      J.b.part[(size_t)w * gridDim.x + blockIdx.x] = uni[w];
}

// distinct sums of the normal equations (order: 1, x, y, xx, xy, yy, u, v,
// xu, yu, xv, yv, xxu, xyu, yyu, xxv, xyv, yyv, xq, yq, xxq, xyq, yyq with
// q = u^2 + v^2), and a zero
constexpr int kSums = 24;

// The terms of degree two and more of one match, products of two in type T.
template <typename T>
__device__ inline void add_terms(long long (&s)[kSums], T x, T y, T u, T v) {
  const T xx = x * x, xy = x * y, yy = y * y, q = u * u + v * v;
  auto mad = [](long long& acc, T p, T r) { acc += (long long)p * (long long)r; };
  s[3] += xx; s[4] += xy; s[5] += yy;
  mad(s[8], x, u);   mad(s[9], y, u);   mad(s[10], x, v);  mad(s[11], y, v);
  mad(s[12], xx, u); mad(s[13], xy, u); mad(s[14], yy, u);
  mad(s[15], xx, v); mad(s[16], xy, v); mad(s[17], yy, v);
  mad(s[18], x, q);  mad(s[19], y, q);
  mad(s[20], xx, q); mad(s[21], xy, q); mad(s[22], yy, q);
}

// One step of summing N values over the wave: the lanes' halves (bit OFF)
// keep half of the values each. Returns the values left per lane.
template <int OFF, int N>
__device__ inline void halve_sums(long long (&s)[kSums]) {
  constexpr int H = (N + 1) / 2;
  const bool hi = (threadIdx.x & OFF) != 0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const long long up = i + H < N ? s[i + H] : 0;
    const long long keep = hi ? up : s[i], give = hi ? s[i] : up;
    s[i] = keep + __shfl_xor(give, OFF);
  }
}

// The wave's totals of s[0, 24) into out[24] (exact int64, order-free): 25
// exchanges of one value instead of 6 for each of the 24.
__device__ inline void wave_sums(long long (&s)[kSums], long long* out) {
  halve_sums<32, 24>(s);
  halve_sums<16, 12>(s);
  halve_sums<8, 6>(s);
  halve_sums<4, 3>(s);
  halve_sums<2, 2>(s);
  s[0] += __shfl_xor(s[0], 1);
  const int l = threadIdx.x;
  const int k = (l & 4 ? 2 : 0) + (l & 2 ? 1 : 0);
  if (!(l & 1) && k < 3) out[(l & 32 ? 12 : 0) + (l & 16 ? 6 : 0) + (l & 8 ? 3 : 0) + k] = s[0];
}

// polynomial degree of unknown i (h11 h12 h13 h21 h22 h23 h31 h32) in the
// coordinates, for the power-of-two scaling
__device__ inline int deg_of(int i) { return (i == 2 || i == 5) ? 0 : (i >= 6 ? 2 : 1); }

// Row r of the normal equations A^T A | A^T b of the rows
// (x, y, 1, 0, 0, 0, -xu, -yu | u) and (0, 0, 0, x, y, 1, -xv, -yv | v) as
// codes of six bits from entry 0 up: the sum's index, plus 32 where negated
// (23: the zero).
constexpr unsigned long long row_code(const int (&e)[9]) {
  unsigned long long c = 0ull;
  for (int j = 0; j < 9; ++j) c |= (unsigned long long)e[j] << (6 * j);
  return c;
}
constexpr int kZ = 23, kM = 32;
constexpr int kRow[8][9] = {
    {3, 4, 1, kZ, kZ, kZ, kM + 12, kM + 13, 8},
    {4, 5, 2, kZ, kZ, kZ, kM + 13, kM + 14, 9},
    {1, 2, 0, kZ, kZ, kZ, kM + 8, kM + 9, 6},
    {kZ, kZ, kZ, 3, 4, 1, kM + 15, kM + 16, 10},
    {kZ, kZ, kZ, 4, 5, 2, kM + 16, kM + 17, 11},
    {kZ, kZ, kZ, 1, 2, 0, kM + 10, kM + 11, 7},
    {kM + 12, kM + 13, kM + 8, kM + 15, kM + 16, kM + 10, 20, 21, kM + 18},
    {kM + 13, kM + 14, kM + 9, kM + 16, kM + 17, kM + 11, 21, 22, kM + 19}};
constexpr unsigned long long kCode[8] = {row_code(kRow[0]), row_code(kRow[1]), row_code(kRow[2]),
                                         row_code(kRow[3]), row_code(kRow[4]), row_code(kRow[5]),
                                         row_code(kRow[6]), row_code(kRow[7])};

// The level fit from the sums (LDS: tot as doubles, msel of them), by the
// first wave of a block, then H_l = Hbase o G with Hbase = H_{l+1} (matches
// relative to the warped source) or the identity (absolute matches);
// H_l = H_{l+1} when fewer than 4 matches were fitted or the solve fails.
// A lane per row of the system, then a lane per entry of the product: lane
// 3 i + j holds Hprev[i][j] in hp and row i of Hbase in hb.
__device__ inline void solve_level(const WeedJob& J, const double* tot, int msel, double hp,
                                   const double (&hb)[3]) {
  const int w = J.w, h = J.h, lane = threadIdx.x & 63, row = lane & 7;
  const int ox = w / 2, oy = h / 2;
  const int mx = max(max(ox, oy), 1);
  const int k = mx > 1 ? 32 - __clz(mx - 1) : 0;  // 2^k >= mx
  unsigned long long code = kCode[0];
#pragma unroll
  for (int r = 1; r < 8; ++r) code = row == r ? kCode[r] : code;
  const int dr = -k * deg_of(row);
  double A[9];
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const int e = (int)(code >> (6 * j)) & 63;
    const double v = tot[e & 31];
    A[j] = ldexp(e & 32 ? -v : v, dr - k * (j < 8 ? deg_of(j) : 1));
  }
  double hs[8];
  const bool ok = solve8_rows(A, hs);
  double G[9];
#pragma unroll
  for (int i = 0; i < 8; ++i) G[i] = ldexp(hs[i], k * (1 - deg_of(i)));
  G[8] = 1.0;
  // H = Hbase ((P G) Q), every entry's sum left to right as mat3_mul forms it
  const double pox = (double)(2 * ox - (w - 1)), poy = (double)(2 * oy - (h - 1));
  const double Pm[9] = {2, 0, pox, 0, 2, poy, 0, 0, (double)w};
  double T[9];
  mat3_mul(Pm, G, T);
  const int j = min(lane, 8) % 3;
  const double q0 = j == 0 ? (double)w : j == 2 ? -pox : 0.0;
  const double q1 = j == 1 ? (double)w : j == 2 ? -poy : 0.0;
  const double q2 = j == 2 ? 2.0 : 0.0;
  double c[3];  // column j of (P G) Q
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    c[m] = T[3 * m] * q0;
    c[m] = c[m] + T[3 * m + 1] * q1;
    c[m] = c[m] + T[3 * m + 2] * q2;
  }
  double t = hb[0] * c[0];
  t = t + hb[1] * c[1];
  t = t + hb[2] * c[2];
  const double d = __shfl(t, 8);
  const double hn = t / d;
  const bool take = msel >= 4 && ok && d != 0.0 && !__any(lane < 9 && !isfinite(hn));
  if (lane < 9) J.Hout[lane] = take ? hn : hp;
  if (lane == 0) J.counts[1] = msel;
}

// Block x owns tile words [x wpb, (x + 1) wpb): the union M over the nhyp blocks
// of k_hyp (per iterations a turn; in chunks: over the hypotheses, whose keys
// are the chunks' with the counts added up), flags 4 (in M) and 8 (in the fit)
// of its tiles and their least-squares terms; the level's only block
// then solves, several leave their sums to k_solve. One block is enough for
// kFitOne words (2048 tiles, four per thread); beyond, its one CU is the
// limit (4860 tiles: 20 us in one block, 7.5 us in five and 5.6 for k_solve).
// 7.6 us at 300 tiles, where a union over all the iterations' inlier rows and
// a one-lane solve in a launch of its own took 10.1 + 6.6.
template <bool JOBS, int SLOTS>
__global__ __launch_bounds__(kFitThreads) void k_fit(WeedJob one,
                                                     const WeedJob* __restrict__ jobs,
                                                     WeedArgs a, int per, int nhyp, int chunks,
                                                     int wpb) {
  const WeedJob J = JOBS ? jobs[blockIdx.z] : one;
  const int ntiles = J.ntiles, words = J.words;
  const int w0 = blockIdx.x * wpb, w1 = min(words, w0 + wpb);
  if (blockIdx.x > 0 && w0 >= words) return;  // past this job's words
  const int32_t* __restrict__ cxy = J.cxy;
  const int32_t* __restrict__ disp = J.disp;
  uint8_t* __restrict__ flags = J.flags;
  constexpr int NW = kFitThreads / 64;
  __shared__ __align__(16) double Gs[SLOTS * 8];
  __shared__ unsigned long long M[kFitOne];
  __shared__ uint32_t csum[NW][SLOTS];
  __shared__ long long part[NW][kSums];
  __shared__ double tot[kSums];
  __shared__ int msel;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ox = J.w / 2, oy = J.h / 2;
  // everything that does not depend on the keys is in flight with them: this
  // thread's first tile, the best hypotheses, the unions' first words
  const int tc0 = min(w0 * 64 + tid, max(ntiles - 1, 0));
  uint8_t f0 = 0;
  int4 m0 = make_int4(0, 0, 0, 0);
  if (ntiles > 0) {
    f0 = flags[tc0];
    m0 = tile_match(cxy, disp, tc0, ox, oy);
  }
  const int N = *J.b.nmatch;
  constexpr int NK = SLOTS / 64;             // hypothesis blocks per lane
  constexpr int NC = SLOTS * 8 / kFitThreads;  // coefficients per thread
  unsigned long long key[NK];
#pragma unroll
  for (int u = 0; u < NK; ++u) {
    const int b = lane + 64 * u;
    key[u] = J.b.key[min(b, nhyp - 1)];
    if (b >= nhyp) key[u] = 0ull;
  }
  double gr[NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) gr[u] = J.b.G[min(tid + u * kFitThreads, nhyp * 8 - 1)];
  // word wd's unions, a block per lane
  unsigned long long pr[NK];
  auto fetch = [&](int wd) {
    const unsigned long long* p = J.b.part + (size_t)wd * nhyp;
#pragma unroll
    for (int u = 0; u < NK; ++u) pr[u] = p[min(lane + 64 * u, nhyp - 1)];
  };
  if (w0 + wave < w1) fetch(w0 + wave);
  double hp = 0.0, hb[3] = {0.0, 0.0, 0.0};
  if (wave == 0) {
    const int e = min(lane, 8);
    hp = J.Hprev[e];
#pragma unroll
    for (int i = 0; i < 3; ++i) hb[i] = J.Hbase[e / 3 * 3 + i];
  }
  if (chunks > 1) {
    // a wave adds up every NW-th chunk's counts, all of them in flight
    const int wpc = split_words(words, chunks), used = (words + wpc - 1) / wpc;
    constexpr int PW = kSplitChunks / NW;
#pragma unroll
    for (int u = 0; u < NK; ++u) {
      if (64 * u >= nhyp) break;
      unsigned long long k[PW];
#pragma unroll
      for (int i = 0; i < PW; ++i)
        k[i] = J.b.key[(size_t)min(wave + i * NW, used - 1) * nhyp + min(lane + 64 * u, nhyp - 1)];
      uint32_t c = 0;
#pragma unroll
      for (int i = 0; i < PW; ++i) c += wave + i * NW < used ? (uint32_t)(k[i] >> 32) : 0u;
      csum[wave][64 * u + lane] = c;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NK; ++u) {
      if (64 * u >= nhyp) break;
      uint32_t c = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) c += csum[w][64 * u + lane];
      if (lane + 64 * u < nhyp)
        key[u] = (unsigned long long)c << 32 | (key[u] & 0xffffffffull);
    }
  }
  const int delta = weed_delta(N, a);
  unsigned long long bkey = key[0];
#pragma unroll
  for (int u = 1; u < NK; ++u) bkey = key[u] > bkey ? key[u] : bkey;
  bkey = wave_max_u64(bkey);
  const int bc = bkey ? (int)(bkey >> 32) : -1;
  const int bi = bkey ? (int)(~(uint32_t)(bkey & 0xffffffffull)) : -1;
  const int bb = bkey ? bi / per % nhyp : 0;  // the block that solved iteration bi
  const bool fit = bc > delta;
  if (blockIdx.x == 0 && tid == 0) {
    J.counts[0] = N;
    J.counts[2] = bc;
    J.counts[3] = bi;
  }
  // M, a wave per word: the union over the blocks with an accepted hypothesis
  for (int wd = w0 + wave; wd < w1; wd += NW) {
    unsigned long long v = 0ull;
#pragma unroll
    for (int u = 0; u < NK; ++u)
      if ((int)(key[u] >> 32) > delta) v |= pr[u];
    if (wd + NW < w1) fetch(wd + NW);
    v = wave_or_u64(v);
    if (lane == 0) M[wd - w0] = v;
  }
#pragma unroll
  for (int u = 0; u < NC; ++u) Gs[tid + u * kFitThreads] = gr[u];
  __syncthreads();
  double g[8];  // the best hypothesis
#pragma unroll
  for (int i = 0; i < 8; ++i) g[i] = Gs[bb * 8 + i];
  const bool plain = needs_plain(g);
  long long s[kSums];
#pragma unroll
  for (int i = 0; i < kSums; ++i) s[i] = 0;
  for (int t0 = w0 * 64; t0 < w1 * 64; t0 += kFitThreads) {
    const int t = t0 + tid, word = t >> 6;
    if (word >= w1) break;  // whole waves
    const bool first = t0 == w0 * 64;
    const int tc = max(min(t, ntiles - 1), 0);
    uint8_t tf = f0;
    int4 m = m0;
    if (!first) {
      tf = flags[tc];
      m = tile_match(cxy, disp, tc, ox, oy);
    }
    if (t >= ntiles || !(tf & 2)) continue;
    const bool inM = (M[word - w0] >> lane) & 1ull;
    const bool sel = fit && (plain ? is_inlier<true>(g, m, a.eps2)
                                   : is_inlier<false>(g, m, a.eps2));
    flags[t] = (uint8_t)((tf & 0x13) | (inM ? 4 : 0) | (sel ? 8 : 0));
    if (sel) {
      // normal equations of G: (x, y) -> (u, v), reference side to source side
      const int x = m.z, y = m.w, u = m.x, v = m.y;
      s[0] += 1; s[1] += x; s[2] += y; s[6] += u; s[7] += v;
      if (max(max(abs(x), abs(y)), max(abs(u), abs(v))) <= 32767) {
        // products of two coordinates (and q) stay below 2^31: 32 x 32 -> 64
        // bit multiply-adds
        add_terms<int>(s, x, y, u, v);
      } else {  // a caller's matches far outside any image
        add_terms<long long>(s, x, y, u, v);
      }
    }
  }
  if (__ballot(s[0] != 0)) {
    wave_sums(s, part[wave]);
  } else if (lane < kSums) {
    part[wave][lane] = 0;
  }
  __syncthreads();
  if (wave == 0) {
    if (lane < kSums) {
      long long z = 0;
#pragma unroll
      for (int q = 0; q < NW; ++q) z += part[q][lane];
      tot[lane] = (double)z;
      if (lane == 0) msel = (int)z;
      if (gridDim.x > 1) J.b.psum[(size_t)blockIdx.x * kSums + lane] = z;
    }
    if (gridDim.x > 1) return;
    wave_lds_order();
    solve_level(J, tot, msel, hp, hb);
  } else if (gridDim.x == 1 && J.clear_vb) {  // the next level's search sets bits
    for (int i = tid - 64; i < J.clear_words; i += kFitThreads - 64) J.clear_vb[i] = 0ull;
  }
}

// The fit of a level whose sums several k_fit blocks left.
template <bool JOBS>
__global__ __launch_bounds__(64) void k_solve(WeedJob one, const WeedJob* __restrict__ jobs,
                                              int wpb) {
  const WeedJob J = JOBS ? jobs[blockIdx.z] : one;
  __shared__ double tot[kSums];
  __shared__ int msel;
  const int lane = threadIdx.x, e = min(lane, 8);
  const double hp = J.Hprev[e];
  const double hb[3] = {J.Hbase[e / 3 * 3], J.Hbase[e / 3 * 3 + 1], J.Hbase[e / 3 * 3 + 2]};
  if (lane < kSums) {
    long long z = 0;
#pragma unroll 8
    for (int b = 0; b < (J.words + wpb - 1) / wpb; ++b) z += J.b.psum[(size_t)b * kSums + lane];
    tot[lane] = (double)z;
    if (lane == 0) msel = (int)z;
  }
  if (J.clear_vb)
    for (int i = lane; i < J.clear_words; i += 64) J.clear_vb[i] = 0ull;
  wave_lds_order();
  solve_level(J, tot, msel, hp, hb);
}

WeedArgs weed_args(const lnr_params& p, int level) {
  WeedArgs a;
  a.iters = p.weed_iters;
  a.level = level;
  a.delta_min = p.weed_delta_min;
  a.delta_pct = p.weed_delta_pct;
  a.eps2 = p.weed_eps * p.weed_eps;
  a.seed = p.seed;
  return a;
}

}  // namespace

namespace {
// k_hyp, k_fit and, for a level of more than one k_fit block, k_solve over
// njobs jobs of at most ntiles tiles.
template <bool JOBS, int IPB, int NT, HypMode MODE>
hipError_t launch_hyp(const WeedJob& one, const WeedJob* jobs, int njobs, int words,
                      const WeedArgs& a, const HypForm& f, hipStream_t st) {
  const size_t lds = hyp_lds(words, MODE == kSplitHyp ? 0 : IPB, MODE == kManyHyp ? f.per : 0);
  if (lds > 64 * 1024) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hyp<JOBS, IPB, NT, MODE>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  LNR_LAUNCH((k_hyp<JOBS, IPB, NT, MODE>), dim3(f.blocks, f.chunks, njobs), dim3(NT), lds, st, one,
             jobs, a, f.per);
  return hipGetLastError();
}

template <bool JOBS>
hipError_t launch_weed(const WeedJob& one, const WeedJob* jobs, int njobs, int ntiles,
                       const WeedArgs& a, hipStream_t st) {
  const int words = ntiles > 0 ? (ntiles + 63) / 64 : 1;
  if (words > kMaxWords || a.iters > kMaxIters) return hipErrorInvalidValue;
  const HypForm f = hyp_form(a.iters, ntiles, words, njobs);
  const bool many = f.per > (f.wide ? 4 : 8);
  hipError_t e =
      f.chunks > 1 ? launch_hyp<JOBS, 4, 512, kSplitHyp>(one, jobs, njobs, words, a, f, st)
      : f.wide     ? many ? launch_hyp<JOBS, 4, 512, kManyHyp>(one, jobs, njobs, words, a, f, st)
                          : launch_hyp<JOBS, 4, 512, kUsualHyp>(one, jobs, njobs, words, a, f, st)
      : many       ? launch_hyp<JOBS, 8, 256, kManyHyp>(one, jobs, njobs, words, a, f, st)
                   : launch_hyp<JOBS, 8, 256, kUsualHyp>(one, jobs, njobs, words, a, f, st);
  if (e != hipSuccess) return e;
  const int wpb = words <= kFitOne ? kFitOne : kFitWords;
  const int blocks = (words + wpb - 1) / wpb;
  const int per = f.chunks > 1 ? 1 : f.per, slots = f.chunks > 1 ? a.iters : f.blocks;
  if (slots <= kWeedBlocks)
    LNR_LAUNCH((k_fit<JOBS, kWeedBlocks>), dim3(blocks, 1, njobs), dim3(kFitThreads), 0, st, one,
               jobs, a, per, slots, f.chunks, wpb);
  else
    LNR_LAUNCH((k_fit<JOBS, kSplitIters>), dim3(blocks, 1, njobs), dim3(kFitThreads), 0, st, one,
               jobs, a, per, slots, f.chunks, wpb);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (blocks > 1) {
    LNR_LAUNCH(k_solve<JOBS>, dim3(1, 1, njobs), dim3(64), 0, st, one, jobs, wpb);
    e = hipGetLastError();
  }
  return e;
}
}  // namespace

hipError_t launch_weed_fit(const int32_t* corner_xy, const int32_t* disp, uint8_t* flags,
                           int ntiles, int w, int h, int level, const lnr_params& p,
                           const double* H_prev, double* H_out, int32_t* counts,
                           const WeedBufs& b, hipStream_t st, bool vb_ready,
                           const double* H_base, int clear_words) {
  WeedJob J;
  J.cxy = corner_xy; J.disp = disp; J.flags = flags;
  J.ntiles = ntiles; J.w = w; J.h = h; J.words = ntiles > 0 ? (ntiles + 63) / 64 : 1;
  J.b = b;
  J.Hprev = H_prev; J.Hbase = H_base ? H_base : H_prev; J.Hout = H_out; J.counts = counts;
  J.clear_vb = clear_words > 0 ? b.vb : nullptr;
  J.clear_words = clear_words;
  if (J.words > kMaxWords) return hipErrorInvalidValue;
  if (!vb_ready) {  // else the level's search set the bits
    LNR_LAUNCH(k_valid, dim3((J.words + kValidThreads / 64 - 1) / (kValidThreads / 64)),
               dim3(kValidThreads), 0, st, flags, ntiles, J.words, b.vb);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return launch_weed<false>(J, nullptr, 1, ntiles, weed_args(p, level), st);
}

hipError_t launch_weed_jobs(const WeedJob* jobs, int njobs, int max_tiles, int level,
                            const lnr_params& p, hipStream_t st) {
  if (njobs < 1) return hipSuccess;
  return launch_weed<true>(WeedJob{}, jobs, njobs, max_tiles, weed_args(p, level), st);
}

}  // namespace lnr

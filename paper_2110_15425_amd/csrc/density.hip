// density.hip -- exact first-passage distribution of the discretised DDM.
//
// Instead of simulating thousands of runs, propagate the probability density
// of the walk's state: the Distill paper notes that a drift-diffusion model
// has an analytical solution and that recognising one saves thousands of
// model executions (Sec. 1, Sec. 4.4).  For the Euler-Maruyama walk
// x_n = x_{n-1} + a + b z_n with absorbing bounds +-theta, the survivor mass
// on M cells of (-theta, theta) evolves by a Gaussian transition kernel: the
// mass moving from cell i to cell j depends only on j - i (a Toeplitz
// matrix T), and the mass absorbed at either bound from cell i is a Gaussian
// tail.  The first step leaves the exact start point; later steps leave cell
// centres (midpoint rule, error O(h^2)).
//
// Where the step's width allows it the mass is propagated by its samples on a
// coarser grid, 16 steps at a time (the coarse form below); else one workgroup
// per setting keeps the kernel row and the mass vectors in LDS for all steps.  The product T m is a dense contraction on the FP64 matrix
// cores: with cells grouped in blocks of 16, block-diagonal d of T is one
// 16x16 matrix F_d (F_d[alpha][gamma] = f(16 d + alpha - gamma)), so
//   y_block(a) = sum_d F_d m_block(a - d),
// i.e. for every d a 16x16 by 16 x (blocks) product.  Each 16x16x4 product
// takes its F_d fragment straight from the kernel row in LDS and its mass
// fragment from the (zero-padded) mass vector.  Block-diagonals whose
// entries are all below 2^-60 (the Gaussian's far tails, at most 2^-60 of a
// row's mass each) are skipped, as are blocks whose mass columns lie outside
// the grid.  Wavefront (tile t, group g) accumulates the output columns
// 16 t .. 16 t + 15 over its share (the g-th of G contiguous ranges) of the
// block-diagonals; the groups' partial sums are added in group order
// through LDS.
#include "internal.hpp"

namespace cm {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxThreads = 1024;
constexpr int kBS = 17;  // LDS slots per 16-cell block of a mass vector (one pad)
constexpr int kWin = 16; // steps whose sums are reduced together

__device__ __forceinline__ double Phi(double x) { return 0.5 * erfc(-x * 0.70710678118654752440); }

// A double from another lane: DPP patterns within 16-lane rows (swap pairs,
// swap pairs of pairs, mirror within 8, mirror within 16), lane shuffles
// across rows.  Round r joins the halves of aligned groups of 2^(r+1) lanes.
template <int R>
__device__ __forceinline__ double partner(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  constexpr int ctrl = R == 0 ? 0xB1 : R == 1 ? 0x4E : R == 2 ? 0x141 : 0x140;
  if constexpr (R < 4) {
    lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, ctrl, 0xF, 0xF, false);
    hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, ctrl, 0xF, 0xF, false);
  } else {
    lo = (uint32_t)__shfl_xor((int)lo, 1 << R, 64);
    hi = (uint32_t)__shfl_xor((int)hi, 1 << R, 64);
  }
  return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}

// Sum over the wavefront, the same value in every lane (all lanes active).
__device__ __forceinline__ double wave_sum(double v) {
  v += partner<0>(v);
  v += partner<1>(v);
  v += partner<2>(v);
  v += partner<3>(v);
  v += partner<4>(v);
  v += partner<5>(v);
  return v;
}

// Sum over the 16-lane row, the same value in every lane of the row.
__device__ __forceinline__ double row_sum(double v) {
  v += partner<0>(v);
  v += partner<1>(v);
  v += partner<2>(v);
  v += partner<3>(v);
  return v;
}

__device__ __forceinline__ int floor_div16(int v) { return v >= 0 ? v / 16 : -((15 - v) / 16); }
__device__ __forceinline__ int ceil_div16(int v) { return -floor_div16(-v); }

}  // namespace

// Launch geometry of M cells: NB blocks of 16 cells, NT output tiles of 16
// blocks, G wavefronts per tile (W = NT G, 6 to 12; measured on MI355X at
// 1000 cells, four tiles: with every fragment read from LDS, 2 per tile 5 %
// faster than 4 and 1 per tile 25 % slower; with the kernel fragments of
// the first diagonals in registers, 3 per tile (12 diagonals each) 2 %
// faster than 2 (24 each) and 4 (6 each)), the
// kernel row's offset
// FOFF (entry of displacement 0) and width FW, and CB blocks per mass vector
// (NB zero blocks on either side of the 16 NT output blocks).
struct DensityGeo {
  uint32_t M, NB, NT, G, W, FOFF, FW, CB;
};
__host__ __device__ inline DensityGeo density_geo(uint32_t M) {
  DensityGeo g;
  g.M = M;
  g.NB = (M + 15u) / 16u;
  g.NT = (g.NB + 15u) / 16u;
  g.G = g.NT == 4u ? 3u : 8u / g.NT > 2u ? 8u / g.NT : 2u;
  g.W = g.NT * g.G;
  g.FOFF = 16u * g.NB + 16u;
  g.FW = 2u * g.FOFF + 1u;
  g.CB = 16u * g.NT + 2u * g.NB;
  return g;
}

namespace {

// ---------------------------------------------------------------------------
// Coarse propagation.
//
// After one step the survivor mass is a superposition of Gaussians of the
// step's width b, so its spectrum above 8.9 / b is below 2^-57 of the whole:
// as a function of the position it is determined by its samples s cells
// apart, with s h <= pi b / 8.9 (h the cell width).  With those r samples v as
// the state -- over the grid and 8.3 b beyond it, where the function has died
// away -- a step is one r x r matrix,
//   v' = B v,  B[p][q] = sum over cells i of f(X_p - i) sinc((i - X_q) / s),
// f the kernel row, X_p = s (p - mg) the sample positions in cells: the mass of
// cell i is interpolated from the samples and moved to sample p, the same sum
// over cells as the full product (r is about 110 for 1000 cells where b is a
// 20th of the range).  Up to 128 cells the samples are the cells themselves.
// The sum over all integers i would be s f(X_p - X_q) by the sampling theorem,
// so B is that minus the sums over the cells that are not there, i < 0 and
// i >= M, and only rows within 8.7 b of a bound take any product.
//
// B, its squares and the powers up to B^16 are products on the FP64 matrix
// cores from LDS; the outputs of 16 steps are W v with W's 48 rows w B^k (w
// the absorption at either bound and the total, k = 0..15), built beside the
// squarings by doubling.  One pass over (B^16, W), held in registers, then
// advances 16 steps: 3000 steps are 188 passes.  The first steps, while the
// mass at a bound is so small that the samples' absolute rounding would show
// in it, are taken on the full grid.
//
// Precision: f comes from a Hermite expansion of the Gaussian's cell integral
// (no cancellation), and the rounding of f and of B's Toeplitz part is corrected
// so that they conserve mass, or a systematic relative error of 10^-16 per step
// would grow with the steps.  Against an 80-bit propagation (14 cases of 120 to
// 1300 cells; norm of the error over the norm of the result) 7.8e-16 on average
// and 3.2e-15 at most, the full-grid form 8.1e-16 and 3.5e-15.  An entry is off by less
// than 2^-52 of the mass that is left before its step, besides 10^-13 of itself.
//
// Bound by the FP64 matrix cores of one compute unit per setting and, in the
// passes, by latency.  64 drifts x 3000 steps x 1000 cells: 0.48 ms against
// 20.4 on the full grid, of which the squarings 0.19, the passes 0.13 (0.7 us
// each), B 0.08, the seven full-grid steps 0.05.
// ---------------------------------------------------------------------------
constexpr int kCoarse = 128;        // most samples (rows of B)
constexpr int kCoarseThreads = 512;
constexpr int kCoarsePow = 16;      // steps per pass
constexpr int kCoarseSlots = 3;     // cells of a thread in the full-grid steps

// Static LDS beside the dynamic one.
struct CoarseShared {
  double red[3][kCoarseThreads / 64];
  double resid;
  double first[2][32];  // outputs of the full-grid steps
};

struct CoarsePlan {
  bool ok;
  int s, mg, r;  // sample spacing (cells), samples beyond either end, samples
  int E;         // displacement (cells) beyond which f is nothing
  int direct;    // steps taken on the full grid
};

// LDS layout (doubles): the preparation's arrays, later overlaid by the powers.
struct CoarseGeo {
  int FO, SM;  // f table: displacements -FO .. FO; sinc table: 0 .. SM
  int o_st, o_m0, o_m1, o_part, prep;
};
__host__ __device__ inline CoarseGeo coarse_geo(const DensityGeo& g, const CoarsePlan& p) {
  CoarseGeo c;
  const int need = p.E + 16 * p.s + 16;
  c.FO = (int)g.FOFF > need ? (int)g.FOFF : need;
  c.SM = (int)g.M + 2 * p.E + 2 * p.s + 16;
  c.o_st = 2 * c.FO + 1;
  c.o_m0 = c.o_st + c.SM + 1;
  c.o_m1 = c.o_m0 + (int)g.CB * kBS;
  c.o_part = c.o_m1 + (int)g.CB * kBS;
  c.prep = c.o_part + 8 * 256;
  return c;
}
constexpr int kWRows = 3 * kCoarsePow;                      // output rows
constexpr int kVSeg = 34;                                    // LDS slots per 32 samples (two pads)
constexpr int kOffW = kCoarse * kCoarse;                     // W's first 24 rows, behind B
constexpr int kOffV = kOffW + (kWRows / 2) * kCoarse;        // [2][4 * kVSeg] samples
constexpr int kCoarseLds = kOffV + 2 * 4 * kVSeg;            // doubles
constexpr int kRing = 256;                                   // passes whose outputs LDS holds
static_assert(kRing * kWRows <= kOffW, "the outputs fit over B");

// Whether a setting propagates its samples instead of its cells: the samples
// must be few enough and the kernel wide enough in cells, and neither bound so
// unlikely (drift over noise) that its probabilities fall to the samples'
// absolute rounding.  A NaN fails every test.
//
// Nor may the propagation end so soon that the preparation costs more than the
// full-grid steps it replaces: the survivor mass falls like (4 / pi) e^-(lambda n), lambda =
// pi^2 b^2 / 8 (th + 0.583 b)^2 + as^2 / 2 b^2 (the bounds as a walk in steps meets them),
// and is below tol after tol_log / lambda steps, tol_log = log(4 / (pi tol)); the full grid
// then goes on for half a window and has its own start.  Fitted to measured times, us: a
// full-grid step 1.6 at 48 to 128 cells, 2.2 at 333, 6.8 at 1,000, 12 at 1,300; the
// preparation 51 at 48 samples, 120 at 80, 254 at 128, of 333 cells 209 at 84 and 284 at 123,
// of 1,000 302, of 1,300 386.  With tol 0.5, us, full grid and coarse: 128 cells at noise 2.4
// 41 and 262, 333 at 2.0 107 and 219, 333 at 1.0 230 and 306, 1,000 at 1.0 672 and 353.
__host__ __device__ inline CoarsePlan coarse_plan(uint32_t cells, double th, double b, double as, double start,
                                                  double tol_log) {
  CoarsePlan p{};
  const double h = (2.0 * th) / (double)cells, bc = b / h, ac = fabs(as) / h;
  if (!(bc >= 4.0) || !(2.0 * th >= 8.0 * b) || !(2.0 * fabs(as) * th <= 4.0 * b * b) || !(bc < 400.0)) return p;
  if (cells <= (uint32_t)kCoarse) {
    p.s = 1;
    p.mg = 0;
  } else {
    p.s = (int)(3.14159265358979 * bc / 8.9);
    if (p.s > 7) p.s -= 1 - (p.s & 1);  // odd: the strided reads of the tables spread over the LDS banks
    if (p.s < 1) return p;
    p.mg = (int)ceil((8.3 * bc + ac) / p.s);
  }
  p.r = ((int)cells - 1 + p.s - 1) / p.s + 1 + 2 * p.mg;
  p.E = (int)ceil(8.7 * bc + ac) + 1;
  const double far = (th + fabs(start)) / (3.8 * b), d = ceil(far * far);
  p.direct = d < 1.0 ? 1 : d > 31.0 ? 31 : (int)d;
  const double wide = th + 0.583 * b, lambda = 1.2337 * (b * b) / (wide * wide) + 0.5 * (as * as) / (b * b);
  const double M = (double)cells, step_us = 1.6 + (M / 440.0) * (M / 440.0);
  const double prep_us = 20.0 + 0.015 * (p.r * p.r) + (p.mg ? 40.0 + 0.13 * M : 0.0);
  const DensityGeo g = density_geo(cells);
  p.ok = tol_log >= (p.direct - 14.0 + prep_us / step_us) * lambda && p.r <= kCoarse && d <= 31.0 && 256u * g.NT <= (uint32_t)(kCoarseSlots * kCoarseThreads) &&
         coarse_geo(g, p).prep <= kCoarseLds;
  return p;
}

// Slot of element (i, j) of a 128-column matrix: rows rotated against each
// other by an exclusive or, so that a column of 16 rows spreads over the banks.
__device__ __forceinline__ int mat_at(int i, int j) { return i * kCoarse + (j ^ ((i & 15) << 1)); }
__device__ __forceinline__ int seg_at(int q) { return (q >> 5) * kVSeg + (q & 31); }

// Gaussian mass of the unit cell at displacement d cells: the integral of the
// normal density over [z - e/2, z + e/2], z = (d h - as) / b, e = h / b, as its
// expansion in e (even Hermite polynomials; e <= 1/4, next term below 2^-55 of
// the centre's value).
__device__ double cell_mass(double d, double h, double as, double b) {
  const double z = (d * h - as) / b, e = h / b, x = z * z, t = 0.25 * e * e;
  const double h2 = x - 1.0, h4 = (x - 6.0) * x + 3.0, h6 = ((x - 15.0) * x + 45.0) * x - 15.0;
  const double h8 = (((x - 28.0) * x + 210.0) * x - 420.0) * x + 105.0;
  const double h10 = ((((x - 45.0) * x + 630.0) * x - 3150.0) * x + 4725.0) * x - 945.0;
  double v = h10 * (t * (1.0 / 39916800.0));
  v = t * (h8 * (1.0 / 362880.0) + v);
  v = t * (h6 * (1.0 / 5040.0) + v);
  v = t * (h4 * (1.0 / 120.0) + v);
  v = t * (h2 * (1.0 / 6.0) + v);
  return exp(-0.5 * x) * (0.39894228040143267794 * e) * (1.0 + v);
}

__global__ __launch_bounds__(kCoarseThreads) void ddm_density_coarse_kernel(DensityArgs a) {
  extern __shared__ double sh[];
  __shared__ CoarseShared shared;
  auto& red = shared.red;
  auto& first = shared.first;
  double& resid_s = shared.resid;
  const DensityGeo geo = density_geo(a.cells);
  const int tid = (int)threadIdx.x, lane = tid & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = (int)__builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
  const uint64_t st = blockIdx.x;
  const double drift = a.n_signals ? a.grid[st * a.n_signals] : a.drift;
  const double as = drift * a.dt, b = a.b, th = a.thresh, h = (2.0 * th) / (double)a.cells;
  CoarsePlan pl = coarse_plan(a.cells, th, b, as, a.start, a.tol_log);
  if (!pl.ok) {  // the full-grid kernel's setting: no probability is negative
    if (tid == 0) a.out[st * 2u * a.max_steps] = -1.0;
    return;
  }
  for (int* v : {&pl.s, &pl.mg, &pl.r, &pl.E, &pl.direct}) *v = __builtin_amdgcn_readfirstlane(*v);  // scalars
  const CoarseGeo cg = coarse_geo(geo, pl);
  const int M = (int)a.cells, NB = (int)geo.NB, NT = (int)geo.NT, s = pl.s, r = pl.r, N = (int)a.max_steps;
  double* out_lo = a.out + (st * 2u) * a.max_steps;
  double* out_up = out_lo + a.max_steps;
  double* ft = sh;
  double* sc = sh + cg.o_st;
  double* cur = sh + cg.o_m0;
  double* nxt = sh + cg.o_m1;
  double* part = sh + cg.o_part;

  for (int x = tid; x < 2 * (int)geo.CB * kBS; x += kCoarseThreads) cur[x] = 0.0;
  for (int x = tid; x <= 2 * cg.FO; x += kCoarseThreads) {
    const int d = x - cg.FO;
    ft[x] = d >= -pl.E && d <= pl.E ? cell_mass((double)d, h, as, b) : 0.0;
  }
  for (int x = tid; x <= cg.SM; x += kCoarseThreads)
    sc[x] = x == 0 ? 1.0 : sinpi((double)(x % (2 * s)) / (double)s) * (double)s / (3.14159265358979323846 * (double)x);
  __syncthreads();

  // The mass that rounding leaves out of the kernel's row, 1 - sum of step f(step k),
  // summed exactly by the first wavefront.
  auto missing = [&](int step) {
    double hi = 0.0, lo = 0.0;
    const int kmax = pl.E / step;
    for (int k = -kmax + lane; k <= kmax; k += 64) {
      const double v = (double)step * ft[cg.FO + step * k], t = hi + v, bb = t - hi;
      lo += (hi - (t - bb)) + (v - bb);
      hi = t;
    }
    for (int o = 32; o > 0; o >>= 1) {
      const double ohi = __shfl_xor(hi, o, 64), olo = __shfl_xor(lo, o, 64);
      const double t = hi + ohi, bb = t - hi;
      lo = (lo + olo) + ((hi - (t - bb)) + (ohi - bb));
      hi = t;
    }
    if (lane == 0) resid_s = (1.0 - hi) - lo;
  };
  if (wave == 0) {
    missing(1);
    // to the entries one b either side, where it acts as it does spread over all
    // of them in proportion
    if (lane == 0) {
      const int d1 = (int)(b / h + 0.5);
      ft[cg.FO + d1] += 0.5 * resid_s;
      ft[cg.FO - d1] += 0.5 * resid_s;
    }
  }
  __syncthreads();

  // This thread's cells of the full-grid steps, as in the full-grid kernel.
  constexpr int kSlots = kCoarseSlots;
  double upc[kSlots], loc[kSlots];
  int pos[kSlots], cell[kSlots];
  double sv = 0.0, pu = 0.0, pw = 0.0;
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const int t = tid + k * kCoarseThreads;
    const int tt = t >> 8, rr = (t >> 6) & 3, l = t & 63;
    const int blk = 16 * tt + (l & 15), j = 16 * blk + 4 * rr + (l >> 4);
    cell[k] = t < 256 * NT && j < M ? j : -1;
    pos[k] = t < 256 * NT ? (blk + NB) * kBS + 4 * rr + (l >> 4) : -1;
    upc[k] = loc[k] = 0.0;
    if (cell[k] >= 0) {
      const double c = -th + ((double)j + 0.5) * h;
      upc[k] = Phi(-((th - c) - as) / b);
      loc[k] = Phi(((-th - c) - as) / b);
      const double e0 = -th + (double)j * h, e1 = -th + (double)(j + 1) * h;
      const double v = Phi(((e1 - a.start) - as) / b) - Phi(((e0 - a.start) - as) / b);
      cur[pos[k]] = v;
      pu = fma(v, upc[k], pu);
      pw = fma(v, loc[k], pw);
    }
  }
  // Full-grid steps: the mass after step n in cur, absorbed next in (pu, pw).
  const int dlo = -((pl.E + 15) / 16) - 1, dhi = (pl.E + 15) / 16 + 1;
  const int G = 8 / NT > 1 ? 8 / NT : 1, tile = wave / G, grp = wave - tile * G, c0 = 16 * tile;
  const int dA = max(dlo, c0 - NB + 1), dB = min(dhi, min(c0 + 15, NB - 1));
  const int nd = dB >= dA ? dB - dA + 1 : 0;
  const int dS = dA + (nd * grp) / G, dE = dA + (nd * (grp + 1)) / G;
  if (tid == 0) {
    out_up[0] = Phi(-((th - a.start) - as) / b);
    out_lo[0] = Phi(((-th - a.start) - as) / b);
  }
  int n = 1;
  for (;; ++n) {
    // sums of the mass after step n
    pu = wave_sum(pu);
    pw = wave_sum(pw);
    sv = wave_sum(sv);
    if (lane == 0) {
      red[0][wave] = sv;
      red[1][wave] = pu;
      red[2][wave] = pw;
    }
    __syncthreads();  // sums, and the new mass in cur
    double tv = 0.0, tu = 0.0, tl = 0.0;
    for (int w = 0; w < kCoarseThreads / 64; ++w) {
      tv += red[0][w];
      tu += red[1][w];
      tl += red[2][w];
    }
    if (n >= 2 && tv < a.tol) {  // as the full-grid kernel stops
      for (int k = 1 + tid; k < N; k += kCoarseThreads) {
        out_up[k] = k < n ? first[0][k] : 0.0;
        out_lo[k] = k < n ? first[1][k] : 0.0;
      }
      return;
    }
    if (tid == 0) {
      first[0][n] = tu;
      first[1][n] = tl;
    }
    if (n == pl.direct) break;
    f64x4 C = {0.0, 0.0, 0.0, 0.0};
    if (tile < NT) {
      const double* fa = ft + cg.FO + l16 - l4;
      const double* mb = cur + (c0 + l16 + NB) * kBS + l4;
      for (int d = dS; d < dE; ++d) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          C = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[16 * d - 4 * q], mb[4 * q - d * kBS], C, 0, 0, 0);
      }
      double* pp = part + ((grp * NT + tile) * 4) * 64 + lane;
#pragma unroll
      for (int k = 0; k < 4; ++k) pp[k * 64] = C[k];
    }
    __syncthreads();
    sv = 0.0;
    pu = 0.0;
    pw = 0.0;
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
      if (pos[k] >= 0) {
        const int t = tid + k * kCoarseThreads;
        double v = part[t];
        for (int g = 1; g < G; ++g) v += part[t + g * NT * 256];
        if (cell[k] < 0) v = 0.0;
        nxt[pos[k]] = v;
        sv += v;
        pu = fma(v, upc[k], pu);
        pw = fma(v, loc[k], pw);
      }
    }
    double* t = cur;
    cur = nxt;
    nxt = t;
  }
  __syncthreads();  // every thread has read the sums; nxt is free
  if (tid >= 1 && tid <= n) {  // (the launch rule leaves more steps than these)
    out_up[tid] = first[0][tid];
    out_lo[tid] = first[1][tid];
  }
  double* ua = nxt;  // absorption at either bound by cell, [2][M]
#pragma unroll
  for (int k = 0; k < kSlots; ++k)
    if (cell[k] >= 0) {
      ua[cell[k]] = upc[k];
      ua[M + cell[k]] = loc[k];
    }
  if (wave == 0) missing(s);  // of B's Toeplitz part
  __syncthreads();
  // It goes to the entries one b either side again; what their rounding leaves
  // goes to those three b away, whose own rounding is small.
  const int k1 = (int)(b / (h * s) + 0.5), k3 = (int)(3.0 * b / (h * s));
  const double gu = (double)s * ft[cg.FO + s * k1], gd = (double)s * ft[cg.FO - s * k1];
  const double gur = gu + 0.5 * resid_s, gdr = gd + 0.5 * resid_s;
  const double rest = 0.5 * (resid_s - ((gur - gu) + (gdr - gd)));

  // The samples after the next step, and w in the samples: sums over cells in
  // four parts, one sample or column per thread, by blocks of 16 cells (their
  // rounding is in every output alike).
  const int q = tid & (kCoarse - 1), qc = q < r ? q : r - 1, quarter = tid >> 7;
  const int Xq = s * (qc - pl.mg);
  double v0 = 0.0, w0 = 0.0, w1 = 0.0, w2 = 0.0;
  for (int blk = quarter; blk < NB; blk += 4) {
    const double* mb = cur + (blk + NB) * kBS;
    const int i1 = min(16, M - 16 * blk);
    double bv = 0.0, b0 = 0.0, b1 = 0.0, b2 = 0.0;
    for (int k = 0; k < i1; ++k) {
      const int i = 16 * blk + k, d = Xq - i;
      const int dc = d < -cg.FO ? -cg.FO : d > cg.FO ? cg.FO : d;  // f is 0 at either end of its table
      bv = fma(ft[cg.FO + dc], mb[k], bv);
      const double S = sc[d < 0 ? -d : d];
      b0 = fma(ua[i], S, b0);
      b1 = fma(ua[M + i], S, b1);
      b2 += S;
    }
    v0 += bv;
    w0 += b0;
    w1 += b1;
    w2 += b2;
  }

  // B: this wavefront's 16 rows, in two chains per tile
  f64x4 acc[8], acd[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = acd[c] = f64x4{0.0, 0.0, 0.0, 0.0};
  if (pl.mg) {
    const int Xlo = s * (16 * wave - pl.mg), Xhi = Xlo + 15 * s;
    const double* fr = ft + cg.FO + Xlo + s * l16 - l4;  // fr[-i]: f(X - (i + l4))
    int Xc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int qq = 16 * c + l16;
      Xc[c] = s * ((qq < r ? qq : r - 1) - pl.mg) - l4;
    }
    auto edge = [&](int i0, int steps) {  // cells i0 .. i0 + 4 steps - 1
      for (int t = 0; t < steps; ++t) {
        const int i = i0 + 4 * t;
        const double A = fr[-i];
        if (t & 1) {
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const int dd = i - Xc[c];
            acd[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(A, sc[dd < 0 ? -dd : dd], acd[c], 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const int dd = i - Xc[c];
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(A, sc[dd < 0 ? -dd : dd], acc[c], 0, 0, 0);
          }
        }
      }
    };
    if (16 * wave < r) {
      const int left = min(pl.E, pl.E - Xlo);  // cells -left .. -1 reach these rows
      if (left > 0) edge(-4 * ((left + 3) / 4), (left + 3) / 4);
      const int right = min(pl.E, Xhi + pl.E + 1 - M);  // cells M .. M + right - 1
      if (right > 0) edge(M, (right + 3) / 4);
    }
  }
  // B and W's first rows into LDS, over the preparation's arrays
  double bv[8][4];
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int p = 16 * wave + 4 * k + l4, qq = 16 * c + l16, d = s * (p - qq);
      double v = 0.0;
      if (p < r && qq < r) {
        v = d >= -pl.E && d <= pl.E ? (double)s * ft[cg.FO + d] : 0.0;
        if (p - qq == k1) v = gur;
        if (qq - p == k1) v = gdr;
        if (p - qq == k3 || qq - p == k3) v += rest;
        v -= acc[c][k] + acd[c][k];
      }
      bv[c][k] = v;
    }
  __syncthreads();
  double* P = sh;
  double* W = sh + kOffW;
  double* V = sh + kOffV;
  // (the four parts' sums through P's region first)
  P[tid] = v0;
  P[512 + tid] = w0;
  P[1024 + tid] = w1;
  P[1536 + tid] = w2;
  __syncthreads();
  if (tid < 512) {
    const int kind = tid >> 7;  // v, up, lo, total
    const double* x = P + 512 * kind + q;
    const double v = q < r ? ((x[0] + x[128]) + (x[256] + x[384])) : 0.0;
    if (kind == 0) V[seg_at(q)] = v;
    else W[mat_at(kind - 1, q)] = v;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int k = 0; k < 4; ++k) P[mat_at(16 * wave + 4 * k + l4, 16 * c + l16)] = bv[c][k];
  __syncthreads();

  // Four squarings; W's rows double beside them.  A plain product would round
  // each entry of magnitude 0.1 some twenty times, a systematic error of every
  // later step: the factors are split at 2^-26, so that the products of the
  // upper parts add up exactly (multiples of 2^-52 below 2) and the rest, 2^27
  // times smaller, is added once.
  auto upper = [](double x) { return (x + 0x1.8p26) - 0x1.8p26; };
  const int ksteps = 4 * ((r + 15) / 16);
  f64x4 wa[2];
#pragma unroll 1
  for (int lv = 0; lv < 4; ++lv) {
    const int rows = 3 << lv;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = acd[c] = f64x4{0.0, 0.0, 0.0, 0.0};
    wa[0] = wa[1] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int rw0 = min(l16, rows - 1), rw1 = min(16 + l16, rows - 1);
    if (16 * wave < r) {
#pragma unroll 1
      for (int t = 0; t < ksteps; ++t) {
        const int kk = 4 * t + l4;
        const double A = P[mat_at(16 * wave + l16, kk)], Bw = P[mat_at(kk, 16 * wave + l16)];
        const double Ah = upper(A), Al = A - Ah;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (16 * c < r) {
            const double Bc = P[mat_at(kk, 16 * c + l16)], Bh = upper(Bc);
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ah, Bh, acc[c], 0, 0, 0);
            acd[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ah, Bc - Bh, acd[c], 0, 0, 0);
            acd[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(Al, Bc, acd[c], 0, 0, 0);
          }
        }
        wa[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(W[mat_at(rw0, kk)], Bw, wa[0], 0, 0, 0);
        if (rows > 16) wa[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(W[mat_at(rw1, kk)], Bw, wa[1], 0, 0, 0);
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) P[mat_at(16 * wave + 4 * k + l4, 16 * c + l16)] = acc[c][k] + acd[c][k];
    if (lv < 3) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int row = 4 * k + l4;
        if (row < rows) W[mat_at(rows + row, 16 * wave + l16)] = wa[0][k];
      }
    }
    __syncthreads();
  }
  // B^16 and W into registers: eight threads per row, thread (slot, seg) holding
  // columns 16 seg .. 16 seg + 15 of B^16's rows slot and slot + 64 and of W's
  // row slot (three rows for each read of the samples, which LDS reads bound
  // otherwise).
  double Pr[2][16], Wr[16];
  const int slot = tid >> 3, seg = tid & 7;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    Pr[0][k] = P[mat_at(slot, 16 * seg + k)];
    Pr[1][k] = P[mat_at(slot + 64, 16 * seg + k)];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // W's last 24 rows, over B's region
    const int row = 4 * k + l4;
    P[mat_at(row, 16 * wave + l16)] = wa[0][k];
    if (16 + row < kWRows / 2) P[mat_at(16 + row, 16 * wave + l16)] = wa[1][k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int row = slot < kWRows / 2 ? slot : slot - kWRows / 2;
    Wr[k] = slot < kWRows ? (slot < kWRows / 2 ? W : P)[mat_at(row, 16 * seg + k)] : 0.0;
  }
  __syncthreads();
  // Passes of 16 steps.  Their outputs collect in LDS over B's region and leave
  // it together: a store to HBM in a pass would be waited for at its barrier.
  double* O = sh;  // [kRing][48]
  const int vo = kVSeg * (seg >> 1) + 16 * (seg & 1);
  int par = 0, pass = 0, n0 = pl.direct + 1;  // n0: the ring's first step
  for (;;) {
    const double* v = V + par * 4 * kVSeg + vo;
    double y0 = 0.0, y1 = 0.0, o1 = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const double x = v[k];
      y0 = fma(Pr[0][k], x, y0);
      y1 = fma(Pr[1][k], x, y1);
      o1 = fma(Wr[k], x, o1);
    }
    auto sum8 = [](double x) {
      x += partner<0>(x);
      x += partner<1>(x);
      return x + partner<2>(x);
    };
    y0 = sum8(y0);
    y1 = sum8(y1);
    o1 = sum8(o1);
    if (seg == 0) {
      double* vn = V + (par ^ 1) * 4 * kVSeg;
      vn[seg_at(slot)] = y0;
      vn[seg_at(slot + 64)] = y1;
      if (slot < kWRows) O[pass * kWRows + slot] = o1;
    }
    __syncthreads();
    par ^= 1;
    // the first of the pass's steps whose mass is below tol
    const uint64_t below =
        __builtin_amdgcn_ballot_w64(O[pass * kWRows + 3 * (lane & 15) + 2] < a.tol) & 0xFFFFull;
    const int stop = below ? (int)__builtin_ctzll(below) : kCoarsePow;
    const int end = min(N, n0 + pass * kCoarsePow + stop);  // steps before this one have outputs
    const bool last = stop < kCoarsePow || end >= N;
    if (!last && ++pass < kRing) continue;
    for (int x = n0 + tid; x < end; x += kCoarseThreads) {
      const double* o = O + 3 * (x - n0);  // rows of a pass follow each other by step
      out_up[x] = fmax(o[0], 0.0);  // the samples' sums can fall below 0 once the mass is denormal
      out_lo[x] = fmax(o[1], 0.0);
    }
    if (last) {
      for (int x = end + tid; x < N; x += kCoarseThreads) {
        out_up[x] = 0.0;
        out_lo[x] = 0.0;
      }
      return;
    }
    __syncthreads();
    n0 += kRing * kCoarsePow;
    pass = 0;
  }
}

// MAXT: workgroup size bound; REGD: diagonals per wavefront whose kernel
// fragments stay in registers (at two wavefronts per SIMD a wavefront's 256
// registers hold 24 diagonals' fragments beside the rest, at three 12;
// measured on MI355X at 1000 cells: 6 % faster than reading them from LDS
// every step.
// One wavefront per tile with 48 diagonals in registers and the accumulator
// as the new mass -- no partial sums, one barrier per step -- was 8 % slower
// than reading everything from LDS, with one accumulation chain or two).
template <int MAXT, int REGD>
__global__ __launch_bounds__(MAXT) void ddm_density_kernel(DensityArgs a) {
  extern __shared__ double sh[];
  __shared__ double red[3][kMaxThreads / 64];
  __shared__ double wsum[3][kWin];
  __shared__ int band[2];
  const DensityGeo geo = density_geo(a.cells);
  const uint32_t M = geo.M, NB = geo.NB, NT = geo.NT, G = geo.G;
  const uint32_t tid = threadIdx.x, nt = blockDim.x;
  const int lane = (int)(tid & 63u), wave = (int)(tid >> 6), nw = (int)(nt >> 6);
  double* f = sh;                       // kernel row: f[FOFF + delta], [FW]
  double* m0 = f + geo.FW;              // mass vectors, block c at (c + NB) * kBS
  double* m1 = m0 + geo.CB * kBS;
  double* part = m1 + geo.CB * kBS;     // partial sums [G][NT][4][64]
  // per step of a window: the 16-lane rows' sums of the new mass, and of the
  // mass the next step absorbs at either bound, [kWin][3][rows]
  double* ring = part + G * NT * 256u;
  const uint64_t s = blockIdx.x;
  const double drift = a.n_signals ? a.grid[s * a.n_signals] : a.drift;
  const double as = drift * a.dt, b = a.b, th = a.thresh, h = (2.0 * th) / (double)M;
  double* out_lo = a.out + (s * 2u) * a.max_steps;  // choice 0: lower bound
  double* out_up = out_lo + a.max_steps;             // choice 1: upper bound
  // the coarse kernel's setting (a uniform test: with one per lane the steps below came out
  // 2 to 4 % slower)
  if (a.coarse && __builtin_amdgcn_ballot_w64(out_lo[0] != -1.0) != 0) return;

  if (tid == 0) {
    band[0] = 0x7FFFFFFF;
    band[1] = -0x7FFFFFFF;
  }
  for (uint32_t i = tid; i < 2u * geo.CB * kBS; i += nt) m0[i] = 0.0;
  __syncthreads();
  // kernel row: entry delta is the mass moving delta cells up; the band of
  // displacements whose entries reach 2^-60
  for (uint32_t x = tid; x < geo.FW; x += nt) {
    const int d = (int)x - (int)geo.FOFF;
    double v = 0.0;
    if (d > -(int)M && d < (int)M) {
      const double k = (double)d;
      v = Phi(((k + 0.5) * h - as) / b) - Phi(((k - 0.5) * h - as) / b);
    }
    f[x] = v;
    if (v >= 0x1p-60) {
      atomicMin(&band[0], d);
      atomicMax(&band[1], d);
    }
  }
  // This thread's output slots: slot t is register r of lane l of tile tt's
  // accumulator, cell 16 (16 tt + l % 16) + 4 r + l / 16 (the 16x16x4 FP64
  // accumulator holds row 4 r + l / 16, column l % 16).  Their absorption
  // tables stay in registers; the first step's mass comes from the start
  // point exactly.
  constexpr int kSlots = 2;
  double upc[kSlots], loc[kSlots];
  uint32_t pos[kSlots];
  bool real[kSlots];
  double pu = 0.0, pl = 0.0;
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const uint32_t t = tid + (uint32_t)k * nt;
    const uint32_t tt = t >> 8, r = (t >> 6) & 3u, l = t & 63u;
    const uint32_t blk = 16u * tt + (l & 15u), j = 16u * blk + 4u * r + (l >> 4);
    real[k] = t < 256u * NT && j < M;
    pos[k] = (blk + NB) * kBS + 4u * r + (l >> 4);
    upc[k] = loc[k] = 0.0;
    if (real[k]) {
      const double c = -th + ((double)j + 0.5) * h;
      upc[k] = Phi(-((th - c) - as) / b);
      loc[k] = Phi(((-th - c) - as) / b);
      const double e0 = -th + (double)j * h, e1 = -th + (double)(j + 1) * h;
      const double v = Phi(((e1 - a.start) - as) / b) - Phi(((e0 - a.start) - as) / b);
      m0[pos[k]] = v;
      pu = fma(v, upc[k], pu);
      pl = fma(v, loc[k], pl);
    }
  }
  pu = wave_sum(pu);
  pl = wave_sum(pl);
  if (lane == 0) {
    red[1][wave] = pu;
    red[2][wave] = pl;
  }
  __syncthreads();
  if (tid == 0) {
    out_up[0] = Phi(-((th - a.start) - as) / b);
    out_lo[0] = Phi(((-th - a.start) - as) / b);
    if (a.max_steps >= 2u) {
      double su = 0.0, sl = 0.0;
      for (int w = 0; w < nw; ++w) {
        su += red[1][w];
        sl += red[2][w];
      }
      out_up[1] = su;
      out_lo[1] = sl;
    }
  }
  // Block-diagonals holding an entry of the band (diagonal d covers
  // displacements 16 d - 15 .. 16 d + 15) whose mass blocks a - d, for the
  // columns a of this wavefront's tile, reach the grid: a contiguous range,
  // split into G contiguous shares, one per group.  All wave-uniform.
  // (the lowest d with 16 d + 15 >= band[0], the highest with 16 d - 15 <= band[1])
  const int dlo = ceil_div16(band[0] - 15), dhi = floor_div16(band[1] + 15);
  const uint32_t wv = __builtin_amdgcn_readfirstlane((uint32_t)wave);
  const uint32_t tile = wv / G, grp = wv - tile * G;
  const int nbi = (int)NB, c0 = 16 * (int)tile;
  const int dA = max(dlo, c0 - nbi + 1), dB = min(dhi, min(c0 + 15, nbi - 1));
  const int nd = dB >= dA ? dB - dA + 1 : 0;
  const int dS = dA + (nd * (int)grp) / (int)G, dE = dA + (nd * ((int)grp + 1)) / (int)G;
  const int l16 = lane & 15, l4 = lane >> 4;
  // The kernel row does not change from step to step: the F_d fragments of
  // this wavefront's first REGD diagonals stay in registers, so each step
  // reads only their mass fragments from LDS.
  const double* fa = f + (int)geo.FOFF + l16 - l4;
  double Ar[REGD > 0 ? REGD : 1][4];
#pragma unroll
  for (int i = 0; i < REGD; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) Ar[i][q] = dS + i < dE ? fa[16 * (dS + i) - 4 * q] : 0.0;
  double* cur = m0;
  double* nxt = m1;
  uint32_t n = 2;
  for (; n <= a.max_steps; ++n) {
    // (A) this wavefront's share of T m on the matrix cores; the fragments
    // of the next diagonal are read while the current products run
    f64x4 C = {0.0, 0.0, 0.0, 0.0};
    if (tile < NT) {
      const double* mb = cur + (c0 + l16 + nbi) * kBS + l4;
      double A[4], B[4];
      if (dS < dE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) B[q] = mb[4 * q - dS * kBS];
      }
      // two mass-fragment buffers in turn, so that the next diagonal's
      // fragments are read while this diagonal's products run
      double B1[4];
#pragma unroll
      for (int i = 0; i < REGD; ++i) {
        const int d = dS + i;
        if (d < dE) {
          double* cu = (i & 1) ? B1 : B;
          double* nx = (i & 1) ? B : B1;
          const int dn = d + 1 < dE ? d + 1 : d;
#pragma unroll
          for (int q = 0; q < 4; ++q) nx[q] = mb[4 * q - dn * kBS];
#pragma unroll
          for (int q = 0; q < 4; ++q) C = __builtin_amdgcn_mfma_f64_16x16x4f64(Ar[i][q], cu[q], C, 0, 0, 0);
        }
      }
      if (REGD & 1) {  // the last register diagonal left the next fragments in B1
#pragma unroll
        for (int q = 0; q < 4; ++q) B[q] = B1[q];
      }
      const int dR = dS + REGD;  // the rest, fragments of both operands from LDS
      if (dR < dE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) A[q] = fa[16 * dR - 4 * q];
      }
      for (int d = dR; d < dE; ++d) {
        double An[4], Bn[4];
        const int dn = d + 1 < dE ? d + 1 : d;  // the last diagonal re-reads its own
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          An[q] = fa[16 * dn - 4 * q];
          Bn[q] = mb[4 * q - dn * kBS];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) C = __builtin_amdgcn_mfma_f64_16x16x4f64(A[q], B[q], C, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          A[q] = An[q];
          B[q] = Bn[q];
        }
      }
      double* pw = part + ((grp * NT + tile) * 4u) * 64u + (uint32_t)lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) pw[r * 64] = C[r];
    }
    __syncthreads();
    // (B) the new mass: the groups' partial sums in group order; its total
    // and the mass it will lose at either bound in the next step
    double sv = 0.0;
    pu = 0.0;
    pl = 0.0;
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
      const uint32_t t = tid + (uint32_t)k * nt;
      if (t < 256u * NT) {
        const double* pr = part + t;  // [grp][tile][r][l] with (tile, r, l) = t
        double v = pr[0];
        for (uint32_t g = 1; g < G; ++g) v += pr[g * NT * 256u];
        if (!real[k]) v = 0.0;
        nxt[pos[k]] = v;
        sv += v;
        pu = fma(v, upc[k], pu);
        pl = fma(v, loc[k], pl);
      }
    }
    // 16-lane row sums into the window's ring; whole sums once a window is
    // full (the stop test and the absorbed masses need no per-step barrier
    // of their own)
    const uint32_t rows = nt >> 4, k = (n - 2u) % kWin;
    sv = row_sum(sv);
    pu = row_sum(pu);
    pl = row_sum(pl);
    if ((lane & 15) == 0) {
      double* rw = ring + (k * 3u) * rows + (tid >> 4);
      rw[0] = sv;
      rw[rows] = pu;
      rw[2u * rows] = pl;
    }
    // Reads of this step's partial sums and writes of the new mass come
    // before this barrier; the next step's products read the new mass and
    // overwrite the partial sums after it.
    __syncthreads();
    double* t = cur;
    cur = nxt;
    nxt = t;
    if (k == kWin - 1u || n == a.max_steps) {
      // window steps n0 .. n: whole sums in row order, one per thread
      const uint32_t cnt = k + 1u, n0 = n - k;
      if (tid < 3u * cnt) {
        const uint32_t q = tid / cnt, kk = tid - q * cnt;
        const double* rw = ring + (kk * 3u + q) * rows;
        double v = 0.0;
        for (uint32_t r = 0; r < rows; ++r) v += rw[r];
        wsum[q][kk] = v;
      }
      __syncthreads();
      // the first step of the window whose survivor mass is below tol
      uint32_t stop = cnt;
      for (uint32_t kk = 0; kk < cnt; ++kk)
        if (wsum[0][kk] < a.tol) {
          stop = kk;
          break;
        }
      // absorbed at step m + 1, for the window's steps m before the stop
      if (tid < stop) {
        const uint32_t m = n0 + tid;
        if (m < a.max_steps) {
          out_up[m] = wsum[1][tid];
          out_lo[m] = wsum[2][tid];
        }
      }
      if (stop < cnt) {
        n = n0 + stop;
        break;
      }
    }
  }
  if (n > a.max_steps) n = a.max_steps + 1u;
  // after a stop at step n, steps n + 1 .. N absorb nothing
  for (uint32_t k = n + tid; k < a.max_steps; k += nt) {
    out_up[k] = 0.0;
    out_lo[k] = 0.0;
  }
}

}  // namespace

size_t coarse_lds_bytes() { return kCoarseLds * sizeof(double) + sizeof(CoarseShared); }

// LDS: the kernel row, two zero-padded mass vectors, the partial sums and
// the window's row sums.
size_t density_lds_bytes(uint32_t cells) {
  const DensityGeo g = density_geo(cells);
  return ((size_t)g.FW + 2u * (size_t)g.CB * kBS + (size_t)g.G * g.NT * 256u +
          (size_t)kWin * 3u * (g.W * 64u / 16u)) * sizeof(double);
}

// Fewer steps than this cost less on the full grid than the coarse form's
// preparation does (0.3 ms; a full-grid step costs 1.7 us at 120 cells, 2.3 at
// 333, 3.8 at 537, 6.8 at 1000).
constexpr uint32_t kCoarseSteps = 192;

hipError_t launch_ddm_density(const DensityArgs& args, hipStream_t st) {
  const DensityGeo g = density_geo(args.cells);
  if (args.cells < 16u || g.W * 64u > (uint32_t)kMaxThreads || 2u * g.W * 64u < 256u * g.NT)
    return hipErrorInvalidValue;
  // Which form a setting takes depends on its drift: known here without a
  // grid, else both kernels run, the coarse one marks the settings it leaves and
  // the other takes those.
  DensityArgs a = args;
  const CoarsePlan p = coarse_plan(a.cells, a.thresh, a.b, a.n_signals ? 0.0 : a.drift * a.dt, a.start, a.tol_log);
  a.coarse = args.coarse && p.ok && a.max_steps >= kCoarseSteps;
  if (a.coarse) {
    hipLaunchKernelGGL(ddm_density_coarse_kernel, dim3((uint32_t)a.n_settings), dim3(kCoarseThreads),
                       kCoarseLds * sizeof(double), st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.n_signals) return e;
  }
  if (g.NT == 4u)
    hipLaunchKernelGGL((ddm_density_kernel<768, 12>), dim3((uint32_t)a.n_settings), dim3(g.W * 64u),
                       density_lds_bytes(a.cells), st, a);
  else if (g.W <= 8u)
    hipLaunchKernelGGL((ddm_density_kernel<512, 24>), dim3((uint32_t)a.n_settings), dim3(g.W * 64u),
                       density_lds_bytes(a.cells), st, a);
  else
    hipLaunchKernelGGL((ddm_density_kernel<kMaxThreads, 0>), dim3((uint32_t)a.n_settings), dim3(g.W * 64u),
                       density_lds_bytes(a.cells), st, a);
  return hipGetLastError();
}

}  // namespace cm

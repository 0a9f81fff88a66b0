// rnn.hip -- the recurrent logistic rate network on matrix cores.
//
// Each run steps n logistic rate units coupled by a weight-matrix
// projection (the logistic transfer and projections of Distill, Sec. 3.4.2;
// the simultaneous update reads the previous step's outputs, the
// current/previous output buffers of Sec. 3.3):
//   r = logistic(x);  p = W r;
//   x <- x + dt (-x + p + g u) + b xi;      y <- y + dt R (r - 1/2)
// until max(y) >= theta or the step cap.  u is the run's fixed input drive,
// xi fresh noise per unit and step, y a two-unit readout.
//
// Many runs share W, so the projection of 16 runs is one 16-column matrix
// product per step.  A workgroup of four wavefronts owns 16 run slots; wave
// w owns a quarter of the units of all 16 runs.  In the 16x16 MFMA output
// layout lane j + 16 g holds units 16b + 4g + q (q = 0..3) of run j, so each
// lane updates its own units, evaluates their logistic and publishes them
// through LDS in blocks of 16 units; the bf16 product reads them back as the
// B operand of 16x16x32 MFMAs (two published quads per lane and K block).
//
// bf16 path: each wave keeps its quarter of W (bf16, matrix-core fragment
// order) in registers for the whole kernel; r goes through LDS as bf16 B
// fragments.  FP64 path: W's fp64 fragments stream from L2 (512 KB does not
// fit on chip) and r goes through LDS in fp64.  What bounds a step of the FP64
// kernel at 256 units: 256 products of 64 cycles per wavefront (16,384 cycles),
// then about 1,450 vector instructions, which one wavefront issues at one per
// 7 cycles; two workgroups on a CU fill each other's gaps.  The stream of W must
// keep up with the products (32 bytes per cycle and CU): loads of 16 bytes per
// lane, contiguous over the wavefront (60 bytes per cycle from L2, against 32 with
// 8-byte loads), one K block's at a time right behind its products, the first ones
// of a step during the step before.  The product phase took 24.0 thousand cycles
// with 8-byte loads issued in bursts, 18.2 now; 8,192 runs of 256 units 4.93 ms
// before and 4.37 ms now, 8,192 of 64 units 700 and 616 us.  Loads 8 K blocks ahead
// instead of 4: 4.86 ms (registers spill); eight wavefronts of two blocks each: 5.2
// ms.  Few runs have a kernel of their own.
//
// Run slots are refilled as runs end: a workgroup's runs are handed to slots in
// order of slot index as they free up.  Every wave evaluates the slot
// decisions identically from the same LDS partial sums, so the assignment needs
// no atomics.  Runs are counted in an LDS window.
#include <algorithm>
#include <type_traits>

#include "internal.hpp"
#include "normal64.hpp"
#include "rng.hpp"
#include "window.hpp"

namespace cm {
namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kRnnBlock = 256;
enum { kFormBf16, kFormFp64, kFormFew };  // kernels, each with its own order of W

__device__ __forceinline__ bool near_th(double q, double th, double eps) {
  return fabs(q - th) < eps;
}

__device__ __forceinline__ float logistic_f(float x) {
  // 1 / (1 + e^-x) with the hardware exp2 and reciprocal
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * x));
}

// 1 / (1 + e^-x) in double for |x| < kLogisticMax: E = e^-x = 2^(k / 32) e^f with
// |f| <= ln2 / 64, the power from a 32-entry table (LDS) and an exponent, e^f - 1
// from a minimax polynomial (error below 2^-61 of 1); the hardware's reciprocal of
// 1 + E (good to 2^-24), then one cubic step on its residual (1 - y) - E y, so that
// 1 + E is never rounded.  Mean error 0.32 ulp over [-3, 3], 0.35 over [-30, 30] (exponential
// and division of the library: 0.41 and 0.44) in 24 instructions instead of about 50.  A
// reciprocal in floats is 1.5 % faster a sweep of 64 units, but overflows from x = -88 on,
// and sweeps whose states pass that are 4 to 6 % slower.  Larger |x|, infinities and NaN
// take the library's.
constexpr double kLogisticMax = 700.0;
constexpr int kExpEntries = 32;
__device__ const double kExpTab[kExpEntries] = {
    0x1.0000000000000p+0, 0x1.059b0d3158574p+0, 0x1.0b5586cf9890fp+0, 0x1.11301d0125b51p+0,
    0x1.172b83c7d517bp+0, 0x1.1d4873168b9aap+0, 0x1.2387a6e756238p+0, 0x1.29e9df51fdee1p+0,
    0x1.306fe0a31b715p+0, 0x1.371a7373aa9cbp+0, 0x1.3dea64c123422p+0, 0x1.44e086061892dp+0,
    0x1.4bfdad5362a27p+0, 0x1.5342b569d4f82p+0, 0x1.5ab07dd485429p+0, 0x1.6247eb03a5585p+0,
    0x1.6a09e667f3bcdp+0, 0x1.71f75e8ec5f74p+0, 0x1.7a11473eb0187p+0, 0x1.82589994cce13p+0,
    0x1.8ace5422aa0dbp+0, 0x1.93737b0cdc5e5p+0, 0x1.9c49182a3f090p+0, 0x1.a5503b23e255dp+0,
    0x1.ae89f995ad3adp+0, 0x1.b7f76f2fb5e47p+0, 0x1.c199bdd85529cp+0, 0x1.cb720dcef9069p+0,
    0x1.d5818dcfba487p+0, 0x1.dfc97337b9b5fp+0, 0x1.ea4afa2a490dap+0, 0x1.f50765b6e4540p+0};

__device__ __forceinline__ double logistic_d(double x, const double* tab) {
  const double m = __builtin_fma(x, -0x1.71547652b82fep+5, 0x1.8p52);  // k in its low bits
  const double kd = m - 0x1.8p52;
  const double f = __builtin_fma(kd, -0x1.abc9e3b39803fp-61, __builtin_fma(kd, -0x1.62e42fefa39efp-6, -x));
  const int k = (int)(uint32_t)double_bits(m);
  const uint64_t tb = double_bits(tab[k & (kExpEntries - 1)]);
  const double t = bits_double(tb + ((uint64_t)(uint32_t)((k >> 5) << 20) << 32));
  double h = fma_coef(f, 0x1.6c1718e7568e2p-10, 0x1.11114f8dacd43p-7);
  h = fma_coef(f, h, 0x1.555555554b930p-5);
  h = fma_coef(f, h, 0x1.555555554dd39p-3);
  h = __builtin_fma(f, h, 0.5);
  const double E = __builtin_fma(t, __builtin_fma(f * f, h, f), t);
  const double y = __builtin_amdgcn_rcp(1.0 + E), e = __builtin_fma(-E, y, 1.0 - y);
  return __builtin_fma(y, __builtin_fma(e, e, e), y);
}

// Logistics of a lane's units.  The library's form is a branch of the whole wavefront's,
// rarely taken, in which each unit keeps the form that its own state asks for: a run's
// bits must not depend on the runs beside it.
template <int N>
__device__ __forceinline__ void logistics_d(const double* x, double* r, const double* tab) {
  bool far = false;
#pragma unroll
  for (int i = 0; i < N; ++i) far |= !(fabs(x[i]) < kLogisticMax);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, 0)) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double y = logistic_d(x[i], tab), z = 1.0 / (1.0 + exp(-x[i]));
      r[i] = fabs(x[i]) < kLogisticMax ? y : z;
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = logistic_d(x[i], tab);
  }
}

// A workgroup's runs -- consecutive, or dealt out to the workgroups in turn -- and the
// window in LDS that counts them (counted one by one in global memory, 65,536 runs of 64
// units, bf16, took 1.87 ms, now 1.24 ms).  Workgroups differ by one run at most: rounded up
// alike, 8,300 runs of 256 units gave 483 workgroups a seventeenth run, a round of its own
// (622 us), where 108 of 512 need one (455 us).
template <bool DEALT>
struct Work {
  uint32_t* lds;
  uint64_t r0;
  uint32_t len, s_lo;
  __device__ __forceinline__ explicit Work(const RnnArgs& a) {
    r0 = DEALT ? blockIdx.x : blockIdx.x * a.base + min((uint64_t)blockIdx.x, a.extra);
    len = (uint32_t)(a.base + (blockIdx.x < a.extra));
    s_lo = DEALT ? 0u : (uint32_t)(r0 / a.trials);
    extern __shared__ unsigned long long lds_u64[];
    lds = (uint32_t*)lds_u64;
    for (uint32_t i = threadIdx.x; i < a.window * rec_words(a.n_bins); i += blockDim.x) lds[i] = 0u;
    __syncthreads();
  }
  __device__ __forceinline__ void flush(const RnnArgs& a) const {
    __syncthreads();
    if (!a.direct) flush_window(a, lds, s_lo);
  }
};

// A finished run (one lane per run).
template <bool DEALT>
__device__ __forceinline__ void record_run(const RnnArgs& a, const Work<DEALT>& wk, uint32_t s, uint32_t t,
                                           uint32_t n, int choice, bool flag, double y0, double y1) {
  count_run(a, wk.lds, wk.s_lo, s, t, n, choice, -1, flag, nullptr, 0);
  if (a.run_state) {
    const uint64_t idx = (uint64_t)s * a.trials + t;
    a.run_state[idx * (2u + a.n_units)] = y0;
    a.run_state[idx * (2u + a.n_units) + 1] = y1;
  }
}

// The same in global memory always, for the few-run kernel: its workgroups have eight
// runs at most, and the window's code in its step cost 20 to 35 us a launch (64 units,
// 500 runs 301 and 323 us).
__device__ __forceinline__ void record_few(const RnnArgs& a, uint32_t s, uint32_t t, uint32_t n, int choice,
                                           bool flag, double y0, double y1) {
  uint64_t* st = a.stats + (uint64_t)s * CM_NSTAT;
  const unsigned long long nn = n;
  if (choice >= 0) {
    const uint32_t bin = ((n - 1u) * a.n_bins) / a.max_steps;
    atomicAdd((unsigned long long*)&a.hist[((uint64_t)s * 2u + choice) * a.n_bins + bin], 1ull);
    atomicAdd((unsigned long long*)&st[CM_ST_DEC0 + choice], 1ull);
    atomicAdd((unsigned long long*)&st[CM_ST_SUMN0 + choice], nn);
    atomicAdd((unsigned long long*)&st[CM_ST_SUMSQ0 + choice], nn * nn);
  } else {
    atomicAdd((unsigned long long*)&st[CM_ST_UNDEC], 1ull);
  }
  if (flag) atomicAdd((unsigned long long*)&st[CM_ST_FLAGGED], 1ull);
  if (a.run_choice) {
    const uint64_t idx = (uint64_t)s * a.trials + t;
    a.run_choice[idx] = (int8_t)choice;
    a.run_step[idx] = n;
    a.run_flag[idx] = flag ? 1 : 0;
    if (a.run_state) {
      a.run_state[idx * (2u + a.n_units)] = y0;
      a.run_state[idx * (2u + a.n_units) + 1] = y1;
    }
  }
}

// Per-slot control state, identical in every lane of a slot (and every wave).
struct Slot {
  uint32_t s, t, n;
  bool active, flag;
  double y0, y1;
  float acc0, acc1;  // readout sum of R (r - 1/2) for the next y update
};

// Run k of the workgroup, if there is one.
template <bool DEALT>
__device__ __forceinline__ void slot_begin(const RnnArgs& a, const Work<DEALT>& wk, Slot& S, uint32_t k) {
  S.active = k < wk.len;
  const uint64_t r = wk.r0 + (S.active ? (uint64_t)k * (DEALT ? gridDim.x : 1u) : 0u);
  S.s = (uint32_t)(r / a.trials);
  S.t = (uint32_t)(r - (uint64_t)S.s * a.trials);
  S.n = 0;
  S.flag = false;
  S.y0 = 0.0;
  S.y1 = 0.0;
  S.acc0 = 0.0f;  // r = logistic(0) = 1/2 exactly, so R (r - 1/2) = 0
  S.acc1 = 0.0f;
}

// Decision after the readout update; returns true when the run ends.
__device__ __forceinline__ bool slot_decide(const RnnArgs& a, Slot& S, int& choice) {
  const double th = a.thresh, eps = a.flag_eps;
  if (near_th(S.y0, th, eps) || near_th(S.y1, th, eps)) S.flag = true;
  const double mx = S.y0 > S.y1 ? S.y0 : S.y1;
  if (mx >= th) {
    choice = S.y1 > S.y0 ? 1 : 0;
    if (fabs(S.y0 - S.y1) < eps) S.flag = true;
    return true;
  }
  choice = -1;
  return S.n == a.max_steps;
}

// ---------------------------------------------------------------------------
// bf16 projection, fp32 steps, fp64 accumulators.
// ---------------------------------------------------------------------------
// Workgroups of a CU, as the registers allow (65,536 runs of 128 units: two 2.58 ms,
// four 2.25 ms; of 64 units: two 1.46 ms, five 1.24 ms, 20,000 runs 0.56 and 0.39 ms).
constexpr int bf16_groups(int NB) { return NB > 8 ? 2 : NB > 4 ? 4 : 5; }

template <int NB, bool DEALT>
__global__ __launch_bounds__(kRnnBlock, NB == 8 ? 4 : 2) void rnn_bf16_kernel(RnnArgs a) {
  const Work<DEALT> wk(a);
  constexpr int NBW = NB / 4;  // output blocks per wave
  constexpr int NU = NB * 16;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, j = l & 15, g = l >> 4;
  __shared__ bf16x4 rt[NB][64];  // r of the 16 slots: [16-unit block][lane j + 16 g] = 4 units
  __shared__ float ypart[4][2][16];
  __shared__ float Rs[2][NU];

  // this wave's quarter of W as A fragments: block b = w NBW + bw, K block kb
  // of 32 units
  constexpr int NK = NB / 2;
  bf16x8 A[NBW][NK];
  const bf16x8* wf = (const bf16x8*)a.wfrag;
#pragma unroll
  for (int bw = 0; bw < NBW; ++bw)
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) A[bw][kb] = wf[((w * NBW + bw) * NK + kb) * 64 + l];
  // B operand of K block kb: units 32 kb + 8 g + 0..7 of run j, i.e. the
  // quads published by lanes j + 16 (2 (g & 1)) and j + 16 (2 (g & 1) + 1)
  // for 16-unit block 2 kb + g / 2
  const int bh = g >> 1, bl = j + 32 * (g & 1);
  for (int i = tid; i < 2 * NU; i += kRnnBlock) Rs[i / NU][i % NU] = (float)a.R[i];

  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const float dtf = (float)a.dt, bf = (float)a.b;

  double x[NBW][4];
  float gu[NBW][4];
  Slot S;
  uint32_t knext = 16;  // next run ordinal of this workgroup

  // Initialise a run in this lane's units: x = 0, drive g u, r = 1/2.
  auto begin_units = [&]() {
    const float gf = (float)(a.n_signals ? a.grid[(uint64_t)S.s * a.n_signals] : a.gain);
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) {
      const int b = w * NBW + bw;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t m = (uint32_t)(8 * b + 2 * g + h);  // unit pair (2m, 2m+1)
        const Words wd = philox(m, S.t, S.s, kStreamDrive, k0, k1);
        float u0, u1;
        normals32(wd, u0, u1);
        gu[bw][2 * h] = gf * u0;
        gu[bw][2 * h + 1] = gf * u1;
        x[bw][2 * h] = 0.0;
        x[bw][2 * h + 1] = 0.0;
      }
      rt[b][l] = bf16x4{(__bf16)0.5f, (__bf16)0.5f, (__bf16)0.5f, (__bf16)0.5f};
    }
  };

  slot_begin(a, wk, S, (uint32_t)j);
  begin_units();
  __syncthreads();

  for (;;) {
    // every lane of every wave sees the same slot states
    if (!__any(S.active)) break;

    // (1) projection p = W r for this wave's output blocks and all 16 slots
    f32x4 P[NBW];
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) P[bw] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
      const bf16x4 lo = rt[2 * kb + bh][bl], hi = rt[2 * kb + bh][bl + 16];
      const bf16x8 B = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int bw = 0; bw < NBW; ++bw)
        P[bw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[bw][kb], B, P[bw], 0, 0, 0);
    }
    __syncthreads();  // all reads of rt done

    // (2) unit update, new rates, readout partial sums
    S.n += 1;
    float ya = 0.0f, yb = 0.0f;
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) {
      const int b = w * NBW + bw;
      float r4[4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t m = (uint32_t)(8 * b + 2 * g + h);
        const Words wd = philox(S.n - 1u, S.t, S.s, m, k0, k1);
        float xi[2];
        normals32(wd, xi[0], xi[1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int q = 2 * h + e;
          const float xf = (float)x[bw][q];
          const float inc = fmaf(dtf, (P[bw][q] - xf) + gu[bw][q], bf * xi[e]);
          x[bw][q] = x[bw][q] + (double)inc;
          r4[q] = logistic_f((float)x[bw][q]);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int u = 16 * b + 4 * g + q;
        ya = fmaf(Rs[0][u], r4[q] - 0.5f, ya);
        yb = fmaf(Rs[1][u], r4[q] - 0.5f, yb);
      }
      rt[b][l] = bf16x4{(__bf16)r4[0], (__bf16)r4[1], (__bf16)r4[2], (__bf16)r4[3]};
    }
    ya += __shfl_xor(ya, 16, 64);
    yb += __shfl_xor(yb, 16, 64);
    ya += __shfl_xor(ya, 32, 64);
    yb += __shfl_xor(yb, 32, 64);
    if (g == 0) {
      ypart[w][0][j] = ya;
      ypart[w][1][j] = yb;
    }
    __syncthreads();

    // (3) readout update and decision, replicated in every lane of the slot
    S.y0 = S.y0 + (double)(dtf * S.acc0);
    S.y1 = S.y1 + (double)(dtf * S.acc1);
    S.acc0 = ((ypart[0][0][j] + ypart[1][0][j]) + ypart[2][0][j]) + ypart[3][0][j];
    S.acc1 = ((ypart[0][1][j] + ypart[1][1][j]) + ypart[2][1][j]) + ypart[3][1][j];
    int choice = -1;
    const bool done = S.active && slot_decide(a, S, choice);
    const uint64_t mask = __ballot(done) & 0xFFFFull;  // one bit per slot (lanes 0..15)
    if (mask) {  // uniform across the workgroup
      if (done) {
        if (w == 0 && g == 0) record_run(a, wk, S.s, S.t, S.n, choice, S.flag, S.y0, S.y1);
        if (a.run_state) {
          const uint64_t idx = (uint64_t)S.s * a.trials + S.t;
#pragma unroll
          for (int bw = 0; bw < NBW; ++bw)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              a.run_state[idx * (2u + a.n_units) + 2u + 16u * (w * NBW + bw) + 4u * g + q] = x[bw][q];
        }
        const uint32_t rank = __builtin_popcountll(mask & ((1ull << j) - 1ull));
        slot_begin(a, wk, S, knext + rank);
        begin_units();
      }
      knext += (uint32_t)__builtin_popcountll(mask);
      __syncthreads();  // refilled slots' rt entries visible to the next projection
    }
  }
  wk.flush(a);
}

// ---------------------------------------------------------------------------
// fp64 throughout.  K blocks are (b, q): units 16 b + 4 k + q, k = 0..3, which
// is the B layout of the 16x16x4 fp64 MFMA (lane j + 16 k supplies row k).
// ---------------------------------------------------------------------------
// Blocks of W that a lane's load takes at once (16-byte loads where a wavefront has
// an even number of blocks).
__host__ __device__ constexpr int f64_load(int NB) { return NB / 4 % 2 == 0 ? 2 : 1; }
// Workgroups of a CU, by the registers: at 128 units four of them would spill (8,192
// runs 1.71 ms against 1.45 ms with two).
constexpr int f64_groups(int NB) { return NB > 4 ? 2 : 4; }

template <int NB>
__global__ __launch_bounds__(kRnnBlock, f64_groups(NB)) void rnn_f64_kernel(RnnArgs a) {
  const Work<false> wk(a);
  constexpr int NBW = NB / 4, VW = f64_load(NB), NV = NBW / VW;
  constexpr int NU = NB * 16;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, j = l & 15, g = l >> 4;
  __shared__ double rt[NB * 4][64];  // [K block (b, q)][lane]
  __shared__ double ypart[4][2][16];
  __shared__ double Rs[2][NU];
  __shared__ double exps[kExpEntries];
  __shared__ NormLds<CM_FP64> norm;
  norm.load();
  if (tid < kExpEntries) exps[tid] = kExpTab[tid];
  __syncthreads();
  for (int i = tid; i < 2 * NU; i += kRnnBlock) Rs[i / NU][i % NU] = a.R[i];

  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  struct alignas(8 * VW) Frag {
    double a[VW];
  };
  const Frag* wf = (const Frag*)a.wfrag;

  double x[NBW][4], gu[NBW][4];
  Slot S;
  double acc0 = 0.0, acc1 = 0.0;  // fp64 readout sums (S.acc* unused here)
  uint32_t knext = 16;

  auto begin_units = [&]() {
    const double gd = a.n_signals ? a.grid[(uint64_t)S.s * a.n_signals] : a.gain;
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) {
      const int b = w * NBW + bw;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t m = (uint32_t)(8 * b + 2 * g + h);
        const Words wd = philox(m, S.t, S.s, kStreamDrive, k0, k1);
        double u0, u1;
        normals64(wd, norm.t, u0, u1);
        gu[bw][2 * h] = gd * u0;
        gu[bw][2 * h + 1] = gd * u1;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[bw][q] = 0.0;
        rt[4 * b + q][l] = 0.5;
      }
    }
    acc0 = 0.0;
    acc1 = 0.0;
  };

  // W's fragments, PF K blocks ahead of their products
  constexpr int K = NB * 4, PF = 4;
  const Frag* wbase = wf + w * K * NV * 64 + l;
  Frag Af[PF][NV];
#pragma unroll
  for (int f = 0; f < PF; ++f)
#pragma unroll
    for (int v = 0; v < NV; ++v) Af[f][v] = wbase[(f * NV + v) * 64];

  slot_begin(a, wk, S, (uint32_t)j);
  begin_units();
  __syncthreads();

  for (;;) {
    if (!__any(S.active)) break;

    f64x4 P[NBW];
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) P[bw] = f64x4{0.0, 0.0, 0.0, 0.0};
    double B[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) B[f] = rt[f][l];
#pragma unroll 1
    for (int kb0 = 0; kb0 < K; kb0 += PF) {
      const int kn = kb0 + PF < K ? kb0 + PF : 0;
#pragma unroll
      for (int f = 0; f < PF; ++f) {
#pragma unroll
        for (int bw = 0; bw < NBW; ++bw)
          P[bw] = __builtin_amdgcn_mfma_f64_16x16x4f64(Af[f][bw / VW].a[bw % VW], B[f], P[bw], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < NV; ++v) Af[f][v] = wbase[((kn + f) * NV + v) * 64];
        B[f] = rt[kn + f][l];  // (after the last block: block 0 of this step's r, not used)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();

    S.n += 1;
    double ya = 0.0, yb = 0.0;
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) {
      const int b = w * NBW + bw;
      double r4[4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t m = (uint32_t)(8 * b + 2 * g + h);
        double xi[2];
        normals64(philox(S.n - 1u, S.t, S.s, m, k0, k1), norm.t, xi[0], xi[1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int q = 2 * h + e;
          x[bw][q] = __builtin_fma(a.b, xi[e], __builtin_fma(a.dt, (P[bw][q] - x[bw][q]) + gu[bw][q], x[bw][q]));
        }
      }
      logistics_d<4>(x[bw], r4, exps);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int u = 16 * b + 4 * g + q;
        ya = fma(Rs[0][u], r4[q] - 0.5, ya);
        yb = fma(Rs[1][u], r4[q] - 0.5, yb);
        rt[4 * b + q][l] = r4[q];
      }
    }
    ya += __shfl_xor(ya, 16, 64);
    yb += __shfl_xor(yb, 16, 64);
    ya += __shfl_xor(ya, 32, 64);
    yb += __shfl_xor(yb, 32, 64);
    if (g == 0) {
      ypart[w][0][j] = ya;
      ypart[w][1][j] = yb;
    }
    __syncthreads();

    S.y0 = S.y0 + a.dt * acc0;
    S.y1 = S.y1 + a.dt * acc1;
    acc0 = ((ypart[0][0][j] + ypart[1][0][j]) + ypart[2][0][j]) + ypart[3][0][j];
    acc1 = ((ypart[0][1][j] + ypart[1][1][j]) + ypart[2][1][j]) + ypart[3][1][j];
    int choice = -1;
    const bool done = S.active && slot_decide(a, S, choice);
    const uint64_t mask = __ballot(done) & 0xFFFFull;
    if (mask) {
      if (done) {
        if (w == 0 && g == 0) record_run(a, wk, S.s, S.t, S.n, choice, S.flag, S.y0, S.y1);
        if (a.run_state) {
          const uint64_t idx = (uint64_t)S.s * a.trials + S.t;
#pragma unroll
          for (int bw = 0; bw < NBW; ++bw)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              a.run_state[idx * (2u + a.n_units) + 2u + 16u * (w * NBW + bw) + 4u * g + q] = x[bw][q];
        }
        const uint32_t rank = __builtin_popcountll(mask & ((1ull << j) - 1ull));
        slot_begin(a, wk, S, knext + rank);
        begin_units();
      }
      knext += (uint32_t)__builtin_popcountll(mask);
      __syncthreads();
    }
  }
  wk.flush(a);
}

// ---------------------------------------------------------------------------
// fp64 for launches of few runs: at most eight slots in a workgroup, in groups of
// four, each run in its slot from the start.
//
// The 16x16x4 product costs 64 cycles however many of its columns are runs.  The
// 4x4x4 one (four blocks of 4 x 4) costs 16 at the same rate, so a group of four
// runs is the unit here: A's fragment of 16 units (row i of block b in lane
// i + 4 b + 16 k) against the same four columns in every block.  Output lane
// j + 4 b + 16 g holds row (b, g) of run j, so with rows in order of (wavefront, b,
// g, block of the wavefront) a lane has NBW consecutive units of each of its slots,
// whose pairs share their random words.  What remains at one group is the stream
// of W (512 KB for 256 units, 60 bytes per cycle and CU: 8.5 thousand cycles of a
// step of 11 thousand).  The readout is one more product, of the rates in the
// lane's own registers; y needs only the rates of the step before, so wavefront 0
// decides which runs end while the others are in their products.  When a group
// can be freed, its runs move into holes of the first.
//
// 256 units, 500 runs 2.55 -> 1.08 ms, 2,048 runs 2.55 -> 1.43 ms; 192 units, 1,000
// runs 1.58 -> 0.68 ms (the first figures: the kernel above).  Up to 128 units all
// of W stays in the registers: 128 units, 500 runs 0.85 -> 0.40 -> 0.315 ms, 64 units
// 0.41 -> 0.30 -> 0.26 ms (the middle figures: streamed).  Of 256 units 24 of the 64 K
// blocks would fit: 500 runs 0.95 ms, but 2,048 runs 1.47 ms, from copies between the
// register halves.
// ---------------------------------------------------------------------------
constexpr int few_blocks(int NB) { return NB > 12 ? 4 : 2; }             // blocks of 16 units of a wavefront
constexpr int few_waves(int NB) { return NB / few_blocks(NB); }
// Largest launch, in runs per CU: above it the kernel above is the faster one (256
// units, 3,000 runs 2.45 ms here and 2.56 ms there, 6,000 to 8,192 runs 3.9 to 5.1 and
// 4.4 ms; 192 units, 3,000 runs 1.97 and 1.59 ms; 64 units, 2,048 runs 0.41 and 0.41 ms).
constexpr uint64_t few_runs_per_cu(int NB) { return NB > 4 ? 8 : 4; }

template <int NB>
__global__ __launch_bounds__(64 * few_waves(NB), 2) void rnn_few_kernel(RnnArgs a) {
  constexpr int NBW = few_blocks(NB), NWV = few_waves(NB), kThreads = 64 * NWV;
  constexpr int NP = NBW / 2;              // unit pairs of a lane and slot
  constexpr int kC = 2, kSlots = 4 * kC;
  constexpr int K = NB * 4, PF = 8;        // K blocks of four units; W's fragments are loaded PF ahead
  constexpr int kRow = 16 * kC + 8 / NBW;   // padded so that a wavefront's writes spread over the banks
  constexpr int NU = NB * 16;
  struct alignas(16) Pair {
    double v[2];
  };
  // lane j + 4 b + 16 g holds units u0 .. u0 + NBW - 1 of slot 4 c + j
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int j = l & 3, b = (l >> 2) & 3, g = l >> 4;
  const uint32_t u0 = (uint32_t)(NBW * (16 * w + 4 * b + g));
  __shared__ Pair rt[K / 2][kRow];         // [pair of K blocks (w, b, pair)][16 c + 4 g + j]: two units of a slot
  __shared__ double ypart[NWV][kC][32];
  __shared__ double Rs[NWV][NBW][64];      // readout weights as A fragments (rows 0 and 1)
  __shared__ uint4 state[kSlots];          // steps done, t, s, active | flag << 1
  __shared__ double2 yv[kSlots];
  __shared__ uint4 msg[kSlots];            // step index, t, s, ended | source slot << 8
  __shared__ int ctl[2];                   // groups of the next step, slots move
  __shared__ double exps[kExpEntries];
  __shared__ NormLds<CM_FP64> norm;
  norm.load();
  for (int i = tid; i < kExpEntries; i += kThreads) exps[i] = kExpTab[i];
  {
    // A fragment lane i + 4 b + 16 k: row i, unit (b, k, block)
    const int i = j, k = g;
#pragma unroll
    for (int bw = 0; bw < NBW; ++bw) Rs[w][bw][l] = i < 2 ? a.R[i * NU + NBW * (16 * w + 4 * b + k) + bw] : 0.0;
  }

  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const uint64_t G = gridDim.x, wg = blockIdx.x;
  int C = (int)(((a.total_runs - wg + G - 1) / G + 3) / 4);  // runs wg, wg + G, ...: kSlots at most
  if (tid < kSlots) {
    const uint64_t run = wg + G * (uint64_t)tid, r = run < a.total_runs ? run : 0;
    const uint32_t s = (uint32_t)(r / a.trials);
    state[tid] = uint4{0, (uint32_t)(r - (uint64_t)s * a.trials), s, run < a.total_runs ? 1u : 0u};
    yv[tid] = double2{0.0, 0.0};
  }
  __syncthreads();

  double x[kC][NBW], gu[kC][NBW];
#pragma unroll
  for (int c = 0; c < kC; ++c) {
    const uint4 st = state[4 * c + j];
    const double gd = a.n_signals ? a.grid[(uint64_t)st.z * a.n_signals] : a.gain;
#pragma unroll
    for (int h = 0; h < NP; ++h) {
      double z0, z1;
      normals64(philox(u0 / 2 + h, st.y, st.z, kStreamDrive, k0, k1), norm.t, z0, z1);
      gu[c][2 * h] = gd * z0;
      gu[c][2 * h + 1] = gd * z1;
      x[c][2 * h] = x[c][2 * h + 1] = 0.0;
      rt[(4 * w + b) * NP + h][16 * c + 4 * g + j] = Pair{{0.5, 0.5}};
    }
  }

  // up to 128 units all of W fits in the registers, else PF K blocks do
  constexpr bool kAll = NB <= 8;
  constexpr int KR = kAll ? K : PF;
  const Pair* wbase = (const Pair*)a.wfrag + (uint64_t)w * K * NP * 64 + l;
  Pair Af[KR][NP];
#pragma unroll
  for (int f = 0; f < KR; ++f)
#pragma unroll
    for (int v = 0; v < NP; ++v) Af[f][v] = wbase[(f * NP + v) * 64];

  double P[kC][NBW];
  // p = W r of this wavefront's units for the first CC groups of slots
  auto product = [&](auto cc) {
    constexpr int CC = decltype(cc)::value, PB = PF / 2;
    Pair B[PB][CC];
#pragma unroll
    for (int c = 0; c < CC; ++c)
#pragma unroll
      for (int bw = 0; bw < NBW; ++bw) P[c][bw] = 0.0;
#pragma unroll
    for (int h = 0; h < PB; ++h)
#pragma unroll
      for (int c = 0; c < CC; ++c) B[h][c] = rt[h][16 * c + 4 * g + j];
    auto block = [&](const Pair* A, int kb) {
#pragma unroll
      for (int bw = 0; bw < NBW; ++bw)
#pragma unroll
        for (int c = 0; c < CC; ++c)
          P[c][bw] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[bw / 2].v[bw % 2], B[kb / 2 % PB][c].v[kb % 2], P[c][bw], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (kAll) {
#pragma unroll
      for (int kb = 0; kb < K; ++kb) {
        block(Af[kb], kb);
        if (kb % 2 && kb / 2 + PB < K / 2)
#pragma unroll
          for (int c = 0; c < CC; ++c) B[kb / 2 % PB][c] = rt[kb / 2 + PB][16 * c + 4 * g + j];
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll 1
      for (int kb0 = 0; kb0 < K; kb0 += PF) {
        const int kn = kb0 + PF < K ? kb0 + PF : 0;
#pragma unroll
        for (int f = 0; f < PF; ++f) {
          block(Af[f], f);
#pragma unroll
          for (int v = 0; v < NP; ++v) Af[f][v] = wbase[((kn + f) * NP + v) * 64];
          if (f % 2)  // (after the last block: this step's r once more, not used)
#pragma unroll
            for (int c = 0; c < CC; ++c) B[f / 2][c] = rt[(kn + f) / 2][16 * c + 4 * g + j];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };

  // Readout, decisions and moves of the step that the other wavefronts are computing
  auto control = [&]() {
    const int q = l & 7, ro = (l >> 3) & 1;
    double acc = 0.0;
#pragma unroll
    for (int v = 0; v < NWV; ++v) acc += ypart[v][q >> 2][16 * ro + 4 * (l >> 4) + (q & 3)];
    acc += __shfl_xor(acc, 16, 64);
    acc += __shfl_xor(acc, 32, 64);
    const double oth = __shfl_xor(acc, 8, 64);
    const uint4 st = state[q];
    const double2 y = yv[q];
    Slot S;
    S.n = st.x + 1;
    S.t = st.y;
    S.s = st.z;
    S.active = st.w & 1;
    S.flag = st.w & 2;
    S.y0 = y.x + a.dt * (st.x ? (ro ? oth : acc) : 0.0);
    S.y1 = y.y + a.dt * (st.x ? (ro ? acc : oth) : 0.0);
    int choice = -1;
    const bool done = S.active && slot_decide(a, S, choice);
    const uint32_t mask = (uint32_t)__ballot(done) & 0xFFu;
    uint4 m = uint4{st.x, st.y, st.z, (uint32_t)q << 8};
    int Cn = C, moved = 0;
    if (mask) {
      if (done && l < kSlots) record_few(a, S.s, S.t, S.n, choice, S.flag, S.y0, S.y1);
      S.active = S.active && !done;
      m.w |= done ? 1u : 0u;
      const uint32_t act = (uint32_t)__ballot(S.active) & 0xFFu;
      Cn = (__builtin_popcount(act) + 3) / 4;
      if (Cn < C) {  // the last slots in use move into the holes of the first group
        const uint32_t low = (1u << (4 * Cn)) - 1u, holes = low & ~act;
        uint32_t src = (uint32_t)q, rest = act & ~low;
        if ((holes >> q) & 1u) {
          for (uint32_t r = __builtin_popcount(holes & ((1u << q) - 1u)); r; --r) rest &= rest - 1u;
          if (rest) src = (uint32_t)__builtin_ctz(rest);
        }
        m.w = (m.w & 1u) | src << 8;
        const int from = (int)src + (l & 56);
        S.n = __shfl(S.n, from, 64);
        S.t = __shfl(S.t, from, 64);
        S.s = __shfl(S.s, from, 64);
        S.active = __shfl((int)S.active, from, 64) && q < 4 * Cn;
        S.flag = __shfl((int)S.flag, from, 64);
        S.y0 = __shfl(S.y0, from, 64);
        S.y1 = __shfl(S.y1, from, 64);
        moved = 1;
      }
    }
    if (l < kSlots) {
      state[q] = uint4{S.n, S.t, S.s, (S.active ? 1u : 0u) | (S.flag ? 2u : 0u)};
      yv[q] = double2{S.y0, S.y1};
      msg[q] = m;
      if (l == 0) {
        ctl[0] = Cn;
        ctl[1] = moved;
      }
    }
  };
  __syncthreads();

  while (C > 0) {
    if (w == 0) control();
    if (C == 1)
      product(std::integral_constant<int, 1>{});
    else
      product(std::integral_constant<int, 2>{});
    __syncthreads();  // all reads of rt done, control's words visible

    const int Cn = __builtin_amdgcn_readfirstlane(ctl[0]), moved = __builtin_amdgcn_readfirstlane(ctl[1]);
#pragma unroll
    for (int c = 0; c < kC; ++c) {
      if (c >= C) break;
      const uint4 m = msg[4 * c + j];
#pragma unroll
      for (int h = 0; h < NP; ++h) {
        double z[2];
        normals64(philox(m.x, m.y, m.z, u0 / 2 + h, k0, k1), norm.t, z[0], z[1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int bw = 2 * h + e;
          x[c][bw] = __builtin_fma(a.b, z[e], __builtin_fma(a.dt, (P[c][bw] - x[c][bw]) + gu[c][bw], x[c][bw]));
        }
      }
      if (a.run_state && (m.w & 1u)) {
        double* to = a.run_state + ((uint64_t)m.z * a.trials + m.y) * (2u + a.n_units) + 2u + u0;
#pragma unroll
        for (int bw = 0; bw < NBW; ++bw) to[bw] = x[c][bw];
      }
    }
    if (moved) {  // through this wavefront's own rows of rt
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        double(*v)[NBW] = part ? gu : x;
#pragma unroll
        for (int c = 0; c < kC; ++c)
          if (c < C)
#pragma unroll
            for (int h = 0; h < NP; ++h)
              rt[(4 * w + b) * NP + h][16 * c + 4 * g + j] = Pair{{v[c][2 * h], v[c][2 * h + 1]}};
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kC; ++c)
          if (c < Cn) {
            const uint32_t src = msg[4 * c + j].w >> 8;
#pragma unroll
            for (int h = 0; h < NP; ++h) {
              const Pair q = rt[(4 * w + b) * NP + h][16 * (src >> 2) + 4 * g + (src & 3)];
              v[c][2 * h] = q.v[0];
              v[c][2 * h + 1] = q.v[1];
            }
          }
        __syncthreads();
      }
    }
#pragma unroll
    for (int c = 0; c < kC; ++c) {
      if (c >= Cn) break;
      double r[NBW];
      logistics_d<NBW>(x[c], r, exps);
#pragma unroll
      for (int h = 0; h < NP; ++h) rt[(4 * w + b) * NP + h][16 * c + 4 * g + j] = Pair{{r[2 * h], r[2 * h + 1]}};
      double y = 0.0;
#pragma unroll
      for (int bw = 0; bw < NBW; ++bw) y = __builtin_amdgcn_mfma_f64_4x4x4f64(Rs[w][bw][l], r[bw] - 0.5, y, 0, 0, 0);
      if (l < 32) ypart[w][c][l] = y;
    }
    C = Cn;
    __syncthreads();
  }
}

// W (fp64 row-major n x n) -> matrix-core fragment order.
//  bf16: fragment (b, kb) for 16x16x32 MFMAs, lane l = i + 16 k8 holds
//        W[16b + i][32kb + 8k8 + 0..7].
//  fp64: fragment (b, kb4 = 4 bb + q), lane l = i + 16 k holds
//        W[16b + 4 (i % 4) + i / 4][16bb + 4k + q].
__global__ void rnn_prep_kernel(const double* W, uint32_t n, void* out, int form) {
  const uint32_t NB = n / 16;
  const uint64_t total = (uint64_t)n * n;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * blockDim.x) {
    if (form == kFormBf16) {
      // e enumerates (b, kb, lane, item)
      const uint32_t item = e & 7u, lane = (e >> 3) & 63u, NK = NB / 2u;
      const uint64_t frag = e >> 9;
      const uint32_t kb = (uint32_t)(frag % NK), b = (uint32_t)(frag / NK);
      const uint32_t i = lane & 15u, k8 = lane >> 4;
      const double v = W[(uint64_t)(16u * b + i) * n + 32u * kb + 8u * k8 + item];
      ((__bf16*)out)[e] = (__bf16)(float)v;
    } else if (form == kFormFew) {
      // e enumerates (wavefront w, K block, load v, lane, item).  Lane i + 4 b + 16 k
      // of block bw = 2 v + item holds the row of unit NBW (16 w + 4 b + i) + bw and
      // the column of unit NBW (4 kb' + k) + kw, where the K blocks are numbered
      // NBW kb' + kw.
      const uint32_t NBW = few_blocks((int)NB), NP = NBW / 2u, K = 4u * NB;
      const uint32_t lane = (uint32_t)(e >> 1) & 63u, i = lane & 3u, b = (lane >> 2) & 3u, k = lane >> 4;
      const uint64_t frag = e >> 7;
      const uint32_t bw = 2u * (uint32_t)(frag % NP) + (uint32_t)(e & 1u), kb = (uint32_t)(frag / NP % K);
      const uint32_t w = (uint32_t)(frag / (NP * K));
      const uint32_t row = NBW * (16u * w + 4u * b + i) + bw, col = NBW * (4u * (kb / NBW) + k) + kb % NBW;
      ((double*)out)[e] = W[(uint64_t)row * n + col];
    } else {
      // e enumerates (wavefront, kb4, load, lane, block of the load): what a
      // wavefront reads for a K block is contiguous, so its lines spread over the
      // L2's channels.  The fp64 16x16x4 accumulator holds row 4 reg + lane/16 in
      // register reg of a lane, so row position i of block b stands for unit
      // 16 b + 4 (i % 4) + i / 4: each lane then holds four consecutive units
      // (16 b + 4 g + reg), as in the bf16 layout.
      const uint32_t VW = f64_load((int)NB), NV = NB / 4u / VW, K = 4u * NB;
      const uint32_t lane = (uint32_t)(e / VW) & 63u;
      const uint64_t frag = e / (64u * VW);
      const uint32_t kb4 = (uint32_t)(frag / NV % K);
      const uint32_t b = ((uint32_t)(frag / (NV * K)) * NV + (uint32_t)(frag % NV)) * VW + (uint32_t)(e % VW);
      const uint32_t bb = kb4 >> 2, q = kb4 & 3u, i = lane & 15u, k = lane >> 4;
      const uint32_t row = 16u * b + 4u * (i & 3u) + (i >> 2);
      ((double*)out)[e] = W[(uint64_t)row * n + 16u * bb + 4u * k + q];
    }
  }
}

constexpr bool deals(int NB) { return NB > 8; }  // see plan_nb

template <int NB>
hipError_t launch_nb(int form, const RnnArgs& a, uint32_t groups, hipStream_t st) {
  const size_t lds = (size_t)a.window * rec_words(a.n_bins) * 4u;
  if (form == kFormFew)
    hipLaunchKernelGGL((rnn_few_kernel<NB>), dim3(groups), dim3(64 * few_waves(NB)), lds, st, a);
  else if (form == kFormFp64)
    hipLaunchKernelGGL((rnn_f64_kernel<NB>), dim3(groups), dim3(kRnnBlock), lds, st, a);
  else if (deals(NB) && a.dealt)
    hipLaunchKernelGGL((rnn_bf16_kernel<NB, deals(NB)>), dim3(groups), dim3(kRnnBlock), lds, st, a);
  else
    hipLaunchKernelGGL((rnn_bf16_kernel<NB, false>), dim3(groups), dim3(kRnnBlock), lds, st, a);
  return hipGetLastError();
}

// Consecutive runs fill few windows, but belong to few settings: where settings' runs
// differ in length so do the workgroups, and at two on a CU, all resident from the start,
// nothing evens that out.  So bf16 networks of 192 and 256 units deal runs out in turn from
// three settings on (with one or two, a CU's two workgroups hold both alike), where slots are
// filled four times and more (20,000 runs of 192 units, 2.4 times, 16 gains from 0.5 to 1.5:
// consecutive 1.23 ms, dealt 1.27, from 0.02 to 30 1.27 and 1.24): 65,536 runs of
// 256 units with 16 gains from 0.02 to 30 consecutive 5.02 ms, dealt 4.65, 100 gains 5.03 and
// 4.68, gains from 0.5 to 1.5 5.02 and 5.01, two gains 3.95 and 4.48; 192 units, 16 gains
// falling from 30 to 0.02 3.53 and 3.36.  Smaller networks have four or five workgroups on a
// CU (128 units, 16 gains 2.06 and 2.26 ms), and in FP64 it goes either way (256 units 13.6 and
// 13.6, two gains 11.3 and 12.5, 100 falling gains 13.4 and 12.8).
template <int NB>
RnnPlan plan_nb(int precision, uint64_t settings, uint64_t runs, uint64_t cus) {
  const uint64_t wide = std::min<uint64_t>((runs + 15) / 16, cus * (precision == CM_FP64 ? f64_groups(NB) : bf16_groups(NB)));
  if (precision != CM_FP64) return {kFormBf16, (uint32_t)wide, false, deals(NB) && settings > 2 && runs >= 4u * 16u * wide};
  if (runs > few_runs_per_cu(NB) * cus) return {kFormFp64, (uint32_t)wide, false, false};
  return {kFormFew, (uint32_t)std::min<uint64_t>((runs + 3) / 4, cus), true, false};
}

}  // namespace

hipError_t launch_rnn_prep(const double* W, uint32_t n, void* out, int form, hipStream_t st) {
  const uint64_t total = (uint64_t)n * n;
  const uint32_t grid = (uint32_t)std::min<uint64_t>((total + 255) / 256, 4096);
  hipLaunchKernelGGL(rnn_prep_kernel, dim3(grid), dim3(256), 0, st, W, n, out, form);
  return hipGetLastError();
}

RnnPlan plan_rnn(int precision, uint32_t n_units, uint64_t settings, uint64_t runs, uint32_t cus) {
  switch (n_units) {
    case 64: return plan_nb<4>(precision, settings, runs, cus);
    case 128: return plan_nb<8>(precision, settings, runs, cus);
    case 192: return plan_nb<12>(precision, settings, runs, cus);
    default: return plan_nb<16>(precision, settings, runs, cus);
  }
}

hipError_t launch_rnn(int form, const RnnArgs& a, uint32_t groups, hipStream_t st) {
  switch (a.n_units) {
    case 64: return launch_nb<4>(form, a, groups, st);
    case 128: return launch_nb<8>(form, a, groups, st);
    case 192: return launch_nb<12>(form, a, groups, st);
    case 256: return launch_nb<16>(form, a, groups, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace cm

// lme_flip.hip -- the streamed Liouvillian of spin chains (n = 2^M, 128 or
// 256): every off-diagonal entry of A = -iH - 1/2 sum C^+C is imaginary and
// flips one spin (column i xor 2^b), every collapse operator is real and is
// either diagonal or flips one spin.
//
// A workgroup takes 8 rows of an instance; a thread owns a column j and RT = 4
// consecutive rows, whose elements it keeps in registers and
// shares through LDS.  What the flip structure gives over rows_lindblad():
//   * where a source lies depends on the bit alone, at compile time: a row of
//     the same thread (bits below RB), of the block (below kLB) or of another
//     block (one contiguous row read); columns j xor 1, 2, 8 come from other
//     lanes by DPP, the rest from LDS;
//   * the value the right product reads for row t, y[i][j xor 2^b], is the
//     jump's source for row t xor 2^b: no second read for the thread's bits;
//   * the diagonal collapse operators are one factor per element,
//     sum_k z_k(i) z_k(j), added to the diagonal of the generator;
//   * row-side entries are wavefront-uniform runs of RT doubles (scalar
//     loads); a jump whose row factor vanishes on the block's rows (half of the
//     blocks for a lowering operator on a high bit) is skipped.
// One application of 64 chains of 8 spins (134 MB in and out): 50 us against
// 94 us for apply_rows_kernel (2.7 TB/s; the remote rows add about six times
// the state through L2, and a block's loads, barrier and 80 registers leave
// five wavefronts a SIMD to hide them).  8-row blocks in 512 threads: 16-row
// blocks in 1024 threads 58 us, 8 rows a thread 71 us (spills).  A stage of
// the adaptive step moves up to 536 MB and runs at 3.1 to 3.8 TB/s (108 to 143
// us, loading other blocks' rows one spin ahead; a whole step 0.87 ms against
// 1.3 ms); a single application is faster without (50 against 54 us).
#include <type_traits>

#include "lme_device.h"
#include "lme_internal.h"

namespace lme {

namespace {

constexpr int kFlipR = lme::kFlipRows;
constexpr int kRB = 2;                   // log2 of the rows of a thread
constexpr int kLB = 3;                   // log2 of the rows of a block
// threads of a block of rows of 2^logn elements
constexpr int flip_threads(int logn) { return (kFlipR >> kRB) << logn; }

template <int V>
using Int = std::integral_constant<int, V>;
template <typename T>
using cptr = const T __attribute__((address_space(4))) *;

// lane exchanges of a double2 through DPP
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL>
__device__ __forceinline__ double2 dpp_c(double2 v) {
  return make_double2(dpp_d<CTRL>(v.x), dpp_d<CTRL>(v.y));
}

// Per-instance table (doubles): D [n] complex | FA [M][n], Im A_{i, i xor 2^b}
// | FJ [nf][n], flipping collapse operators ordered by bit | Z [nd][n],
// diagonal ones.
template <int LOGN>
struct FlipTile {
  static constexpr int N = 1 << LOGN, RB = kRB, RT = 1 << RB;
  double2 y[RT];     // the thread's rows of the input

  // Loads and shares the block's rows; the caller synchronises.  rg: the row
  // group, uniform in the wavefront.
  __device__ __forceinline__ void load(const double2 *Yg, double2 *Ys, int r0, int rg, int j) {
#pragma unroll
    for (int t = 0; t < RT; ++t) y[t] = Yg[(r0 + rg * RT + t) * N + j];
#pragma unroll
    for (int t = 0; t < RT; ++t) Ys[(rg * RT + t) * N + j] = y[t];
  }

  // kv[t] = (L y)_ij for the thread's rows.
  template <bool AHEAD>
  __device__ __forceinline__ void apply(const FlipArgs &f, const double *tab, const double2 *Yg,
                                        const double2 *Ys, int r0, int rg, int j,
                                        double2 (&kv)[RT]) const {
    const int i0 = r0 + rg * RT;
    const cptr<double> ct = (cptr<double>)tab;
    const double *FA = tab + 2 * N, *FJ = FA + LOGN * N, *Z = FJ + f.nf * N;
    const cptr<double> cFA = ct + 2 * N, cFJ = cFA + LOGN * N, cZ = cFJ + f.nf * N;
    {
      const double2 dj = reinterpret_cast<const double2 *>(tab)[j];
      double dre[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) dre[t] = ct[2 * (i0 + t)] + dj.x;
      for (int k = 0; k < f.nd; ++k) {
        const double zj = Z[k * N + j];
#pragma unroll
        for (int t = 0; t < RT; ++t) dre[t] = fma(cZ[k * N + i0 + t], zj, dre[t]);
      }
#pragma unroll
      for (int t = 0; t < RT; ++t)
        kv[t] = cmul(make_double2(dre[t], ct[2 * (i0 + t) + 1] - dj.y), y[t]);
    }
    // AHEAD: rows of other blocks are loaded one spin before their use
    double2 l0[RT], l1[RT];
    auto ahead = [&](auto spin, double2 (&l)[RT]) {
      if constexpr (AHEAD && spin.value < LOGN) load_rows<spin.value>(Yg, i0, j, l);
    };
    auto spin = [&](auto b, const double2 (&l)[RT]) {
      if constexpr (b.value < LOGN)
        bit<AHEAD, b.value>(f, FA, FJ, cFA, cFJ, Yg, Ys, i0, rg, j, l, kv);
    };
    ahead(Int<3>{}, l0);
    spin(Int<0>{}, l0);
    spin(Int<1>{}, l0);
    ahead(Int<4>{}, l1);
    spin(Int<2>{}, l0);
    spin(Int<3>{}, l0);
    ahead(Int<5>{}, l0);
    spin(Int<4>{}, l1);
    ahead(Int<6>{}, l1);
    spin(Int<5>{}, l0);
    ahead(Int<7>{}, l0);
    spin(Int<6>{}, l1);
    spin(Int<7>{}, l0);
  }

  // y[i xor 2^B][j] of the thread's rows, another block's
  template <int B>
  __device__ __forceinline__ void load_rows(const double2 *Yg, int i0, int j,
                                            double2 (&l)[RT]) const {
#pragma unroll
    for (int t = 0; t < RT; ++t) l[t] = Yg[((i0 + t) ^ (1 << B)) * N + j];
  }

  // the terms of spin B; far: load_rows<B>() under AHEAD where B >= kLB
  template <bool AHEAD, int B>
  __device__ __forceinline__ void bit(const FlipArgs &f, const double *FA, const double *FJ,
                                      cptr<double> cFA, cptr<double> cFJ, const double2 *Yg,
                                      const double2 *Ys, int i0, int rg, int j,
                                      const double2 (&far)[RT], double2 (&kv)[RT]) const {
    constexpr int MB = 1 << B;
    const int jx = j ^ MB;
    // y[i][j xor 2^B]
    auto right = [&](int t) {
      if constexpr (B == 0) return dpp_c<0xB1>(y[t]);
      else if constexpr (B == 1) return dpp_c<0x4E>(y[t]);
      else if constexpr (B == 3) return dpp_c<0x128>(y[t]);   // row_ror:8
      else return Ys[(rg * RT + t) * N + jx];
    };
    // y[i xor 2^B][jj], a row of the block or of another one
    auto row = [&](int t, int jj) {
      if constexpr (MB < kFlipR) return Ys[((rg * RT + t) ^ MB) * N + jj];
      else return Yg[((i0 + t) ^ MB) * N + jj];
    };
    const double faj = FA[B * N + j];
    // the jump's row factors, and whether one of them is not zero
    const int q0 = f.first[B], q1 = f.first[B + 1];
    bool jump = q1 > q0;
    if (B >= RB && jump) {
      double any = 0.0;
      for (int q = q0; q < q1; ++q)
#pragma unroll
        for (int t = 0; t < RT; ++t) any += fabs(cFJ[q * N + i0 + t]);
      jump = any != 0.0;
    }
    double w[RT];
    if (jump) {
#pragma unroll
      for (int t = 0; t < RT; ++t) w[t] = 0.0;
      for (int q = q0; q < q1; ++q) {
        const double jj = FJ[q * N + j];
#pragma unroll
        for (int t = 0; t < RT; ++t) w[t] = fma(cFJ[q * N + i0 + t], jj, w[t]);
      }
    }
    if constexpr (B < RB) {
      double2 R[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) R[t] = right(t);
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const double fai = cFA[B * N + i0 + t];
        const double2 l = y[t ^ MB];
        kv[t] = make_double2(fma(-fai, l.y, kv[t].x), fma(fai, l.x, kv[t].y));
        kv[t] = make_double2(fma(faj, R[t].y, kv[t].x), fma(-faj, R[t].x, kv[t].y));
      }
      if (jump) {
#pragma unroll
        for (int t = 0; t < RT; ++t) kv[t] = caxpy(w[t], R[t ^ MB], kv[t]);
      }
    } else {
      double2 l[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        if constexpr (AHEAD && B >= kLB) l[t] = far[t];
        else l[t] = row(t, j);
      }
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const double2 R = right(t);
        kv[t] = make_double2(fma(faj, R.y, kv[t].x), fma(-faj, R.x, kv[t].y));
      }
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const double fai = cFA[B * N + i0 + t];
        kv[t] = make_double2(fma(-fai, l[t].y, kv[t].x), fma(fai, l[t].x, kv[t].y));
      }
      if (jump) {
#pragma unroll
        for (int t = 0; t < RT; ++t) l[t] = row(t, jx);
#pragma unroll
        for (int t = 0; t < RT; ++t) kv[t] = caxpy(w[t], l[t], kv[t]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

// workgroup -> tile in the XCD-aware order of lme_kernels.hip
__device__ __forceinline__ int flip_tile_index(int n_tiles) {
  const int per = (n_tiles + 7) / 8;
  return (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
}

// Dormand & Prince (1980), as in lme_kernels.hip, known at compile time here
constexpr double kA[7][6] = {
    {0, 0, 0, 0, 0, 0},
    {1.0 / 5, 0, 0, 0, 0, 0},
    {3.0 / 40, 9.0 / 40, 0, 0, 0, 0},
    {44.0 / 45, -56.0 / 15, 32.0 / 9, 0, 0, 0},
    {19372.0 / 6561, -25360.0 / 2187, 64448.0 / 6561, -212.0 / 729, 0, 0},
    {9017.0 / 3168, -355.0 / 33, 46732.0 / 5247, 49.0 / 176, -5103.0 / 18656, 0},
    {35.0 / 384, 0, 500.0 / 1113, 125.0 / 192, -2187.0 / 6784, 11.0 / 84}};
constexpr double kE[7] = {35.0 / 384 - 5179.0 / 57600, 0.0, 500.0 / 1113 - 7571.0 / 16695,
                          125.0 / 192 - 393.0 / 640, -2187.0 / 6784 - (-92097.0 / 339200),
                          11.0 / 84 - 187.0 / 2100, 0.0 - 1.0 / 40};

}  // namespace

template <int LOGN>
__global__ __launch_bounds__(flip_threads(LOGN), 4) void apply_flip_kernel(FlipArgs f, const double *y,
                                                               double *out) {
  constexpr int N = 1 << LOGN;
  extern __shared__ __align__(16) uint8_t smem[];
  const int tix = flip_tile_index(f.n_tiles);
  if (tix >= f.n_tiles) return;
  const int b = tix / (N / kFlipR), r0 = (tix % (N / kFlipR)) * kFlipR;
  double2 *Ys = reinterpret_cast<double2 *>(smem);
  const double2 *Yg = reinterpret_cast<const double2 *>(y) + (int64_t)b * N * N;
  const int j = threadIdx.x & (N - 1);
  const int rg = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> LOGN));
  FlipTile<LOGN> tl;
  tl.load(Yg, Ys, r0, rg, j);
  __syncthreads();
  double2 kv[FlipTile<LOGN>::RT];
  tl.template apply<false>(f, f.tab + b * f.stride, Yg, Ys, r0, rg, j, kv);
  double2 *o = reinterpret_cast<double2 *>(out) + (int64_t)b * N * N;
#pragma unroll
  for (int t = 0; t < FlipTile<LOGN>::RT; ++t)
    o[(r0 + rg * FlipTile<LOGN>::RT + t) * N + j] = kv[t];
}

// Stage S of the streamed adaptive step (sdp_stage_rows_kernel) on flip
// tiles.  Weights that are zero (the second derivative in the fifth-order
// solution and in the error) are not read.
template <int LOGN, int S>
__global__ __launch_bounds__(flip_threads(LOGN), 4) void sdp_stage_flip_kernel(FlipArgs f, StreamArgs a) {
  constexpr int N = 1 << LOGN, RT = FlipTile<LOGN>::RT;
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ double sh[flip_threads(LOGN) / 64];
  const int tix = flip_tile_index(f.n_tiles);
  if (tix >= f.n_tiles) return;
  const int b = tix / (N / kFlipR), r0 = (tix % (N / kFlipR)) * kFlipR;
  const DpCtl &ctl = a.ctl[b];
  if (!ctl.active) return;
  const double ht = ctl.h_try;
  const bool need = S > 0 || ctl.need_k1;
  const int64_t base = (int64_t)b * N * N, SE = a.state_elems;
  const double2 *rho = reinterpret_cast<const double2 *>(a.rho) + base;
  double2 *yb0 = reinterpret_cast<double2 *>(a.yb0) + base;
  double2 *yb1 = reinterpret_cast<double2 *>(a.yb1) + base;
  double2 *y5 = reinterpret_cast<double2 *>(a.y5) + base;
  double2 *K = reinterpret_cast<double2 *>(a.K) + base;
  const double2 *Yin = S == 0 ? rho : (S == 6 ? y5 : (S & 1) ? yb0 : yb1);
  double2 *Yout = S == 5 ? y5 : (S & 1) ? yb1 : yb0;
  double2 *Ys = reinterpret_cast<double2 *>(smem);
  const int j = threadIdx.x & (N - 1);
  const int rg = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> LOGN));
  const int e0 = (r0 + rg * RT) * N + j;
  double2 kv[RT];
  FlipTile<LOGN> tl;
  if (need) {
    tl.load(Yin, Ys, r0, rg, j);
    __syncthreads();
    tl.template apply<true>(f, f.tab + b * f.stride, Yin, Ys, r0, rg, j, kv);
#pragma unroll
    for (int t = 0; t < RT; ++t) K[S * SE + e0 + t * N] = kv[t];
  } else {
#pragma unroll
    for (int t = 0; t < RT; ++t) kv[t] = K[e0 + t * N];
  }
  // the sum over the stored derivatives (a zero weight is not read)
  double2 acc[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    acc[t] = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const double w = S < 6 ? kA[S < 6 ? S + 1 : 0][S < 6 ? q : 0] : kE[q];
      if (w != 0.0) acc[t] = caxpy(w, K[q * SE + e0 + t * N], acc[t]);
    }
  }
  if constexpr (S < 6) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      acc[t] = caxpy(kA[S + 1][S], kv[t], acc[t]);
      Yout[e0 + t * N] = caxpy(ht, acc[t], rho[e0 + t * N]);
    }
  } else {
    double part = 0.0;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int e = e0 + t * N;
      double2 er = caxpy(kE[6], kv[t], acc[t]);
      er = make_double2(ht * er.x, ht * er.y);
      const double2 p = rho[e], y = tl.y[t];
      const double sc = a.atol + a.rtol * fmax(hypot(p.x, p.y), hypot(y.x, y.y));
      const double q = hypot(er.x, er.y) / sc;
      part += q * q;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
      double tot = 0.0;
      for (int w = 0; w < flip_threads(LOGN) / 64; ++w) tot += sh[w];
      a.tile_part[tix] = tot;
    }
  }
}

}  // namespace lme

// logn 7 or 8; f.n_tiles = instances * n / kFlipRows
extern "C" hipError_t lme_internal_launch_apply_flip(int logn, const lme::FlipArgs *f,
                                                     const double *y, double *out, hipStream_t s) {
  auto k = logn == 8 ? lme::apply_flip_kernel<8> : lme::apply_flip_kernel<7>;
  const int lds = 16 * lme::kFlipR << logn, grid = 8 * ((f->n_tiles + 7) / 8);
  if (logn != 7 && logn != 8) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(grid), dim3(lme::flip_threads(logn)), lds, s, *f, y, out);
  return hipGetLastError();
}

typedef void (*flip_stage_t)(lme::FlipArgs, lme::StreamArgs);
static flip_stage_t flip_stage(int logn, int s) {
#define LME_FS(G)                                                                   \
  {lme::sdp_stage_flip_kernel<G, 0>, lme::sdp_stage_flip_kernel<G, 1>,              \
   lme::sdp_stage_flip_kernel<G, 2>, lme::sdp_stage_flip_kernel<G, 3>,              \
   lme::sdp_stage_flip_kernel<G, 4>, lme::sdp_stage_flip_kernel<G, 5>,              \
   lme::sdp_stage_flip_kernel<G, 6>}
  static const flip_stage_t k[2][7] = {LME_FS(7), LME_FS(8)};
#undef LME_FS
  return k[logn - 7][s];
}

// Stage kernel of the streamed adaptive stepper: prepare sets its dynamic LDS
// limits (outside any graph capture), launch issues stage s.
extern "C" hipError_t lme_internal_sdp_flip_prepare(int logn) {
  if (logn != 7 && logn != 8) return hipErrorInvalidValue;
  for (int s = 0; s < 7; ++s) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(flip_stage(logn, s)),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       16 * lme::kFlipR << logn);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

extern "C" hipError_t lme_internal_launch_sdp_flip(int logn, int s, const lme::FlipArgs *f,
                                                   const lme::StreamArgs *a, hipStream_t st) {
  if (logn < 7 || logn > 8 || s < 0 || s > 6) return hipErrorInvalidValue;
  const int lds = 16 * lme::kFlipR << logn, grid = 8 * ((f->n_tiles + 7) / 8);
  hipLaunchKernelGGL(flip_stage(logn, s), dim3(grid), dim3(lme::flip_threads(logn)), lds, st, *f, *a);
  return hipGetLastError();
}

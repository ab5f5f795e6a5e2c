// lme_mc.hip -- Monte-Carlo wave-function trajectories on gfx950.
//
// What is computed (arXiv:1110.0573, Sec. 3.2, steps I-IV): every trajectory
// evolves a ket under the effective Hamiltonian of Eq. (heff),
//   d psi/dt = A psi,   A = -i H_eff = -i H - 1/2 sum_n C_n^+ C_n,
// until its squared norm falls to the drawn number r (step II), then jumps
// with the collapse operator chosen by the cumulative rule of Eq. (mc3) with
// a second draw r' (Eq. (pcn) gives the probabilities), is renormalised
// (Eq. (project)) and continues with the next draw (step IV).
//
// Integrator: classic RK4 on the grid t0 + m h.  For the autonomous linear
// equation the RK4 step of length s is exactly the degree-4 Taylor polynomial
//   psi(s) = v0 + s v1 + s^2 v2 + s^3 v3 + s^4 v4,  v0 = psi, v_k = A v_{k-1} / k,
// which is how it is evaluated here: the v_k do not depend on s, so
//   * every trajectory of a workgroup can take its own step length (the rest
//     of a grid step after a jump) in one uniform pass, and
//   * the jump time is a root of the scalar polynomial |psi(s)|^2 - r, whose
//     nine coefficients c_d = sum_{j+k=d} Re <v_j|v_k> come from one
//     reduction; bisection on that polynomial replaces repeated integration.
//
// Work decomposition: a workgroup holds P trajectories; G = 2^g threads own
// one trajectory, thread g its rows g, g + G, ... (R rows).  The current
// Taylor vector of every trajectory is staged in LDS (16 n bytes each) so the
// sparse products gather from LDS; the state psi sits in LDS too (read and
// written only by the thread that owns the row) and the running sum in
// registers.  Per-trajectory scalars (threshold, time left, jump count,
// status) are identical in every thread of a group: reductions end with the
// same bits in every lane (xor butterflies, then a fixed-order sum of the
// wave partials), so every decision is taken uniformly without broadcasts.
// Workgroups are persistent and walk the packs of P trajectories.
#include <hip/hip_runtime.h>

#include "../../include/lme.h"
#include "lme_internal.h"

namespace {

using lme::McArgs;

struct __attribute__((aligned(16))) cplx {
  double x, y;
};

__device__ inline cplx cmul(cplx a, cplx b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ inline cplx cfma(cplx a, cplx b, cplx c) {  // a * b + c
  return {fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y))};
}
__device__ inline cplx cscale(double s, cplx a) { return {s * a.x, s * a.y}; }
__device__ inline cplx caxpy(double s, cplx a, cplx c) { return {fma(s, a.x, c.x), fma(s, a.y, c.y)}; }
__device__ inline double cabs2(cplx a) { return fma(a.x, a.x, a.y * a.y); }
// An opaque copy: the compiler cannot prove it equal to its input.
__device__ inline int launder(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ inline double wave_sum(double v);

// Sum of NV values over the G threads of each trajectory group.  Every
// thread of the group gets bitwise the same sums.  red: LDS, NV doubles per
// wave.  Must be called by every thread of the workgroup (it may contain
// barriers).
template <int NV>
__device__ inline void group_sum(double (&v)[NV], int G, double *red) {
  const int lane = threadIdx.x & 63;
  if (G <= 64) {
    for (int off = G >> 1; off > 0; off >>= 1)
#pragma unroll
      for (int q = 0; q < NV; ++q) v[q] += __shfl_xor(v[q], off, 64);
    return;
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = wave_sum(v[q]);
  const int wave = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < NV; ++q) red[wave * NV + q] = v[q];
  __syncthreads();
  const int wpg = G >> 6;                      // waves per group
  const int w0 = (threadIdx.x / G) * wpg;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double s = red[w0 * NV + q];
    for (int w = 1; w < wpg; ++w) s += red[(w0 + w) * NV + q];
    v[q] = s;
  }
  __syncthreads();
}

// Sum over the wavefront, the same bits in every lane: four steps inside each
// row of 16 lanes (quad and row permutes, no LDS), then the four row sums in
// order.
template <int CTRL>
__device__ inline double dpp_add(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline double lane_value(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline double row_sum16(double v) {
  v = dpp_add<0xB1>(v);    // quad_perm 1,0,3,2
  v = dpp_add<0x4E>(v);    // quad_perm 2,3,0,1
  v = dpp_add<0x141>(v);   // row_half_mirror
  return dpp_add<0x140>(v);  // row_mirror
}
__device__ inline double wave_sum(double v) {
  v = row_sum16(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// group_sum() in two halves for whole wavefronts per group (G >= 64): the
// wave partials into red, and after the caller's barrier their sum, in one
// order for every thread.  red: [waves], 16-byte aligned.
__device__ inline void wave_partial(double v, double *red) {
  const double w = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
}
__device__ inline double sum_partials(int G, const double *red) {
  const int wpg = G >> 6;
  const double *r = red + (threadIdx.x / G) * wpg;
  double s = r[0];
  for (int w = 1; w < wpg; ++w) s += r[w];
  return s;
}

// Operator tables read through buffer resources (base and size in scalar
// registers, a 32-bit byte offset per lane): no 64-bit address per row stays
// live across the step loop.
constexpr int kBufferFlags = 0x00020000;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Tabs {
  __amdgpu_buffer_rsrc_t D, Oval, Ocol, Jval, Jcol, Eval, Ecol, vb;
};

__device__ inline __amdgpu_buffer_rsrc_t rsrc(const void *p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, kBufferFlags);
}
__device__ inline cplx ld_c(__amdgpu_buffer_rsrc_t r, uint32_t idx) {
  return __builtin_bit_cast(cplx, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 16u, 0, 0));
}
__device__ inline int ld_i(__amdgpu_buffer_rsrc_t r, uint32_t idx) {
  return (int)__builtin_amdgcn_raw_buffer_load_b32(r, idx * 4u, 0, 0);
}
__device__ inline void st_c(__amdgpu_buffer_rsrc_t r, uint32_t idx, cplx v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, idx * 16u, 0, 0);
}

// y = (A x)_i for row i, x = the group's vector in LDS.
__device__ inline cplx row_apply(const Tabs &t, int n, int wo, const cplx *x, int i) {
  cplx acc = cmul(ld_c(t.D, i), x[i]);
  for (int s = 0; s < wo; ++s) acc = cfma(ld_c(t.Oval, s * n + i), x[ld_i(t.Ocol, s * n + i)], acc);
  return acc;
}

// (C_k x)_i
__device__ inline cplx row_jump(const Tabs &t, int n, int wc, const cplx *x, int k, int i) {
  cplx acc = {0.0, 0.0};
  const int base = k * wc * n;
  for (int s = 0; s < wc; ++s)
    acc = cfma(ld_c(t.Jval, base + s * n + i), x[ld_i(t.Jcol, base + s * n + i)], acc);
  return acc;
}

// (E_m x)_i
__device__ inline cplx row_eop(const Tabs &t, int n, int we, const cplx *x, int m, int i) {
  cplx acc = {0.0, 0.0};
  const int base = m * we * n;
  for (int s = 0; s < we; ++s)
    acc = cfma(ld_c(t.Eval, base + s * n + i), x[ld_i(t.Ecol, base + s * n + i)], acc);
  return acc;
}

constexpr int kMaxNC = lme::kMcMaxNC;

// Largest workgroup of the kernel with R rows per thread.
constexpr int mc_max_threads(int) { return 512; }

template <int R>
__global__ __launch_bounds__(mc_max_threads(R)) void mc_kernel(McArgs a) {
  extern __shared__ double lds[];
  const int G = a.G, P = a.P, n = a.n;
  const int nwaves = (blockDim.x + 63) >> 6;
  double *red = lds;                                     // [nwaves][9] wave partials
  double *wts = lds + nwaves * 9;                        // [P][kMaxNC] jump weights
  cplx *V = reinterpret_cast<cplx *>(lds + ((nwaves * 9 + P * kMaxNC + 1) & ~1));
  const int p = threadIdx.x / G;                         // trajectory slot
  const int g0 = threadIdx.x % G;
  cplx *X = V + (size_t)p * n;                           // this group's Taylor vector
  cplx *PS = V + (size_t)(P + p) * n;                    // this group's state psi
  const bool in_group = p < P;
  const cplx *psi0 = reinterpret_cast<const cplx *>(a.psi0);
  cplx *ex = reinterpret_cast<cplx *>(a.ex_traj);
  const int n_packs = (a.n_traj + P - 1) / P;
  const int64_t dstride = 2LL * (a.max_jumps + 1);
  Tabs tb;
  tb.D = rsrc(a.D, 16LL * n);
  tb.Oval = rsrc(a.Oval, 16LL * a.wo * n);
  tb.Ocol = rsrc(a.Ocol, 4LL * a.wo * n);
  tb.Jval = rsrc(a.Jval, 16LL * a.nc * a.wc * n);
  tb.Jcol = rsrc(a.Jcol, 4LL * a.nc * a.wc * n);
  tb.Eval = rsrc(a.Eval, 16LL * a.ne * a.we * n);
  tb.Ecol = rsrc(a.Ecol, 4LL * a.ne * a.we * n);
  tb.vb = rsrc(a.vbuf + (size_t)blockIdx.x * 8 * P * n, 64LL * P * n);

  for (int pack = blockIdx.x; pack < n_packs; pack += gridDim.x) {
    // g is re-read here, in every sub-step, output and jump (opaque copies),
    // so the row indices and offsets derived from it are recomputed where
    // they are used instead of being hoisted out of the loops and spilled
    int g = launder(g0);
    const int traj = pack * P + p;
    const bool alive0 = in_group && traj < a.n_traj;
    // the initial ket, normalised, into PS (each thread its own rows)
    double nn[1] = {0.0};
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int i = g + q * G;
      if (alive0 && i < n) nn[0] += cabs2(psi0[i]);
    }
    group_sum<1>(nn, G, red);
    const double sc = nn[0] > 0.0 ? 1.0 / sqrt(nn[0]) : 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int i = g + q * G;
      if (in_group && i < n) PS[i] = alive0 ? cscale(sc, psi0[i]) : cplx{0.0, 0.0};
    }
    // outputs of a trajectory that stops early stay zero
    if (alive0)
      for (int e = g; e < a.ne * a.n_t; e += G) ex[(size_t)traj * a.ne * a.n_t + e] = {0.0, 0.0};
    int status = (alive0 && !(nn[0] > 0.0 && isfinite(nn[0]))) ? LME_EINVAL : LME_OK;
    bool alive = alive0 && status == LME_OK;
    int jumps = 0;
    const double *dr = a.draws + (alive0 ? traj * dstride : 0);
    double r = alive ? dr[0] : 0.0;
    int next_out = 0;

    // <psi|E_m|psi> / <psi|psi> of every trajectory at output k (operators
    // reduced two at a time)
    auto record = [&](int k) {
      g = launder(g0);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int i = g + q * G;
        if (in_group && i < n) X[i] = PS[i];
      }
      __syncthreads();
      for (int m0 = 0; m0 < a.ne; m0 += 2) {
        double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = g + q * G;
          if (in_group && i < n) {
            const cplx ps = X[i];
#pragma unroll
            for (int d = 0; d < 2; ++d)
              if (m0 + d < a.ne) {
                const cplx e = row_eop(tb, n, a.we, X, m0 + d, i);
                // conj(psi_i) * (E psi)_i
                v[2 * d] += ps.x * e.x + ps.y * e.y;
                v[2 * d + 1] += ps.x * e.y - ps.y * e.x;
              }
            v[4] += cabs2(ps);
          }
        }
        group_sum<5>(v, G, red);
        if (alive && g == 0)
#pragma unroll
          for (int d = 0; d < 2; ++d)
            if (m0 + d < a.ne)
              ex[((size_t)traj * a.ne + m0 + d) * a.n_t + k] = {v[2 * d] / v[4], v[2 * d + 1] / v[4]};
      }
    };

    for (int st = 0; st <= a.nsteps; ++st) {
      // outputs due at grid point st (output 0 at the initial time)
      while (next_out < a.n_t && (next_out == 0 || a.out_step[next_out] == st)) record(next_out++);
      if (st == a.nsteps) break;
      double t = a.t0 + (double)st * a.h;   // time of the current state
      double left = alive ? a.h : 0.0;      // rest of this grid step
      for (;;) {
        if (!__syncthreads_or(left > 0.0)) break;
        g = launder(g0);
        const double s = left;
        cplx acc[R];
        // Taylor form of the RK4 step of length s: acc = sum_k s^k v_k
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = g + q * G;
          acc[q] = (in_group && i < n) ? PS[i] : cplx{0.0, 0.0};
          if (in_group && i < n) X[i] = acc[q];
        }
        double sk = 1.0;
        for (int k = 1; k <= 4; ++k) {
          __syncthreads();
          cplx y[R];
          const double inv = 1.0 / (double)k;
          sk *= s;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int i = g + q * G;
            y[q] = (in_group && i < n) ? cscale(inv, row_apply(tb, n, a.wo, X, i)) : cplx{0.0, 0.0};
            acc[q] = caxpy(sk, y[q], acc[q]);
          }
          if (k < 4) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < R; ++q) {
              const int i = g + q * G;
              if (in_group && i < n) X[i] = y[q];
            }
          }
        }
        double nt[1] = {0.0};
#pragma unroll
        for (int q = 0; q < R; ++q) nt[0] += cabs2(acc[q]);
        group_sum<1>(nt, G, red);
        bool cross = false;
        if (left > 0.0) {
          if (!isfinite(nt[0])) {
            status = LME_ENONFINITE;
            alive = false;
            left = 0.0;
          } else if (nt[0] > r) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
              const int i = g + q * G;
              if (in_group && i < n) PS[i] = acc[q];
            }
            left = 0.0;
          } else {
            cross = true;
          }
        }
        if (!__syncthreads_or(cross)) continue;
        g = launder(g0);

        // ---- a jump inside this sub-step for at least one trajectory ----
        // recompute v1..v4 from psi (unchanged for the crossing ones), keep
        // them in this workgroup's slice of the scratch buffer
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = g + q * G;
          if (in_group && i < n) X[i] = PS[i];
        }
        for (int k = 1; k <= 4; ++k) {
          __syncthreads();
          cplx y[R];
          const double inv = 1.0 / (double)k;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int i = g + q * G;
            y[q] = (in_group && i < n) ? cscale(inv, row_apply(tb, n, a.wo, X, i)) : cplx{0.0, 0.0};
            if (in_group && i < n) st_c(tb.vb, ((k - 1) * P + p) * n + i, y[q]);
          }
          __syncthreads();
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int i = g + q * G;
            if (in_group && i < n) X[i] = y[q];
          }
        }
        // coefficients of |psi(x)|^2 = sum_d c_d x^d
        double c[9];
#pragma unroll
        for (int d = 0; d < 9; ++d) c[d] = 0.0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = g + q * G;
          if (in_group && i < n) {
            cplx v[5];
            v[0] = PS[i];
#pragma unroll
            for (int k = 1; k <= 4; ++k) v[k] = ld_c(tb.vb, ((k - 1) * P + p) * n + i);
#pragma unroll
            for (int j = 0; j <= 4; ++j) {
              c[2 * j] += cabs2(v[j]);
#pragma unroll
              for (int k = j + 1; k <= 4; ++k)
                c[j + k] += 2.0 * (v[j].x * v[k].x + v[j].y * v[k].y);
            }
          }
        }
        group_sum<9>(c, G, red);
        double tau = 0.0;
        if (cross) {
          // bisection on (0, left]: the norm is above r at 0, at most r at left
          double lo = 0.0, hi = left;
          for (int it = 0; it < 400; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (!(mid > lo && mid < hi)) break;
            double pv = c[8];
            for (int d = 7; d >= 0; --d) pv = fma(pv, mid, c[d]);
            if (pv <= r)
              hi = mid;
            else
              lo = mid;
          }
          tau = hi;
        }
        __syncthreads();
        // psi(tau) by Horner into X (crossing trajectories)
        if (cross)
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int i = g + q * G;
            if (in_group && i < n) {
              cplx h4 = ld_c(tb.vb, (3 * P + p) * n + i);
              for (int k = 3; k >= 1; --k) {
                const cplx vk = ld_c(tb.vb, ((k - 1) * P + p) * n + i);
                h4 = {fma(h4.x, tau, vk.x), fma(h4.y, tau, vk.y)};
              }
              const cplx v0 = PS[i];
              X[i] = {fma(h4.x, tau, v0.x), fma(h4.y, tau, v0.y)};
            }
          }
        __syncthreads();
        // jump weights <psi|C_k^+ C_k|psi> at tau, four operators at a time,
        // into this trajectory's slots of wts
        for (int k0 = 0; k0 < a.nc; k0 += 4) {
          double w4[4] = {0.0, 0.0, 0.0, 0.0};
          if (cross)
#pragma unroll
            for (int q = 0; q < R; ++q) {
              const int i = g + q * G;
              if (in_group && i < n)
#pragma unroll
                for (int d = 0; d < 4; ++d)
                  if (k0 + d < a.nc) w4[d] += cabs2(row_jump(tb, n, a.wc, X, k0 + d, i));
            }
          group_sum<4>(w4, G, red);
          if (g == 0)
#pragma unroll
            for (int d = 0; d < 4; ++d)
              if (k0 + d < a.nc) wts[p * kMaxNC + k0 + d] = w4[d];
        }
        __syncthreads();
        if (cross) {
          if (jumps >= a.max_jumps) {
            status = LME_EDRAWS;
            alive = false;
            left = 0.0;
          } else {
            const double r2 = dr[2 * jumps + 1];
            const double *w = wts + p * kMaxNC;
            double total = 0.0;
            for (int k = 0; k < a.nc; ++k) total += w[k];
            if (!(total > 0.0) || !isfinite(total)) {
              status = LME_ENONFINITE;
              alive = false;
              left = 0.0;
            } else {
              int chosen = -1, last_nonzero = -1;
              double cum = 0.0, w_chosen = 0.0, w_last = 0.0;
              for (int k = 0; k < a.nc; ++k)
                if (chosen < 0) {
                  if (w[k] > 0.0) {
                    last_nonzero = k;
                    w_last = w[k];
                  }
                  cum += w[k] / total;
                  if (cum >= r2 && w[k] > 0.0) {
                    chosen = k;
                    w_chosen = w[k];
                  }
                }
              if (chosen < 0) {
                chosen = last_nonzero;
                w_chosen = w_last;
              }
              // the projected, renormalised state (Eq. (project)) into PS
              const double rs = 1.0 / sqrt(w_chosen);
#pragma unroll
              for (int q = 0; q < R; ++q) {
                const int i = g + q * G;
                if (in_group && i < n) PS[i] = cscale(rs, row_jump(tb, n, a.wc, X, chosen, i));
              }
              t += tau;
              if (g == 0) {
                if (a.jump_t) a.jump_t[(size_t)traj * a.max_jumps + jumps] = t;
                if (a.jump_op) a.jump_op[(size_t)traj * a.max_jumps + jumps] = chosen;
              }
              ++jumps;
              r = dr[2 * jumps];
              left -= tau;
            }
          }
        }
      }
    }
    if (alive0 && g == 0) {
      if (a.n_jumps) a.n_jumps[traj] = jumps;
      if (a.status) a.status[traj] = status;
    }
    __syncthreads();   // PS and X are reused by the next pack
  }
}

__device__ inline Tabs mc_tabs(const McArgs &a) {
  const int64_t n = a.n;
  Tabs t;
  t.D = rsrc(a.D, 16LL * n);
  t.Oval = rsrc(a.Oval, 16LL * a.wo * n);
  t.Ocol = rsrc(a.Ocol, 4LL * a.wo * n);
  t.Jval = rsrc(a.Jval, 16LL * a.nc * a.wc * n);
  t.Jcol = rsrc(a.Jcol, 4LL * a.nc * a.wc * n);
  t.Eval = rsrc(a.Eval, 16LL * a.ne * a.we * n);
  t.Ecol = rsrc(a.Ecol, 4LL * a.ne * a.we * n);
  t.vb = rsrc(a.vbuf + (size_t)blockIdx.x * 8 * a.P * n, 64LL * a.P * n);
  return t;
}

// <psi|E_m|psi> / <psi|psi> of every trajectory of the workgroup at output k,
// psi staged in X (four operators a pass); traj < 0: nothing is written.
__device__ __forceinline__ void mc_record(const McArgs &a, const cplx *X, double *red, int g,
                                          int traj, int k) {
  const Tabs tb = mc_tabs(a);
  const int n = a.n, G = a.G;
  cplx *ex = reinterpret_cast<cplx *>(a.ex_traj);
  for (int m0 = 0; m0 < a.ne; m0 += 4) {
    double v[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int i = g; i < n; i += G) {
      const cplx ps = X[i];
      v[8] += cabs2(ps);
      // conj(psi_i) * (E psi)_i, the operators' entries loaded together
      for (int s = 0; s < a.we; ++s) {
        cplx ev[4];
        int ec[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int at = (min(m0 + d, a.ne - 1) * a.we + s) * n + i;
          ev[d] = ld_c(tb.Eval, at);
          ec[d] = ld_i(tb.Ecol, at);
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const cplx e = cmul(ev[d], X[ec[d]]);
          v[2 * d] += ps.x * e.x + ps.y * e.y;
          v[2 * d + 1] += ps.x * e.y - ps.y * e.x;
        }
      }
    }
    group_sum<9>(v, G, red);
    if (traj >= 0 && g == 0)
#pragma unroll
      for (int d = 0; d < 4; ++d)
        if (m0 + d < a.ne)
          ex[((size_t)traj * a.ne + m0 + d) * a.n_t + k] = {v[2 * d] / v[8], v[2 * d + 1] / v[8]};
  }
}

struct JumpState {
  double r, left, t;   // threshold, rest of the grid step, time
  int jumps, status;
};

// The jump of every crossing trajectory of the workgroup inside the sub-step
// of length st.left that begins at PS (its own rows written by each thread);
// the state after the jump goes back to PS.  X: work vector, as PS in LDS.
// Every thread of the workgroup calls it.
__device__ __forceinline__ JumpState mc_jump(const McArgs &a, cplx *X, cplx *PS, double *red,
                                             double *wts, int p, int g, int traj, bool cross,
                                             JumpState st) {
  const Tabs tb = mc_tabs(a);
  const int n = a.n, G = a.G, P = a.P;
  const int lim = p < P ? n : 0;
  // the Taylor vectors v_k = A v_{k-1} / k of psi, kept in this workgroup's
  // slice of the scratch buffer
  for (int i = g; i < lim; i += G) X[i] = PS[i];
  for (int k = 1; k <= 4; ++k) {
    __syncthreads();
    const double inv = 1.0 / (double)k;
    for (int i = g; i < lim; i += G)
      st_c(tb.vb, ((k - 1) * P + p) * n + i, cscale(inv, row_apply(tb, n, a.wo, X, i)));
    __syncthreads();
    if (k < 4)
      for (int i = g; i < lim; i += G) X[i] = ld_c(tb.vb, ((k - 1) * P + p) * n + i);
  }
  // coefficients of |psi(x)|^2 = sum_d c_d x^d
  double c[9];
#pragma unroll
  for (int d = 0; d < 9; ++d) c[d] = 0.0;
  for (int i = g; i < lim; i += G) {
    cplx v[5];
    v[0] = PS[i];
#pragma unroll
    for (int k = 1; k <= 4; ++k) v[k] = ld_c(tb.vb, ((k - 1) * P + p) * n + i);
#pragma unroll
    for (int j = 0; j <= 4; ++j) {
      c[2 * j] += cabs2(v[j]);
#pragma unroll
      for (int k = j + 1; k <= 4; ++k) c[j + k] += 2.0 * (v[j].x * v[k].x + v[j].y * v[k].y);
    }
  }
  group_sum<9>(c, G, red);
  double tau = 0.0;
  if (cross) {
    // bisection on (0, left]: the norm is above r at 0, at most r at left
    double lo = 0.0, hi = st.left;
    for (int it = 0; it < 400; ++it) {
      const double mid = 0.5 * (lo + hi);
      if (!(mid > lo && mid < hi)) break;
      double pv = c[8];
#pragma unroll
      for (int d = 7; d >= 0; --d) pv = fma(pv, mid, c[d]);
      if (pv <= st.r)
        hi = mid;
      else
        lo = mid;
    }
    tau = hi;
    // psi(tau) by Horner into X
    for (int i = g; i < lim; i += G) {
      cplx h4 = ld_c(tb.vb, (3 * P + p) * n + i);
#pragma unroll
      for (int k = 3; k >= 1; --k) {
        const cplx vk = ld_c(tb.vb, ((k - 1) * P + p) * n + i);
        h4 = {fma(h4.x, tau, vk.x), fma(h4.y, tau, vk.y)};
      }
      const cplx v0 = PS[i];
      X[i] = {fma(h4.x, tau, v0.x), fma(h4.y, tau, v0.y)};
    }
  }
  __syncthreads();
  // jump weights <psi|C_k^+ C_k|psi> at tau, four operators at a time, into
  // this trajectory's slots of wts
  for (int k0 = 0; k0 < a.nc; k0 += 4) {
    double w4[4] = {0.0, 0.0, 0.0, 0.0};
    if (cross)
      for (int i = g; i < lim; i += G)
#pragma unroll
        for (int d = 0; d < 4; ++d)
          if (k0 + d < a.nc) w4[d] += cabs2(row_jump(tb, n, a.wc, X, k0 + d, i));
    group_sum<4>(w4, G, red);
    if (p < P && g == 0)
#pragma unroll
      for (int d = 0; d < 4; ++d)
        if (k0 + d < a.nc) wts[p * kMaxNC + k0 + d] = w4[d];
  }
  __syncthreads();
  if (!cross) return st;
  if (st.jumps >= a.max_jumps) {
    st.status = LME_EDRAWS;
    st.left = 0.0;
    return st;
  }
  const double *dr = a.draws + 2LL * (a.max_jumps + 1) * traj;
  const double r2 = dr[2 * st.jumps + 1];
  const double *w = wts + p * kMaxNC;
  double total = 0.0;
  for (int k = 0; k < a.nc; ++k) total += w[k];
  if (!(total > 0.0) || !isfinite(total)) {
    st.status = LME_ENONFINITE;
    st.left = 0.0;
    return st;
  }
  int chosen = -1, last_nonzero = -1;
  double cum = 0.0, w_chosen = 0.0, w_last = 0.0;
  for (int k = 0; k < a.nc; ++k)
    if (chosen < 0) {
      if (w[k] > 0.0) {
        last_nonzero = k;
        w_last = w[k];
      }
      cum += w[k] / total;
      if (cum >= r2 && w[k] > 0.0) {
        chosen = k;
        w_chosen = w[k];
      }
    }
  if (chosen < 0) {
    chosen = last_nonzero;
    w_chosen = w_last;
  }
  // the projected, renormalised state (Eq. (project)) into PS
  const double rs = 1.0 / sqrt(w_chosen);
  for (int i = g; i < lim; i += G) PS[i] = cscale(rs, row_jump(tb, n, a.wc, X, chosen, i));
  st.t += tau;
  if (g == 0) {
    if (a.jump_t) a.jump_t[(size_t)traj * a.max_jumps + st.jumps] = st.t;
    if (a.jump_op) a.jump_op[(size_t)traj * a.max_jumps + st.jumps] = chosen;
  }
  ++st.jumps;
  st.r = dr[2 * st.jumps];
  st.left -= tau;
  return st;
}

// ---------------------------------------------------------------------------
// The same trajectories with A in registers: systems whose A has at most two
// off-diagonal entries a row, all of them real or all imaginary (a real or
// an imaginary Hamiltonian with diagonal C^+C; AS below).  mc_kernel reads 56
// bytes of operator tables per row and product through the caches, 275 KB a
// stage at n = 4913, which bounds it; here a thread loads its rows' entries
// once between two outputs or jumps (7 to 9 registers a row) and a product
// costs only its LDS gathers and one store.  The RK4 step is evaluated by Horner's rule,
//   psi(s) = psi + s A (psi + s/2 A (psi + s/3 A (psi + s/4 A psi))),
// so a row keeps psi and the current vector (8 registers) and no running
// sum.  Seven rows fit the 256 registers of a 512-thread workgroup; from eight
// on some spill (ten rows of two real entries: 56, about twenty reloads a step;
// of two imaginary ones or under a complex diagonal: 86).  Five rows in 1024
// threads of 128 registers spill more: 58.2 ms for the figures below.  psi
// being in registers, the LDS that held it is the second buffer of the
// current vector: one barrier per product.  The norm of the new psi costs
// none of its own: its wave partials are published by the barrier that also
// publishes the new psi for the next step's first product, and psi is
// replaced only after the sum has been looked at.
// n = 4913, 1000 trajectories x 1000 steps, 201 outputs: 37.4 ms against
// 98.9 ms; a step takes 6.4 us (4 products of 3 LDS accesses a row, 3.2 us of
// the LDS pipe at 128 bytes a cycle; two wavefronts a SIMD leave part of the
// gathers' latency and the five barriers uncovered), an output 12 us, of
// which 5 us load the entries again.
// ---------------------------------------------------------------------------
// structure of A: all real; imaginary off-diagonal; real off-diagonal with a
// complex diagonal
enum { kAReal = 0, kAOffImag = 1, kAOffReal = 2 };
constexpr int kRegThreads = 512;   // largest workgroup: 256 registers a thread

template <int R, int WO, int AS>
__global__ __launch_bounds__(kRegThreads) void mc_reg_kernel(McArgs a) {
  extern __shared__ __align__(16) double lds[];
  constexpr bool OIM = AS == kAOffImag, DRE = AS == kAReal;
  const int G = a.G, P = a.P, n = a.n;
  const int nwaves = (blockDim.x + 63) >> 6;
  double *red = lds;                                     // [nwaves][9] wave partials
  double *wts = lds + nwaves * 9;                        // [P][kMaxNC] jump weights
  cplx *V = reinterpret_cast<cplx *>(lds + ((nwaves * 9 + P * kMaxNC + 1) & ~1));
  const int p = threadIdx.x / G;                         // trajectory slot (the launch has P G threads)
  const int g0 = threadIdx.x % G;
  cplx *X = V + (size_t)p * n;                           // this group's vector, buffer 0
  const int flip = P * n;                                // distance of buffer 1
  const cplx *psi0 = reinterpret_cast<const cplx *>(a.psi0);
  cplx *ex = reinterpret_cast<cplx *>(a.ex_traj);
  const int n_packs = (a.n_traj + P - 1) / P;
  const int64_t dstride = 2LL * (a.max_jumps + 1);

  // This thread's rows are g0 + q G.  Only the last slot can lie past the last
  // row ((R - 1) G < n: the launch rule): it is row n - 1 once more, computes
  // and stores that row's value again, so the step has no branches, and is
  // left out of the norm.
  const bool last_own = g0 + (R - 1) * G < n;
  const int last_row = last_own ? g0 + (R - 1) * G : n - 1;
  auto row = [&](int g, int q) { return q == R - 1 ? last_row : g + q * G; };
  // a condition any group of the workgroup meets (one group: it is the same
  // in every thread); not a barrier
  auto any = [&](bool c) { return P == 1 ? c : (bool)__syncthreads_or(c); };

  for (int pack = blockIdx.x; pack < n_packs; pack += gridDim.x) {
    const int traj = pack * P + p;
    const bool alive0 = traj < a.n_traj;
    // the initial ket, normalised, into buffer 1
    double nn[1] = {0.0};
    for (int i = g0; i < n; i += G)
      if (alive0) nn[0] += cabs2(psi0[i]);
    group_sum<1>(nn, G, red);
    const double sc = nn[0] > 0.0 ? 1.0 / sqrt(nn[0]) : 0.0;
    for (int i = g0; i < n; i += G)
      X[flip + i] = alive0 ? cscale(sc, psi0[i]) : cplx{0.0, 0.0};
    // outputs of a trajectory that stops early stay zero
    if (alive0)
      for (int e = g0; e < a.ne * a.n_t; e += G) ex[(size_t)traj * a.ne * a.n_t + e] = {0.0, 0.0};
    int status = (alive0 && !(nn[0] > 0.0 && isfinite(nn[0]))) ? LME_EINVAL : LME_OK;
    bool alive = alive0 && status == LME_OK;
    int jumps = 0;
    const double *dr = a.draws + (alive0 ? traj * dstride : 0);
    double r = alive ? dr[0] : 0.0;
    int next_out = 0, st = 0;             // st: grid steps done
    double t = a.t0;                      // time of the current state
    double left = alive ? a.h : 0.0;      // rest of this grid step

    // Between two outputs or jumps the operator entries and psi are in
    // registers; an output or a jump takes psi from buffer 1 (each thread its
    // own rows) and leaves it there, and the entries are loaded again after
    // it: alive across that code as well they would not fit.
    for (;;) {
      while (next_out < a.n_t && (next_out == 0 || a.out_step[next_out] == st)) {
        __syncthreads();
        mc_record(a, X + flip, red, g0, alive ? traj : -1, next_out++);
      }
      if (st == a.nsteps) break;
      const int due = next_out < a.n_t ? a.out_step[next_out] : a.nsteps;

      double d[R][DRE ? 1 : 2], o[R][WO];
      uint32_t col[R];
      cplx psi[R], x[R];
      int g = launder(g0);
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int i = row(g, q);
        d[q][0] = a.D[2 * i];
        if (!DRE) d[q][DRE ? 0 : 1] = a.D[2 * i + 1];
        col[q] = 0;
#pragma unroll
        for (int w = 0; w < WO; ++w) {
          o[q][w] = 0.0;
          if (w < a.wo) {
            o[q][w] = a.Oval[2 * ((size_t)w * n + i) + (OIM ? 1 : 0)];
            col[q] |= (uint32_t)a.Ocol[(size_t)w * n + i] << (16 * w);
          }
        }
        psi[q] = X[flip + i];
        X[i] = psi[q];
      }
      __syncthreads();
      // (A x)_i of row slot q; own = x_i, xs = the group's vector
      auto apply = [&](int q, cplx own, const cplx *xs) {
        uint32_t c = col[q];
        asm volatile("" : "+v"(c));   // no unpacked address kept across the steps
        cplx y = DRE ? cscale(d[q][0], own) : cmul(cplx{d[q][0], d[q][DRE ? 0 : 1]}, own);
#pragma unroll
        for (int w = 0; w < WO; ++w) {
          const cplx v = xs[w == 0 ? (c & 0xffffu) : (c >> 16)];
          y = OIM ? cplx{fma(-o[q][w], v.y, y.x), fma(o[q][w], v.x, y.y)}
                  : cplx{fma(o[q][w], v.x, y.x), fma(o[q][w], v.y, y.y)};
        }
        return y;
      };

      bool cross = false, jump = false;
      for (;;) {
#pragma unroll
        for (int q = 0; q < R; ++q) x[q] = psi[q];
        // four products, buffer 0 -> 1 -> 0 -> 1 -> 0: the last leaves the
        // new psi in buffer 0, its readers done since the barrier before
#pragma unroll
        for (int k = 4; k >= 1; --k) {
          const cplx *xs = (k & 1) ? X + flip : X;
          cplx *xd = (k & 1) ? X : X + flip;
          const double sk = left / (double)k;
          const int gk = launder(g0);
#pragma unroll
          for (int q = 0; q < R; ++q) {
            x[q] = caxpy(sk, apply(q, x[q], xs), psi[q]);
            xd[row(gk, q)] = x[q];
            // two rows' gathers in flight at a time
            if (q & 1) __builtin_amdgcn_sched_barrier(0);
          }
          if (k > 1) __syncthreads();
        }
        double nt[1] = {0.0};
#pragma unroll
        for (int q = 0; q < R; ++q) nt[0] += q < R - 1 || last_own ? cabs2(x[q]) : 0.0;
        if (G >= 64) {
          wave_partial(nt[0], red);
          __syncthreads();
          nt[0] = sum_partials(G, red);
        } else {
          group_sum<1>(nt, G, red);
          __syncthreads();
        }
        if (left > 0.0) {
          if (!isfinite(nt[0])) {
            status = LME_ENONFINITE;
            alive = false;
            left = 0.0;
          } else if (nt[0] > r) {
#pragma unroll
            for (int q = 0; q < R; ++q) psi[q] = x[q];
            left = 0.0;
          } else {
            cross = true;
          }
        }
        jump = any(cross);
        if (jump) break;
        // no trajectory of the workgroup has a rest left: the next grid step
        ++st;
        t = a.t0 + (double)st * a.h;
        left = alive ? a.h : 0.0;
        if (st == due || !any(alive)) break;
      }
      // psi into buffer 1, last read by the fourth product
#pragma unroll
      for (int q = 0; q < R; ++q) X[flip + row(g, q)] = psi[q];
      if (jump) {
        const JumpState js = mc_jump(a, X, X + flip, red, wts, p, g0, traj, cross,
                                     JumpState{r, left, t, jumps, status});
        if (cross) {
          r = js.r;
          left = js.left;
          t = js.t;
          jumps = js.jumps;
          status = js.status;
          alive = status == LME_OK;
        }
        __syncthreads();
        // every rest done (a draw that ran out, a norm that vanished): on to
        // the next grid step
        if (!any(left > 0.0)) {
          ++st;
          t = a.t0 + (double)st * a.h;
          left = alive ? a.h : 0.0;
        }
      } else if (st != due) {   // no trajectory is alive any more
        st = due;
        t = a.t0 + (double)st * a.h;
      }
    }
    if (alive0 && g0 == 0) {
      if (a.n_jumps) a.n_jumps[traj] = jumps;
      if (a.status) a.status[traj] = status;
    }
    __syncthreads();   // the buffers are reused by the next pack
  }
}

// expect[m][k] = (sum over trajectories, in order, of ex_traj[b][m][k]) / n_traj
__global__ void mc_average_kernel(const double *ex_traj, double *expect, int n_traj, int per) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= per) return;
  double sx = 0.0, sy = 0.0;
#pragma unroll 8
  for (int b = 0; b < n_traj; ++b) {
    sx += ex_traj[2 * ((size_t)b * per + e)];
    sy += ex_traj[2 * ((size_t)b * per + e) + 1];
  }
  expect[2 * e] = sx / (double)n_traj;
  expect[2 * e + 1] = sy / (double)n_traj;
}

template <int R>
hipError_t launch_r(const McArgs *a, int grid, int lds, hipStream_t s) {
  auto k = mc_kernel<R>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(grid), dim3(a->P * a->G), lds, s, *a);
  return hipGetLastError();
}

template <int R, int WO, int AS>
hipError_t launch_reg(const McArgs *a, int grid, int lds, hipStream_t s) {
  auto k = mc_reg_kernel<R, WO, AS>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(grid), dim3(a->P * a->G), lds, s, *a);
  return hipGetLastError();
}

template <int R, int AS>
hipError_t launch_reg_w(const McArgs *a, int grid, int lds, hipStream_t s) {
  return a->wo <= 1 ? launch_reg<R, 1, AS>(a, grid, lds, s) : launch_reg<R, 2, AS>(a, grid, lds, s);
}

template <int R>
hipError_t launch_reg_r(int as, const McArgs *a, int grid, int lds, hipStream_t s) {
  switch (as) {
    case kAReal: return launch_reg_w<R, kAReal>(a, grid, lds, s);
    case kAOffImag: return launch_reg_w<R, kAOffImag>(a, grid, lds, s);
    case kAOffReal: return launch_reg_w<R, kAOffReal>(a, grid, lds, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Rows per thread and largest workgroup of the kernel with A in registers.
extern "C" int lme_internal_mc_reg_rows() { return 10; }
extern "C" int lme_internal_mc_reg_threads() { return kRegThreads; }

// wo <= 2, structure of A `as` (0 all real, 1 imaginary off-diagonal, 2 real
// off-diagonal), P * G <= lme_internal_mc_reg_threads(), (R - 1) G < n <= R G.
extern "C" hipError_t lme_internal_launch_mc_reg(int R, int as, const McArgs *a, int grid,
                                                 int lds, hipStream_t s) {
  if (a->wo > 2 || R * a->G < a->n || (R - 1) * a->G >= a->n || a->P * a->G > lme_internal_mc_reg_threads())
    return hipErrorInvalidValue;
  switch (R) {
    case 1: return launch_reg_r<1>(as, a, grid, lds, s);
    case 2: return launch_reg_r<2>(as, a, grid, lds, s);
    case 3: return launch_reg_r<3>(as, a, grid, lds, s);
    case 4: return launch_reg_r<4>(as, a, grid, lds, s);
    case 5: return launch_reg_r<5>(as, a, grid, lds, s);
    case 6: return launch_reg_r<6>(as, a, grid, lds, s);
    case 7: return launch_reg_r<7>(as, a, grid, lds, s);
    case 8: return launch_reg_r<8>(as, a, grid, lds, s);
    case 9: return launch_reg_r<9>(as, a, grid, lds, s);
    case 10: return launch_reg_r<10>(as, a, grid, lds, s);
    default: return hipErrorInvalidValue;
  }
}

// Rows per thread the Monte-Carlo kernel is compiled for (ascending) and the
// largest workgroup of each.
extern "C" int lme_internal_mc_rows(int *rows, int *max_threads, int cap) {
  static const int kR[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
  const int nr = (int)(sizeof kR / sizeof kR[0]);
  for (int i = 0; i < nr && i < cap; ++i) {
    rows[i] = kR[i];
    max_threads[i] = mc_max_threads(kR[i]);
  }
  return nr;
}

// Dynamic LDS of a workgroup of T threads holding P vectors of dimension n.
extern "C" int lme_internal_mc_lds_bytes(int T, int P, int n) {
  const int nwaves = (T + 63) / 64;
  return 8 * ((nwaves * 9 + P * kMaxNC + 1) & ~1) + 32 * P * n;   // + X and psi
}

extern "C" hipError_t lme_internal_launch_mc(int R, const McArgs *a, int grid, int lds,
                                             hipStream_t s) {
  switch (R) {
    case 1: return launch_r<1>(a, grid, lds, s);
    case 2: return launch_r<2>(a, grid, lds, s);
    case 3: return launch_r<3>(a, grid, lds, s);
    case 4: return launch_r<4>(a, grid, lds, s);
    case 5: return launch_r<5>(a, grid, lds, s);
    case 6: return launch_r<6>(a, grid, lds, s);
    case 8: return launch_r<8>(a, grid, lds, s);
    case 10: return launch_r<10>(a, grid, lds, s);
    case 12: return launch_r<12>(a, grid, lds, s);
    case 16: return launch_r<16>(a, grid, lds, s);
    default: return hipErrorInvalidValue;
  }
}

extern "C" hipError_t lme_internal_launch_mc_average(const double *ex_traj, double *expect,
                                                     int n_traj, int per, hipStream_t s) {
  const int T = 256;
  hipLaunchKernelGGL(mc_average_kernel, dim3((per + T - 1) / T), dim3(T), 0, s, ex_traj, expect,
                     n_traj, per);
  return hipGetLastError();
}

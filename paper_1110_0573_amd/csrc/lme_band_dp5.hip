// lme_band_dp5.hip -- resident Dormand-Prince 5(4) under banded operators
// (those of lme_band.hip), any state, along diagonals.
//
// One workgroup integrates one pack with per-instance step control, as
// dp5_resident_kernel, with its arithmetic in its order: the same steps and
// the same bits.  What differs is where things live:
//   * thread (g, j) owns consecutive diagonals of column j: elements (i, j),
//     i = j + d mod n.  Every operand lies at a fixed distance in LDS rows of
//     n columns (contiguous in the wavefront); the wrap from diagonal n - 1 to
//     0 concerns a thread's first and last diagonal only;
//   * row-side operator entries come from three LDS tables, 16 bytes each,
//     read at consecutive rows (the row kernel's blobs cost five reads and
//     their addresses);
//   * the stage derivatives stay in registers, four at a time: k5 takes k2's
//     place once the sixth stage's input is formed (nothing later weighs k2),
//     and after k6 the error's sum so far takes k3's; k1 stays for a rejected
//     step.  dp5_resident_kernel keeps all seven in memory: 1.2 MB read and
//     0.4 MB written a step at n = 60, about 25 thousand cycles of one CU's
//     share of the L2;
//   * two buffers of the stage input, one barrier a stage; an accepted state
//     is already in the buffer that its outputs are taken from;
//   * the controller's power function is called, not inlined: only the
//     wavefronts that take step decisions save registers around it.
// Bound by LDS reads (seven of 16 bytes an element and stage: 3640 cycles of a
// stage at n = 60, 9 us of a step) and the latency that two or three wavefronts
// a SIMD leave open, at n = 60 also by spilled registers (267 to 460 by operator
// shape in eight diagonals a thread, about 25 reloads a stage; the column form
// of 1024 threads 68 to 74).  One step of a driven Kerr system, dp5_resident_kernel's column
// form -> here: n = 15 11.0 -> 4.4 us, n = 31 15.0 -> 7.8, n = 45 27.2 -> 13.1,
// n = 60 38.5 -> 30.1.  Batches gain more, with three collapse operators as with
// two (30 attempts, 512 systems of n = 60: Kerr 4.60 -> 2.66 ms, thermal
// Jaynes-Cummings 4.52 -> 2.63; of n = 20 those 1.78 -> 0.77 in 60 attempts).
// At n = 60 a wavefront set aside for the decisions (448
// threads of 9 diagonals) takes 38.0 us; k1 partly in LDS changes nothing.
#include "lme_device.h"
#include "lme_internal.h"

namespace lme {

namespace {

// Dormand & Prince (1980): stage matrix and error weights b - bhat.  Read from
// memory where they are used (opaque offsets below): kept in registers over
// the step loop, the 25 numbers and the addresses derived from the thread's
// place spill.
__constant__ double kDpA[7][6] = {
    {0, 0, 0, 0, 0, 0},
    {1.0 / 5, 0, 0, 0, 0, 0},
    {3.0 / 40, 9.0 / 40, 0, 0, 0, 0},
    {44.0 / 45, -56.0 / 15, 32.0 / 9, 0, 0, 0},
    {19372.0 / 6561, -25360.0 / 2187, 64448.0 / 6561, -212.0 / 729, 0, 0},
    {9017.0 / 3168, -355.0 / 33, 46732.0 / 5247, 49.0 / 176, -5103.0 / 18656, 0},
    {35.0 / 384, 0, 500.0 / 1113, 125.0 / 192, -2187.0 / 6784, 11.0 / 84}};
__constant__ double kDpE[7] = {35.0 / 384 - 5179.0 / 57600, 0.0, 500.0 / 1113 - 7571.0 / 16695,
                          125.0 / 192 - 393.0 / 640, -2187.0 / 6784 - (-92097.0 / 339200),
                          11.0 / 84 - 187.0 / 2100, 0.0 - 1.0 / 40};

// Sum over each instance's n2 entries of buf (LDS doubles) -> out[b];
// waves take instances round-robin, lanes stride the entries, then a
// butterfly: the order of dp5_resident_kernel's sum.
__device__ __forceinline__ void per_instance_sum_waves(const double *buf, int m, int n2, double *out,
                                              int waves) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int b = wave; b < m; b += waves) {
    double v = 0.0;
#pragma unroll 8
    for (int e = lane; e < n2; e += 64) v += buf[b * n2 + e];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) out[b] = v;
  }
}

struct DpLds {
  uint8_t *buf;        // two buffers
  uint8_t *tab;        // row tables
  DpCtl *ctl;
  double *sums;        // [2 m]
  int32_t *flags;      // [0] active instances, [1] attempt with an output due
  int64_t *off;
  int32_t *ids;
};

__device__ __forceinline__ DpLds carve_dp(uint8_t *smem, int n, int m, int nc) {
  DpLds p;
  p.buf = smem;
  p.tab = smem + 2 * band_dp_buffer_bytes(n, m);
  uint8_t *q = p.tab + band_dp_tables(nc) * 32 * m * n;
  p.ctl = reinterpret_cast<DpCtl *>(q);
  q += align16(m * (int32_t)sizeof(DpCtl));
  p.sums = reinterpret_cast<double *>(q);
  p.flags = reinterpret_cast<int32_t *>(q + 16 * m);
  q += 16 * m + 16;
  p.off = reinterpret_cast<int64_t *>(q);
  p.ids = reinterpret_cast<int32_t *>(q + align16(8 * m));
  return p;
}

// Sets up the next attempt of an active instance (dp5_resident_kernel's step
// set-up); c.hs holds the next stop point.
__device__ void dp_next_attempt(DpCtl &c, const Dp5Args &a) {
  if (!c.active) return;
  if (c.n_acc + c.n_rej >= a.max_steps) {
    c.status = 3;  // LME_EMAXSTEPS
    c.active = 0;
  } else if (c.h < a.h_min) {
    c.status = 4;  // LME_ESTEPUNDERFLOW
    c.active = 0;
  } else {
    const double ts = c.hs;
    c.landing = c.h >= ts - c.t;
    c.h_try = c.landing ? ts - c.t : c.h;
  }
}

__device__ __attribute__((noinline)) double dp_pow(double x, double y) { return pow(x, y); }

// The starting step's length; c.hs and c.t hold the trial step and d1.
__device__ __forceinline__ void dp_start(DpCtl &c, const Dp5Args &a, double sum, int n2) {
  const double hs = c.hs, d1 = c.t;
  const double d2 = sqrt(sum / n2) / hs;
  const double dm = fmax(d1, d2);
  const double h1 = (dm <= 1e-15) ? fmax(1e-6, hs * 1e-3) : dp_pow(0.01 / dm, 0.2);
  c.h = fmin(100.0 * hs, h1);
  c.t = a.t0;
}

// The decision on an attempted step (dp5_resident_kernel's rules).
__device__ __forceinline__ void dp_decide(DpCtl &c, const Dp5Args &a, double sum, int n2,
                                          int attempt, int32_t *flags) {
  c.accept = 0;
  if (!c.active) return;
  const double err = sqrt(sum / n2);
  if (!isfinite(err)) {
    c.status = 5;  // LME_ENONFINITE
    c.active = 0;
  } else if (err <= 1.0) {
    c.accept = 1;
    ++c.n_acc;
    double fac = (err == 0.0) ? 10.0 : 0.9 * dp_pow(err, -0.2);
    fac = fmin(10.0, fmax(0.2, fac));
    if (c.prev_rej && fac > 1.0) fac = 1.0;
    c.prev_rej = 0;
    c.h = c.h_try * fac;
    if (c.landing) {
      c.t = c.hs;
      c.out_due = a.stop_out[c.stop];
      if (c.out_due >= 0) flags[1] = attempt;
      if (++c.stop == a.n_stops) c.active = 0;
      else c.hs = a.stops[c.stop];
    } else {
      c.t += c.h_try;
    }
  } else {
    ++c.n_rej;
    c.prev_rej = 1;
    c.h = c.h_try * fmax(0.2, 0.9 * dp_pow(err, -0.2));
  }
  dp_next_attempt(c, a);
  if (!c.active) atomicAdd(&flags[0], -1);
}

// Expectation values of the instances with an output due, rho in buffer 0.
__device__ void dp_band_outputs(const Dp5Args &a, int n, int m, const DpLds &L) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  for (int task = wave; task < m * a.n_e; task += waves) {
    const int b = task / a.n_e, e = task - b * a.n_e;
    const int k = L.ctl[b].out_due;
    if (k < 0) continue;
    const int id = L.ids[b];
    const InstDesc &d = a.inst[id];
    const int we = d.we;
    const int32_t *Ec = reinterpret_cast<const int32_t *>(a.eops + d.eops_off);
    const double2 *Ev = reinterpret_cast<const double2 *>(
        a.eops + d.eops_off + eops_val_offset(n, we, a.n_e));
    const double2 *Y = reinterpret_cast<const double2 *>(L.buf) + b * n * n;
    double2 part = make_double2(0.0, 0.0);
    for (int i = lane; i < n; i += 64)
      for (int w = 0; w < we; ++w) {
        const int idx = (e * we + w) * n + i;
        int q = Ec[idx] - i;
        q = q < 0 ? q + n : q;
        part = cfma(Ev[idx], Y[q * n + i], part);
      }
    part = wave_sum(part);
    if (lane == 0) {
      double *dst = a.expect + 2 * (((int64_t)id * a.n_e + e) * a.n_t + k);
      dst[0] = part.x;
      dst[1] = part.y;
    }
  }
}

}  // namespace

// One pack whose threads own at most EPT diagonals (EPT or EPT - 1 each).
template <int EPT, int NW, int NC>
__device__ __forceinline__ void dp5_band_pack(const Dp5Args &a, const PackDesc &pk, uint8_t *smem) {
  const int n = pk.n, n2 = n * n, m = pk.m, C = m * n, G = pk.G, n16 = 16 * n;
  const DpLds L = carve_dp(smem, n, m, NC);
  const int bufb = band_dp_buffer_bytes(n, m);
  const int tid = threadIdx.x, T = blockDim.x;
  const int64_t SE = a.state_elems;

  const bool active = tid < C * G;
  const int g = active ? tid / C : 0;
  const int c = active ? tid - g * C : 0;
  const int b = c / n, j = c - b * n;
  const int q0 = n / G, rem = n - q0 * G;
  const int d0 = g * q0 + min(g, rem);
  const int nown = !active ? 0 : g < rem ? q0 + 1 : q0;
  const uint32_t yb = (uint32_t)(16 * b * n2);
  auto wrap = [&](int x) { return x < 0 ? x + n : (x >= n ? x - n : x); };
  // byte address, in a buffer, of diagonal d (wrapped) of column cc
  auto at = [&](int d, int cc) { return yb + (uint32_t)(wrap(d) * n + wrap(cc)) * 16u; };
  const int dl = d0 + max(nown, 1) - 1;   // last diagonal

  // column-j entries
  const OpView op = make_view(a.ops + a.inst[L.ids[b]].ops_off,
                              blob_layout(n, pk.wo, pk.nb, pk.wb, pk.nc, pk.wc));
  const double2 dj = cconj(op.D[j]);
  double qr[NW], jv[NC];
  // right neighbours: diagonal d + dd, column j - dd, dd = 1 (w = 0) and -1 or,
  // with one per row, whichever the row has; linear in d but for the wrap
  int dd[NW];
  uint32_t aj[NC];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    qr[w] = 0.0;
    dd[w] = NW == 2 ? (w == 0 ? 1 : -1) : 0;
  }
  for (int w = 0; w < pk.wo; ++w) {
    const int cc = op.Ocol[w * n + j];
    if (cc == j) continue;   // ELL padding
    const double v = -op.Oval[w * n + j].y;
    if (NW == 1) {
      qr[0] = v;
      dd[0] = j - cc;
    } else {
      qr[cc < j ? 0 : NW - 1] = v;
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    jv[k] = op.Jval[k * n + j].x;
    aj[k] = at(d0, j + band_offset(a.band_off[k], n));
  }
  const uint32_t own = at(d0, j), aprev = at(d0 - 1, j), anext = at(dl + 1, j);
  uint32_t ar[NW], af[NW], al[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    af[w] = at(d0 + dd[w], j - dd[w]);
    al[w] = at(dl + dd[w], j - dd[w]);
    ar[w] = yb + (uint32_t)((d0 + dd[w]) * n + wrap(j - dd[w])) * 16u;
  }
  // row tables of the instance at row j + d0 (rows 0 .. 2 n - 1, the second
  // half repeating the first): D | (A_{i,i-1}, A_{i,i+1}) | J_0, J_1 | J_2
  const uint32_t tab = (uint32_t)(L.tab - smem) + 16u * (uint32_t)(b * 2 * n + j + d0);
  const uint32_t tstep = 32 * m * n;
  const int64_t goff = L.off[b];
  auto element = [&](int r) { return wrap(j + d0 + r) * n + j; };   // r < nown

  double2 rho[EPT], k1[EPT], k2[EPT], k3[EPT], k4[EPT];
  const double2 zero = make_double2(0.0, 0.0);
  const double2 *rho0 = reinterpret_cast<const double2 *>(a.rho0) + goff;
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    rho[r] = k1[r] = k2[r] = k3[r] = k4[r] = zero;
    if (r < nown) rho[r] = rho0[element(r)];
  }
  // element of slot r into the buffer at dst
  auto store = [&](uint32_t dst, int r, double2 v) __attribute__((always_inline)) {
    if (r < EPT - 1 ? active : r < nown)
      *reinterpret_cast<double2 *>(smem + dst + own + (uint32_t)(r * n16)) = v;
  };
  // f(r, y, (L y)) of the thread's diagonals, y in the buffer at src
  auto apply = [&](uint32_t src, auto &&f) __attribute__((always_inline)) {
    uint32_t so = src + own, sr[NW], sj[NC], to = tab;
    asm volatile("" : "+v"(so), "+v"(to));
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      sr[w] = src + ar[w];
      asm volatile("" : "+v"(sr[w]));
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      sj[k] = src + aj[k];
      asm volatile("" : "+v"(sj[k]));
    }
    auto Y = [&](uint32_t addr) { return *reinterpret_cast<const double2 *>(smem + addr); };
    double2 prev = Y(src + aprev), y = Y(so);
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const uint32_t o = (uint32_t)(r * n16);
      const bool end = r >= EPT - 2 && r == nown - 1;
      const double2 di = Y(to + 16 * r), oi = Y(to + tstep + 16 * r),
                    ji = Y(to + 2 * tstep + 16 * r);
      uint32_t an = so + o + n16;
      if (r >= EPT - 2) an = end ? src + anext : an;
      const double2 next = Y(an);
      double2 vr[NW], vj[NC];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        uint32_t x = r == 0 ? src + af[w] : sr[w] + o;
        if (r >= EPT - 2) x = end ? src + al[w] : x;
        vr[w] = Y(x);
      }
#pragma unroll
      for (int k = 0; k < NC; ++k) vj[k] = Y(sj[k] + o);
      double2 kv = cmul(cadd(di, dj), y);
      kv = make_double2(fma(-oi.x, prev.y, kv.x), fma(oi.x, prev.x, kv.y));
      kv = make_double2(fma(-oi.y, next.y, kv.x), fma(oi.y, next.x, kv.y));
#pragma unroll
      for (int w = 0; w < NW; ++w)
        kv = make_double2(fma(-qr[w], vr[w].y, kv.x), fma(qr[w], vr[w].x, kv.y));
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        double p;
        if (k < 2) p = (k == 0 ? ji.x : ji.y) * jv[k];
        else p = *reinterpret_cast<const double *>(smem + to + 3 * tstep + 16 * r) * jv[k];
        kv = make_double2(fma(p, vj[k].x, kv.x), fma(p, vj[k].y, kv.y));
      }
      f(r, y, kv);
      prev = y;
      y = next;
      if ((r & 1) || EPT > 3) __builtin_amdgcn_sched_barrier(0);
    }
  };
  // outputs of the instances with one due, their rho in buffer 0
  auto outputs = [&]() {
    const int k = L.ctl[b].out_due;
    if (a.states && k >= 0)
#pragma unroll
      for (int r = 0; r < EPT; ++r)
        if (r < nown)
          reinterpret_cast<double2 *>(a.states)[(int64_t)k * SE + goff + element(r)] = rho[r];
    if (a.expect && a.n_e > 0) dp_band_outputs(a, n, m, L);
    __syncthreads();
    for (int bb = tid; bb < m; bb += T) L.ctl[bb].out_due = -1;
    __syncthreads();
  };
  double *red = reinterpret_cast<double *>(smem + bufb);   // sums' operands: buffer 1
  const int red_at = b * n2;
  auto sum_wide = [&](const double *src, double *out) {
    per_instance_sum_waves(src, m, n2, out, T >> 6); };

#pragma unroll
  for (int r = 0; r < EPT; ++r) store(0, r, rho[r]);
  __syncthreads();
  outputs();
  if (a.n_stops > 0) {
    apply(0, [&](int r, double2, double2 kv) { k1[r] = kv; });
    // Starting step (Hairer, Norsett & Wanner, Solving ODEs I, Sec. II.4) in
    // the scaled RMS norm, exponent 1/5, as in dp5_resident_kernel
    if (a.h0 <= 0.0) {
#pragma unroll
      for (int r = 0; r < EPT; ++r)
        if (r < nown) {
          const double sc = a.atol + a.rtol * hypot(rho[r].x, rho[r].y);
          const double r0 = hypot(rho[r].x, rho[r].y) / sc, r1 = hypot(k1[r].x, k1[r].y) / sc;
          red[red_at + element(r)] = r0 * r0;
          red[m * n2 + red_at + element(r)] = r1 * r1;
        }
      __syncthreads();
      sum_wide(red, L.sums);
      sum_wide(red + m * n2, L.sums + m);
      __syncthreads();
      for (int bb = tid; bb < m; bb += T) {
        const double d0s = sqrt(L.sums[bb] / n2), d1 = sqrt(L.sums[m + bb] / n2);
        L.ctl[bb].hs = (d0s < 1e-5 || d1 < 1e-5) ? 1e-6 : 0.01 * d0s / d1;
        L.ctl[bb].t = d1;  // keep d1 until h is set
      }
      __syncthreads();
      const double hs = L.ctl[b].hs;
#pragma unroll
      for (int r = 0; r < EPT; ++r) store(bufb, r, caxpy(hs, k1[r], rho[r]));
      __syncthreads();
      apply(bufb, [&](int r, double2, double2 kv) { k2[r] = kv; });
      __syncthreads();
#pragma unroll
      for (int r = 0; r < EPT; ++r)
        if (r < nown) {
          const double sc = a.atol + a.rtol * hypot(rho[r].x, rho[r].y);
          const double r2 = hypot(k2[r].x - k1[r].x, k2[r].y - k1[r].y) / sc;
          red[red_at + element(r)] = r2 * r2;
        }
      __syncthreads();
      sum_wide(red, L.sums);
      __syncthreads();
      for (int bb = tid; bb < m; bb += T) dp_start(L.ctl[bb], a, L.sums[bb], n2);
    }
    for (int bb = tid; bb < m; bb += T) {
      L.ctl[bb].hs = a.stops[0];
      dp_next_attempt(L.ctl[bb], a);
      if (L.ctl[bb].active) atomicAdd(&L.flags[0], 1);
    }
    __syncthreads();

    // row s of the stage matrix, the error weights
    auto weights = [&](int row, double (&w)[6]) {
      int z = 0;
      asm volatile("" : "+s"(z));
#pragma unroll
      for (int q = 0; q < 6; ++q) w[q] = kDpA[row][q + z];
    };
    auto error_weights = [&](double (&w)[7]) {
      int z = 0;
      asm volatile("" : "+s"(z));
#pragma unroll
      for (int q = 0; q < 7; ++q) w[q] = kDpE[q + z];
    };
    for (int attempt = 1; L.flags[0] > 0; ++attempt) {
      const bool act = L.ctl[b].active;
      const double ht = L.ctl[b].h_try;
      double A[6], E[7];
      // the next stage's input from the weighted sum of the derivatives so far
      auto input = [&](uint32_t dst, int r, double2 acc) {
        store(dst, r, caxpy(ht, acc, rho[r]));
      };
      weights(1, A);
#pragma unroll
      for (int r = 0; r < EPT; ++r) input(bufb, r, caxpy(A[0], k1[r], zero));
      __syncthreads();
      weights(2, A);
      apply(bufb, [&](int r, double2, double2 kv) {
        k2[r] = kv;
        input(0, r, caxpy(A[1], kv, caxpy(A[0], k1[r], zero)));
      });
      __syncthreads();
      weights(3, A);
      apply(0, [&](int r, double2, double2 kv) {
        k3[r] = kv;
        input(bufb, r, caxpy(A[2], kv, caxpy(A[1], k2[r], caxpy(A[0], k1[r], zero))));
      });
      __syncthreads();
      weights(4, A);
      apply(bufb, [&](int r, double2, double2 kv) {
        k4[r] = kv;
        input(0, r, caxpy(A[3], kv,
                          caxpy(A[2], k3[r], caxpy(A[1], k2[r], caxpy(A[0], k1[r], zero)))));
      });
      __syncthreads();
      weights(5, A);
      apply(0, [&](int r, double2, double2 kv) {
        input(bufb, r,
              caxpy(A[4], kv,
                    caxpy(A[3], k4[r],
                          caxpy(A[2], k3[r], caxpy(A[1], k2[r], caxpy(A[0], k1[r], zero))))));
        k2[r] = kv;   // k5
      });
      __syncthreads();
      weights(6, A);
      error_weights(E);
      apply(bufb, [&](int r, double2, double2 kv) {
        input(0, r,
              caxpy(A[5], kv,
                    caxpy(A[4], k2[r],
                          caxpy(A[3], k4[r], caxpy(A[2], k3[r], caxpy(A[0], k1[r], zero))))));
        // the error's sum so far
        k3[r] = caxpy(E[5], kv,
                      caxpy(E[4], k2[r],
                            caxpy(E[3], k4[r], caxpy(E[2], k3[r], caxpy(E[0], k1[r], zero)))));
      });
      __syncthreads();
      error_weights(E);
      int jd = j + d0;
      asm volatile("" : "+v"(jd));
      apply(0, [&](int r, double2 y, double2 kv) {
        k4[r] = kv;   // k7
        const double2 e = caxpy(E[6], kv, k3[r]);
        const double2 eh = make_double2(ht * e.x, ht * e.y);
        const double sc = a.atol + a.rtol * fmax(hypot(rho[r].x, rho[r].y), hypot(y.x, y.y));
        const double q = hypot(eh.x, eh.y) / sc;
        if (r < nown) red[red_at + wrap(jd + r) * n + j] = act ? q * q : 0.0;
      });
      __syncthreads();
      sum_wide(red, L.sums);
      __syncthreads();
      for (int bb = tid; bb < m; bb += T) dp_decide(L.ctl[bb], a, L.sums[bb], n2, attempt, L.flags);
      __syncthreads();
      // accepted instances move to the fifth-order solution; k7 -> k1
      if (L.ctl[b].accept) {
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
          rho[r] = *reinterpret_cast<const double2 *>(smem + own + (uint32_t)(r * n16));
          k1[r] = k4[r];
        }
      }
      if (L.flags[1] == attempt) outputs();
    }
  }

  if (a.rho_out) {
#pragma unroll
    for (int r = 0; r < EPT; ++r)
      if (r < nown) reinterpret_cast<double2 *>(a.rho_out)[goff + element(r)] = rho[r];
  }
  for (int bb = tid; bb < m; bb += T) {
    const int id = L.ids[bb];
    if (a.counts) {
      a.counts[2 * (int64_t)id] = L.ctl[bb].n_acc;
      a.counts[2 * (int64_t)id + 1] = L.ctl[bb].n_rej;
    }
    if (a.status) a.status[id] = L.ctl[bb].status;
  }
}

template <int T, int EPT, int NW, int NC>
__global__ __launch_bounds__(T) void dp5_band_kernel(Dp5Args a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const PackDesc pk = a.packs[blockIdx.x];
  const int n = pk.n, m = pk.m;
  const DpLds L = carve_dp(smem, n, m, NC);
  for (int b = threadIdx.x; b < m; b += blockDim.x) {
    const int id = a.order[pk.first + b];
    L.ids[b] = id;
    L.off[b] = a.inst[id].rho_off;
    if (a.status) a.status[id] = 0;
    DpCtl c;
    c.t = a.t0;
    c.h = a.h0;
    c.h_try = 0.0;
    c.hs = 0.0;
    c.n_acc = c.n_rej = 0;
    c.stop = 0;
    c.status = 0;
    c.active = a.n_stops > 0;
    c.accept = c.landing = 0;
    c.seg = -1;
    c.k1_seg = -2;
    c.prev_rej = 0;
    c.out_due = 0;   // the initial state is output 0
    c.need_k1 = 1;
    L.ctl[b] = c;
  }
  if (threadIdx.x == 0) L.flags[0] = L.flags[1] = 0;
  // diagonals that nothing stores are read with zero coefficients
  for (int e = threadIdx.x; e < band_dp_buffer_bytes(n, m) / 8; e += blockDim.x)
    reinterpret_cast<double2 *>(L.buf)[e] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * m * n; e += blockDim.x) {
    const int b = e / (2 * n), i = (e - b * 2 * n) % n;
    const OpView op = make_view(a.ops + a.inst[L.ids[b]].ops_off,
                                blob_layout(n, pk.wo, pk.nb, pk.wb, pk.nc, pk.wc));
    double2 *tb = reinterpret_cast<double2 *>(L.tab) + e;
    const int step = 2 * m * n;
    double dn = 0.0, up = 0.0;
    for (int w = 0; w < pk.wo; ++w) {
      const int cc = op.Ocol[w * n + i];
      if (cc == i - 1) dn = op.Oval[w * n + i].y;
      if (cc == i + 1) up = op.Oval[w * n + i].y;
    }
    tb[0] = op.D[i];
    tb[step] = make_double2(dn, up);
    tb[2 * step] = make_double2(op.Jval[i].x, op.Jval[n + i].x);
    if (NC > 2) tb[3 * step] = make_double2(op.Jval[(NC - 1) * n + i].x, 0.0);
  }
  __syncthreads();
  switch (pk.ept) {
    case 1: dp5_band_pack<1, NW, NC>(a, pk, smem); break;
    case 2: dp5_band_pack<2, NW, NC>(a, pk, smem); break;
    case 3: dp5_band_pack<3, NW, NC>(a, pk, smem); break;
    default:
      if constexpr (EPT > 3) {
        if (pk.ept == 4) dp5_band_pack<4, NW, NC>(a, pk, smem);
        if (pk.ept == 5) dp5_band_pack<5, NW, NC>(a, pk, smem);
        if (pk.ept == 6) dp5_band_pack<6, NW, NC>(a, pk, smem);
        if (pk.ept == 7) dp5_band_pack<7, NW, NC>(a, pk, smem);
        if (pk.ept == 8) dp5_band_pack<8, NW, NC>(a, pk, smem);
      }
  }
}

}  // namespace lme

template <int CFG>
static void (*band_dp_kernel(int nw, int nc))(lme::Dp5Args) {
  constexpr int T = lme::kBandDpCfg[CFG][0], E = lme::kBandDpCfg[CFG][1];
  if (nw == 1 && nc == 2) return lme::dp5_band_kernel<T, E, 1, 2>;
  if (nw == 1 && nc == 3) return lme::dp5_band_kernel<T, E, 1, 3>;
  if (nw == 2 && nc == 2) return lme::dp5_band_kernel<T, E, 2, 2>;
  return nullptr;
}

// Configuration cfg of kBandDpCfg; (nw, nc) one of (1, 2), (1, 3), (2, 2);
// `threads` (a multiple of 64) covers every pack's m n G.
extern "C" hipError_t lme_internal_launch_dp5_band(int cfg, int nw, int nc, const lme::Dp5Args *a,
                                                   int n_packs, int threads, int lds,
                                                   hipStream_t s) {
  void (*k)(lme::Dp5Args) = cfg == 0 ? band_dp_kernel<0>(nw, nc) : band_dp_kernel<1>(nw, nc);
  if (!k || threads < 64 || threads > lme::kBandDpCfg[cfg == 0 ? 0 : 1][0])
    return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_packs), dim3(threads), lds, s, *a);
  return hipGetLastError();
}

// lme_band.hip -- resident fixed-step RK4 of Hermitian states under banded
// operators, along diagonals.
//
// Operators: every off-diagonal entry of A = -iH - 1/2 sum C^+C is imaginary
// and next to the diagonal, every collapse operator is real with all its
// entries on one diagonal (offset delta_k), no control terms.  That is the
// Jaynes-Cummings family (delta = 2, 1 and, at a temperature, -2) and every
// single bosonic mode (Kerr, thermal cavity: delta = 1, -1).
//
// Layout.  Thread (g, j) owns column j of one instance and the consecutive
// diagonals d = g e .. g e + e - 1 of it: elements (i, j), i = j + d mod n,
// d <= n/2, which is every unordered pair {i, j} once (for even n the pair at
// d = n/2 belongs to the smaller column).  In these coordinates every operand
// of an element sits at a fixed distance:
//   y[i -+ 1][j]          diagonal d -+ 1, the same column: the thread's own
//                         registers, but for its first and last diagonal
//   y[i][j -+ 1]          diagonal d +- 1, column j -+ 1
//   y[i + delta][j + delta]   the same diagonal, column j + delta
// LDS holds the stage input by diagonals, rows of n columns, so the lanes of
// one run of columns access contiguous addresses (1.3 conflict cycles an LDS
// instruction on the sweep, from wavefronts that span several columns' runs
// and from wrapped neighbours; 2.1 in rk4_herm_kernel) and each operand is
// addressed by a register plus a uniform offset per diagonal.  Besides the owned diagonals
// it holds their neighbours -1 and n/2 + 1 (conjugates of diagonals 1 and
// n - n/2 - 1, stored by their owners).  Half the matrix leaves room for two
// buffers: a stage reads one and writes the other, one barrier per stage.
//
// The generator is constant and linear, so the RK4 step is the degree-4 Taylor
// polynomial and is evaluated by Horner's rule,
//   x <- rho + h/k L x,   k = 4, 3, 2, 1, from x = rho,
// which needs no running sum (20 registers a diagonal instead of 24; with the
// sum the 768-thread configuration spills in its stages and takes 40.3 ms
// instead of 36.6; as it is, 13 to 31 registers by operator shape spill, 7 to 17
// reloads a step and none in a stage).  Rounding: the last stage's input enters
// the result with h L, the classic form's three with h L / 3, / 3 and / 6.
// Against an 80-bit RK4 the root mean square error is 1.1 to 1.7 times the
// classic form's, the largest entry's 0.95 to 1.3 times (400 steps, n = 10 to
// 40, 24 systems each: 0.7e-16 to 5.7e-16 of a trace of one).
//
// What bounds it (4096 Jaynes-Cummings instances of n = 10 to 80, 1000 steps:
// 36.6 ms; rk4_herm_kernel, whose mirrored full matrix and per-lane rows cost
// two stores, 2.1 conflict cycles an access and a third more VALU, 43.8 ms):
// about 27 VALU instructions and 4.6 LDS accesses a wavefront and diagonal,
// each pipe close to half busy at three wavefronts a SIMD.  A pack that fills
// a fraction of a CU is bound by the latency of a stage, about 250 ns at one
// diagonal a thread (one instance of n = 20: 1.08 ms per 1000 steps against
// 1.97 ms).
#include "lme_device.h"
#include "lme_internal.h"

namespace lme {

namespace {

// y = x where c (by values: a conditional of the two objects would select
// their addresses)
__device__ __forceinline__ void take(bool c, double2 x, double2 &y) {
  y.x = c ? x.x : y.x;
  y.y = c ? x.y : y.y;
}

struct BandLds {
  double2 *Y;        // two buffers of m instances
  int64_t *off;
  int32_t *ids;
};

__device__ __forceinline__ BandLds carve_band(uint8_t *smem, int n, int m) {
  BandLds p;
  p.Y = reinterpret_cast<double2 *>(smem);
  uint8_t *q = smem + 2 * band_buffer_bytes(n, m) + 16 * n * kBandSlack;
  p.off = reinterpret_cast<int64_t *>(q);
  p.ids = reinterpret_cast<int32_t *>(q + align16(8 * m));
  return p;
}

// Expectation values at output k from the diagonals in buffer 0: the sums of
// write_outputs() in its order.
__device__ void band_outputs(const Rk4Args &a, int n, int m, const BandLds &L, int k) {
  const int D = n / 2, S = band_rows(n) * n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  for (int task = wave; task < m * a.n_e; task += waves) {
    const int b = task / a.n_e, e = task - b * a.n_e;
    const int id = L.ids[b];
    const InstDesc &d = a.inst[id];
    const int we = d.we;
    const int32_t *Ec = reinterpret_cast<const int32_t *>(a.eops + d.eops_off);
    const double2 *Ev = reinterpret_cast<const double2 *>(
        a.eops + d.eops_off + eops_val_offset(n, we, a.n_e));
    const double2 *Y = L.Y + b * S;
    double2 part = make_double2(0.0, 0.0);
    for (int i = lane; i < n; i += 64)
      for (int w = 0; w < we; ++w) {
        const int idx = (e * we + w) * n + i;
        // element (r, i)
        const int r = Ec[idx];
        int q = r - i;
        q = q < 0 ? q + n : q;
        const bool low = q <= D;
        double2 y = Y[low ? (q + 1) * n + i : (n - q + 1) * n + r];
        if (!low) y = cconj(y);
        part = cfma(Ev[idx], y, part);
      }
    part = wave_sum(part);
    if (lane == 0) {
      double *dst = a.expect + 2 * (((int64_t)id * a.n_e + e) * a.n_t + k);
      dst[0] = part.x;
      dst[1] = part.y;
      if (!cfinite(part) && a.status) a.status[id] = 5;  // LME_ENONFINITE
    }
  }
}

}  // namespace

// All steps of one pack whose threads own at most EPT diagonals.
// NW: off-diagonal entries per row of A (1: the neighbour differs from row to
// row); NC collapse operators at offsets a.band_off[k].
template <int EPT, int NW, int NC>
__device__ __forceinline__ void band_pack(const Rk4Args &a, const PackDesc &pk, uint8_t *smem) {
  const int n = pk.n, D = n / 2, C = pk.m * n, G = pk.G, n16 = 16 * n;
  const int rows = band_rows(n), bufb = band_buffer_bytes(n, pk.m);
  const BandLds L = carve_band(smem, n, pk.m);
  const int tid = threadIdx.x;

  // Thread (g, column c of the pack); the D + 1 diagonals go to the G groups
  // in runs of EPT or EPT - 1.  For even n the columns j >= n/2 leave their
  // last diagonal, n/2, to column j - n/2.
  const bool active = tid < C * G;
  const int g = active ? tid / C : 0;
  const int c = active ? tid - g * C : 0;
  const int b = c / n, j = c - b * n;
  const int q = (D + 1) / G, rem = (D + 1) - q * G;
  const int d0 = g * q + min(g, rem);
  const int nown = !active ? 0 : (g < rem ? q + 1 : q) -
                                     ((n & 1) == 0 && 2 * j >= n && g == G - 1 ? 1 : 0);
  const uint32_t yb = (uint32_t)(16 * b * rows * n);
  auto wrap = [&](int x) { return x < 0 ? x + n : (x >= n ? x - n : x); };
  // byte address of diagonal d0 + dd of column cc
  auto at = [&](int dd, int cc) { return yb + (uint32_t)((d0 + dd + 1) * n + wrap(cc)) * 16u; };

  // column-j and per-diagonal coefficients (zero for what is not owned)
  const OpView op = make_view(a.ops + a.inst[L.ids[b]].ops_off,
                              blob_layout(n, pk.wo, pk.nb, pk.wb, pk.nc, pk.wc));
  const double2 dj = cconj(op.D[j]);
  double qr[NW];            // Im conj(A_{j,c}), c the column of gather w
  uint32_t ar[NW], aj[NC];
  double jv[NC];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    qr[w] = 0.0;
    ar[w] = NW == 2 ? at(w == 0 ? 1 : -1, w == 0 ? j - 1 : j + 1) : at(0, j);
  }
  for (int w = 0; w < pk.wo; ++w) {
    const int cc = op.Ocol[w * n + j];
    if (cc == j) continue;   // ELL padding
    const double v = -op.Oval[w * n + j].y;
    if (NW == 1) {
      qr[0] = v;
      ar[0] = at(j - cc, cc);
    } else {
      qr[cc < j ? 0 : NW - 1] = v;
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    jv[k] = op.Jval[k * n + j].x;
    aj[k] = at(0, j + band_offset(a.band_off[k], n));
  }
  double2 dsum[EPT];
  double odn[EPT], oup[EPT], p[EPT][NC];
  const uint32_t own = at(0, j);
  bool mirrors = false;     // some diagonal of this thread is stored twice
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    dsum[r] = make_double2(0.0, 0.0);
    odn[r] = oup[r] = 0.0;
#pragma unroll
    for (int k = 0; k < NC; ++k) p[r][k] = 0.0;
    if (r < nown) {
      const int d = d0 + r, i = wrap(j + d);
      dsum[r] = cadd(op.D[i], dj);
      for (int w = 0; w < pk.wo; ++w) {
        const int cc = op.Ocol[w * n + i];
        if (cc == i - 1) odn[r] = op.Oval[w * n + i].y;
        if (cc == i + 1) oup[r] = op.Oval[w * n + i].y;
      }
#pragma unroll
      for (int k = 0; k < NC; ++k) p[r][k] = op.Jval[k * n + i].x * jv[k];
      mirrors |= d == 1 || (d > 0 && n - d <= D + 1);
    }
  }
  // what a thread does not own it stores past the diagonals (no branch)
  const uint32_t waste = (uint32_t)(2 * bufb + 16 * min(tid & 31, n - 1));
  const bool wave_on = __builtin_amdgcn_readfirstlane((int)(__ballot(active) != 0)) != 0;
  // the copies of its diagonals that other columns' neighbours read: the
  // conjugate of 1 as -1, of the last ones as n/2 and n/2 + 1
  auto put_mirrors = [&](uint32_t buf, const auto &v) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const int d = d0 + r;
      if (r < nown && d == 1)
        *reinterpret_cast<double2 *>(smem + buf + yb + 16 * wrap(j + 1)) = cconj(v[r]);
      if (r < nown && d > 0 && n - d <= D + 1)
        *reinterpret_cast<double2 *>(smem + buf + yb + 16 * ((n - d + 1) * n + wrap(j + d))) =
            cconj(v[r]);
    }
  };
  // element (i, j) and its mirror into global memory
  auto put_global = [&](double2 *dst, int r, double2 v) {
    const int i = wrap(j + d0 + r);
    dst[i * n + j] = v;
    if (i != j) dst[j * n + i] = cconj(v);
  };

  double2 rho[EPT], yn[EPT + 1];
  const double2 *rho0 = reinterpret_cast<const double2 *>(a.rho0) + L.off[b];
  bool not_herm = false;
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    rho[r] = make_double2(0.0, 0.0);
    if (r < nown) {
      const int i = wrap(j + d0 + r);
      const double2 x = rho0[i * n + j], y = rho0[j * n + i];
      const double dx = x.x - y.x, dy = x.y + y.y;
      not_herm |= dx * dx + dy * dy > 2e-24 * (x.x * x.x + x.y * x.y + y.x * y.x + y.y * y.y);
      rho[r] = make_double2(0.5 * (x.x + y.x), 0.5 * (x.y - y.y));
      *reinterpret_cast<double2 *>(smem + own + (uint32_t)(r * n16)) = rho[r];
    }
  }
  if (mirrors) put_mirrors(0, rho);
  if (not_herm && a.status) a.status[L.ids[b]] = 9;  // LME_ENOTHERM
  __syncthreads();

  const bool want_expect = a.expect != nullptr && a.n_e > 0;
  int next_out = 0, due = a.out_step[0];
  const double h = a.h, h3 = h / 3.0;
  for (int st = 0;; ++st) {
    // outputs due after st steps (st = 0: the initial state), from buffer 0
    while (due == st) {
      if (a.states)
#pragma unroll
        for (int r = 0; r < EPT; ++r)
          if (r < nown)
            put_global(reinterpret_cast<double2 *>(a.states) + (int64_t)next_out * a.state_elems +
                           L.off[b], r, rho[r]);
      if (want_expect) band_outputs(a, n, pk.m, L, next_out);
      ++next_out;
      due = next_out < a.n_t ? a.out_step[next_out] : -1;
    }
    if (st == a.nsteps) break;
#pragma unroll
    for (int r = 0; r < EPT; ++r) yn[r] = rho[r];
    // four products, each from one buffer to the other; the last leaves the
    // new rho in buffer 0
#pragma unroll(EPT <= 3 ? 4 : 1)
    for (int k4 = 4; k4 >= 1; --k4) {
      const uint32_t src = (k4 & 1) ? bufb : 0, dst = (k4 & 1) ? 0 : bufb;
      const double hk = k4 == 1 ? h : k4 == 2 ? 0.5 * h : k4 == 3 ? h3 : 0.25 * h;
      if (wave_on) {
        // opaque copies: no address per diagonal is kept across the stages
        uint32_t so = src + own, to = active ? dst + own : waste, sr[NW], sj[NC];
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
        // the neighbours of the thread's first and last diagonal (a run of
        // EPT, EPT - 1 or EPT - 2)
        double2 prev = Y(so - n16);
        const double2 next = Y(so + (uint32_t)mul24(nown, n16));
        yn[EPT] = next;
        if constexpr (EPT >= 2) take(nown == EPT - 1, next, yn[EPT - 1]);
        if constexpr (EPT >= 3) take(nown == EPT - 2, next, yn[EPT - 2]);
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
          const uint32_t o = (uint32_t)(r * n16);
          double2 vr[NW], vj[NC];
#pragma unroll
          for (int w = 0; w < NW; ++w) vr[w] = Y(sr[w] + o);
#pragma unroll
          for (int k = 0; k < NC; ++k) vj[k] = Y(sj[k] + o);
          const double2 y = yn[r];
          double2 kv = cmul(dsum[r], y);
          kv = make_double2(fma(-odn[r], prev.y, kv.x), fma(odn[r], prev.x, kv.y));
          kv = make_double2(fma(-oup[r], yn[r + 1].y, kv.x), fma(oup[r], yn[r + 1].x, kv.y));
#pragma unroll
          for (int w = 0; w < NW; ++w)
            kv = make_double2(fma(-qr[w], vr[w].y, kv.x), fma(qr[w], vr[w].x, kv.y));
#pragma unroll
          for (int k = 0; k < NC; ++k)
            kv = make_double2(fma(p[r][k], vj[k].x, kv.x), fma(p[r][k], vj[k].y, kv.y));
          // the diagonal of L(y) is real for Hermitian y: drop the rounding
          // residue of its imaginary part
          if (r == 0) kv.y = d0 == 0 ? 0.0 : kv.y;
          prev = y;
          yn[r] = caxpy(hk, kv, rho[r]);
          uint32_t w = to + o;
          if (r >= EPT - 2) w = r < nown ? w : waste;
          *reinterpret_cast<double2 *>(smem + w) = yn[r];
          if (r & 1) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (mirrors) put_mirrors(dst, yn);
      __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < EPT; ++r) rho[r] = yn[r];
  }

  if (a.rho_out) {
#pragma unroll
    for (int r = 0; r < EPT; ++r)
      if (r < nown) put_global(reinterpret_cast<double2 *>(a.rho_out) + L.off[b], r, rho[r]);
  }
}

// The body compiled for each run length, so that its loops have no branches:
// a pack runs the one of its pk.ept.
template <int T, int EPT, int NW, int NC>
__global__ __launch_bounds__(T) void rk4_band_kernel(Rk4Args a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const PackDesc pk = a.packs[blockIdx.x];
  const BandLds L = carve_band(smem, pk.n, pk.m);
  for (int bb = threadIdx.x; bb < pk.m; bb += blockDim.x) {
    const int id = a.order[pk.first + bb];
    L.ids[bb] = id;
    L.off[bb] = a.inst[id].rho_off;
    if (a.status) a.status[id] = 0;
    if (a.counts) {
      a.counts[2 * (int64_t)id] = a.nsteps;
      a.counts[2 * (int64_t)id + 1] = 0;
    }
  }
  // diagonals that nothing stores are read with zero coefficients
  const int cells = band_buffer_bytes(pk.n, pk.m) / 8 + pk.n * kBandSlack;
  for (int e = threadIdx.x; e < cells; e += blockDim.x) L.Y[e] = make_double2(0.0, 0.0);
  __syncthreads();
  switch (pk.ept) {
    case 1: band_pack<1, NW, NC>(a, pk, smem); break;
    case 2: band_pack<2, NW, NC>(a, pk, smem); break;
    case 3: band_pack<3, NW, NC>(a, pk, smem); break;
    case 4: band_pack<4, NW, NC>(a, pk, smem); break;
    default:
      if constexpr (EPT >= 5)
        if (pk.ept == 5) band_pack<5, NW, NC>(a, pk, smem);
      if constexpr (EPT >= 7) {
        if (pk.ept == 6) band_pack<6, NW, NC>(a, pk, smem);
        if (pk.ept == 7) band_pack<7, NW, NC>(a, pk, smem);
      }
  }
}

}  // namespace lme

template <int T, int EPT, int NW, int NC>
static hipError_t launch_band_t(const lme::Rk4Args &a, int n_packs, int threads, int lds,
                                hipStream_t s) {
  auto k = lme::rk4_band_kernel<T, EPT, NW, NC>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_packs), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template <int T, int EPT>
static hipError_t launch_band_cfg(int nw, int nc, const lme::Rk4Args &a, int n_packs, int threads,
                                  int lds, hipStream_t s) {
  if (threads < 64 || threads > T) return hipErrorInvalidValue;
  switch (10 * nw + nc) {
    case 12: return launch_band_t<T, EPT, 1, 2>(a, n_packs, threads, lds, s);
    case 13: return launch_band_t<T, EPT, 1, 3>(a, n_packs, threads, lds, s);
    case 22: return launch_band_t<T, EPT, 2, 2>(a, n_packs, threads, lds, s);
    default: return hipErrorInvalidValue;
  }
}

// Configuration cfg of kBandCfg; nw 1 or 2, nc 1 to 3; `threads` (a multiple
// of 64) covers every pack's m n G.
extern "C" hipError_t lme_internal_launch_rk4_band(int cfg, int nw, int nc, const lme::Rk4Args *a,
                                                   int n_packs, int threads, int lds,
                                                   hipStream_t s) {
  return cfg == 0 ? launch_band_cfg<lme::kBandCfg[0][0], lme::kBandCfg[0][1]>(nw, nc, *a, n_packs,
                                                                              threads, lds, s)
                  : launch_band_cfg<lme::kBandCfg[1][0], lme::kBandCfg[1][1]>(nw, nc, *a, n_packs,
                                                                              threads, lds, s);
}

// lme_device.h -- device helpers shared by the gfx950 kernels of the library:
// complex FP64 arithmetic, the operator view of an op blob, wavefront sums.
#pragma once
#include <hip/hip_runtime.h>

#include "lme_internal.h"

namespace lme {

// ---------------------------------------------------------------------------
// complex helpers (double2 = re, im)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 cadd(double2 a, double2 b) {
  return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
// a * b with the product fused into each sum written out: left to the
// compiler, which product of a.x b.y + a.y b.x it fuses depends on the
// surrounding code, and two kernels evaluating the same element could round
// it differently
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
// c + a * b
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
// c + conj(a) * b
__device__ __forceinline__ double2 cfma_conj(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(a.y, b.y, c.x)), fma(a.x, b.y, fma(-a.y, b.x, c.y)));
}
// c + s * a  (s real)
__device__ __forceinline__ double2 caxpy(double s, double2 a, double2 c) {
  return make_double2(fma(s, a.x, c.x), fma(s, a.y, c.y));
}
__device__ __forceinline__ bool cfinite(double2 a) { return isfinite(a.x) && isfinite(a.y); }

// ---------------------------------------------------------------------------
// operator view of one instance's op blob
// ---------------------------------------------------------------------------
struct OpView {
  const double2 *D, *Oval, *Jval, *DB, *OBval;
  const int32_t *Ocol, *Jcol, *OBcol;
  int n, wo, nb, wb, nc, wc;
};

__device__ __forceinline__ OpView make_view(const uint8_t *blob, const BlobLayout &L) {
  OpView v;
  v.D = reinterpret_cast<const double2 *>(blob + L.offD);
  v.Oval = reinterpret_cast<const double2 *>(blob + L.offOval);
  v.Ocol = reinterpret_cast<const int32_t *>(blob + L.offOcol);
  v.Jval = reinterpret_cast<const double2 *>(blob + L.offJval);
  v.Jcol = reinterpret_cast<const int32_t *>(blob + L.offJcol);
  v.DB = reinterpret_cast<const double2 *>(blob + L.offDB);
  v.OBval = reinterpret_cast<const double2 *>(blob + L.offOBval);
  v.OBcol = reinterpret_cast<const int32_t *>(blob + L.offOBcol);
  v.n = L.n; v.wo = L.wo; v.nb = L.nb; v.wb = L.wb; v.nc = L.nc; v.wc = L.wc;
  return v;
}

// Deterministic butterfly sum over the 64 lanes of a wavefront.
__device__ __forceinline__ double2 wave_sum(double2 v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.x += __shfl_xor(v.x, off, 64);
    v.y += __shfl_xor(v.y, off, 64);
  }
  return v;
}

// 24-bit multiply: full rate on CDNA (a 32-bit multiply is quarter rate);
// every product here is below 2^24.
__device__ __forceinline__ int mul24(int a, int b) { return (int)__umul24((unsigned)a, (unsigned)b); }

}  // namespace lme

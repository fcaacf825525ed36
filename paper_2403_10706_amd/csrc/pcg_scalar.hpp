// Scalar recurrences of the PCG shared by the stepped form (pcg.hip) and the resident form
// (pcg_resident.hip).  Included after `#pragma clang fp contract(off)`: both forms round alike.
#pragma once

#include "rgp_internal.hpp"

namespace rgp {

__device__ __forceinline__ float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Slot of iteration it >= 1 from the running slot of iteration it-1 and the block sums t of
// iteration it-1: [0] p.w, [1] r.w/d, [2] w.w/d, [3] r.w, [4] w.w, [5] r.r/d and [6] r.r of the
// residual that iteration stored (at it == 1 the right-hand side, whose r.r is |rhs|^2).  `fin`
// is set when the solve ends here.
__device__ __forceinline__ PcgSlot pcg_advance(const PcgSlot& prev, const double (&t)[7], int it,
                                               int maxit, double rtol, bool& fin) {
  PcgSlot cur = prev;
  const double rz = t[5], rr = t[6];
  const double bn = it == 1 ? t[6] : prev.bnorm2;
  const double pw = t[0];
  cur.bnorm2 = bn;
  if (!(bn > 0.0) || !(pw > 0.0)) {  // zero right-hand side or p^T H p <= 0: keep x
    cur.status = kPcgDone;
    cur.iters = it - 1;
    cur.relres = it == 1 ? (bn > 0.0 ? 1.0 : 0.0) : prev.relres;
    fin = true;
    return cur;
  }
  const double a2 = rz / pw;
  const double rzn = rz - 2.0 * a2 * t[1] + a2 * a2 * t[2];
  const double rrn = rr - 2.0 * a2 * t[3] + a2 * a2 * t[4];
  cur.alpha = a2;
  cur.beta = rzn / rz;
  cur.rz = rzn;
  cur.rr = rrn;
  cur.iters = it;
  cur.relres = sqrt(fmax(rrn, 0.0) / bn);
  fin = cur.relres < rtol || it >= maxit;
  cur.status = fin ? kPcgFinish : kPcgRunning;
  return cur;
}

}  // namespace rgp

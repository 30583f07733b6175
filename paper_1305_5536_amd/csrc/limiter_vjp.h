// Transpose of the slope limiter (Sec. 2.5) on a Cartesian cell: what one
// limited variable hands back to its gradients, its mean and the one neighbour
// mean that set its bound.
#pragma once

#include <hip/hip_runtime.h>

#include "dg_math.h"

namespace dg {

// The limiter's decision for one variable of a cell: alpha = min(1, D / dm) with
// D the distance of the mean to the nearer bound and dm the largest
// |gradient| h/2.  Ties take the first argument in the order self, -x, +x, -y,
// +y(, -z, +z), the upper bound before the lower, x before y before z.
template <typename T>
struct LimDecision {
  T alpha, dm;
  bool act;    // alpha = D / dm (dm > D), else 1
  bool lower;  // D is phi - lo
  int nbr;     // the neighbour that set the bound, 0 the cell itself, else 1 + direction
  int axis;    // the axis that set dm
};

template <typename T, int DIM>
__device__ __forceinline__ LimDecision<T> limiter_decide(T phi, const T* nbm, const T* g,
                                                         const T* half) {
  T hi = phi, lo = phi;
  int ihi = 0, ilo = 0;
#pragma unroll
  for (int f = 0; f < 2 * DIM; ++f) {
    const bool up = nbm[f] > hi, dn = nbm[f] < lo;
    hi = up ? nbm[f] : hi;
    ihi = up ? f + 1 : ihi;
    lo = dn ? nbm[f] : lo;
    ilo = dn ? f + 1 : ilo;
  }
  LimDecision<T> r;
  const T Du = hi - phi, Dl = phi - lo;
  r.lower = Dl < Du;
  const T Dd = r.lower ? Dl : Du;
  r.nbr = r.lower ? ilo : ihi;
  r.dm = fabs(g[0]) * half[0];
  r.axis = 0;
#pragma unroll
  for (int d = 1; d < DIM; ++d) {
    const T x = fabs(g[d]) * half[d];
    r.axis = x > r.dm ? d : r.axis;
    r.dm = x > r.dm ? x : r.dm;
  }
  r.act = r.dm > Dd;
  r.alpha = r.act ? div_small(Dd, r.dm) : T(1);
  return r;
}

// The derivative of that alpha with cotangent ab: adds the gradient part to gb,
// returns the cotangent of the bound that entered D (the neighbour r.nbr gets
// it; the cell's mean gets its negative).  alpha = 1 has none.
template <typename T, int DIM>
__device__ __forceinline__ T limiter_bar(const LimDecision<T>& r, T ab, const T* g, const T* half,
                                         T* gb) {
  const T Db = r.act ? div_small(ab, r.dm) : T(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const T x = -r.alpha * Db * half[d];
    gb[d] += d == r.axis ? (g[d] < T(0) ? -x : x) : T(0);
  }
  return r.lower ? -Db : Db;
}

}  // namespace dg

// Least-squares gradient of one cell (App. B): the sums over its stencil and
// their solution.
#pragma once

#include <hip/hip_runtime.h>

#include "wave_ops.h"

namespace vofpc {

// least-squares sums of one cell: G (6 components) and b
struct LsqSums {
  double xx = 0, yy = 0, zz = 0, xy = 0, xz = 0, yz = 0, b0 = 0, b1 = 0, b2 = 0;
  __device__ __forceinline__ void add(double r0, double r1, double r2, double dv, int weight) {
    double w = 1.0;
    if (weight == 1) w = 1.0 / sqrt(r0 * r0 + r1 * r1 + r2 * r2);
    else if (weight == 2) w = 1.0 / (r0 * r0 + r1 * r1 + r2 * r2);
    const double w0 = w * r0, w1 = w * r1, w2 = w * r2;
    xx += w0 * r0; yy += w1 * r1; zz += w2 * r2; xy += w0 * r1; xz += w0 * r2; yz += w1 * r2;
    b0 += w0 * dv; b1 += w1 * dv; b2 += w2 * dv;
  }
};

// Sums over a group of W lanes.
template <int W>
__device__ __forceinline__ void lsq_reduce(LsqSums &L) {
  L.xx = gsum<W>(L.xx); L.yy = gsum<W>(L.yy); L.zz = gsum<W>(L.zz);
  L.xy = gsum<W>(L.xy); L.xz = gsum<W>(L.xz); L.yz = gsum<W>(L.yz);
  L.b0 = gsum<W>(L.b0); L.b1 = gsum<W>(L.b1); L.b2 = gsum<W>(L.b2);
}

// Solution by the adjugate; false (and zero) when the matrix is singular,
// det <= 1e-12 (tr/3)^3.
__device__ __forceinline__ bool lsq_solve(const LsqSums &L, double &g0, double &g1, double &g2) {
  const double xx = L.xx, yy = L.yy, zz = L.zz, xy = L.xy, xz = L.xz, yz = L.yz;
  const double c00 = yy * zz - yz * yz, c01 = xz * yz - xy * zz, c02 = xy * yz - xz * yy;
  const double c11 = xx * zz - xz * xz, c12 = xy * xz - xx * yz, c22 = xx * yy - xy * xy;
  const double det = xx * c00 + xy * c01 + xz * c02;
  const double tr = (xx + yy + zz) * (1.0 / 3.0);
  if (det > 1e-12 * tr * tr * tr) {
    const double id = 1.0 / det;
    g0 = (c00 * L.b0 + c01 * L.b1 + c02 * L.b2) * id;
    g1 = (c01 * L.b0 + c11 * L.b1 + c12 * L.b2) * id;
    g2 = (c02 * L.b0 + c12 * L.b1 + c22 * L.b2) * id;
    return true;
  }
  g0 = g1 = g2 = 0.0;
  return false;
}

}  // namespace vofpc

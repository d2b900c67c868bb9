// Volume-matched iso-polygon reconstruction with a group of G lanes per mixed
// cell (G = 4 or 16) and up to 64/G cells per wavefront.
//
// A lane owns a few edges, faces and vertices of its cell for the whole
// search and keeps them in registers: an edge's end values, its liquid end,
// direction and whole-edge volume term, a face's fan point and two edge masks, a
// vertex's value and adjacency mask.  The cut of an isovalue is described by
// bit masks over the cell's edges and vertices, gathered with wavefront
// ballots, so an evaluation reads LDS only for the crossing points of the
// faces that are cut.
//
// One volume evaluation at isovalue s (divergence theorem, each face's
// liquid polygon fanned from a point of its plane, one of its vertices):
//   - per edge, held from its end of larger value u to the other end v (the
//     liquid end of a cut edge is always u): the two faces' terms of the
//     whole edge, D_e = det(c1, u, v) + det(c2, v, u), are fixed per cell; an
//     evaluation adds D_e times the edge's liquid fraction (1, 0, or for a
//     cut edge the fraction from its liquid end, which scales both faces'
//     liquid pieces of the edge alike) and stores the crossing point of a cut
//     edge (Eq. edge_intersection) once, so both faces get the same point;
//     the ballots of the cut edges give the cell's cut mask;
//   - per face, the iso-curve leaves through the cut edges its loop runs
//     along from u to v and enters through the others: two static masks
//     and'ed with the cut mask.  A face with two crossings has one chord,
//     exit -> entry; a face with four or more pairs each exit with the next
//     entry in loop order when the face-mean vertex value is >= s, else with
//     the previous one (the oracle's rule); the chord closes the face's
//     liquid polygon;
//   - per chord, the terms of its iso-loop: a loop is the chain of chords
//     (the chord entering through edge e follows the chord leaving through
//     e), and fanning a loop from its length-weighted polyline centroid k
//     gives volume k . Y / 6 and area vector -Y / 2 with Y = sum over its
//     chords of (entry point x exit point), the centroid from sum l and
//     sum l (entry + exit): chord-local sums, taken about a reference
//     vertex of the cell.
// The loops of a cut bound the connected pieces of the liquid and the vapour
// part of the cell's surface, one loop fewer than there are pieces; when no
// face has more than two crossings the pieces are the connected components of
// the liquid and of the vapour vertices under the cell's edges.  A flood
// fill of the vertex masks (ballots, no memory) therefore shows that there is
// one loop, the usual case, and its result is kept while the liquid vertices
// stay the same, which they do once the search is inside one interval of the
// vertex values.  Otherwise the chords are linked through LDS, the loops
// labelled and their sums gathered loop by loop in a second pass.
//
// What bounds it: instruction issue and the latency of dependent FP64
// operations, not memory.  Holding the edges in registers and the cut in
// masks, against cells staged in LDS and walked through byte tables (the
// evaluation before), whole plain steps on one chip: 24,042 Voronoi cells cut
// of 351k in 241 instead of 395 us, 31,948 hexahedra of 1.33M in 190 instead of
// 249 us; with few cells the teams below: 2,832 of 195k Voronoi cells in 106
// instead of 165 us (one cell per wavefront, recon.hip), 5,000 of 422k
// hexahedra in 62 instead of 143 us.
//
// Search: the root of r(s) = V(s)/V_P - alpha in a bracket of [phi_min,
// phi_max] whose ends straddle it.  The first cut is the quantile of alpha in a
// model of the cell's volume over phi (quantile()), the second moves by the
// difference of the quantiles of the volume found and of alpha; then the secant
// and the inverse quadratic interpolation through the last three cuts, wherever
// the bracket's other end is; the midpoint when the estimate leaves the bracket
// or does not shrink fast enough (the rule of Brent 1973, ch. 4).  One evaluation
// per step, the stopping rule of the wavefront kernel.  The mean number of cuts
// is 5.2 for hexahedra and 6.1 for Voronoi cells (Brent's method from the ends of
// the bracket: 8.8), the largest of 31,886 hexahedra 14 (41): a wavefront
// waits for its slowest cell.  31,886 hexahedra, label pass: 114 us (174 us);
// 24,431 Voronoi cells: 230 us (280 us).
// A narrowed bracket [h_lo, h_hi] starts with a cut at its centre (the network's
// predicted isovalue; a team: and at its ends).  A step that would leave the
// bracket cuts the end it would pass instead; an isovalue found outside has the
// status LEARNED_FALLBACK.  So the flag says that a cut at the end is short of
// the root, as if both ends had been cut, and most cells cut none.
//
// Scheduling: a wavefront takes up to 64/G consecutive mixed entries (a
// batch), stages them together, runs their searches side by side until the
// last one stops, writes them out and claims the next batch.  The batches go
// to the XCDs in runs of consecutive batches (neighbouring cells share an
// L2), and each XCD's wavefronts claim its batches from a counter of its own
// that wraps back to zero after the XCD's last claim.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "recon_common.h"
#include "mlp_core.h"

namespace vofpc {
namespace {

// ---------------------------------------------------------- group reductions
// Sums, minima and maxima over the G consecutive lanes of a group by DPP quad,
// half-row and row butterflies; every lane of the group ends with the same
// bits.
template <int G>
__device__ __forceinline__ double tsum(double v) {
  if constexpr (G >= 2) v += dpp_d<kQuadXor1>(v);
  if constexpr (G >= 4) v += dpp_d<kQuadXor2>(v);
  if constexpr (G >= 8) v += dpp_d<kHalfMirror>(v);
  if constexpr (G >= 16) v += dpp_d<kRowMirror>(v);
  return v;
}
template <int G>
__device__ __forceinline__ int tmin_i(int v) {
  if constexpr (G >= 2) v = min(v, dpp_i<kQuadXor1>(v));
  if constexpr (G >= 4) v = min(v, dpp_i<kQuadXor2>(v));
  if constexpr (G >= 8) v = min(v, dpp_i<kHalfMirror>(v));
  if constexpr (G >= 16) v = min(v, dpp_i<kRowMirror>(v));
  return v;
}
template <int G>
__device__ __forceinline__ double tmin(double v) {
  if constexpr (G >= 2) v = fmin(v, dpp_d<kQuadXor1>(v));
  if constexpr (G >= 4) v = fmin(v, dpp_d<kQuadXor2>(v));
  if constexpr (G >= 8) v = fmin(v, dpp_d<kHalfMirror>(v));
  if constexpr (G >= 16) v = fmin(v, dpp_d<kRowMirror>(v));
  return v;
}
template <int G>
__device__ __forceinline__ double tmax(double v) {
  if constexpr (G >= 2) v = fmax(v, dpp_d<kQuadXor1>(v));
  if constexpr (G >= 4) v = fmax(v, dpp_d<kQuadXor2>(v));
  if constexpr (G >= 8) v = fmax(v, dpp_d<kHalfMirror>(v));
  if constexpr (G >= 16) v = fmax(v, dpp_d<kRowMirror>(v));
  return v;
}

// ------------------------------------------------------------ fast division
// Quotient a/b from the hardware reciprocal, refined by two Newton steps and
// one residual correction (within an ulp of the rounded quotient; b finite
// and nonzero): a few instructions instead of the IEEE division sequence.
__device__ __forceinline__ double qdiv(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  r = fma(fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}
// Square root of x >= 0 from the hardware reciprocal square root, refined by
// two Newton steps and one residual correction (0 for x = 0).
__device__ __forceinline__ double qsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * fma(-0.5 * x * y, y, 1.5);
  y = y * fma(-0.5 * x * y, y, 1.5);
  const double t = x * y;
  return x > 0.0 ? fma(fma(-t, t, x), 0.5 * y, t) : 0.0;
}
// Root of the inverse quadratic through three (isovalue, residual) points,
// about x0 over one common denominator; NaN or infinite when two residuals
// coincide.
__device__ __forceinline__ double iqi1(double x0, double f0, double x1, double f1, double x2, double f2) {
  const double d01 = f0 - f1, d02 = f0 - f2, d12 = f1 - f2;
  return x0 + qdiv((x2 - x0) * f0 * f1 * d01 - (x1 - x0) * f0 * f2 * d02, d01 * d02 * d12);
}

// Where a fraction x of a cell's volume lies above, in widths of [phi_min,
// phi_max] from the mean vertex value: a quantile function with the contact of
// a corner (x ~ distance^(1/0.3)) at both ends.  Fitted to the reconstructed
// isovalues of hexahedra and Voronoi cells cut by bubbles: a mean error of
// 0.03 and 0.06 widths, against 0.15 and 0.23 of the line through the ends.
__device__ __forceinline__ float quantile_power(float x) { return __builtin_amdgcn_exp2f(0.3f * __builtin_amdgcn_logf(x)); }
__device__ __forceinline__ float quantile(double x) {
  const float hi = quantile_power((float)fmin(fmax(x, 0.0), 1.0)), lo = quantile_power((float)fmin(fmax(1.0 - x, 0.0), 1.0));
  return 0.6f * (lo - hi);
}

// Sum over the group of one value per slot (item q + G t in slot t), added
// in the order of the wavefront kernel's reductions (its lane i holds item
// i): within rows of 16 items, then rows 0 + 1, then the rest, so both
// kernels feed the network the same bits.
template <int G, int K>
__device__ __forceinline__ double items_sum(const double (&v)[K]) {
  static_assert(G == 4 || G == 16, "a DPP quad or row per group");
  constexpr int R = (K * G + 15) / 16;   // rows of 16 items
  double r[R];
  if constexpr (G == 16) {
#pragma unroll
    for (int t = 0; t < R; ++t) r[t] = tsum<16>(v[t]);
  } else {
    double s[4 * R];
#pragma unroll
    for (int t = 0; t < 4 * R; ++t) s[t] = t < K ? tsum<4>(v[t < K ? t : 0]) : 0.0;
#pragma unroll
    for (int t = 0; t < R; ++t) r[t] = (s[4 * t] + s[4 * t + 1]) + (s[4 * t + 2] + s[4 * t + 3]);
  }
  double a = r[0];
  if constexpr (R > 1) a += r[1];
  if constexpr (R > 2) {
    double b = r[2];
    if constexpr (R > 3) b += r[3];
    a += b;
  }
  return a;
}
// The group's bits of a wavefront ballot, the group's first lane in bit 0.
template <int G>
__device__ __forceinline__ uint32_t group_bits(bool b, int base) {
  return (uint32_t)(__ballot(b) >> base) & ((1u << G) - 1u);
}

template <int N>
using mask_t = std::conditional_t<(N <= 32), uint32_t, uint64_t>;
__device__ __forceinline__ int count_bits(uint32_t m) { return __popc(m); }
__device__ __forceinline__ int count_bits(uint64_t m) { return __popcll(m); }
__device__ __forceinline__ int first_bit(uint32_t m) { return __ffs((int)m) - 1; }
__device__ __forceinline__ int first_bit(uint64_t m) { return __ffsll((long long)m) - 1; }
__device__ __forceinline__ void or_lds(uint32_t *p, uint32_t v) { atomicOr(p, v); }
__device__ __forceinline__ void or_lds(uint64_t *p, uint64_t v) {
  atomicOr(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}

// ----------------------------------------------------------------- LDS layout
// The staged cells of one wavefront, item-major and cell-slot-minor; the
// 8-byte arrays have an odd slot stride CP, so the lanes of a group, which
// read different items of one cell, spread over the LDS banks.
//
// Network scratch (learned form): a row of inputs and of hidden activations
// per cell (BF16 values held as floats; rows padded by one 16-byte word
// against bank conflicts), the face sums before the activations, and the
// vertex ranks.
template <int C, int NV>
struct NetRows {
  alignas(16) float x[C][net::kIn + 4];
  union {
    alignas(16) float h[C][net::kHid + 4];
    double sum[C][19];
  };
  uint8_t rank[NV][C];   // vertex of each rank
};

template <int C, int CP, int NV, int NF, int NL, int NE>
struct GroupCells {
  double phi[NV][CP];   // vertex field
  double X[NV][CP][3];  // vertex positions relative to the cell centroid
  union {
    // while a cell's registers are filled
    struct {
      mask_t<NE> out[NF][CP], in[NF][CP];   // edges the face's loop runs along u -> v, v -> u
      mask_t<NV> adj[NV][CP];               // vertices joined to each vertex by an edge
      uint32_t fan[NF][CP];                 // smallest vertex of each face: its fan point
    } st;
    NetRows<C, NV> net;   // network phase of the learned form
    // one evaluation
    struct {
      double pt[NE][CP][3];   // crossing point of each cut edge
      uint8_t part[NE][C];    // entry edge of the chord leaving through each cut edge (several loops)
      uint8_t lab[NE][C];     // loop of each cut edge (several loops)
    } ev;
  };
  uint8_t lv[NL][C], eid[NL][C];   // vertex and edge of each loop position (faces with several chords)
  double hint[3][C];    // narrowed bracket of each cell: first cut, lower end, upper end
  double smp[2][C];     // a team's isovalues and residuals
  double fin[9][C];     // what a search ended with: V / V_P, its loops' sums S, A, A k, and whether they failed
};

// per-lane sums of the chords of one loop (or of all loops)
struct ChordAcc {
  double L, M0, M1, M2, Y0, Y1, Y2;
};

template <int G>
__device__ __forceinline__ void reduce_acc(ChordAcc &a) {
  a.L = tsum<G>(a.L);
  a.M0 = tsum<G>(a.M0); a.M1 = tsum<G>(a.M1); a.M2 = tsum<G>(a.M2);
  a.Y0 = tsum<G>(a.Y0); a.Y1 = tsum<G>(a.Y1); a.Y2 = tsum<G>(a.Y2);
}

// The chord from exit point x to entry point e as a loop segment, from its
// entry point u to its exit point w, both relative to the cell's reference
// point r (near a small cut piece, so the cross products of a small loop do
// not cancel).
__device__ __forceinline__ void add_segment(ChordAcc &acc, double r0, double r1, double r2, double x0, double x1,
                                            double x2, double e0, double e1, double e2) {
  const double u0 = e0 - r0, u1 = e1 - r1, u2 = e2 - r2;
  const double w0 = x0 - r0, w1 = x1 - r1, w2 = x2 - r2;
  const double d0 = w0 - u0, d1 = w1 - u1, d2 = w2 - u2;
  const double l = qsqrt(d0 * d0 + d1 * d1 + d2 * d2);
  acc.L += l;
  acc.M0 += l * (u0 + w0);
  acc.M1 += l * (u1 + w1);
  acc.M2 += l * (u2 + w2);
  acc.Y0 += u1 * w2 - u2 * w1;
  acc.Y1 += u2 * w0 - u0 * w2;
  acc.Y2 += u0 * w1 - u1 * w0;
}

// Centroid of a loop from its length sums, k = r + M/(2L) (a loop of zero
// length has zero area: its centre does not matter).
__device__ __forceinline__ void loop_centre(const ChordAcc &a, double r0, double r1, double r2, double &k0, double &k1,
                                            double &k2) {
  k0 = r0; k1 = r1; k2 = r2;
  if (a.L > 0) {
    const double h = qdiv(0.5, a.L);
    k0 += a.M0 * h; k1 += a.M1 * h; k2 += a.M2 * h;
  }
}

// Add one loop's fan: volume k . Y, area vector -Y/2.
__device__ __forceinline__ void finish_loop(const ChordAcc &a, double r0, double r1, double r2, double &Vi, double &S0,
                                            double &S1, double &S2, double &A, double &cw0, double &cw1, double &cw2) {
  double k0, k1, k2;
  loop_centre(a, r0, r1, r2, k0, k1, k2);
  Vi += k0 * a.Y0 + k1 * a.Y1 + k2 * a.Y2;
  const double t0 = -0.5 * a.Y0, t1 = -0.5 * a.Y1, t2 = -0.5 * a.Y2;
  const double Ak = qsqrt(t0 * t0 + t1 * t1 + t2 * t2);
  S0 += t0; S1 += t1; S2 += t2;
  A += Ak;
  cw0 += Ak * k0; cw1 += Ak * k1; cw2 += Ak * k2;
}

// The cell's vertices (positions relative to xP, when WANT_X) and their
// inverse-distance vertex field (or the caller's override) into LDS; lane q
// of a group takes vertices q, q + G, ...  Each lane works KV vertices per
// round with the loads of a round issued together level by level (vertex
// ids; positions and incidence ranges; incidences four at a time; neighbour
// alphas) and sums each vertex's incidences in order.  lo/hi: the lane's
// smallest and largest vertex value.
template <int G, int KV, bool WANT_X, class TM>
__device__ __forceinline__ void stage_vertex_field(TM &M, const DevMesh &m, const ReconParams &p, int sl, int q,
                                                   int64_t v0, int nv, double xP0, double xP1, double xP2, double &lo,
                                                   double &hi) {
  const double *w = p.vertex_mode ? m.vc_wmean : m.vc_w;
  for (int i0 = q; i0 < nv; i0 += KV * G) {
    int gv[KV];
    int64_t jb[KV], je[KV];
    double px[KV], py[KV], pz[KV], ph[KV];
#pragma unroll
    for (int t = 0; t < KV; ++t) {
      const int i = i0 + t * G;
      gv[t] = i < nv ? m.cv_gid[v0 + i] : -1;
    }
#pragma unroll
    for (int t = 0; t < KV; ++t) {
      const bool in = gv[t] >= 0;
      if constexpr (WANT_X) {
        px[t] = in ? m.xyz[gv[t]] : 0.0;
        py[t] = in ? m.xyz[m.n_verts + gv[t]] : 0.0;
        pz[t] = in ? m.xyz[2 * m.n_verts + gv[t]] : 0.0;
      }
      ph[t] = 0.0;
      if (p.phi_override) {
        ph[t] = in ? p.phi_override[gv[t]] : 0.0;
        jb[t] = je[t] = 0;
      } else {
        jb[t] = in ? m.vc_off[gv[t]] : 0;
        je[t] = in ? m.vc_off[gv[t] + 1] : 0;
      }
    }
    bool more = true;
    for (int c4 = 0; more; c4 += 4) {
      int cc[KV][4];
      double ww[KV][4], aa[KV][4];
#pragma unroll
      for (int t = 0; t < KV; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t jj = jb[t] + c4 + u;
          const bool in = jj < je[t];
          cc[t][u] = in ? m.vc_cell[jj] : 0;
          ww[t][u] = in ? w[jj] : 0.0;
        }
#pragma unroll
      for (int t = 0; t < KV; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) aa[t][u] = (jb[t] + c4 + u < je[t]) ? p.alpha[cc[t][u]] : 0.0;
      more = false;
#pragma unroll
      for (int t = 0; t < KV; ++t) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (jb[t] + c4 + u < je[t]) ph[t] += ww[t][u] * aa[t][u];
        more = more || jb[t] + c4 + 4 < je[t];
      }
    }
#pragma unroll
    for (int t = 0; t < KV; ++t) {
      const int i = i0 + t * G;
      if (i < nv) {
        if constexpr (WANT_X) {
          M.X[i][sl][0] = px[t] - xP0;
          M.X[i][sl][1] = py[t] - xP1;
          M.X[i][sl][2] = pz[t] - xP2;
        }
        M.phi[i][sl] = ph[t];
        lo = fmin(lo, ph[t]);
        hi = fmax(hi, ph[t]);
      }
    }
  }
}


// The 32 network inputs of the cell in slot sl (the definitions of the
// features entry point) into its row: face sums over the group's faces, the
// vertex values ordered by rank (ties by index).  Sums in the wavefront
// kernel's order (items_sum).
template <int G, int KF, int KV, class TM>
__device__ __forceinline__ void cell_features(TM &M, int sl, int q, const ReconParams &p, int P, double a, int nv,
                                              int nf, int64_t f0, double pmin, double Wd) {
  double A[KF], n0[KF], n1[KF], n2[KF], da[KF], t[KF];
  double amin = __builtin_inf(), amax = -__builtin_inf();
  double *ns = &M.net.sum[sl][0];
  {
    double aq[KF], in[KF];
#pragma unroll
    for (int k = 0; k < KF; ++k) {
      const int f = q + k * G;
      A[k] = n0[k] = n1[k] = n2[k] = da[k] = aq[k] = in[k] = 0.0;
      if (f < nf) {
        const NetFace g = load_net_face(p, P, a, f0 + f);
        A[k] = sqrt(g.S0 * g.S0 + g.S1 * g.S1 + g.S2 * g.S2);
        n0[k] = g.S0 / A[k]; n1[k] = g.S1 / A[k]; n2[k] = g.S2 / A[k];
        da[k] = A[k] * (g.aQ - a);
        if (g.inner) {
          aq[k] = g.aQ;
          in[k] = 1.0;
          amin = fmin(amin, g.aQ);
          amax = fmax(amax, g.aQ);
        }
      }
    }
    const double s16 = items_sum<G>(aq), s17 = items_sum<G>(in), s0 = items_sum<G>(A);
    if (q == 0) {
      ns[0] = s0;
      ns[16] = s16;
      ns[17] = s17;
    }
  }
  amin = tmin<G>(amin);
  amax = tmax<G>(amax);
  auto red = [&](int i) {
    const double s = items_sum<G>(t);
    if (q == 0) ns[i] = s;
  };
#define NET_SUM(i, expr)                         \
  _Pragma("unroll") for (int k = 0; k < KF; ++k) t[k] = (expr); \
  red(i);
  NET_SUM(1, da[k] * n0[k])
  NET_SUM(2, da[k] * n1[k])
  NET_SUM(3, da[k] * n2[k])
  NET_SUM(4, da[k] * n0[k] * n0[k])
  NET_SUM(5, da[k] * n1[k] * n1[k])
  NET_SUM(6, da[k] * n2[k] * n2[k])
  NET_SUM(7, da[k] * n0[k] * n1[k])
  NET_SUM(8, da[k] * n0[k] * n2[k])
  NET_SUM(9, da[k] * n1[k] * n2[k])
  NET_SUM(10, A[k] * n0[k] * n0[k])
  NET_SUM(11, A[k] * n1[k] * n1[k])
  NET_SUM(12, A[k] * n2[k] * n2[k])
  NET_SUM(13, A[k] * n0[k] * n1[k])
  NET_SUM(14, A[k] * n0[k] * n2[k])
  NET_SUM(15, A[k] * n1[k] * n2[k])
#undef NET_SUM
  // ranks of the vertex values
  double v[KV];
  int r[KV];
#pragma unroll
  for (int k = 0; k < KV; ++k) {
    v[k] = q + k * G < nv ? M.phi[q + k * G][sl] : 0.0;
    r[k] = 0;
  }
#pragma unroll 4
  for (int j = 0; j < nv; ++j) {
    const double u = M.phi[j][sl];
#pragma unroll
    for (int k = 0; k < KV; ++k) r[k] += (u < v[k]) || (u == v[k] && j < q + k * G);
  }
#pragma unroll
  for (int k = 0; k < KV; ++k)
    if (q + k * G < nv) M.net.rank[r[k]][sl] = (uint8_t)(q + k * G);
  const double lsum = items_sum<G>(v);
  wave_sync();
  // (ranks of values that are not numbers are not all written)
  auto sorted = [&](int i) { return M.phi[min((int)M.net.rank[i][sl], nv - 1)][sl]; };
  for (int i = q; i < net::kIn; i += G)
    M.net.x[sl][i] = net::from_bf16(net::to_bf16(net::feature(i, a, sorted, nv, lsum, pmin, Wd, ns, amin, amax, nf)));
}

// ------------------------------------------------------------- the network
// Output 0 of the network for the cells of a wavefront, every sum in the order
// of the wavefront kernel's row_forward, so all flavours predict the same bits.
// The products go through the FP32 matrix instructions of one step (K = 1): each
// result is one fused multiply-add a step, as the chain of v_fma_f32 that
// row_forward runs (BF16 weights and activations are exact in FP32; compared
// over ordinary, wide, denormal and cancelling operands: no bit differs).
// Lane l holds the weights of unit l as operand A, so a wavefront reads the
// weights once for all its cells and unpacks each once.  With the units dealt to
// a cell's lanes and the products on the vector ALU a step over 113,584 cells took
// 777 us, now 673; one over 366,598 cells 2,141 us, now 1,905 (the class
// kernels alone: 151,485 hexahedra 419, now 303; 214,287 Voronoi cells 1,392, now
// 1,278).

// the two BF16 values of a word
__device__ __forceinline__ float bf16_low(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_high(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// z += W x over one layer of K inputs: w the weights of unit `lane`, x the row
// of this lane's column (4 or 16 cells); step(a, b, z) one matrix instruction
template <int K, class Acc, class Step>
__device__ __forceinline__ void net_layer(const uint16_t *wts, const float *x, int lane, Acc &z, Step step) {
  const uint4 *w = reinterpret_cast<const uint4 *>(wts + lane * K);
  uint4 r[K / 8];
#pragma unroll
  for (int i = 0; i < K / 8; ++i) r[i] = w[i];
#pragma unroll
  for (int i = 0; i < K / 8; ++i) {
    const float4 xa = *reinterpret_cast<const float4 *>(x + 8 * i), xb = *reinterpret_cast<const float4 *>(x + 8 * i + 4);
    step(bf16_low(r[i].x), xa.x, z);
    step(bf16_high(r[i].x), xa.y, z);
    step(bf16_low(r[i].y), xa.z, z);
    step(bf16_high(r[i].y), xa.w, z);
    step(bf16_low(r[i].z), xb.x, z);
    step(bf16_high(r[i].z), xb.y, z);
    step(bf16_low(r[i].w), xb.z, z);
    step(bf16_high(r[i].w), xb.w, z);
  }
}
__device__ __forceinline__ float net_act(float z) { return net::from_bf16(net::to_bf16(net::act_tanh(z))); }

// sum over the four units 4i .. 4i + 3 of the third layer's terms
__device__ __forceinline__ float net_quad(const uint16_t *wb, const float *master, int u, const float (&z)[4]) {
  using namespace net;
  const f32x4 b = *reinterpret_cast<const f32x4 *>(master + oB2 + u);
  const uint2 w = *reinterpret_cast<const uint2 *>(wb + oW3 + u);
  return (bf16_low(w.x) * net_act(z[0] + b[0]) + bf16_high(w.x) * net_act(z[1] + b[1])) +
         (bf16_low(w.y) * net_act(z[2] + b[2]) + bf16_high(w.y) * net_act(z[3] + b[3]));
}

// Four cells, v_mfma_f32_4x4x1_16b_f32: lane l has cell l % 4 (its rows x and
// h) and, as results, the units 4 (l / 4) + j, j = 0 .. 3.
__device__ __forceinline__ float net_four(const float *x, float *h, int lane, const uint16_t *wb, const float *master) {
  using namespace net;
  auto step = [](float a, float b, f32x4 &z) { z = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, z, 0, 0, 0); };
  const int u = lane & ~3;
  f32x4 z = {0.f, 0.f, 0.f, 0.f};
  net_layer<kIn>(wb + oW1, x, lane, z, step);
  const f32x4 b1 = *reinterpret_cast<const f32x4 *>(master + oB1 + u);
  f32x4 a;
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = net_act(z[j] + b1[j]);
  *reinterpret_cast<f32x4 *>(h + u) = a;
  wave_sync();
  z = f32x4{0.f, 0.f, 0.f, 0.f};
  net_layer<kHid>(wb + oW2, h, lane, z, step);
  const float zq[4] = {z[0], z[1], z[2], z[3]};
  // the quads of units are 4 lanes apart: sums over lanes l ^ 4, l ^ 8 (two
  // mirrors each), and the rows of 16 lanes
  auto mirror = [](float v, auto ctrl) {
    return __builtin_bit_cast(float, dpp_i<decltype(ctrl)::value>(__builtin_bit_cast(int, v)));
  };
  std::integral_constant<int, kHalfMirror> half;
  std::integral_constant<int, kRowMirror> whole;
  std::integral_constant<int, 0x1B> quad;   // lanes 3, 2, 1, 0 of each quad
  float v = net_quad(wb, master, u, zq);
  v += mirror(mirror(v, half), quad);
  v += mirror(mirror(v, whole), half);
  return cross_sum_f<32>(cross_sum_f<16>(v)) + master[oB3];
}

// Sixteen cells, v_mfma_f32_16x16x1_4b_f32: lane l has cell l % 16 and the units
// 16 b + 4 (l / 16) + j.
__device__ __forceinline__ float net_sixteen(const float *x, float *h, int lane, const uint16_t *wb,
                                             const float *master) {
  using namespace net;
  typedef float f32x16 __attribute__((ext_vector_type(16)));
  auto step = [](float a, float b, f32x16 &z) { z = __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, z, 0, 0, 0); };
  const int u = 4 * (lane >> 4);
  f32x16 z = 0.f;
  net_layer<kIn>(wb + oW1, x, lane, z, step);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const f32x4 b1 = *reinterpret_cast<const f32x4 *>(master + oB1 + 16 * b + u);
    f32x4 a;
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = net_act(z[4 * b + j] + b1[j]);
    *reinterpret_cast<f32x4 *>(h + 16 * b + u) = a;
  }
  wave_sync();
  z = 0.f;
  net_layer<kHid>(wb + oW2, h, lane, z, step);
  float row[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const float zq[4] = {z[4 * b], z[4 * b + 1], z[4 * b + 2], z[4 * b + 3]};
    row[b] = cross_sum_f<32>(cross_sum_f<16>(net_quad(wb, master, 16 * b + u, zq)));
  }
  return ((row[0] + row[1]) + (row[2] + row[3])) + master[oB3];
}

// One cell, one unit a lane: the vector ALU (a matrix instruction has four cells
// at least).
__device__ __forceinline__ float net_one(const float *x, float *h, int lane, const uint16_t *wb, const float *master) {
  using namespace net;
  auto step = [](float a, float b, float &z) { z = __builtin_fmaf(a, b, z); };
  float z = 0.f;
  net_layer<kIn>(wb + oW1, x, lane, z, step);
  h[lane] = net_act(z + master[oB1 + lane]);
  wave_sync();
  z = 0.f;
  net_layer<kHid>(wb + oW2, h, lane, z, step);
  return wave_sum_f(from_bf16(wb[oW3 + lane]) * net_act(z + master[oB2 + lane])) + master[oB3];
}

// Largest cell of a build (vertices, faces, loop positions, edges), its
// group size and the slot stride of its LDS arrays.
template <int G_, int NV_, int NF_, int NL_, int NE_, int CP_ = (64 / G_) | 1>
struct Build {
  static constexpr int G = G_, NV = NV_, NF = NF_, NL = NL_, NE = NE_;
  using Mem = GroupCells<64 / G_, CP_, NV_, NF_, NL_, NE_>;
  static __device__ __host__ bool fits(int64_t nv, int64_t nf, int64_t nl) {
    return nv <= NV && nf <= NF && nl <= NL && nl / 2 <= NE;
  }
};

// The groups of a wavefront: cw cells per batch, ts groups (a team) per cell.
struct Team {
  int lane, sl, q, base;   // lane, its group, its place in the group, the group's first lane
  int cw, ts, g, lead;     // g: the group's place in its team, lead: the team's first group
  int weight;              // evaluations a step of the search counts as
};

// A mixed entry and its cell's place in the mesh arrays.
struct CellRef {
  int64_t k = 0, f0 = 0, v0 = 0, l0 = 0;
  int P = 0, nf = 0, nv = 0, nl = 0;
  double a = 0.0;
};

// The active groups' cells: staging, bracket, search and outputs.
template <class Caps, bool NET>
__device__ __forceinline__ void solve_cells(const ReconParams &p, typename Caps::Mem &M, const Team &tm,
                                            const CellRef &cell, bool active) {
  constexpr int G = Caps::G, C = 64 / G, NV = Caps::NV, NE = Caps::NE;
  constexpr int KE = (NE + G - 1) / G, KF = (Caps::NF + G - 1) / G, KV = (NV + G - 1) / G,
                KL = (Caps::NL + G - 1) / G;
  using EM = mask_t<NE>;
  using VM = mask_t<NV>;
  const int lane = tm.lane, sl = tm.sl, q = tm.q, base = tm.base, cw = tm.cw, ts = tm.ts, g = tm.g, lead = tm.lead;
  const DevMesh &m = p.m;
  const int64_t N = m.n_cells, cap = p.out.cap;
  // ---- phase 1, per cell: checks and staging
  const int64_t k = cell.k, f0 = cell.f0, v0 = cell.v0, l0 = cell.l0;
  const int P = cell.P, nf = cell.nf, nv = cell.nv, ne = cell.nl / 2;   // a closed surface uses every edge twice
  const double a = cell.a;
  int st = VOFPC_CELL_OK, it = 0;
  double VP = 1.0, pmin = 0.0, pmax = 0.0;
  bool have_field = false;
  double s_out = __builtin_nan(""), A_out = 0, d_out = 0, n0 = 0, n1 = 0, n2 = 0, ag = a;
  uint32_t ew[KE];   // the lane's edge records
  uint32_t fl[KF];   // and its faces' loops: first position, positions << 16
  if (active) {
    if (!(a >= 0.0 && a <= 1.0)) {
      st = VOFPC_CELL_BAD_INPUT;
    } else if (!(a > p.eps && a < 1.0 - p.eps)) {
      st = VOFPC_CELL_NOT_MIXED;
    } else if (!Caps::fits(nv, nf, cell.nl)) {
      st = VOFPC_CELL_BAD_INPUT;   // cannot happen: the launcher sizes the build by the class
    } else {
      const double xP0 = m.xc[P], xP1 = m.xc[N + P], xP2 = m.xc[2 * N + P];
      VP = m.V[P];
#pragma unroll
      for (int t = 0; t < KE; ++t) {
        const int e = q + t * G;
        ew[t] = e < ne ? m.ce[(l0 >> 1) + e] : 0u;
      }
      uint8_t tl[KL], te[KL];
#pragma unroll
      for (int t = 0; t < KL; ++t) {
        const int i = q + t * G;
        tl[t] = i < cell.nl ? m.cl_lv[l0 + i] : (uint8_t)0;
        te[t] = i < cell.nl ? (uint8_t)m.cl_eid[l0 + i] : (uint8_t)0;
      }
#pragma unroll
      for (int t = 0; t < KF; ++t) {
        const int f = q + t * G;
        fl[t] = f < nf ? (uint32_t)m.cf_loff[f0 + f] | (uint32_t)m.cf_lsz[f0 + f] << 16 : 0u;
      }
      // the vertices with the inverse-distance vertex field, level by
      // level (ids, positions and incidence ranges, incidences, neighbour
      // alphas), so the latencies of a level's loads overlap
      constexpr int KS = KV < 2 ? KV : 2;   // vertices per lane per round
      double lo_phi = __builtin_inf(), hi_phi = -__builtin_inf();
      stage_vertex_field<G, KS, true>(M, m, p, sl, q, v0, nv, xP0, xP1, xP2, lo_phi, hi_phi);
#pragma unroll
      for (int t = 0; t < KL; ++t) {
        const int i = q + t * G;
        if (i < cell.nl) {
          M.lv[i][sl] = tl[t];
          M.eid[i][sl] = te[t];
        }
      }
      pmin = tmin<G>(lo_phi);
      pmax = tmax<G>(hi_phi);
      have_field = true;
      wave_sync();
      if (pmax - pmin <= 1e-12) {
        // degenerate vertex field: linear alpha from the plain least-squares
        // gradient over the interior face neighbours
        st = VOFPC_CELL_DEGENERATE;
        double gxx = 0, gyy = 0, gzz = 0, gxy = 0, gxz = 0, gyz = 0, b0 = 0, b1 = 0, b2 = 0;
        for (int f = q; f < nf; f += G) {
          const int qq = m.cf_nbr[f0 + f];
          if (qq < 0) continue;
          const double r0 = m.xc[qq] - xP0, r1 = m.xc[N + qq] - xP1, r2 = m.xc[2 * N + qq] - xP2;
          const double dv = p.alpha[qq] - a;
          gxx += r0 * r0; gyy += r1 * r1; gzz += r2 * r2; gxy += r0 * r1; gxz += r0 * r2; gyz += r1 * r2;
          b0 += r0 * dv; b1 += r1 * dv; b2 += r2 * dv;
        }
        gxx = tsum<G>(gxx); gyy = tsum<G>(gyy); gzz = tsum<G>(gzz);
        gxy = tsum<G>(gxy); gxz = tsum<G>(gxz); gyz = tsum<G>(gyz);
        b0 = tsum<G>(b0); b1 = tsum<G>(b1); b2 = tsum<G>(b2);
        const double c00 = gyy * gzz - gyz * gyz, c01 = gxz * gyz - gxy * gzz, c02 = gxy * gyz - gxz * gyy;
        const double c11 = gxx * gzz - gxz * gxz, c12 = gxy * gxz - gxx * gyz, c22 = gxx * gyy - gxy * gxy;
        const double det = gxx * c00 + gxy * c01 + gxz * c02;
        const double tr = (gxx + gyy + gzz) / 3.0;
        double g0 = 0, g1 = 0, g2 = 0;
        if (det > 1e-12 * tr * tr * tr) {
          g0 = (c00 * b0 + c01 * b1 + c02 * b2) / det;
          g1 = (c01 * b0 + c11 * b1 + c12 * b2) / det;
          g2 = (c02 * b0 + c12 * b1 + c22 * b2) / det;
        }
        lo_phi = __builtin_inf();
        hi_phi = -__builtin_inf();
        for (int i = q; i < nv; i += G) {
          const double ph = a + (g0 * M.X[i][sl][0] + g1 * M.X[i][sl][1] + g2 * M.X[i][sl][2]);
          M.phi[i][sl] = ph;
          lo_phi = fmin(lo_phi, ph);
          hi_phi = fmax(hi_phi, ph);
        }
        pmin = tmin<G>(lo_phi);
        pmax = tmax<G>(hi_phi);
        if (pmax - pmin <= 1e-12) have_field = false;
        wave_sync();
      }
    }
  }
  // ---- phase 2: the narrowed bracket of every cell with a vertex field,
  // from the network or the caller (a fixed isovalue has no search and none)
  bool hint = false;
  if constexpr (NET) {
    double nlo = __builtin_nan(""), nhi = __builtin_nan("");   // none where the network does not run
    const bool row = active && have_field && st == VOFPC_CELL_OK;   // degenerate fields skip the network
    const double Wd = pmax - pmin;
    if (row) cell_features<G, KF, KV>(M, sl, q, p, P, a, nv, nf, f0, pmin, Wd);
    wave_sync();
    // all lanes: the cells of a tile are its columns, each by itself, and those
    // without a row are not used
    float u = 0.f;
    if (__any(row)) {
      if (cw == 1) {
        u = net_one(M.net.x[0], M.net.h[0], lane, p.net_wb, p.net_master);
      } else if (cw == 4) {
        const int at = (lane & 3) * ts;
        u = __shfl(net_four(M.net.x[at], M.net.h[at], lane, p.net_wb, p.net_master), lead / ts);
      } else {
        if constexpr (C == 16)
          u = __shfl(net_sixteen(M.net.x[lane & 15], M.net.h[lane & 15], lane, p.net_wb, p.net_master), sl);
      }
    }
    if (row) {
      if (!isnan(u)) {
        const double uc = u < 0.f ? 0.0 : (u > 1.f ? 1.0 : (double)u);
        const double sh = pmin + uc * Wd, dl = p.net_delta * Wd;
        nlo = sh - dl;
        nhi = sh + dl;
        const double hl = nlo > pmin ? nlo : pmin, hh = nhi < pmax ? nhi : pmax;
        hint = hl <= hh && !p.fixed_iso;
        M.hint[0][sl] = sh < hl ? hl : (sh > hh ? hh : sh);
        M.hint[1][sl] = hl;
        M.hint[2][sl] = hh;
      }
    }
    if (active && q == 0 && g == 0 && p.net_lo) {
      p.net_lo[k] = nlo;
      p.net_hi[k] = nhi;
    }
    wave_sync();
  } else {
    if (active && have_field && p.use_hint && !p.fixed_iso) {
      double hl = p.hint_lo[k], hh = p.hint_hi[k];
      if (!isnan(hl) && !isnan(hh)) {
        hl = hl > pmin ? hl : pmin;
        hh = hh < pmax ? hh : pmax;
        hint = hl <= hh;
        M.hint[0][sl] = hl + (hh - hl) / 2.0;
        M.hint[1][sl] = hl;
        M.hint[2][sl] = hh;
      }
    }
  }
  // ---- phase 3, per cell: registers of the search, the search, the outputs
  if (active && have_field) {
    // edges from their end of larger value u (liquid whenever the edge is
    // cut) to v: values, 1/(phi_v - phi_u), and the whole-edge volume term
    // of its two faces' fans, det(c1, u, v) + det(c2, v, u); the face whose
    // loop runs u -> v takes the edge as an exit of the iso-curve, the other
    // one as an entry.  Missing edges are never liquid and never cut.
    double pu[KE], pv[KE], iv[KE], D[KE];
    EM fo[KF], fi[KF];
    int fc[KF];       // fan vertex of each face
    double pw[KV];
    VM adj[KV];
    int rv;           // reference vertex of the loop sums
    for (int f = q; f < nf; f += G) {
      M.st.out[f][sl] = 0;
      M.st.in[f][sl] = 0;
      M.st.fan[f][sl] = 0xffffffffu;
    }
    for (int i = q; i < nv; i += G) M.st.adj[i][sl] = 0;
    wave_sync();
#pragma unroll
    for (int t = 0; t < KE; ++t) {
      const int e = q + t * G;
      pu[t] = pv[t] = -__builtin_inf();
      iv[t] = D[t] = 0.0;
      if (e < ne) {
        const uint32_t wv = ew[t];
        int u = (int)(wv & 0xffu), v = (int)((wv >> 8) & 0xffu), f1 = (int)((wv >> 16) & 0xffu), f2 = (int)(wv >> 24);
        pu[t] = M.phi[u][sl];
        pv[t] = M.phi[v][sl];
        if (pv[t] > pu[t]) {
          const double x = pu[t];
          pu[t] = pv[t];
          pv[t] = x;
          int i = u;
          u = v;
          v = i;
          i = f1;
          f1 = f2;
          f2 = i;
          ew[t] = (uint32_t)u | (uint32_t)v << 8 | (uint32_t)f1 << 16 | (uint32_t)f2 << 24;
        }
        iv[t] = qdiv(1.0, pv[t] - pu[t]);   // not used when the values are equal
        or_lds(&M.st.out[f1][sl], (EM)1 << e);
        or_lds(&M.st.in[f2][sl], (EM)1 << e);
        or_lds(&M.st.adj[u][sl], (VM)1 << v);
        or_lds(&M.st.adj[v][sl], (VM)1 << u);
        const uint32_t lowv = (uint32_t)(u < v ? u : v);
        atomicMin(&M.st.fan[f1][sl], lowv);
        atomicMin(&M.st.fan[f2][sl], lowv);
      }
    }
    wave_sync();
#pragma unroll
    for (int t = 0; t < KE; ++t) {
      if (q + t * G >= ne) continue;
      const double *c1 = M.X[M.st.fan[(ew[t] >> 16) & 0xffu][sl]][sl], *c2 = M.X[M.st.fan[ew[t] >> 24][sl]][sl];
      const double *u = M.X[ew[t] & 0xffu][sl], *v = M.X[(ew[t] >> 8) & 0xffu][sl];
      D[t] = det3(c1[0] - c2[0], c1[1] - c2[1], c1[2] - c2[2], u[0], u[1], u[2], v[0], v[1], v[2]);
    }
#pragma unroll
    for (int t = 0; t < KF; ++t) {
      const int f = q + t * G;
      const bool in = f < nf;
      fo[t] = in ? M.st.out[f][sl] : 0;
      fi[t] = in ? M.st.in[f][sl] : 0;
      fc[t] = in ? (int)M.st.fan[f][sl] : 0;
    }
    // reference point of the loop sums: the vertex of largest value when
    // the cell is mostly vapour (a small liquid piece sits at it), else
    // the vertex of smallest value (the smallest index among ties)
    {
      const double want = a < 0.5 ? pmax : pmin;
      int cand = 0x7fffffff;
#pragma unroll
      for (int t = KV - 1; t >= 0; --t) {
        const int i = q + t * G;
        pw[t] = i < nv ? M.phi[i][sl] : -__builtin_inf();
        adj[t] = i < nv ? M.st.adj[i][sl] : 0;
        if (i < nv && pw[t] == want) cand = i;
      }
      rv = tmin_i<G>(cand);
    }
    wave_sync();   // the staging masks give way to the evaluations' points
    const VM all = (VM)(~(VM)0) >> (8 * (int)sizeof(VM) - nv);
    VM seen = 0;           // liquid vertices of the last flood fill
    bool single = false;   // and whether it found one loop
    uint32_t many = 0;     // the lane's faces with four or more crossings at the last evaluation (bit per slot)
    const double far = 0.01 * (pmax - pmin);

    // face-mean vertex value of the lane's face in slot t (vertex values
    // added in loop order)
    auto face_mean = [&](int t) {
      const int o = (int)(fl[t] & 0xffffu), n = (int)(fl[t] >> 16);
      double fm = 0.0;
      for (int i = 0; i < n; ++i) fm += M.phi[M.lv[o + i][sl]][sl];
      return fm / (double)n;
    };
    // One evaluation site; the phase decides where the next one is: the
    // fixed isovalue, the first estimate, the search's, or the bracket end
    // kept when the search cannot stop.
    enum { kFixed, kStart, kSearch, kFinal };
    const double iVP = 1.0 / VP;
    const double tol = p.tol_rel * (a < 1.0 - a ? a : 1.0 - a);
    // The search on the residual r(s) = V(s)/V_P - alpha: [xa, xb] is the
    // bracket (r > 0 at xa); one cell per group remembers its last three cuts
    // (the newest is a bracket end, (xc, fcv) and (xd, fd) the two before it)
    // and takes the inverse quadratic interpolation through them, with two
    // cuts the secant, with one the distance between the quantiles of its
    // volume and of alpha, with none the quantile of alpha; the midpoint of
    // the bracket when that falls outside it or does not shrink fast enough
    // against the steps before (the rule of Brent 1973, ch. 4).  In a team,
    // (xc, fcv) is the cut of smallest residual off the bracket.
    double xa = pmin, fa = 1.0 - a, xb = pmax, fb = -a, xc = 0, fcv = 0, xd = 0, fd = 0;
    int cuts = 0;
    bool bis = false;
    const float qa = quantile(a);
    if (!hint) {
      double ps = 0.0;
#pragma unroll
      for (int t = 0; t < KV; ++t)
        if (q + t * G < nv) ps += pw[t];
      const double W = pmax - pmin;
      double guess = tsum<G>(ps) / (double)nv + W * (double)qa;
      guess = fmin(guess, pmax - 0.3 * W * (double)quantile_power((float)a));
      guess = fmax(guess, pmin + 0.3 * W * (double)quantile_power((float)(1.0 - a)));
      M.hint[0][sl] = guess;   // the first cut, in the place of a narrowed bracket's centre
    }
    // a jump of V: where a face with four or more crossings switches its
    // pairing (at its vertex-value mean) or a loop pinches at a vertex
    // (at that vertex's value), V may step over alpha V_P and the search
    // bisects down to two ulps.  From the second bisection step in a row
    // on a bracket narrower than a hundredth of [phi_min, phi_max], such
    // a value inside the bracket (the one nearest the bisection point)
    // is cut instead, then the adjacent double on the root's side: a
    // sign change between the two pins the bracket to one ulp (at most
    // four tries per cell).
    double xj = 0.0;
    int jtries = 0, nbis = 0;   // nbis in a team: steps in a row that hardly lowered the residual
    bool jnext = false, jpin = false, above = false;   // above: the last residual was positive
    int ph = p.fixed_iso ? kFixed : kStart;
    double se;
    while (true) {
      if (ph >= kStart) {
        const double big = fabs(xa) > fabs(xb) ? fabs(xa) : fabs(xb);
        const bool collapsed = fabs(xb - xa) <= 2.0 * ulp_of(big);
        if (collapsed || it >= p.max_iter) {
          // no isovalue meets the tolerance: the end of smaller residual
          const bool b = fabs(fb) <= fabs(fa) && !(ts > 1 && fabs(fa) == fabs(fb));
          se = b ? xb : xa;
          if (!collapsed) st = VOFPC_CELL_MAX_ITER;
          else if (fabs(b ? fb : fa) > 1e-10) st = VOFPC_CELL_NO_ROOT;
          ph = kFinal;
        } else {
          const double blo = xa, bhi = xb, w = xb - xa, mid = xa + w * 0.5;
          // the points of the estimate: a group's last cuts; a team's bracket
          // ends and its third point
          const double x1 = ts == 1 && above ? xa : xb, f1 = ts == 1 && above ? fa : fb;
          const double x2 = ts == 1 ? xc : xa, f2 = ts == 1 ? fcv : fa, x3 = ts == 1 ? xd : xc, f3 = ts == 1 ? fd : fcv;
          const bool three = f1 != f3 && f2 != f3 && (ts > 1 || cuts > 2);
          const double sec = x1 - f1 * qdiv(x1 - x2, f1 - f2);
          const double qi = iqi1(x2, f2, x1, f1, x3, f3);
          bool look = false;
          ph = ts == 1 ? kSearch : ph;
          if (ts == 1) {
            if (jnext) {
              // the double next to the tried value, on the root's side
              jnext = false;
              se = above ? next_up(xj) : -next_up(-xj);
            }
            if (!(jpin && se > blo && se < bhi)) {
              se = three ? qi : sec;
              if (cuts < 2)
                se = cuts == 0 ? M.hint[0][sl] : x1 + (pmax - pmin) * (double)(qa - quantile(f1 + a));
              const double lastd = bis ? fabs(x1 - x2) : fabs(x2 - x3);
              bis = !(se > blo && se < bhi) || nbis >= 3 ||
                    (cuts > 2 && (fabs(se - x1) >= 0.5 * lastd || lastd < 4.0 * ulp_of(x1)));
              if (bis) {
                // at a residual of rounding noise (the tolerance of a small
                // alpha is below it): close in on the root from its near side,
                // in growing steps, before halving the bracket
                const bool near_a = fabs(fa) <= fabs(fb);
                const double d = ldexp(ulp_of(x1), 3 + 2 * (nbis < 16 ? nbis : 16));
                const bool noise = fmin(fabs(fa), fabs(fb)) < 0x1p-46 && d < 0.5 * w;
                se = noise ? (near_a ? xa + d : xb - d) : mid;
              }
              look = nbis >= 2;
            }
            jpin = false;
          } else {
            // a team's isovalues: the estimate; pairs of points around it at
            // distances spread over the scale of its correction of the secant
            // (a sixteenth of it with four isovalues, 8 times it down to a
            // 4096th with sixteen); and points that divide the bracket evenly,
            // in place of those that fall outside it, and of all but the
            // estimate after a step that hardly lowered the residual
            double e0 = ph == kStart ? M.hint[0][sl] : (three ? qi : sec);
            if (!(e0 > blo && e0 < bhi)) e0 = sec;
            if (!(e0 > blo && e0 < bhi)) e0 = mid;
            const int pairs = ts == 4 ? 1 : 6;
            const double du = 16.0 * ulp_of(e0);
            double d = ldexp(fabs(e0 - sec), ts == 4 ? -4 : 3 - 3 * ((g - 1) >> 1));
            if (ph == kStart) {   // what the first estimate is worth
              d = hint ? 0.25 * (M.hint[2][sl] - M.hint[1][sl]) : 0.12 * w;
              d = ldexp(d, ts == 4 ? 0 : 1 - ((g - 1) >> 1));
            }
            d = d > du ? d : du;
            const bool even = nbis >= 1;
            se = g == 0 ? e0 : ((g & 1) ? e0 - d : e0 + d);
            const double part = (even || g <= 2 * pairs) ? (double)g / (double)ts
                                                         : (double)(g - 2 * pairs) / (double)(ts - 2 * pairs);
            if ((even && g > 0) || g > 2 * pairs || !(se > blo && se < bhi)) se = blo + w * part;
            look = nbis >= 2;
            ph = kSearch;
          }
          if (look && jtries < 4 && w <= far) {
            // candidates: the means of the faces with four or more
            // crossings at the last evaluation, and the vertex values
            double bd = __builtin_inf(), bv = __builtin_inf();
            auto candidate = [&](double sj) {
              const double d = fabs(sj - mid);
              if (sj > blo && sj < bhi && sj != xj && (d < bd || (d == bd && sj < bv))) {
                bd = d;
                bv = sj;
              }
            };
#pragma unroll
            for (int t = 0; t < KF; ++t)
              if ((many >> t) & 1) candidate(face_mean(t));
#pragma unroll
            for (int t = 0; t < KV; ++t)
              if (q + t * G < nv) candidate(pw[t]);
            double bdm = tmin<G>(bd);
            double cj = tmin<G>(bd == bdm ? bv : __builtin_inf());
            if (ts > 1) {
              // (the groups' last cuts, and so their face means, differ)
              if (q == 0) {
                M.smp[0][sl] = cj;
                M.smp[1][sl] = bdm;
              }
              wave_sync();
              const int i = lead + (lane & (ts - 1));
              bd = M.smp[1][i];
              bv = M.smp[0][i];
              bdm = tmin<16>(bd);
              cj = tmin<16>(bd == bdm ? bv : __builtin_inf());
              wave_sync();
            }
            if (cj < __builtin_inf()) {
              if (ts == 1 || g == 0) se = cj;
              if (ts > 1 && g == 1) se = next_up(cj);
              if (ts > 1 && g == 2) se = -next_up(-cj);
              xj = cj;
              jnext = jpin = ts == 1;
              ++jtries;
            }
          }
          if (hint) {
            // a step that would leave the narrowed bracket cuts its end first:
            // the bracket ends then meet the tolerance, hold the root or are
            // known to be short of it.  A team cuts both ends in its first step.
            const double hl = M.hint[1][sl], hh = M.hint[2][sl];
            const bool lo_open = hl > blo && hl < bhi, hi_open = hh > blo && hh < bhi;
            const bool at_lo = lo_open && (ts == 1 ? se < hl : g == 1), at_hi = hi_open && (ts == 1 ? se > hh : g == 2);
            if (at_lo || at_hi) {
              se = at_lo ? hl : hh;
              jnext = jpin = false;
            }
          }
        }
      } else {
        se = p.iso;
      }
      // ---- the evaluation at se: edges
      double vf = 0.0;
      EM cut = 0;
#pragma unroll
      for (int t = 0; t < KE; ++t) {
        const bool lv = pv[t] >= se, c = pu[t] >= se && !lv;
        const double lam = (se - pu[t]) * iv[t];
        vf = fma(lv ? 1.0 : (c ? lam : 0.0), D[t], vf);
        if (c) {
          const double *u = M.X[ew[t] & 0xffu][sl], *v = M.X[(ew[t] >> 8) & 0xffu][sl];
          double *x = M.ev.pt[q + t * G][sl];
          const double u0 = u[0], u1 = u[1], u2 = u[2];
          x[0] = u0 + lam * (v[0] - u0);
          x[1] = u1 + lam * (v[1] - u1);
          x[2] = u2 + lam * (v[2] - u2);
        }
        cut |= (EM)group_bits<G>(c, base) << (t * G);
      }
      // one loop or several: flood fill when the liquid vertices changed
      VM lm = 0;
#pragma unroll
      for (int t = 0; t < KV; ++t) lm |= (VM)group_bits<G>(pw[t] >= se, base) << (t * G);
      lm &= all;
      if (__any(lm != seen)) {
        const VM vm = ~lm & all;
        VM r = (lm & (~lm + 1)) | (vm & (~vm + 1));
        bool grow = true;
        while (__any(grow)) {
          VM nr = r;
#pragma unroll
          for (int t = 0; t < KV; ++t) {
            const VM same = pw[t] >= se ? lm : vm;
            nr |= (VM)group_bits<G>((adj[t] & same & r) != 0, base) << (t * G);
          }
          grow = nr != r;
          r = nr;
        }
        single = r == all;
        seen = lm;
      }
      wave_sync();
      // faces with one chord
      ChordAcc acc{0, 0, 0, 0, 0, 0, 0};
      const double r0 = M.X[rv][sl][0], r1 = M.X[rv][sl][1], r2 = M.X[rv][sl][2];
      many = 0;
#pragma unroll
      for (int t = 0; t < KF; ++t) {
        const EM ex = cut & fo[t], en = cut & fi[t];
        if ((ex | en) == 0) continue;
        if (ex == 0 || en == 0 || ((ex & (ex - 1)) | (en & (en - 1))) != 0) {
          many |= 1u << t;
          continue;
        }
        const double *xe = M.ev.pt[first_bit(ex)][sl], *ee = M.ev.pt[first_bit(en)][sl];
        const double *c = M.X[fc[t]][sl];
        const double x0 = xe[0], x1 = xe[1], x2 = xe[2], e0 = ee[0], e1 = ee[1], e2 = ee[2];
        vf += det3(c[0], c[1], c[2], x0, x1, x2, e0, e1, e2);
        add_segment(acc, r0, r1, r2, x0, x1, x2, e0, e1, e2);
      }
      bool bad = false;
      const bool one = single && group_bits<G>(many != 0, base) == 0;
      double Vi = 0.0;
      if (one) {
        vf = tsum<G>(vf);
        reduce_acc<G>(acc);
        double k0, k1, k2;
        loop_centre(acc, r0, r1, r2, k0, k1, k2);
        Vi = k0 * acc.Y0 + k1 * acc.Y1 + k2 * acc.Y2;
      } else {
        // several loops: the chords' entry edges by exit edge, and the
        // volume terms that the faces with several chords still owe
#pragma unroll
        for (int t = 0; t < KF; ++t) {
          const EM ex = cut & fo[t], en = cut & fi[t];
          if ((ex | en) == 0) continue;
          if (count_bits(ex) != count_bits(en)) {
            bad = true;   // a closed loop alternates exits and entries
          } else if (((many >> t) & 1) == 0) {
            M.ev.part[first_bit(ex)][sl] = (uint8_t)first_bit(en);
          } else {
            // exits and entries as bits over the loop's positions; each exit
            // goes with the next entry or the previous one
            const bool conn = face_mean(t) >= se;
            const int o = (int)(fl[t] & 0xffffu), n = (int)(fl[t] >> 16);
            uint64_t xb = 0, nb = 0;
            for (int i = 0; i < n; ++i) {
              const int e = M.eid[o + i][sl];
              xb |= (uint64_t)((ex >> e) & 1) << i;
              nb |= (uint64_t)((en >> e) & 1) << i;
            }
            const double *c = M.X[fc[t]][sl];
            for (uint64_t left = xb; left != 0; left &= left - 1) {
              const int i = first_bit(left);
              const uint64_t after = i == 63 ? 0 : nb >> (i + 1) << (i + 1), before = nb & ~after;
              const int r = conn ? first_bit(after ? after : nb) : 63 - __clzll((long long)(before ? before : nb));
              const int e = M.eid[o + i][sl], er = M.eid[o + r][sl];
              M.ev.part[e][sl] = (uint8_t)er;
              const double *xe = M.ev.pt[e][sl], *x = M.ev.pt[er][sl];
              vf += det3(c[0], c[1], c[2], xe[0], xe[1], xe[2], x[0], x[1], x[2]);
            }
          }
        }
        bad = group_bits<G>(bad, base) != 0;
        vf = tsum<G>(vf);
        wave_sync();
        // label the loops by following the chords, then add up each loop
        int nloop = 0;
        for (EM left = cut; left != 0 && !bad; ++nloop) {
          const int t0 = first_bit(left);
          int u = t0;
          do {
            M.ev.lab[u][sl] = (uint8_t)nloop;
            left &= ~((EM)1 << u);
            u = M.ev.part[u][sl];
          } while ((left >> u) & 1);
          bad = u != t0;
        }
        wave_sync();
        double S0 = 0, S1 = 0, S2 = 0, A = 0, cw0 = 0, cw1 = 0, cw2 = 0;
        for (int lp = 0; lp < nloop && !bad; ++lp) {
          acc = ChordAcc{0, 0, 0, 0, 0, 0, 0};
          for (int e = q; e < ne; e += G) {
            if (!((cut >> e) & 1) || M.ev.lab[e][sl] != lp) continue;
            const double *xe = M.ev.pt[e][sl], *en = M.ev.pt[M.ev.part[e][sl]][sl];
            add_segment(acc, r0, r1, r2, xe[0], xe[1], xe[2], en[0], en[1], en[2]);
          }
          reduce_acc<G>(acc);
          finish_loop(acc, r0, r1, r2, Vi, S0, S1, S2, A, cw0, cw1, cw2);
        }
        M.fin[1][sl] = S0; M.fin[2][sl] = S1; M.fin[3][sl] = S2;
        M.fin[4][sl] = A;
        M.fin[5][sl] = cw0; M.fin[6][sl] = cw1; M.fin[7][sl] = cw2;
      }
      wave_sync();
      // the liquid fraction, V / V_P by the reciprocal and one correction
      // (the value reported is the one the tolerance was tested on)
      const double V = (vf + Vi) * (1.0 / 6.0);
      double frac = V * iVP;
      frac = fma(fma(-VP, frac, V), iVP, frac);
      it += ph == kSearch ? tm.weight : 1;   // a fixed isovalue and the end kept are one cut
      const double r = frac - a;
      bool done = ph == kFixed || ph == kFinal;
      int win = g;   // the group whose cut ends the search
      if (ts == 1) {
        done = done || fabs(r) <= tol;
      } else {
        if (q == 0) {
          M.smp[0][sl] = se;
          M.smp[1][sl] = r;
        }
        wave_sync();
        // sample i of the team on the lanes i, i + ts, ... of every row
        const int i = lane & (ts - 1);
        const double sx = M.smp[0][lead + i], sr = M.smp[1][lead + i], ar = fabs(sr);
        // reductions over the samples, and the first sample of which c holds;
        // a row repeats four samples, so its quads have all of them
        const int row = lane & ~15;
        auto row_min = [&](double x) { return G == 16 || ts == 4 ? tmin<4>(x) : tmin<16>(x); };
        auto row_max = [&](double x) { return G == 16 || ts == 4 ? tmax<4>(x) : tmax<16>(x); };
        auto sample = [&](bool c) { return first_bit(group_bits<16>(c, row)) & (ts - 1); };
        if (done) {
          win = 0;
        } else {
          if (!done && group_bits<16>(ar <= tol, row) != 0) {
            done = true;
            // (the smallest residual; inside the narrowed bracket if one is)
            const bool in = ar <= tol && !(hint && (sx < M.hint[1][sl] || sx > M.hint[2][sl]));
            const double least = group_bits<16>(in, row) != 0 ? row_min(in ? ar : __builtin_inf()) : row_min(ar);
            win = sample(ar == least && (in || group_bits<16>(in, row) == 0));
          }
        }
        if (!done) {
          // the tightest sign change becomes the bracket [xa, xb]; the third
          // point of the estimate is the one of smallest residual off it
          const double inf = __builtin_inf();
          const double plo = xa, pfl = fa, phi_ = xb, pfh = fb;
          const bool pos = sr > 0 && sx > plo && sx < phi_;
          const double slo = row_max(pos ? sx : -inf);
          if (slo > plo) {
            fa = M.smp[1][lead + sample(pos && sx == slo)];
            xa = slo;
          }
          const bool neg = !(sr > 0) && sx > xa && sx < phi_;
          const double shi = row_min(neg ? sx : inf);
          if (shi < phi_) {
            fb = M.smp[1][lead + sample(neg && sx == shi)];
            xb = shi;
          }
          const bool off = sx != xa && sx != xb;
          double m3 = row_min(off ? ar : inf);
          if (m3 < inf) {
            xc = row_min(off && ar == m3 ? sx : inf);
            fcv = M.smp[1][lead + sample(off && sx == xc)];
          }
          if (xa != plo && fabs(pfl) < m3) {
            m3 = fabs(pfl);
            xc = plo; fcv = pfl;
          }
          if (xb != phi_ && fabs(pfh) < m3) {
            xc = phi_; fcv = pfh;
          }
          nbis = fmin(fabs(fa), fabs(fb)) > 0.25 * fmin(fabs(pfl), fabs(pfh)) ? nbis + 1 : 0;
          wave_sync();
          continue;
        }
      }
      if (done) {
        // the cut that ends the search, in the slot of the cell's first group
        if (one) {
          double vi = 0.0, S0 = 0, S1 = 0, S2 = 0, A = 0, cw0 = 0, cw1 = 0, cw2 = 0;
          finish_loop(acc, r0, r1, r2, vi, S0, S1, S2, A, cw0, cw1, cw2);
          M.fin[1][sl] = S0; M.fin[2][sl] = S1; M.fin[3][sl] = S2;
          M.fin[4][sl] = A;
          M.fin[5][sl] = cw0; M.fin[6][sl] = cw1; M.fin[7][sl] = cw2;
        }
        M.fin[0][sl] = frac;
        M.fin[8][sl] = bad ? 1.0 : 0.0;
        wave_sync();
        if (ts > 1) {
          se = M.smp[0][lead + win];
          if (g == win && g != 0)
            for (int i = q; i < 9; i += G) M.fin[i][lead] = M.fin[i][sl];
          wave_sync();
        }
        break;
      }
      // the cut becomes the bracket end of its sign and the newest of the
      // remembered ones
      xd = xc; fd = fcv;
      xc = above ? xa : xb; fcv = above ? fa : fb;
      ++cuts;
      nbis = fabs(r) > 0.5 * fmin(fabs(fa), fabs(fb)) ? nbis + 1 : 0;
      above = r > 0;
      if (above) {
        xa = se; fa = r;
      } else {
        xb = se; fb = r;
      }
    }
    // the narrowed bracket did not hold the root
    if (hint && st == VOFPC_CELL_OK && (se < M.hint[1][sl] || se > M.hint[2][sl])) st = VOFPC_CELL_LEARNED_FALLBACK;
    if (M.fin[8][lead] != 0.0) {
      st = VOFPC_CELL_BAD_INPUT;
    } else {
      s_out = se;
      ag = M.fin[0][lead];
      A_out = M.fin[4][lead];
      const double S0 = M.fin[1][lead], S1 = M.fin[2][lead], S2 = M.fin[3][lead];
      const double Sm = sqrt(S0 * S0 + S1 * S1 + S2 * S2);
      if (Sm > 0) {
        n0 = S0 / Sm; n1 = S1 / Sm; n2 = S2 / Sm;
        d_out = -(n0 * M.fin[5][lead] + n1 * M.fin[6][lead] + n2 * M.fin[7][lead]) / A_out;
      }
    }
  }
  if (active && q == 0 && g == 0) {
    if (p.mf.gradT) {
      // mass transfer of the entry (one-sided form, as vofpc_mass_transfer)
      double md = 0.0;
      if (A_out > 0.0) {
        const double gn = p.mf.gradT[P] * n0 + p.mf.gradT[N + P] * n1 + p.mf.gradT[2 * N + P] * n2;
        const double gl = (a >= 0.5) ? gn : 0.0, gv = (a >= 0.5) ? 0.0 : gn;
        const double ql = p.mf.k_l * gl * A_out;
        const double qv = -p.mf.k_v * gv * A_out;
        md = (ql + qv) / (p.mf.h_lv * m.V[P]);
      }
      p.mf.mdot[k] = md;
      p.mf.Qdot[k] = -md * p.mf.h_lv;
    }
    p.out.s[k] = s_out;
    p.out.n[k] = n0; p.out.n[cap + k] = n1; p.out.n[2 * cap + k] = n2;
    p.out.A[k] = A_out;
    p.out.d[k] = d_out;
    p.out.alpha_got[k] = ag;
    p.out.status[k] = st;
    p.out.iters[k] = it;
  }
}

// A wavefront's groups work as teams while the wavefronts still take them in
// this many rounds: a step of a team costs what a step of one cell does, and
// the groups it joins had no cells of their own.  Builds of 16 lanes a cell:
// two rounds of teams of four; of four lanes a cell: one round of teams of
// sixteen, then one of teams of four.  Whole label passes on 2,048 wavefronts:
// 3,342 Voronoi cells 92 us in two rounds of teams, 99 us without teams; 2,832
// with the network 117 and 116; 226 hexahedra in teams of sixteen 38 us, 53 us
// without; 3,200 hexahedra in teams of four 60 us, of sixteen (two rounds)
// 73 us; 10,251 without teams 83 us, in two rounds of teams of four 102 us.
template <int C>
__device__ __forceinline__ int cells_per_wave(int64_t count, int64_t waves) {
  if (C == 16) return count <= waves ? 1 : (count <= 4 * waves ? 4 : 16);
  return count <= 2 * waves ? 1 : C;
}

// Waves per SIMD a build's register budget is sized for: at most 2 (256
// VGPRs).  A third one leaves 168 VGPRs and spills in the search: 24,042
// Voronoi cells reconstructed in 224 us against 202 us, 31,948 hexahedra in
// 159 against 146 us.
constexpr int group_occupancy(int bytes) {
  const int w = (160 * 1024) / bytes / 4;
  return w >= 2 ? 2 : 1;
}

// LDS of a wavefront: the larger of the builds it runs (Big: void for one).
template <class Main, class Big>
struct WaveMem {
  union {
    typename Main::Mem a;
    typename Big::Mem b;
  };
};
template <class Main>
struct WaveMem<Main, void> {
  typename Main::Mem a;
};

// The cells of a launch.  With Big, cells that do not fit Main are solved by
// the wavefront that meets them in the Big build, after its other cells.
template <class Main, class Big, bool NET>
__global__ __launch_bounds__(64, (group_occupancy((int)sizeof(WaveMem<Main, Big>))))
void recon_group_kernel(ReconParams p) {
  constexpr int G = Main::G, C = 64 / G;
  __shared__ WaveMem<Main, Big> M;
  const DevMesh &m = p.m;
  int64_t count = p.entries ? (int64_t)*p.entry_count : (int64_t)p.counts[0];
  if (count > p.out.cap) count = p.out.cap;
  Team tm;
  tm.lane = threadIdx.x;
  tm.sl = tm.lane / G;
  tm.q = tm.lane % G;
  tm.base = tm.lane & ~(G - 1);
  // cells per batch, cw, and groups per cell, ts: with few cells the groups
  // of a wavefront form teams that cut one cell at ts isovalues per step
  tm.cw = cells_per_wave<C>(count, gridDim.x);
  tm.ts = C / tm.cw;
  tm.g = tm.sl & (tm.ts - 1);
  tm.lead = tm.sl - tm.g;
  // a step of 4 or 16 isovalues narrows the bracket as 2 or 4 halvings do and
  // counts as that many evaluations
  tm.weight = tm.ts == 16 ? 4 : (tm.ts == 4 ? 2 : 1);
  const int64_t nbatch = (count + tm.cw - 1) / tm.cw;
  // this XCD's batches (runs of kRunCells cells for full batches): the first
  // one per workgroup by its index, the rest claimed from the XCD's counter
  constexpr int kRun = kRunCells / C;
  const int xcd = (int)(blockIdx.x % kXcd);
  const int64_t nx = xcd_count<kRun>(nbatch, xcd);
  const int64_t wx = ((int64_t)gridDim.x - xcd + kXcd - 1) / kXcd;
  unsigned int *claim = reinterpret_cast<unsigned int *>(p.queue + (1 + xcd) * kQueueStride);
  for (int64_t ix = blockIdx.x / kXcd; ix < nx;) {
    const int64_t j = xcd_batch<kRun>(ix, xcd) * tm.cw + tm.sl / tm.ts;
    const bool active = j < count;
    CellRef cell;
    if (active) {
      cell.k = p.entries ? (int64_t)p.entries[j] : j;
      cell.P = p.mixed[cell.k];
      cell.a = p.alpha[cell.P];
      cell.f0 = m.cell_face_off[cell.P];
      cell.nf = (int)(m.cell_face_off[cell.P + 1] - cell.f0);
      cell.v0 = m.cv_off[cell.P];
      cell.nv = (int)(m.cv_off[cell.P + 1] - cell.v0);
      cell.l0 = m.cl_off[cell.P];
      cell.nl = (int)(m.cl_off[cell.P + 1] - cell.l0);
    }
    if constexpr (std::is_void_v<Big>) {
      solve_cells<Main, NET>(p, M.a, tm, cell, active);
    } else {
      const bool fits = Main::fits(cell.nv, cell.nf, cell.nl);
      solve_cells<Main, NET>(p, M.a, tm, cell, active && fits);
      if (__any(active && !fits)) {
        wave_sync();
        solve_cells<Big, NET>(p, M.b, tm, cell, active && !fits);
      }
    }
    // next batch: a wrapping increment, so the XCD's nx claims (one per
    // batch done) bring its counter back to zero
    int nb = 0;
    if (tm.lane == 0) nb = (int)atomicInc(claim, (unsigned int)(nx - 1));
    ix = wx + __builtin_amdgcn_readfirstlane(nb);
    wave_sync();
  }
}

template <class Main, class Big, bool NET>
vofpc_status launch_net(vofpc_ctx ctx, const ReconParams &p, int64_t n_entries) {
  int blocks_per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks_per_cu, recon_group_kernel<Main, Big, NET>, 64, 0);
  if (e != hipSuccess || blocks_per_cu <= 0) blocks_per_cu = 1;
  int64_t grid = (int64_t)ctx->n_cu * blocks_per_cu;
  if (grid > n_entries) grid = n_entries;
  if (grid < 1) grid = 1;
  recon_group_kernel<Main, Big, NET><<<(unsigned)grid, 64, 0, ctx->stream>>>(p);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

// the plain build, or the build that runs the network (learned form)
template <class Main, class Big = void>
vofpc_status launch_t(vofpc_ctx ctx, const ReconParams &p, int64_t n_entries) {
  if (p.net_wb) return launch_net<Main, Big, true>(ctx, p, n_entries);
  return launch_net<Main, Big, false>(ctx, p, n_entries);
}

// The builds: class 0 in two sizes (hexahedra and smaller; the class caps),
// classes 1 and 2 at their caps.  The group is the smallest whose lanes hold
// a cell's edges in registers.
using HexBuild = Build<4, 8, 6, 24, 12>;
using SmallBuild = Build<4, 16, 8, 48, 24>;
using UsualBuild = Build<16, 32, 20, 96, 48>;
using LargeBuild = Build<16, 48, 32, 128, 64, 4>;   // unpadded: beside UsualBuild it must not cost wavefronts

template <class B>
__host__ bool fits(const int64_t cmax[4]) {
  return B::fits(cmax[0], cmax[1], cmax[2]) && cmax[3] <= B::NE;
}

}  // namespace

bool thin_available(int c, int G, const int64_t cmax[4]) {
  if (c == 0) return fits<HexBuild>(cmax) ? (G == 1 || G == 2 || G == 4) : ((G == 2 || G == 4) && fits<SmallBuild>(cmax));
  if (c == 1) return (G == 4 || G == 8 || G == 16) && fits<UsualBuild>(cmax);
  if (c == 2) return (G == 4 || G == 8 || G == 16) && fits<LargeBuild>(cmax);
  return false;
}

vofpc_status launch_thin(vofpc_ctx ctx, const ReconParams &p, int64_t n_entries, int c, int G, const int64_t cmax[4],
                         bool with_large) {
  VOFPC_REQUIRE(thin_available(c, G, cmax), VOFPC_E_INVALID_ARG, "reconstruct: no group build for this class");
  if (c == 0) return fits<HexBuild>(cmax) ? launch_t<HexBuild>(ctx, p, n_entries) : launch_t<SmallBuild>(ctx, p, n_entries);
  if (c == 1)
    return with_large ? launch_t<UsualBuild, LargeBuild>(ctx, p, n_entries) : launch_t<UsualBuild>(ctx, p, n_entries);
  return launch_t<LargeBuild>(ctx, p, n_entries);
}

}  // namespace vofpc

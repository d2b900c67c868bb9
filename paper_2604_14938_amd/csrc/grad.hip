// Interface-modified least-squares temperature gradient (App. B with the
// modification of Sec. 2.4.4) and the mass transfer rate (Eq. mass_transfer,
// Eq. latent_source).
//
// A group of lanes per cell, faces dealt round the lanes.  The gradient gathers,
// for every face of the cell, the neighbour centroid (one 32-byte record), alpha
// and T, or the boundary face centroid and value, and accumulates the
// least-squares matrix beside the right-hand side; solving it in registers is
// cheaper than reading a stored inverse (48 bytes a cell).  Every cell of
// 1,953,125 hexahedra: 66 us, 3.2 TB/s of the 211 MB it must move (197 us with
// eight lanes a cell, of which two idled, the centroids in three arrays, the
// inverse read and each third cache line stored by one lane of eight).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lsq.h"
#include "vofpc_internal.h"
#include "wave_ops.h"

namespace vofpc {

struct GradParams {
  DevMesh m;
  const double *T, *Tb, *alpha;
  double T_sat;
  const int32_t *band, *counts;
  int scope, variant;   // base variant (VOFPC_GRAD_MODIFIED/STANDARD/PRINTED)
  int weight;           // 0 uniform, 1 inverse distance, 2 inverse distance squared
  const int64_t *xn_off;   // vertex-neighbour stencil (null: face neighbours)
  const int32_t *xn_cell;
  double *grad;
  int32_t *status;
};

// Gradient of cell P by a group of W lanes: lane j takes faces j, j + W, ...,
// kAhead of them at a time, whose gathers are in flight together; the
// least-squares sums are reduced over the group.
template <int W>
__device__ __forceinline__ void grad_cell(const GradParams &p, int P, int j) {
  constexpr int kAhead = W >= 8 ? 2 : 4;   // (two rounds of eight: most polyhedra)
  const DevMesh &m = p.m;
  const int64_t N = m.n_cells, NF = m.n_faces;
  const double4 xP = m.xr[P];
  const double aP = p.alpha[P], TP = p.T[P];
  const bool modify = p.variant != VOFPC_GRAD_STANDARD;
  const bool printed = p.variant == VOFPC_GRAD_PRINTED;
  LsqSums L;
  auto walk = [&](const int32_t *nbr, int64_t i0, int64_t i1, bool inner, bool bounds) {
    for (int64_t i = i0 + j; i < i1; i += W * kAhead) {
      int q[kAhead];
      double4 x[kAhead];
      double aQ[kAhead], tQ[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) q[k] = i + k * W < i1 ? nbr[i + k * W] : -3;
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const int c = q[k] >= 0 ? q[k] : P;   // (the cell itself: read, not used)
        x[k] = m.xr[c];
        aQ[k] = p.alpha[c];
        tQ[k] = p.T[c];
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        if (q[k] >= 0) {
          if (!inner) continue;
          // the centre connection, shortened to the alpha-interpolated
          // crossing held at T_sat where the interface cuts it
          double r0 = x[k].x - xP.x, r1 = x[k].y - xP.y, r2 = x[k].z - xP.z, val = tQ[k];
          if (modify && (aP - 0.5) * (aQ[k] - 0.5) < 0.0) {
            const double t = printed ? fabs(aQ[k] - 0.5) / fabs(aP - aQ[k]) : (aP - 0.5) / (aP - aQ[k]);
            r0 *= t; r1 *= t; r2 *= t;
            val = p.T_sat;
          }
          L.add(r0, r1, r2, val - TP, p.weight);
        } else if (q[k] == -1 && bounds) {
          const int f = m.cell_face[i + k * W];
          L.add(m.xf[f] - xP.x, m.xf[NF + f] - xP.y, m.xf[2 * NF + f] - xP.z, p.Tb[f] - TP, p.weight);
        }
      }
    }
  };
  if (p.xn_off) walk(p.xn_cell, p.xn_off[P], p.xn_off[P + 1], true, false);
  // (no boundary values given: interior neighbours only)
  if (!p.xn_off || p.Tb) walk(m.cf_nbr, m.cell_face_off[P], m.cell_face_off[P + 1], !p.xn_off, p.Tb != nullptr);
  lsq_reduce<W>(L);
  if (j != 0) return;
  double g0, g1, g2;
  const int st = lsq_solve(L, g0, g1, g2) ? VOFPC_CELL_OK : VOFPC_CELL_G_SINGULAR;
  p.grad[P] = g0;
  p.grad[N + P] = g1;
  p.grad[2 * N + P] = g2;
  if (p.status) p.status[P] = st;
}

// A block of 256 lanes serves 256 / W cells at a time; every lane of a group
// iterates the same cells, so the group's reductions see all its lanes.  Blocks
// go to the XCDs in turn (block b to XCD b % 8), so the blocks of one XCD take
// one eighth of the cells in order: a neighbour's record is then mostly in
// that XCD's own L2.
template <int W>
__global__ __launch_bounds__(256) void grad_kernel(GradParams p) {
  const int64_t n = (p.scope == VOFPC_SCOPE_ALL) ? p.m.n_cells : (int64_t)p.counts[1];
  constexpr int kCells = 256 / W;
  const int j = threadIdx.x % W;
  const int64_t units = (n + kCells - 1) / kCells;
  const int x = blockIdx.x % kXcd, per = (int)(gridDim.x / kXcd);   // gridDim.x is a multiple of kXcd
  const int64_t last = units * (x + 1) / kXcd;
  for (int64_t u = units * x / kXcd + blockIdx.x / kXcd; u < last; u += per) {
    const int64_t k = u * kCells + threadIdx.x / W;
    if (k < n) grad_cell<W>(p, (p.scope == VOFPC_SCOPE_ALL) ? (int)k : p.band[k], j);
  }
}

static vofpc_status grad_params(vofpc_mesh M, const double *T, const double *Tb, double T_sat, const double *alpha,
                                const int32_t *band, const int32_t *counts, int32_t scope, int32_t variant,
                                double *grad, int32_t *status, GradParams &p) {
  VOFPC_REQUIRE(T && alpha && grad, VOFPC_E_INVALID_ARG, "grad_T: null argument");
  VOFPC_REQUIRE(scope == VOFPC_SCOPE_BAND || scope == VOFPC_SCOPE_ALL, VOFPC_E_INVALID_ARG, "grad_T: unknown scope");
  VOFPC_REQUIRE(scope == VOFPC_SCOPE_ALL || (band && counts), VOFPC_E_INVALID_ARG,
                "grad_T: band scope needs band_idx and counts");
  const int base = variant & 0xf, flags = variant & ~0xf;
  VOFPC_REQUIRE(base >= VOFPC_GRAD_MODIFIED && base <= VOFPC_GRAD_PRINTED &&
                    (flags & ~(VOFPC_GRAD_W_INV_DIST | VOFPC_GRAD_W_INV_DIST2 | VOFPC_GRAD_VERTEX_STENCIL)) == 0 &&
                    (flags & (VOFPC_GRAD_W_INV_DIST | VOFPC_GRAD_W_INV_DIST2)) !=
                        (VOFPC_GRAD_W_INV_DIST | VOFPC_GRAD_W_INV_DIST2),
                VOFPC_E_INVALID_ARG, "grad_T: unknown variant");
  VOFPC_REQUIRE(!(flags & VOFPC_GRAD_VERTEX_STENCIL) || M->xn_off, VOFPC_E_STATE,
                "grad_T: the vertex stencil of this mesh is not built");
  p.m = M->d;
  p.T = T; p.Tb = Tb; p.alpha = alpha; p.T_sat = T_sat;
  p.band = band; p.counts = counts;
  p.scope = scope; p.variant = base;
  p.weight = (flags & VOFPC_GRAD_W_INV_DIST) ? 1 : (flags & VOFPC_GRAD_W_INV_DIST2) ? 2 : 0;
  p.xn_off = (flags & VOFPC_GRAD_VERTEX_STENCIL) ? M->xn_off : nullptr;
  p.xn_cell = (flags & VOFPC_GRAD_VERTEX_STENCIL) ? M->xn_cell : nullptr;
  p.grad = grad; p.status = status;
  return VOFPC_OK;
}

template <int W>
static void grad_launch(vofpc_ctx ctx, const GradParams &p, int64_t cells) {
  int64_t grid = ((cells + 256 / W - 1) / (256 / W) + kXcd - 1) / kXcd;   // blocks per XCD
  const int64_t cap = (int64_t)ctx->n_cu * 8 / kXcd;
  if (grid > cap) grid = cap;
  grad_kernel<W><<<(unsigned)std::max<int64_t>(grid, 1) * kXcd, 256, 0, ctx->stream>>>(p);
}

vofpc_status launch_grad(vofpc_ctx ctx, vofpc_mesh M, const double *T, const double *Tb, double T_sat,
                         const double *alpha, const int32_t *band, const int32_t *counts, int32_t scope,
                         int32_t variant, double *grad, int32_t *status) {
  GradParams p;
  vofpc_status st = grad_params(M, T, Tb, T_sat, alpha, band, counts, scope, variant, grad, status, p);
  if (st) return st;
  // Lanes per cell.  Every cell: one where the cells have about six faces and
  // lie in order (their gathers coalesce), two for polyhedra; twice that for a
  // mesh too small to fill the chip so.  The band: eight; its cells are few and
  // scattered, a chain of gathers.  Microseconds with 1 / 2 / 4 / 8 lanes:
  //   1,953,125 hexahedra, all cells   66 / 69 / 125 / 167
  //   410,758 Voronoi cells, all       51 / 41 /  47 /  53
  //   16,000 Voronoi cells, all        13 /  8 /   6 /   6
  //   43,463 Voronoi cells of a band   15 / 11 / 9.4 / 10.2
  //   the same, vertex stencil         21 / 16 / 13.3 / 13.6
  const int64_t N = M->d.n_cells;
  if (scope != VOFPC_SCOPE_ALL) {
    grad_launch<8>(ctx, p, N);
  } else {
    const bool even = M->ncf <= 8 * N, small = N < 32768;
    if (even && !small) grad_launch<1>(ctx, p, N);
    else if (even || !small) grad_launch<2>(ctx, p, N);
    else grad_launch<4>(ctx, p, N);
  }
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

// ------------------------------------------------------------ mass transfer
struct MdotParams {
  const double *V, *alpha;
  int64_t n_cells;
  const int32_t *mixed, *counts;
  vofpc_interface itf;
  const double *gradT, *gl, *gv;
  double k_l, k_v, h_lv;
  double *mdot, *Qdot, *mdot_c, *Qdot_c;
};

__global__ __launch_bounds__(256) void fill_zero_kernel(double *a, double *b, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride) {
    if (a) a[i] = 0.0;
    if (b) b[i] = 0.0;
  }
}

__global__ __launch_bounds__(256) void mdot_kernel(MdotParams p) {
  int64_t n = p.counts[0];
  if (n > p.itf.cap) n = p.itf.cap;
  const int64_t N = p.n_cells, cap = p.itf.cap;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += stride) {
    const int P = p.mixed[k];
    const double A = p.itf.A[k];
    double md = 0.0;
    if (A > 0.0) {
      const double n0 = p.itf.n[k], n1 = p.itf.n[cap + k], n2 = p.itf.n[2 * cap + k];
      double gl = 0.0, gv = 0.0;  // projections on n
      if (p.gl && p.gv) {
        gl = p.gl[P] * n0 + p.gl[N + P] * n1 + p.gl[2 * N + P] * n2;
        gv = p.gv[P] * n0 + p.gv[N + P] * n1 + p.gv[2 * N + P] * n2;
      } else {
        const double gn = p.gradT[P] * n0 + p.gradT[N + P] * n1 + p.gradT[2 * N + P] * n2;
        if (p.alpha[P] >= 0.5) gl = gn; else gv = gn;
      }
      const double ql = p.k_l * gl * A;
      const double qv = -p.k_v * gv * A;
      md = (ql + qv) / (p.h_lv * p.V[P]);
    }
    p.mdot[k] = md;
    p.Qdot[k] = -md * p.h_lv;
    if (p.mdot_c) p.mdot_c[P] = md;
    if (p.Qdot_c) p.Qdot_c[P] = -md * p.h_lv;
  }
}

vofpc_status launch_mass_transfer(vofpc_ctx ctx, vofpc_mesh M, const double *alpha, const int32_t *mixed,
                                  const int32_t *counts, const vofpc_interface *itf, const double *gradT,
                                  const double *gl, const double *gv, double k_l, double k_v, double h_lv,
                                  double *mdot, double *Qdot, double *mdot_c, double *Qdot_c) {
  VOFPC_REQUIRE(alpha && mixed && counts && itf && mdot && Qdot, VOFPC_E_INVALID_ARG, "mass_transfer: null argument");
  VOFPC_REQUIRE(itf->n && itf->A && itf->cap > 0, VOFPC_E_INVALID_ARG, "mass_transfer: interface record incomplete");
  VOFPC_REQUIRE((gl == nullptr) == (gv == nullptr), VOFPC_E_INVALID_ARG,
                "mass_transfer: give both phase gradients or neither");
  VOFPC_REQUIRE(gradT || gl, VOFPC_E_INVALID_ARG, "mass_transfer: no gradient given");
  VOFPC_REQUIRE(h_lv != 0.0, VOFPC_E_INVALID_ARG, "mass_transfer: h_lv must be nonzero");
  const int64_t N = M->d.n_cells;
  hipStream_t s = ctx->stream;
  if (mdot_c || Qdot_c) {
    int64_t g = (N + 255) / 256;
    if (g > ctx->n_cu * 8) g = ctx->n_cu * 8;
    fill_zero_kernel<<<(unsigned)g, 256, 0, s>>>(mdot_c, Qdot_c, N);
  }
  MdotParams p;
  p.V = M->d.V; p.alpha = alpha; p.n_cells = N;
  p.mixed = mixed; p.counts = counts; p.itf = *itf;
  p.gradT = gradT; p.gl = gl; p.gv = gv;
  p.k_l = k_l; p.k_v = k_v; p.h_lv = h_lv;
  p.mdot = mdot; p.Qdot = Qdot; p.mdot_c = mdot_c; p.Qdot_c = Qdot_c;
  int64_t grid = (std::min<int64_t>(N, itf->cap) + 255) / 256;
  if (grid > ctx->n_cu * 8) grid = ctx->n_cu * 8;
  if (grid < 1) grid = 1;
  mdot_kernel<<<(unsigned)grid, 256, 0, s>>>(p);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

}  // namespace vofpc
